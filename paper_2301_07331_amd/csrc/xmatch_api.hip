// xmatch_api.hip -- the single-call entry points: hlc_xmatch (and its
// self-match mode), hlc_xmatch_radii (eq. (4) per-source radii) and
// hlc_xmatch_quad (the paper's HEALPix + quad-direction partition, emulated).
#include <hip/hip_runtime.h>

#include <cstring>
#include <new>

#include "host.hpp"

namespace hlc {
namespace {

int xmatch_impl(const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
                const double* b_dec, int64_t nb, double r_arcsec, hlc_pair* out_pairs,
                double* out_sep, const hlc_opts* o, Caps& caps, bool* again, const Radii& rad) {
  *again = false;
  Device* dev = nullptr;
  HLC_CHECK(get_device(&dev));
  hipStream_t s = (hipStream_t)o->stream;
  const bool prof = (o->flags & HLC_PROFILE) != 0;
  const int plevel = prof_level(o->flags);
  const bool fp32 = o->precision == HLC_FP32_RECHECK;
  const bool self = (o->flags & HLC_SELF) != 0;
  dev->ordered = false;
  if (prof) HLC_TRY(hipEventRecord(dev->ev[0], s));
  const int64_t na_frame = self ? 0 : na;
  const uint32_t nB = (uint32_t)nb;
  // self-match: A's entries are B's (halo copies included)
  const uint32_t nA = self ? 2 * nB : (uint32_t)na;
  const Slots slB = prof ? Slots{1, 2, 3, 4} : NO_SLOTS;
  const Slots slA = prof ? Slots{5, -1, 6, 7} : NO_SLOTS;

  Side A, B;
  A.plan = plan_sort(na, caps.digit_sort);
  B.plan = plan_sort(nb, caps.digit_sort);
  // what the speculative keygens assume of the crowding (calls that do not ask
  // neither take it from the last that did nor change it for the next; set before
  // A's: the number of radix passes decides which buffer that keygen writes)
  const bool crowd = !B.plan.K && std::max(na, nb) >= CROWD_MIN;
  const bool assumed = crowd && dev->last_crowded;
  Geom g = make_geom(r_arcsec, tuned_height(o), na, nb, tuned_bins(o), Frame{}, assumed);
  // B's windows are cut at sub-bin resolution when its sort orders those bits
  // too: the bucket sort always does. A's digit sort orders them only where the
  // sources are crowded: its groups' windows take the least and largest of their
  // fractions in any order (10M x 1M: 647 us a call with that pass, 595 without)
  Geom gA;
  auto sub_bins = [&](bool crowded) {
    gA = g;
    gA.frac_sorted = crowded || tuned_fraction_sort(o) ? 1 : 0;
    g.frac_sorted = B.plan.K || gA.frac_sorted ? 1 : 0;
  };
  sub_bins(assumed);
  SortScratch sc, scA;
  MatchWs w;
  // FP32: B in the sorted certification layout when the last FP32 call on
  // this device had that many candidates per B entry
  const bool sorted_b = fp32 && !B.plan.K && dev->cand_per_b >= SORTED_RADEC_MIN;
  // both sides through the bucket sort in the same form: in the same launches,
  // all on the caller's stream (two streams' events cost more than running side
  // by side gains: 2,000 a side 99 us against 137, 300k 201 against 213, 1.4M
  // the same)
  const bool both = !self && !prof && same_form(A.plan, B.plan);
  auto lay = [&](Carve& c) {
    // A is read in place: the filter gathers its records itself
    if (!self) {
      carve_side(c, A, nA, !fp32, fp32, nA, false);
      carve_sort(c, scA, nA, A);
    }
    carve_side(c, B, 2 * nB, !fp32, fp32, nB, true, sorted_b);
    carve_sort(c, sc, 2 * nB, B);
    carve_order_ahead(c, w, *dev, o, na, nb);
    carve_match_ws(c, w, nA, g, caps, true);
  };
  // While the host waits for the sample, A's and B's keys under the
  // whole-sphere frame are computed if the previous call on this device had
  // that frame and the workspace already fits it (the places of their
  // buffers do not depend on the frame). They are kept if the sample
  // confirms the frame, else computed again.
  bool spec = false;
  Carve guess{nullptr};
  lay(guess);
  const bool fits = guess.off + 256 <= dev->ws_bytes;
  if (dev->last_full) spec = fits;
  // what the counters' clearing reaches: places that depend on the workspace
  // and the sizes, not on the frame
  struct Cleared {
    size_t ws_bytes;
    void* at[4];
    bool operator==(const Cleared& o) const {
      return ws_bytes == o.ws_bytes && std::memcmp(at, o.at, sizeof at) == 0;
    }
  };
  auto cleared = [&]() { return Cleared{dev->ws_bytes, {dev->ws, A.bws.fine, B.bws.fine, w.reg.cfill}}; };
  auto clear = [&]() { launch_zero_counters(dev->cnt, s, A.bws.fine, B.bws.fine, &w.reg); };
  Cleared early{};
  FrameQuery fq;
  if (spec) {
    Carve c{(char*)dev->ws};
    lay(c);
    if (prof) HLC_TRY(hipEventRecord(dev->ev[14], s));
    clear();
    // B's on the caller's stream, launched first (B's chain is the longer
    // one); the sample and A's keygen beside it on the side stream, where A's
    // sort follows (the places of B's buffers do not depend on the frame
    // either)
    HLC_TRY(hipEventRecord(dev->fork, s));
    // (a self-match's one keygen goes ahead of the sample: 4M, 442 us a call
    // before, 420; with two, A's would wait for the sample beside B's: no gain)
    if (self) partition_keys(*dev, b_ra, b_dec, nB, g, true, !fp32, fp32, sc, 2u, B, slB, s);
    HLC_TRY(hipStreamWaitEvent(dev->side, dev->fork, 0));
    fq = frame_begin(*dev, a_ra, a_dec, na_frame, b_ra, b_dec, nb, crowd, dev->side);
    if (both) {
      partition_keys_both(*dev, a_ra, a_dec, nA, scA, A, b_ra, b_dec, nB, sc, B, g, s);
    } else {
      if (!self) partition_keys(*dev, b_ra, b_dec, nB, g, true, !fp32, fp32, sc, 2u, B, slB, s);
      if (!self) partition_keys(*dev, a_ra, a_dec, nA, gA, false, !fp32, fp32, scA, 1u, A, slA, dev->side);
    }
  } else {
    fq = frame_begin(*dev, a_ra, a_dec, na_frame, b_ra, b_dec, nb, crowd, s);
    if (fits && !prof) {
      // cleared while the host waits for the frame
      Carve c{(char*)dev->ws};
      lay(c);
      early = cleared();
      clear();
    }
  }
  Frame f;
  bool crowded = false;
  HLC_CHECK(frame_finish(*dev, fq, a_ra, a_dec, na_frame, b_ra, b_dec, nb, s, spec ? dev->side : s, &f, &crowded));
  dev->last_full = is_full(f);
  if (crowd) dev->last_crowded = crowded;
  g = make_geom(r_arcsec, tuned_height(o), na, nb, tuned_bins(o), f, crowded);
  sub_bins(crowded);
  const bool keep = spec && dev->last_full && crowded == assumed;  // the speculative keys stand
  Carve sizing{nullptr};
  lay(sizing);
  HLC_CHECK(ensure_ws(*dev, sizing.off + 256));
  Carve c{(char*)dev->ws};
  lay(c);

  if (!keep) {
    if (spec) {
      // the speculative keys are dropped: their kernel ends before the
      // counters are cleared again
      HLC_TRY(hipEventRecord(dev->prepped, dev->side));
      HLC_TRY(hipStreamWaitEvent(s, dev->prepped, 0));
    }
    if (prof) HLC_TRY(hipEventRecord(dev->ev[14], s));
    if (spec || !(early == cleared())) clear();
  }
  // A's partition on the side stream, B's on the caller's, the two keygens
  // side by side; the ranges run on the side stream once both are sorted,
  // beside B's gather (separate sort scratch, disjoint counter fields)
  // (B's keygen launched first: B's chain is the longer one)
  hipStream_t ms = s;  // the stream that the match runs and ends on
  if (both) {
    if (!keep) partition_keys_both(*dev, a_ra, a_dec, nA, scA, A, b_ra, b_dec, nB, sc, B, g, s);
    partition_sort_both(*dev, g, scA, A, sc, B, s);
  } else {
    if (!keep) {
      if (!self) HLC_TRY(hipEventRecord(dev->fork, s));
      partition_keys(*dev, b_ra, b_dec, nB, g, true, !fp32, fp32, sc, 2u, B, slB, s);
      if (!self) {
        HLC_TRY(hipStreamWaitEvent(dev->side, dev->fork, 0));
        partition_keys(*dev, a_ra, a_dec, nA, gA, false, !fp32, fp32, scA, 1u, A, slA, dev->side);
      }
    }
    if (self) mark(*dev, slA.keygen, s);
    if (!self) HLC_CHECK(partition_sort(*dev, gA, !fp32, fp32, scA, A, slA, dev->side));
    HLC_CHECK(partition_sort(*dev, g, !fp32, fp32, sc, B, slB, s, dev->bsorted));
    if (self) {
      // one partition serves both roles; its halo copies are skipped as A
      for (int k : {slA.sort, slA.layout}) mark(*dev, k, s);
      A = B;
    }
    HLC_TRY(hipStreamWaitEvent(dev->side, dev->bsorted, 0));
    mark(*dev, prof ? 12 : -1, dev->side);
    ms = dev->side;
  }
  match(*dev, A, B, g, r_arcsec, fp32, self, self, rad, w, out_pairs,
        (o->flags & HLC_NO_SEP) ? nullptr : out_sep, (uint64_t)o->capacity, plevel, tuned_items(o), s, ms);
  // (on the side stream: after every kernel of the call on s)
  HLC_CHECK(finish_match(*dev, A, B, r_arcsec, rad, w, prof, ms));

  const Counters& h = *dev->cnt_host;
  if (h.err) {
    *o->n_pairs = 0;
    return HLC_E_INVAL;
  }
  if (h.sort_over) {
    dev->overflows.add(na, nb);
    caps.digit_sort = true;
    *again = true;
    return HLC_OK;
  }
  if (regrow(*dev, h, (uint64_t)o->capacity, caps)) {
    *again = true;
    return HLC_OK;
  }
  fill_stats(h, na, nb, nb + (int64_t)h.n_halo, g);
  if (prof) fill_times(*dev, true);
  else if (plevel == PROF_FILTER) g_stats.t_match_ms = elapsed(dev->ev[13], dev->ev[9]);
  HLC_CHECK(finish_order_ahead(*dev, w, (uint64_t)h.n_pairs, na, ms));
  if (fp32) dev->cand_per_b = (double)h.n_cand / (double)std::max<unsigned long long>(1, nb + h.n_halo);
  *o->n_pairs = (int64_t)h.n_pairs;
  return h.n_pairs > (unsigned long long)o->capacity ? HLC_E_OVERFLOW : HLC_OK;
}

// xmatch_impl with the work-buffer retry.
int xmatch_core(const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
                const double* b_dec, int64_t nb, double r_arcsec, hlc_pair* out_pairs,
                double* out_sep, const hlc_opts* o, const Radii& rad = Radii{nullptr, nullptr, 0.0}) {
  Device* dev = nullptr;
  HLC_CHECK(get_device(&dev));
  Caps caps = initial_caps(*dev, (uint64_t)(na + nb), (uint64_t)o->capacity, true, false);
  caps.digit_sort = dev->overflows.take(na, nb);
  for (int attempt = 0; attempt < 4; ++attempt) {
    bool again = false;
    int st = xmatch_impl(a_ra, a_dec, na, b_ra, b_dec, nb, r_arcsec, out_pairs, out_sep, o, caps, &again, rad);
    if (!again) return st;
  }
  return HLC_E_NOMEM;
}

}  // namespace
}  // namespace hlc

using namespace hlc;

extern "C" {

int hlc_xmatch(const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
               const double* b_dec, int64_t nb, double r_arcsec, hlc_pair* out_pairs,
               double* out_sep_arcsec, const hlc_opts* opts) {
  int st = check_common(r_arcsec, na, nb, opts);
  if (st) return st;
  if ((na > 0 && (!a_ra || !a_dec)) || (nb > 0 && (!b_ra || !b_dec))) return HLC_E_INVAL;
  if (opts->capacity > 0 && (!out_pairs || (!(opts->flags & HLC_NO_SEP) && !out_sep_arcsec)))
    return HLC_E_INVAL;
  if ((opts->flags & HLC_SELF) && (a_ra != b_ra || a_dec != b_dec || na != nb)) return HLC_E_INVAL;
  try {
    if (na == 0 || nb == 0) return validate_only(a_ra, a_dec, na, b_ra, b_dec, nb, r_arcsec, opts);
    return sort_output(xmatch_core(a_ra, a_dec, na, b_ra, b_dec, nb, r_arcsec, out_pairs, out_sep_arcsec, opts),
                       out_pairs, out_sep_arcsec, opts, na, nb);
  } catch (const std::bad_alloc&) {
    return HLC_E_NOMEM;
  } catch (...) {
    return HLC_E_DEVICE;
  }
}

int hlc_xmatch_radii(const double* a_ra, const double* a_dec, const double* a_err, int64_t na,
                     const double* b_ra, const double* b_dec, const double* b_err, int64_t nb,
                     double k_sigma, hlc_pair* out_pairs, double* out_sep_arcsec, const hlc_opts* opts) {
  int st = check_common(1.0, na, nb, opts);
  if (st) return st;
  if (!(k_sigma > 0.0) || !(k_sigma < 1e300)) return HLC_E_INVAL;
  if ((na > 0 && (!a_ra || !a_dec || !a_err)) || (nb > 0 && (!b_ra || !b_dec || !b_err))) return HLC_E_INVAL;
  if (opts->capacity > 0 && (!out_pairs || (!(opts->flags & HLC_NO_SEP) && !out_sep_arcsec)))
    return HLC_E_INVAL;
  if (opts->flags & HLC_SELF) return HLC_E_UNSUPPORTED;
  try {
    if (na == 0 || nb == 0) return validate_only(a_ra, a_dec, na, b_ra, b_dec, nb, 1.0, opts);
    // largest radius: filter radius of the whole call (one read-back)
    Device* dev = nullptr;
    HLC_CHECK(get_device(&dev));
    hipStream_t s = (hipStream_t)opts->stream;
    const uint32_t nc = launch_err_max(a_err, (uint32_t)na, b_err, (uint32_t)nb, dev->msg_dev->err, s);
    HLC_TRY(hipStreamSynchronize(s));
    HLC_TRY(hipGetLastError());
    unsigned long long ca = 0ull, cb = 0ull;
    for (uint32_t i = 0; i < nc; ++i) {
      ca = std::max(ca, dev->msg->err[2 * i]);
      cb = std::max(cb, dev->msg->err[2 * i + 1]);
    }
    if (ca == ERR_BAD || cb == ERR_BAD) return HLC_E_INVAL;
    double ea, eb;
    std::memcpy(&ea, &ca, 8);
    std::memcpy(&eb, &cb, 8);
    double rmax = k_sigma * std::sqrt(ea * ea + eb * eb) * (1.0 + 1e-12);
    if (!(rmax <= 3600.0)) return HLC_E_INVAL;
    // all errors zero: only identical positions match; any positive filter
    // radius finds them
    rmax = std::max(rmax, 1e-6);
    return sort_output(xmatch_core(a_ra, a_dec, na, b_ra, b_dec, nb, rmax, out_pairs, out_sep_arcsec, opts,
                                   Radii{a_err, b_err, k_sigma}),
                       out_pairs, out_sep_arcsec, opts, na, nb);
  } catch (const std::bad_alloc&) {
    return HLC_E_NOMEM;
  } catch (...) {
    return HLC_E_DEVICE;
  }
}

int hlc_xmatch_quad(const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
                    const double* b_dec, int64_t nb, double r_arcsec, int32_t order, hlc_pair* out_pairs,
                    double* out_sep_arcsec, const hlc_opts* opts) {
  int st = check_common(r_arcsec, na, nb, opts);
  if (st) return st;
  if (order < 0 || order > 13) return HLC_E_INVAL;
  if (na >= (int64_t(1) << 28) || nb >= (int64_t(1) << 28)) return HLC_E_INVAL;  // 5 entries each
  if ((na > 0 && (!a_ra || !a_dec)) || (nb > 0 && (!b_ra || !b_dec))) return HLC_E_INVAL;
  if (opts->capacity > 0 && (!out_pairs || (!(opts->flags & HLC_NO_SEP) && !out_sep_arcsec)))
    return HLC_E_INVAL;
  if (opts->flags & HLC_SELF) return HLC_E_UNSUPPORTED;
  try {
    if (na == 0 || nb == 0) return validate_only(a_ra, a_dec, na, b_ra, b_dec, nb, r_arcsec, opts);
    Device* dev = nullptr;
    HLC_CHECK(get_device(&dev));
    hipStream_t s = (hipStream_t)opts->stream;
    const uint32_t capA = 5u * (uint32_t)na, capB = 5u * (uint32_t)nb;
    Caps caps = initial_caps(*dev, (uint64_t)capA + capB, (uint64_t)opts->capacity, true, true);
    for (int attempt = 0; attempt < 3; ++attempt) {
      Side A, B;
      SortScratch sc;
      MatchWs w;
      uint32_t *msplit = nullptr, *lb = nullptr;
      Geom g{};
      set_radius(g, r_arcsec);
      g.rb = 0;  // keys are pixels: a candidate must share the A entry's pixel
      g.nz = 1;
      auto lay = [&](Carve& c) {
        carve_side(c, A, capA, true, false);
        carve_side(c, B, capB, true, false);
        A.radec = c.take<double2>(capA);  // sorted (ra, dec): pixel tests
        B.radec = c.take<double2>(capB);
        carve_sort(c, sc, std::max(capA, capB));
        carve_match_ws(c, w, capA, g, caps, false);
        msplit = c.take<uint32_t>(merge_splits_len(capA, capB));
        lb = c.take<uint32_t>(capA);
      };
      Carve sz{nullptr};
      lay(sz);
      HLC_CHECK(ensure_ws(*dev, sz.off + 256));
      Carve c{(char*)dev->ws};
      lay(c);
      launch_zero_counters(dev->cnt, s);
      const double R = r_arcsec / 3600.0;
      launch_hp_keygen(a_ra, a_dec, (uint32_t)na, order, R, 1u, A.keys, A.vals, &dev->cnt->aux[0], dev->cnt, s);
      launch_hp_keygen(b_ra, b_dec, (uint32_t)nb, order, R, 2u, B.keys, B.vals, &dev->cnt->aux[1], dev->cnt, s);
      A.cnt = DevCount{0, capA, &dev->cnt->aux[0]};
      B.cnt = DevCount{0, capB, &dev->cnt->aux[1]};
      A.ra = a_ra; A.dec = a_dec; B.ra = b_ra; B.dec = b_dec;
      const int kb = 2 * order + 4;  // 12 * 4^order < 2^(2 order + 4)
      radix_sort(A.keys, A.vals, A.cnt, kb, sc, s);
      radix_sort(B.keys, B.vals, B.cnt, kb, sc, s);
      launch_layout64(A.vals, A.cnt, a_ra, a_dec, A.r64, s);
      launch_layout64(B.vals, B.cnt, b_ra, b_dec, B.r64, s);
      launch_radec_gather(A.vals, A.cnt, a_ra, a_dec, A.radec, s);
      launch_radec_gather(B.vals, B.cnt, b_ra, b_dec, B.radec, s);
      launch_merge_lb(A.keys, A.cnt, B.keys, B.cnt, msplit, lb, s);
      launch_equal_ranges(A.keys, A.cnt, lb, B.keys, B.cnt, w.ranges, s);
      const Thresholds th = thresholds(r_arcsec);
      MatchArgs ma{};
      ma.ranges = w.ranges;
      ma.na = A.cnt;
      ma.recA64 = A.r64;
      ma.recB64 = B.r64;
      ma.t_lo64 = th.t_lo64;
      ma.t_hi64 = th.t_hi64;
      ma.radecA = A.radec;
      ma.radecB = B.radec;
      ma.keysA = A.keys;
      ma.keysB = B.keys;
      ma.valsA = A.vals;
      ma.valsB = B.vals;
      ma.geom = g;
      ma.H_lo = th.H_lo;
      ma.H_hi = th.H_hi;
      ma.hp_order = order;
      ma.hp_R = R;
      const OutArgs oa = out_args(out_pairs, (opts->flags & HLC_NO_SEP) ? nullptr : out_sep_arcsec,
                                  (uint64_t)opts->capacity, w.band, w.band_cap, w.reg, dev->cnt);
      launch_regions_reset(oa, s);
      launch_filter(ma, oa, false, 1, s);
      launch_cand(ma, oa, false, s);
      launch_certify({a_ra, a_dec}, {b_ra, b_dec}, r_arcsec, th.H_lo, th.H_hi, Radii{nullptr, nullptr, 0.0}, oa, s);
      launch_compact(oa, s);
      HLC_CHECK(read_counters(*dev, s, false));
      const Counters& h = *dev->cnt_host;
      if (h.err) return HLC_E_INVAL;
      if (regrow(*dev, h, (uint64_t)opts->capacity, caps)) continue;
      std::memset(&g_stats, 0, sizeof(g_stats));
      g_stats.na = na;
      g_stats.nb = nb;
      g_stats.nb_halo = (int64_t)h.aux[1];  // B entries (records with their copies)
      g_stats.n_pairs = (int64_t)h.n_pairs;
      g_stats.n_candidates = (int64_t)h.n_cand;
      g_stats.n_band = (int64_t)h.n_band;
      g_stats.n_ties = (int64_t)h.n_ties;
      *opts->n_pairs = (int64_t)h.n_pairs;
      return sort_output(h.n_pairs > (unsigned long long)opts->capacity ? HLC_E_OVERFLOW : HLC_OK, out_pairs,
                         out_sep_arcsec, opts, na, nb);
    }
    return HLC_E_NOMEM;
  } catch (const std::bad_alloc&) {
    return HLC_E_NOMEM;
  } catch (...) {
    return HLC_E_DEVICE;
  }
}

}  // extern "C"
