// host.hpp -- host-side pieces that the entry points of libhlc share: the
// per-device context and workspace, the partition geometry and frame, the
// thresholds of the decision, and the two phases of a call:
//   partition(): keygen -> radix sort -> working layout of ONE catalogue
//                (section 4.2's first-level partition, on the GPU);
//   match():     B zone tables -> key index -> group ranges -> filter ->
//                candidate certification -> band list -> packing (section 4.3).
// Each form's own host logic lives in its file: xmatch_api.hip (single
// calls), part_api.hip (reusable partitions), batch_api.hip + tune_cache.hip
// (batched form), stream_api.hip (pinned host catalogues).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/hlc.h"
#include "hlc_kernels.hpp"

namespace hlc {

constexpr int MAX_DEVICES = 64;
constexpr double U64 = 1.1102230246251565e-16;
constexpr double ETA64 = 4e-15;  // bound on |chord_fp64 - chord| (unit sphere)

// ---------------------------------------------------------------------------
// per-device context (context.hip)
// ---------------------------------------------------------------------------
// Written by kernels, read by the host.
struct HostMsg {
  ExtentSlot ext[EXTENT_SLOTS];              // the footprint passes' slots (polled)
  ExtentSlot sample;                         // the sample's (polled); pad_[0]: its shared cells
  unsigned long long err[2 * EXTENT_SLOTS];  // the largest error radii
  unsigned long long order;                  // what the pair ordering left to do
  Counters cnt;                              // a call's counters,
  unsigned long long cnt_seq;                // once this is its number (polled)
};

// Memory of freed partitions, kept for the next one: hipFree wipes what it
// returns, so a program that partitions, matches and frees in a loop was held
// to about 35 GB/s of freed memory (2M sources: 9.0 ms a pass, 0.5 with the
// block reused). At most POOL_BLOCKS blocks and POOL_BYTES bytes a device; a
// block serves requests of half its size or more; given back by hlc_shutdown
// and whenever an allocation fails. A block is put here only once no kernel
// uses it any more.
struct PoolBlock {
  void* p = nullptr;
  size_t bytes = 0;
};
constexpr int POOL_BLOCKS = 2;
constexpr size_t POOL_BYTES = size_t(2) << 30;

// Sizes of calls in which a bucket outgrew its block: calls of these sizes take
// the digit sort at once for a number of times, twice as many whenever they
// overflow again, so that a crowded catalogue matched over and over rarely pays
// for the attempt and calls of other sizes never for it. (A partition's second
// size is -1.)
struct OverflowNotes {
  static constexpr int KEPT = 4, FIRST = 15, MOST = 1000;
  struct Note {
    int64_t na = -1, nb = -1;
    int left = 0, next = FIRST;
  } at[KEPT];
  int newest = 0;
  Note* find(int64_t na, int64_t nb) {
    for (Note& n : at)
      if (n.na == na && n.nb == nb) return &n;
    return nullptr;
  }
  // the call takes the digit sort
  bool take(int64_t na, int64_t nb) {
    Note* n = find(na, nb);
    if (!n || n->left == 0) return false;
    --n->left;
    return true;
  }
  void add(int64_t na, int64_t nb) {
    Note* n = find(na, nb);
    if (!n) {
      newest = (newest + 1) % KEPT;
      n = &at[newest];
      *n = Note();
      n->na = na;
      n->nb = nb;
    }
    n->left = n->next;
    n->next = std::min(2 * n->next, MOST);
  }
};

struct Device {
  bool init = false;
  PoolBlock pool[POOL_BLOCKS];  // under the pool's lock
  void* ws = nullptr;
  size_t ws_bytes = 0;
  Counters* cnt = nullptr;        // device
  Counters* cnt_host = nullptr;   // pinned host mirror
  hipEvent_t ev[15] = {};
  // streaming form: device and pinned host arenas kept between calls
  // (grow-only; released by hlc_shutdown)
  void* sarena[2] = {nullptr, nullptr};
  size_t sarena_bytes[2] = {0, 0};
  void* harena = nullptr;
  size_t harena_bytes = 0;
  // streaming form: A sources cross-matched per second by the last
  // streaming call's slabs (0: not measured yet)
  double stream_rate = 0.0;
  // A's partition runs on `side` beside B's on the caller's stream
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr;
  // B sorted (the ranges start) and ranges done (the filter may start)
  hipEvent_t bsorted = nullptr, prepped = nullptr;
  // staging sizes that earlier calls needed (grow-only), so a repeated
  // workload does not pay the overflow re-run again
  uint64_t hint_stage = 0, hint_cand = 0;
  // FP32 candidates per B entry of the last FP32 single call: at
  // SORTED_RADEC_MIN or more the next one uses the sorted certification
  // layout for B (see carve_side)
  double cand_per_b = 0.0;
  int ncu = 0;  // compute units (persistent grids)
  bool last_full = true;  // the last call's frame was the whole sphere
  int large_partial = 0;  // calls of more than EXACT_FIRST_MAX sources since one whose frame was
  OverflowNotes overflows;
  bool last_crowded = false;  // the sources of the last call that asked were crowded
  // mapped host memory: what kernels tell the host without a copy
  HostMsg* msg = nullptr;
  HostMsg* msg_dev = nullptr;  // its device address
  bool ordered = false;  // the call's output is in order already (sort_output has nothing left to do)
  unsigned long long fseq = 0;
};

extern Device g_dev[MAX_DEVICES];
// statistics of the last call made on the calling thread
extern thread_local hlc_stats g_stats;

inline int map_err(hipError_t e) {
  if (e == hipSuccess) return HLC_OK;
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) return HLC_E_NOMEM;
  return HLC_E_DEVICE;
}

#define HLC_TRY(x)                            \
  do {                                        \
    hipError_t e_ = (x);                      \
    if (e_ != hipSuccess) return map_err(e_); \
  } while (0)

#define HLC_CHECK(x)             \
  do {                           \
    int s_ = (x);                \
    if (s_ != HLC_OK) return s_; \
  } while (0)

int get_device(Device** out, int* dev_id = nullptr);
// HLC_TEST_FAIL_ALLOC=<bytes>: allocations of at least that size fail
// (failure-injection tests)
bool alloc_fails(size_t bytes);
int dev_alloc(void** p, size_t bytes);
int ensure_ws(Device& d, size_t bytes);
// at least `bytes` of device memory, from the pool or newly allocated (*got:
// its size), and its return
int pool_take(Device& d, size_t bytes, void** p, size_t* got);
void pool_put(Device& d, void* p, size_t bytes);
void pool_release(Device& d);
int read_counters(Device& dev, hipStream_t s, bool prof);
float elapsed(hipEvent_t a, hipEvent_t b);
void fill_stats(const Counters& h, int64_t na, int64_t nb, int64_t nbh, const Geom& g);
void fill_times(Device& dev, bool with_partition);
// releases the batched form's per-device state (batch_api.hip)
void batch_release_all();

// Bump allocator over a device buffer (base == nullptr: sizing pass).
struct Carve {
  char* base;
  size_t off = 0;
  template <class T>
  T* take(size_t n) {
    off = (off + 255) & ~size_t(255);
    T* p = reinterpret_cast<T*>(base ? base + off : nullptr);
    off += n * sizeof(T);
    return p;
  }
};

// ---------------------------------------------------------------------------
// geometry, frame and thresholds (geometry.hip)
// ---------------------------------------------------------------------------
inline int ceil_log2(uint64_t v) {
  int b = 0;
  while ((uint64_t(1) << b) < v) ++b;
  return b;
}

inline int zone_bits(int64_t nz) { return std::max(1, ceil_log2((uint64_t)nz)); }

inline void set_radius(Geom& g, double r_arcsec) {
  g.r_deg = r_arcsec / 3600.0;
  g.rpad_deg = g.r_deg * (1.0 + 1e-9) + 1e-12;
}

// The region the zones and RA bins cover: the whole sphere, or a box around
// the data (every valid source inside it; an RA span under 180 deg, so no
// pair crosses the box's RA edges).
struct Frame {
  bool full_ra = true;
  double dec_lo = -90.0, dec_hi = 90.0;
  double ra_lo = 0.0, ra_span = 360.0;
};

// Partition geometry: zone height h_as (arcsec; <= 0 = automatic from the
// data density), radius r (halo and windows), frame f.
Geom make_geom(double r_arcsec, double h_as, int64_t na, int64_t nb, int ra_bits, const Frame& f = Frame{},
               bool crowded = false);

inline double ext_value(unsigned long long code) {
  double v;
  std::memcpy(&v, &code, 8);
  return v;
}

// Bounding box of the valid sources from the footprint codes (any: at least
// one valid source).
struct Box {
  bool any;
  double dlo, dhi, rlo, rhi;
};
inline Box read_box(const ExtentSlot* slots, uint32_t n) {
  unsigned long long v[4] = {0ull, 0ull, 0ull, 0ull};
  for (uint32_t i = 0; i < n; ++i)
    for (int k = 0; k < 4; ++k) v[k] = std::max(v[k], slots[i].v[k]);
  Box b;
  b.any = v[1] != 0ull;
  b.dlo = ext_value(~v[0]) - 90.0;
  b.dhi = ext_value(v[1]) - 90.0;
  b.rlo = ext_value(~v[2]);
  b.rhi = ext_value(v[3]);
  return b;
}

// The frame of a call's data. When the last call's frame was the whole sphere,
// a sample of both catalogues first: where its box covers over a quarter of
// the sphere the whole sphere is the frame, otherwise one pass over every
// source gives the exact box. After a call with a smaller frame that pass runs
// at once (a sample would only add a round trip). Above EXACT_FIRST_MAX sources,
// where it takes longer than the sample, only once two such calls in a row had
// smaller frames: 10M x 10M over the whole sphere after a patch 1,037 us a call
// with the sample first, 1,091 with the pass; patches of 4M x 4M one after the
// other 517 and 497; 1M x 1M after a patch 200 either way.
constexpr int64_t EXACT_FIRST_MAX = 1 << 22;
struct FrameQuery {
  unsigned long long seq;
  uint32_t slots;
  bool exact;
  bool crowd;  // the sample also says how crowded the sources are
};
// Sources of the larger side from which it does: below, the crowded tests that
// a fourth radix pass saves (500 an A source: 50 us at 2^19) cost no more than
// the pass and the 10 us that the count adds to the sample.
constexpr int64_t CROWD_MIN = 1 << 19;
FrameQuery frame_begin(Device& dev, const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
                       const double* b_dec, int64_t nb, bool crowd, hipStream_t s);
// (qs: the stream that frame_begin was given)
int frame_finish(Device& dev, FrameQuery q, const double* a_ra, const double* a_dec, int64_t na,
                 const double* b_ra, const double* b_dec, int64_t nb, hipStream_t s, hipStream_t qs, Frame* out,
                 bool* crowded);
// the exact box of every valid source of both catalogues
int exact_box(Device& dev, const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
              const double* b_dec, int64_t nb, hipStream_t s, Box* out);
// the box covers over a quarter of the sphere (the whole sphere is the frame)
bool quarter_sky(const Box& b);
// the frame of an exact box of every valid source (a small margin added)
Frame frame_of_box(const Box& b);
inline bool is_full(const Frame& f) { return f.full_ra && f.dec_lo == -90.0 && f.dec_hi == 90.0; }

inline int key_bits(const Geom& g) { return zone_bits(g.nz) + g.rb + g.fb; }

struct Thresholds {
  double c_r, t_lo64, t_hi64, H_lo, H_hi;
  float c_r32;  // c_r rounded up to FP32
};
Thresholds thresholds(double r_arcsec);

inline int check_opts(const hlc_opts* o) {
  if (!o || !o->n_pairs) return HLC_E_INVAL;
  if (o->capacity < 0) return HLC_E_INVAL;
  if (o->precision != HLC_FP32_RECHECK && o->precision != HLC_FP64) return HLC_E_INVAL;
  if (o->tuning && (o->tuning->ra_bins_log2 < 0 || o->tuning->ra_bins_log2 > 30)) return HLC_E_INVAL;
  return HLC_OK;
}

// Largest catalogue: B's entries (sources plus halo copies, up to twice the
// sources) and every grid rounded up to whole tiles stay below 2^32.
constexpr int64_t MAX_SOURCES = (int64_t(1) << 31) - (int64_t(1) << 16);

inline int check_common(double r_arcsec, int64_t na, int64_t nb, const hlc_opts* o) {
  HLC_CHECK(check_opts(o));
  if (!(r_arcsec > 0.0) || !(r_arcsec <= 3600.0)) return HLC_E_INVAL;
  if (na < 0 || nb < 0 || na > MAX_SOURCES || nb > MAX_SOURCES) return HLC_E_INVAL;
  return HLC_OK;
}

inline double tuned_height(const hlc_opts* o) {
  return (o->tuning && o->tuning->zone_height_arcsec > 0) ? o->tuning->zone_height_arcsec : 0.0;
}
inline int tuned_bins(const hlc_opts* o) { return o->tuning ? o->tuning->ra_bins_log2 : 0; }
inline bool tuned_fraction_sort(const hlc_opts* o) { return o->tuning && o->tuning->fraction_sort == 1; }
// lowest key bit the radix sort orders: 0 when the sub-bin bits are sorted too
inline int sort_lo(const Geom& g) { return g.frac_sorted ? 0 : g.fb; }
inline int tuned_items(const hlc_opts* o) {
  return (o->tuning && o->tuning->filter_items > 0) ? o->tuning->filter_items : 1;
}

// ---------------------------------------------------------------------------
// the two phases of a call (pipeline.hip)
// ---------------------------------------------------------------------------
// One partitioned catalogue.
struct Side {
  BucketPlan plan{};  // K > 0: the bucket sort (else the digit sort)
  BucketWs bws{};
  uint32_t n_src = 0, n_cap = 0;  // sources; entry capacity (2 n_src with a halo)
  DevCount cnt{0, 0, nullptr};    // entries, halo copies included (device-side)
  uint32_t *keys = nullptr, *vals = nullptr;
  Rec64* r64 = nullptr;
  CellRec32* r32 = nullptr;
  // sorted (ra, dec): with the bucket sort, of a side read in place and of an
  // FP32 side; with the digit sort, in the sorted certification layout (see
  // carve_side); and for the paper-scheme emulation's pixel tests
  double2* radec = nullptr;
  // (ra, dec) of each source, 16 B, written by the keygen in input order
  // (nullptr: the layout reads the caller's coordinates): the sorted records
  // of a gathered side are computed from it, the filter reads a side in
  // place from it, and the certification reads B's positions from it
  double2* srcrad = nullptr;
  const double *ra = nullptr, *dec = nullptr;  // original coordinates (for the band list),
  uint32_t stride = 1;                         // stride elements apart
};

// Profiling event slots (HLC_PROFILE): per partition, {after keygen,
// before sort, after sort, after layout}; -1 = not recorded.
struct Slots {
  int keygen, sort_begin, sort, layout;
};
constexpr Slots NO_SLOTS{-1, -1, -1, -1};

inline void mark(Device& dev, int slot, hipStream_t s) {
  if (slot >= 0) (void)hipEventRecord(dev.ev[slot], s);
}

// Partition of one side in two steps (the keygen can run on another stream
// than the sort): keys (and the per-source records) first, then the sort and
// the sorted layout. l64 / l32: the side's records are FP64 / FP32; without
// a sorted layout (sd.r64 / sd.r32 null) the per-source records stay in
// input order and the kernels read them through vals. sorted_ev (optional)
// is recorded once the keys are sorted, before the records are gathered.
void partition_keys(Device& dev, const double* ra, const double* dec, uint32_t n, const Geom& g, bool halo,
                    bool l64, bool l32, const SortScratch& sc, uint32_t err_bit, Side& sd, const Slots& sl,
                    hipStream_t s);
// Both sides of a call whose bucket sorts have the same form, in the same
// launches: their keys, then their order.
void partition_keys_both(Device& dev, const double* a_ra, const double* a_dec, uint32_t na, const SortScratch& scA,
                         Side& A, const double* b_ra, const double* b_dec, uint32_t nb, const SortScratch& scB,
                         Side& B, const Geom& g, hipStream_t s);
void partition_sort_both(Device& dev, const Geom& g, const SortScratch& scA, Side& A, const SortScratch& scB, Side& B,
                         hipStream_t s);
int partition_sort(Device& dev, const Geom& g, bool l64, bool l32, const SortScratch& sc, Side& sd,
                   const Slots& sl, hipStream_t s, hipEvent_t sorted_ev = nullptr);
int partition(Device& dev, const double* ra, const double* dec, uint32_t n, const Geom& g, bool halo,
              bool l64, bool l32, const SortScratch& sc, uint32_t err_bit, Side& sd, const Slots& sl,
              hipStream_t s, hipEvent_t sorted_ev = nullptr);

// Coarse index of B's sorted keys: one entry per 2^shift keys, at most 2^18
// (never finer than the sorted key bits: the low fb bits of a sorted key
// array are in input order within a bin, so the index is exact only on
// multiples of 2^fb)
// Below about two FP32 candidates per B entry, reading each candidate's B
// (ra, dec) at random from a 16-B array in input order costs less than
// gathering every entry's into sorted order (measured at 10M x 10M,
// 0.4 per entry: 10 us slower with the gather; at 20M x 20M, 8.7 per entry:
// 0.35-0.5 ms faster).
constexpr double SORTED_RADEC_MIN = 2.0;

struct KeyIndex {
  int shift;
  uint32_t T;
};
inline KeyIndex key_index_dims(const Geom& g) {
  const int kb = key_bits(g);
  const int shift = std::max(std::max(6, kb - 18), sort_lo(g));
  return KeyIndex{shift, (uint32_t)((1ull << std::max(kb - shift, 0)) + 1)};
}

struct MatchWs {
  uint32_t* kidx;
  GroupRanges* ranges;
  int32_t* zmarg;
  double* zdelta;
  uint32_t* zstartB;  // nullptr: computed here into zstart_buf
  uint32_t* zstart_buf;
  uint2* band;
  uint64_t band_cap;
  Regions reg;
  uint64_t ahead_na = 0;
  PairOrderAhead ahead{};  // HLC_SORTED: the ordering enqueued behind the match
  OutArgs out{};  // what the match wrote to (for a band list's decision)
};

// Sizes of the spill-prone work buffers of a call: the band list, the pair
// slots per output region and the candidate slots per candidate region (0:
// candidates are not staged). All start from estimates; a call whose counts
// exceed them runs again with the counted sizes (the counts are
// deterministic, so the second run fits).
struct Caps {
  uint64_t band;
  uint64_t stage;
  uint64_t cand;
  bool digit_sort = false;
};

// pair_regions: pairs staged in regions and compacted (else written straight
// into the caller's buffer by the certification: no pair slots)
Caps initial_caps(const Device& d, uint64_t entries, uint64_t cap, bool stage_cand, bool pair_regions);
void carve_regions(Carve& c, Regions& r, const Caps& k, bool sep);
// True when the call must run again: its band list overflowed, a candidate
// region overflowed, or a pair region overflowed although the caller's
// buffer holds every pair.
bool regrow(Device& d, const Counters& h, uint64_t cap, Caps& k);
OutArgs out_args(hlc_pair* pairs, double* sep, uint64_t cap, uint2* band, uint64_t band_cap,
                 const Regions& reg, Counters* cnt);
// Everything after the partition: ranges, match, certification. With ps the
// ranges run there (ordered by the caller after both sorts), beside B's
// gather on s, and the filter and what follows end on ps. prof: 0 no
// events, PROF_FILTER the filter's two events, PROF_ALL every stage's.
constexpr int PROF_FILTER = 1, PROF_ALL = 2;
void match(Device& dev, const Side& A, const Side& B, const Geom& g, double r_arcsec, bool fp32,
           bool skip_halo_a, bool self_only, const Radii& rad, MatchWs& w, hlc_pair* out_pairs,
           double* out_sep, uint64_t cap, int prof, int filter_items, hipStream_t s, hipStream_t ps = nullptr);
// The ordering of a call's output enqueued behind its match, where the number
// of pairs can be expected to suit (carved with the match's workspace); whether
// it was done, and if not quite, its last step.
void carve_order_ahead(Carve& c, MatchWs& w, Device& dev, const hlc_opts* o, int64_t na, int64_t nb);
int finish_order_ahead(Device& dev, const MatchWs& w, uint64_t n, int64_t na, hipStream_t s);
int finish_match(Device& dev, const Side& A, const Side& B, double r_arcsec, const Radii& rad, const MatchWs& w,
                 bool prof, hipStream_t s);
// the profiling level of a call's flags
inline int prof_level(uint32_t flags) {
  return (flags & HLC_PROFILE) ? PROF_ALL : ((flags & HLC_TIME_FILTER) ? PROF_FILTER : 0);
}
size_t carve_match_ws(Carve& c, MatchWs& w, uint32_t na_entries, const Geom& g, const Caps& caps,
                      bool need_zstart);
// cap entries; n_src > 0 also carves the per-source records of the keygen;
// without `layout` no sorted records are carved (the side is read in place).
// FP32, gathered: with sorted_radec the sorted certification layout (32-B
// per-source records, gathered into sorted cell records and sorted (ra, dec):
// the certification reads a candidate's B (ra, dec) at its sorted position),
// else 16-B cell records and (ra, dec) in separate input-order arrays (the
// gather and the certification then read at random from arrays half the
// size).
void carve_side(Carve& c, Side& sd, uint32_t cap, bool l64, bool l32, uint32_t n_src = 0, bool layout = true,
                bool sorted_radec = false);
void carve_sort(Carve& c, SortScratch& sc, uint32_t nmax);
// the scratch of the sort that sd.plan names
void carve_sort(Carve& c, SortScratch& sc, uint32_t nmax, Side& sd);
// the sort of a side of n sources: through buckets, or digit by digit beyond
// BS_MAX sources or when the call asks for it
inline BucketPlan plan_sort(int64_t n, bool digit_sort) {
  return digit_sort || n < 1 || n > (int64_t)BS_MAX ? BucketPlan{} : bucket_plan((uint32_t)n);
}
// the coordinates checked (no pairs: one side is empty)
int validate_only(const double* a_ra, const double* a_dec, int64_t na, const double* b_ra,
                  const double* b_dec, int64_t nb, double r_arcsec, const hlc_opts* o);
inline int bits_for(int64_t n) { return std::max(1, ceil_log2((uint64_t)std::max<int64_t>(n, 2))); }
// HLC_SORTED: the call's pairs, already in the caller's buffers, ordered by
// (a, b) (indices below na and nb).
int sort_output(int st, hlc_pair* pairs, double* sep, const hlc_opts* o, int64_t na, int64_t nb);

}  // namespace hlc
