// bucket_sort.hip -- one catalogue's entries ordered by their 32-bit keys and
// laid out for the match, for up to BS_MAX sources.
//
// The entries take one pass through K buckets of consecutive keys, carrying
// their (ra, dec), and each bucket is then ordered in LDS by one block, which
// writes the sorted keys, indices and working records. The digit sort is nine
// to twelve launches and a layout that fetches each record from a random
// line; this is four, or one for a catalogue that one block takes, all 32 bits
// are sorted at no extra cost (the bins' RA fractions included), and the
// filter reads A's positions along memory. It is bound by its launches and by
// each block's chain of barriers up to about a million sources. Beyond, the
// ordering blocks hold a CU's LDS without using its memory paths well: 10M
// sources a side took 1,597 us a call against 1,320 by the digit sort, so the
// line lies where the two meet. Whole calls, digit sort and this: 2,000 a
// side 186 and 157 us, 300k 264 and 233, 700k 283 and 256, 1.4M 338 and 295,
// 2.0M 389 and 395, 2.8M 474 and 505.
//   k_keygen       keys; every 2^k-th source is counted by which of 8,192 equal
//                  parts of the key space it lies in
//   k_bs_count     part -> bucket, about equally filled; entries per bucket and
//                  chunk, exactly, which are then scanned over the chunks
//   k_bs_scatter   tiles grouped by bucket in LDS, runs written out
//   k_bs_bucket    the order in LDS and the output
// A catalogue that fits one block (8,192 sources) goes straight from its keys
// to the last kernel. A bucket that outgrows its block (2,000 entries or more
// in one part) sets Counters::sort_over: the sides then count as empty for
// what follows both sorts, and the call runs again with the digit sort.
#include <hip/hip_runtime.h>

#include "bucket_order.hpp"
#include "hlc_kernels.hpp"

namespace hlc {

namespace {

constexpr uint32_t BS_TILE = 6144;      // entries grouped in LDS per scatter tile
constexpr uint32_t BS_THREADS = 1024;
constexpr uint32_t BS_CHUNKS = 256;     // counted and scattered by a block each
constexpr uint32_t BS_CHUNK_MIN = 2048;
constexpr uint32_t BS_CAP = 4096;       // entries of an ordering block

// Entries per bucket and chunk. Each block first makes the map from parts of
// the key space to buckets, the sample's running share times K (an empty
// sample, no valid source, puts everything into bucket 0); block 0 keeps it for
// the scatter.
// The kernels take one side or two, the second's blocks after the first's.
__global__ __launch_bounds__(BS_THREADS) void k_bs_count(BucketSide first, BucketSide second,
                                                         unsigned long long fmul) {
  const bool other = blockIdx.x >= first.p.chunks;
  const BucketSide& S = other ? second : first;
  const uint32_t blk = other ? blockIdx.x - first.p.chunks : blockIdx.x;
  const uint32_t* __restrict__ keys = S.in.keys;
  const uint32_t* __restrict__ fine = S.w.fine;
  uint16_t* __restrict__ map = S.w.map;
  uint32_t* __restrict__ counts = S.w.counts;
  const uint32_t K = S.p.K;
  constexpr uint32_t PER = BS_FINE / BS_THREADS;
  __shared__ uint32_t s_c[BS_BUCKETS];
  __shared__ uint16_t s_map[BS_FINE];
  __shared__ uint32_t s_w[BS_THREADS / 64];
  const uint32_t t = threadIdx.x, n = S.in.cnt.get(), chunk = (n + S.p.chunks - 1u) / S.p.chunks;
  for (uint32_t d = t; d < K; d += BS_THREADS) s_c[d] = 0u;
  {
    uint32_t c[PER], sum = 0u, all;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      c[k] = fine[t * PER + k];
      sum += c[k];
    }
    uint32_t run = scan_block<BS_THREADS / 64>(sum, &all, s_w);
    const float share = all ? (float)K / (float)all : 0.0f;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      const uint16_t b = (uint16_t)min((uint32_t)((float)run * share), K - 1u);
      s_map[t * PER + k] = b;
      if (blk == 0) map[t * PER + k] = b;
      run += c[k];
    }
  }
  __syncthreads();
  const uint32_t b0 = min(n, blk * chunk), b1 = min(n, b0 + chunk);
#pragma unroll 8
  for (uint32_t i = b0 + t; i < b1; i += BS_THREADS) atomicAdd(&s_c[s_map[bucket_fine(keys[i], fmul)]], 1u);
  __syncthreads();
  for (uint32_t d = t; d < K; d += BS_THREADS) counts[(size_t)blk * K + d] = s_c[d];
}

// A chunk's entries into their buckets, a tile at a time, as (key, index) and
// (ra, dec): each entry's rank in its bucket from an LDS counter, the tile
// grouped by bucket in LDS (first the one, then the other, through the same
// words) and written out in runs. Entries from n_src on are Dec-halo copies:
// their index is in vals, their position read by it. starts[0..K] are the
// buckets' first places.
__global__ __launch_bounds__(BS_THREADS) void k_bs_scatter(BucketSide first, BucketSide second,
                                                           unsigned long long fmul, Counters* cnt) {
  const bool other = blockIdx.x >= first.p.chunks;
  const BucketSide& S = other ? second : first;
  const uint32_t blk = other ? blockIdx.x - first.p.chunks : blockIdx.x;
  const uint32_t* __restrict__ keys = S.in.keys;
  const uint32_t* __restrict__ vals = S.in.vals;
  const double* __restrict__ ra = S.in.ra;
  const double* __restrict__ dec = S.in.dec;
  const uint16_t* __restrict__ map = S.w.map;
  const uint32_t* __restrict__ counts = S.w.counts;
  const uint32_t* __restrict__ totals = S.w.totals;
  uint32_t* __restrict__ starts = S.w.starts;
  uint2* __restrict__ kv = S.w.kv;
  double2* __restrict__ rd = S.w.rd;
  const uint32_t n_src = S.in.n_src, K = S.p.K, cap = S.p.cap;
  constexpr uint32_t NW = BS_THREADS / 64, PER = BS_TILE / BS_THREADS, BPT = BS_BUCKETS / BS_THREADS;
  __shared__ double2 s_rd[BS_TILE];
  __shared__ uint16_t s_map[BS_FINE];
  __shared__ uint16_t s_b[BS_TILE];
  __shared__ uint32_t s_cnt[BS_BUCKETS];
  __shared__ uint32_t s_goff[BS_BUCKETS];
  __shared__ uint16_t s_start[BS_BUCKETS];
  __shared__ uint32_t s_w[NW];
  uint2* s_kv = reinterpret_cast<uint2*>(s_rd);
  const uint32_t t = threadIdx.x, n = S.in.cnt.get(), chunk = (n + S.p.chunks - 1u) / S.p.chunks;
  // thread t's buckets are t BPT .. t BPT + BPT - 1
  auto scan_buckets = [&](const uint32_t (&c)[BPT], uint32_t (&st)[BPT]) {
    uint32_t sum = 0u, all;
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) sum += c[u];
    uint32_t run = scan_block<NW>(sum, &all, s_w);
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) {
      st[u] = run;
      run += c[u];
    }
    return all;
  };
  for (uint32_t f = t; f < BS_FINE; f += BS_THREADS) s_map[f] = map[f];
  {
    uint32_t c[BPT], st[BPT];
    bool over = false;
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) {
      const uint32_t d = t * BPT + u;
      c[u] = d < K ? totals[d] : 0u;
      over = over || c[u] > cap;
    }
    scan_buckets(c, st);
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) {
      const uint32_t d = t * BPT + u;
      if (d < K) {
        s_goff[d] = st[u] + counts[(size_t)blk * K + d];
        if (blk == 0) starts[d] = st[u];
      }
    }
    if (blk == 0) {
      if (over) atomicOr(&cnt->sort_over, 1u);
      if (t == 0) starts[K] = n;
    }
  }
  const uint32_t b0 = min(n, blk * chunk), b1 = min(n, b0 + chunk);
  uint32_t key[PER], val[PER];
  double pa[PER], pd[PER];
  auto load = [&](uint32_t base) {
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      const uint32_t i = base + k * BS_THREADS + t;
      key[k] = i < b1 ? keys[i] : 0u;
      val[k] = i < n_src ? i : (i < b1 ? vals[i] : 0u);
      const uint32_t q = val[k] & IDX_MASK;
      pa[k] = i < b1 ? ra[q] : 0.0;
      pd[k] = i < b1 ? dec[q] : 0.0;
    }
  };
  if (b0 < b1) load(b0);
  for (uint32_t base = b0; base < b1; base += BS_TILE) {
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) s_cnt[t * BPT + u] = 0u;
    __syncthreads();
    uint32_t bk[PER], at[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      bk[k] = s_map[bucket_fine(key[k], fmul)];
      at[k] = base + k * BS_THREADS + t < b1 ? atomicAdd(&s_cnt[bk[k]], 1u) : 0u;
    }
    __syncthreads();
    uint32_t c[BPT], st[BPT];
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) c[u] = s_cnt[t * BPT + u];
    const uint32_t tot = scan_buckets(c, st);
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) s_start[t * BPT + u] = (uint16_t)st[u];
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      if (base + k * BS_THREADS + t >= b1) continue;
      at[k] += s_start[bk[k]];
      s_b[at[k]] = (uint16_t)bk[k];
      s_kv[at[k]] = make_uint2(key[k], val[k]);
    }
    __syncthreads();
    uint32_t g[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      const uint32_t i = k * BS_THREADS + t;
      if (i >= tot) continue;
      const uint32_t d = s_b[i];
      g[k] = s_goff[d] + (i - s_start[d]);
      kv[g[k]] = s_kv[i];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k)
      if (base + k * BS_THREADS + t < b1) s_rd[at[k]] = make_double2(pa[k], pd[k]);
    if (base + BS_TILE < b1) load(base + BS_TILE);
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      const uint32_t i = k * BS_THREADS + t;
      if (i < tot) rd[g[k]] = s_rd[i];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) s_goff[t * BPT + u] += c[u];  // (this thread's buckets only)
  }
}

// A bucket in order (one too full for the block is left: the call runs again).
// Keys, indices and places pass through LDS to leave in
// whole lines; the (ra, dec) are read from the bucket's stretch.
template <uint32_t CAP, uint32_t T, bool DIRECT>
__global__ __launch_bounds__(T, CAP <= 4096 ? 8 : 4) void k_bs_bucket(BucketSide first, BucketSide second) {
  const bool other = blockIdx.x >= first.p.K;
  const BucketIn& in = other ? second.in : first.in;
  const BucketOut& out = other ? second.out : first.out;
  const uint32_t blk = other ? blockIdx.x - first.p.K : blockIdx.x;
  constexpr uint32_t PER = CAP / T;
  __shared__ OrderLds<CAP, T> L;
  const uint32_t t = threadIdx.x;
  uint32_t s0 = 0u, m;
  if constexpr (DIRECT) {
    m = in.cnt.get();
  } else {
    s0 = in.starts[blk];
    m = in.starts[blk + 1] - s0;
  }
  if (m == 0u || m > CAP) return;
  uint32_t key[PER], val[PER];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    const uint32_t i = t + j * T;
    if constexpr (DIRECT) {
      key[j] = i < m ? in.keys[i] : 0u;
      val[j] = i < in.n_src ? i : (i < m ? in.vals[i] : 0u);
    } else {
      const uint2 e = i < m ? in.kv[s0 + i] : make_uint2(0u, 0u);
      key[j] = e.x;
      val[j] = e.y;
    }
  }
  uint32_t at[PER];
  order_block<CAP, T>(L, key, at, m);
  auto through_lds = [&](auto value, auto put) {
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
      if (t + j * T < m) L.key[at[j]] = value(j);
    __syncthreads();
#pragma unroll 4
    for (uint32_t p = t; p < m; p += T) put(p, L.key[p]);
  };
  through_lds([&](uint32_t j) { return key[j]; }, [&](uint32_t p, uint32_t v) { out.keys[s0 + p] = v; });
  auto record = [&](uint32_t p, uint32_t v, double2 q) {
    if (out.radec) out.radec[s0 + p] = q;
    if (out.r64 || out.r32) {
      double x, y, z;
      unit_vector(q.x, q.y, x, y, z);
      if (out.r64) out.r64[s0 + p] = Rec64{x, y, z, v, 0u};
      if (out.r32) out.r32[s0 + p] = encode_cell(x, y, z);
    }
  };
  if constexpr (DIRECT) {
    through_lds([&](uint32_t j) { return val[j]; }, [&](uint32_t p, uint32_t v) {
      out.vals[s0 + p] = v;
      const uint32_t i = v & IDX_MASK;
      record(p, v, make_double2(in.ra[i], in.dec[i]));
    });
  } else {
    through_lds([&](uint32_t j) { return val[j]; }, [&](uint32_t p, uint32_t v) { out.vals[s0 + p] = v; });
    // (r64 carries the index as well: it is read back from the line just written)
    through_lds([&](uint32_t j) { return t + j * T; }, [&](uint32_t p, uint32_t i) {
      record(p, out.r64 ? in.kv[s0 + i].y : 0u, in.rd[s0 + i]);
    });
  }
}

}  // namespace

// One block up to 8,192 sources (with as many Dec-halo copies at the most);
// beyond, as many buckets of 1,024 to 1,792 sources as keep a scatter tile's
// runs at six entries or more (1,024 buckets). The ordering blocks take 4,096:
// four of them share a CU, and twice the mean is left for the sample's error,
// the parts' grain and the copies.
BucketPlan bucket_plan(uint32_t n) {
  if (n <= 2048u) return BucketPlan{1u, 1u, 4096u, true};
  if (n <= 8192u) return BucketPlan{1u, 1u, 16384u, true};
  BucketPlan p{};
  p.K = std::min(BS_BUCKETS, (n + 1023u) / 1024u);
  p.chunks = std::min(BS_CHUNKS, std::max(1u, (n + BS_CHUNK_MIN - 1u) / BS_CHUNK_MIN));
  p.cap = BS_CAP;
  return p;
}

// 64 to 128 sampled sources a bucket: a bucket's share is then within 62 % of
// the mean at five standard deviations.
uint32_t bucket_sample_mask(uint32_t n, const BucketPlan& p) {
  uint32_t stride = 1u;
  while (n / (2u * stride) >= 64u * p.K) stride *= 2u;
  return stride - 1u;
}

void launch_bucket_sort(const BucketSide& a, const BucketSide* b, unsigned long long fine_mul, Counters* cnt,
                        hipStream_t s) {
  BucketSide first = a, second = b ? *b : BucketSide{};
  for (BucketSide* x : {&first, &second}) {
    x->in.starts = x->w.starts;
    x->in.kv = x->w.kv;
    x->in.rd = x->w.rd;
  }
  const uint32_t K = first.p.K + second.p.K, chunks = first.p.chunks + second.p.chunks;
  if (first.p.direct) {
    if (first.p.cap == 4096u) k_bs_bucket<4096, 1024, true><<<K, 1024, 0, s>>>(first, second);
    else k_bs_bucket<16384, 1024, true><<<K, 1024, 0, s>>>(first, second);
    return;
  }
  k_bs_count<<<chunks, BS_THREADS, 0, s>>>(first, second, fine_mul);
  launch_bucket_scan(BucketScan{first.w.counts, first.p.chunks, first.p.K, first.w.totals},
                     BucketScan{second.w.counts, second.p.chunks, second.p.K, second.w.totals}, s);
  k_bs_scatter<<<chunks, BS_THREADS, 0, s>>>(first, second, fine_mul, cnt);
  k_bs_bucket<BS_CAP, 512, false><<<K, 512, 0, s>>>(first, second);
}

}  // namespace hlc
