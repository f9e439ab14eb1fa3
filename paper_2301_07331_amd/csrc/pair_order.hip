// pair_order.hip -- HLC_SORTED: a call's pairs and separations ordered by
// (a, b) in the caller's buffers.
//
// Up to PAIR_ORDER_LDS pairs are ordered by one block in LDS, one launch. More
// go through one bucket pass: K <= 1024 buckets of equal ranges of a, counted
// per chunk (k_po_count), scanned over the chunks (k_po_scan), scattered as
// 16-B records (k_po_scatter) and ordered by one block per bucket in LDS
// (k_po_bucket), which writes its stretch of the caller's buffers. Each pair
// crosses memory twice; the digit sort of (key, index) that takes over for the
// largest lists crosses it once per digit of b and of a and then gathers the
// pairs at random places. The scatter is bound by its stores: written straight
// from the lanes into 4,000 buckets, 16 B at a time, it took 91 us for 4.07M
// pairs (each partial line costs a whole one on the way to memory), so a tile
// of 8,192 records is first grouped in LDS and leaves in runs of 8 records
// (128 B) or more; that sets K <= 1024 until the buckets outgrow LDS.
// Measured (kernels alone): 4.07M pairs of 10M sources 89 us (count 12, scan 4,
// scatter 33, buckets 39) against 480 us for the digit sort; 17.4M pairs of
// 20M sources 488 against 2,080; 360,000 pairs 25 us, bound by its launches;
// 700 pairs 8 us, bound by one block's chain of barriers, against 160.
#include <hip/hip_runtime.h>

#include "bucket_order.hpp"
#include "hlc_kernels.hpp"

namespace hlc {

namespace {

// mean pairs per bucket up to PO_RUNS buckets (a self-match, i < j, has twice that first)
constexpr uint32_t PO_MEAN = 768;
constexpr uint32_t PO_RUNS = 1024;       // buckets up to which a scatter tile leaves in runs of 8 records
constexpr uint32_t PO_MEAN_L = 10240;    // mean that more buckets keep, up to PO_BUCKETS of them
constexpr uint32_t PO_BUCKETS = 2048;
constexpr uint32_t PO_TILE = 8192;       // records that a scatter block groups in LDS
constexpr uint32_t PO_CHUNKS = 256;      // most chunks (one block each)
constexpr uint32_t PO_CHUNK_MIN = 2048;  // pairs per chunk before there are that many
constexpr uint32_t PO_CHUNK_THREADS = 1024;
constexpr uint32_t PO_BIN_MAX = 48;      // a fuller bin: compare-exchange network instead of ranks
constexpr uint32_t PO_OUTER = 1024;      // bins that split a bucket too large for LDS
// The ordering blocks, by the buckets' mean: 2,048 pairs by 512 threads (four
// blocks per CU hide each other's barriers) up to 1,000; 6,144 by 1,024 (two
// per CU) up to 5,120; 12,288 by 1,024 beyond.
constexpr uint32_t PO_CAP_S = 2048, PO_THREADS_S = 512, PO_MEAN_S = 1000;
constexpr uint32_t PO_CAP_M = 6144, PO_MEAN_M = 5120;
constexpr uint32_t PO_CAP_L = 12288, PO_THREADS_L = 1024;
constexpr uint32_t PO_OVER = 65536;      // a larger bucket (16-bit places in it): digit sort

using u64 = unsigned long long;

__device__ inline u64 pair_key(uint2 p) { return ((u64)p.x << 32) | p.y; }

// Bucket of a first index: equal ranges of a, monotone in a (mul = K 2^32 / na).
__device__ inline uint32_t bucket_of(uint32_t a, u64 mul, uint32_t K) {
  return min((uint32_t)(((u64)a * mul) >> 32), K - 1u);
}

__host__ __device__ inline uint32_t bucket_count(uint32_t n, uint64_t na) {
  uint64_t k = n / PO_MEAN;
  if (k > PO_RUNS) {
    k = n / PO_MEAN_L;
    k = k > PO_BUCKETS ? PO_BUCKETS : k;
    k = k < PO_RUNS ? PO_RUNS : k;
  }
  k = k > na ? na : k;
  return k < 1 ? 1u : (uint32_t)k;
}
__host__ __device__ inline uint32_t chunk_count(uint32_t n) {
  const uint32_t c = (n + PO_CHUNK_MIN - 1) / PO_CHUNK_MIN;
  return c > PO_CHUNKS ? PO_CHUNKS : c < 1 ? 1u : c;
}

// What the kernels of a bucket pass work on. With cnt the pairs are not
// counted on the host yet: the kernels take the count and the plan from it, in
// grids for the most, and leave the pairs alone (K = 0) when they are few
// enough for one block, more than `most` or the buffer, or crowded.
struct PairRun {
  uint2* pairs;
  double* sep;
  u64 na;
  PairOrderWs w;
  u64* over;
  uint32_t cap;  // pairs that an ordering block takes
  uint32_t n, K, chunks, chunk;
  u64 mul;
  const Counters* cnt;
  u64 most;
};
struct PairPlan {
  uint32_t n, K, chunks, chunk;
  u64 mul;
};
__host__ __device__ inline PairPlan pair_plan(uint32_t n, u64 na) {
  PairPlan p;
  p.n = n;
  p.K = bucket_count(n, na);
  p.chunks = chunk_count(n);
  p.chunk = (n + p.chunks - 1) / p.chunks;
  p.mul = ((u64)p.K << 32) / na;
  return p;
}
__device__ inline PairPlan plan_of(const PairRun& r) {
  if (!r.cnt) return PairPlan{r.n, r.K, r.chunks, r.chunk, r.mul};
  const u64 n = r.cnt->n_pairs;
  PairPlan p{0u, 0u, 0u, 0u, 0ull};
  if (n > PAIR_ORDER_LDS && n <= r.most) {
    p = pair_plan((uint32_t)n, r.na);
    if (p.n / p.K > PO_MEAN_S) p = PairPlan{0u, 0u, 0u, 0u, 0ull};
  }
  return p;
}

template <uint32_t CAP, uint32_t T>
struct PairLds {
  static constexpr int LOG_BINS = 12;
  static constexpr uint32_t BINS = 1u << LOG_BINS;
  u64 key[CAP];
  uint32_t cnt[BINS];
  uint16_t src[CAP];  // each key's place in its bucket
  u64 red[2][T / 64];
  uint32_t w[T / 64];
  uint32_t full;
};

// smallest and largest of the block's values (every thread gets both)
template <uint32_t T>
__device__ inline void block_min_max(u64& lo, u64& hi, u64 (*red)[T / 64]) {
  for (int d = 32; d > 0; d >>= 1) {
    lo = min(lo, (u64)__shfl_xor(lo, d));
    hi = max(hi, (u64)__shfl_xor(hi, d));
  }
  if ((threadIdx.x & 63u) == 0) {
    red[0][threadIdx.x >> 6] = lo;
    red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  for (uint32_t k = 0; k < T / 64; ++k) {
    lo = min(lo, red[0][k]);
    hi = max(hi, red[1][k]);
  }
}

// shift that leaves at most `want` leading bits of a difference
__device__ inline int shift_to(u64 diff, int want) {
  const int bits = diff ? 64 - __clzll((long long)diff) : 0;
  return bits > want ? bits - want : 0;
}

// Orders m <= CAP pairs into pairs[0, m) and sep[0, m); thread t's are number
// t + j T: key[j], place src[j] and separation sp[j]. The keys are grouped in
// LDS by their leading bits between the smallest and the largest (about one
// key per bin where the indices are spread evenly); a key's rank is its bin's
// start and the number of smaller keys in the bin. That is O(1) steps a key;
// where a bin is fuller than PO_BIN_MAX (indices in dense clusters) a
// compare-exchange network of log^2 steps takes over, and the separations are
// fetched by place (sep_at). Equal keys (a pair that two overlapping jobs of a
// batch both report) stay in any order. Keys, then separations, pass through
// LDS to leave in whole lines: fetched from the records by place in rank
// order, the separations cost a line each (54 us for 4.07M pairs).
template <uint32_t CAP, uint32_t T, class SepAt>
__device__ inline void order_pairs(PairLds<CAP, T>& L, const u64 (&key)[CAP / T], const uint32_t (&src)[CAP / T],
                                   const double (&sp)[CAP / T], uint32_t m, uint2* __restrict__ pairs, double* sep,
                                   SepAt sep_at) {
  constexpr uint32_t PER = CAP / T, BINS = PairLds<CAP, T>::BINS;
  const uint32_t t = threadIdx.x;
  for (uint32_t i = t; i < BINS; i += T) L.cnt[i] = 0u;
  if (t == 0) L.full = 0u;
  u64 lo = ~0ull, hi = 0ull;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      lo = min(lo, key[j]);
      hi = max(hi, key[j]);
    }
  block_min_max<T>(lo, hi, L.red);
  const int sh = shift_to(hi - lo, PairLds<CAP, T>::LOG_BINS);
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m && atomicAdd(&L.cnt[(uint32_t)((key[j] - lo) >> sh)], 1u) >= PO_BIN_MAX) L.full = 1u;
  __syncthreads();
  if (L.full) {
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
      if (t + j * T < m) {
        L.key[t + j * T] = key[j];
        L.src[t + j * T] = (uint16_t)src[j];
      }
    __syncthreads();
    // every exchange puts the smaller key first, so the places from m on
    // (larger than any key) need not exist
    auto exchange = [&](uint32_t x, uint32_t y) {
      if (y >= m) return;
      const u64 kx = L.key[x], ky = L.key[y];
      const uint16_t ix = L.src[x], iy = L.src[y];
      if (kx > ky || (kx == ky && ix > iy)) {
        L.key[x] = ky;
        L.key[y] = kx;
        L.src[x] = iy;
        L.src[y] = ix;
      }
    };
    uint32_t n2 = 2;
    while (n2 < m) n2 <<= 1;
    for (uint32_t k = 2; k <= n2; k <<= 1) {
      for (uint32_t p = t; p < n2 / 2; p += T) {
        const uint32_t i = p & (k / 2 - 1u), base = (p - i) * 2u;
        exchange(base + i, base + k - 1u - i);
      }
      __syncthreads();
      for (uint32_t j = k >> 2; j > 0; j >>= 1) {
        for (uint32_t p = t; p < n2 / 2; p += T) {
          const uint32_t x = 2u * p - (p & (j - 1u));
          exchange(x, x + j);
        }
        __syncthreads();
      }
    }
    double v[PER];
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      const uint32_t p = t + j * T;
      v[j] = (sep && p < m) ? sep_at((uint32_t)L.src[p]) : 0.0;
    }
    __syncthreads();  // (the places may lie in the output itself)
    for (uint32_t p = t; p < m; p += T) pairs[p] = make_uint2((uint32_t)(L.key[p] >> 32), (uint32_t)L.key[p]);
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
      if (sep && t + j * T < m) sep[t + j * T] = v[j];
    return;
  }
  {
    constexpr uint32_t PB = BINS / T;
    uint32_t c[PB], sum = 0u, tot;
#pragma unroll
    for (uint32_t k = 0; k < PB; ++k) {
      c[k] = L.cnt[t * PB + k];
      sum += c[k];
    }
    uint32_t run = scan_block<T / 64>(sum, &tot, L.w);
#pragma unroll
    for (uint32_t k = 0; k < PB; ++k) {
      L.cnt[t * PB + k] = run;
      run += c[k];
    }
  }
  __syncthreads();
  uint32_t at[PER];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      at[j] = atomicAdd(&L.cnt[(uint32_t)((key[j] - lo) >> sh)], 1u);
      L.key[at[j]] = key[j];
    }
  __syncthreads();
  // cnt[f] is now the end of bin f, the start of bin f + 1
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      const u64 k = key[j];
      const uint32_t f = (uint32_t)((k - lo) >> sh);
      const uint32_t b0 = f ? L.cnt[f - 1u] : 0u, b1 = L.cnt[f];
      uint32_t r = b0;
      for (uint32_t q = b0; q < b1; ++q) {
        const u64 ko = L.key[q];
        r += (ko < k || (ko == k && q < at[j])) ? 1u : 0u;
      }
      at[j] = r;
    }
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) L.key[at[j]] = key[j];
  __syncthreads();
  for (uint32_t p = t; p < m; p += T) pairs[p] = make_uint2((uint32_t)(L.key[p] >> 32), (uint32_t)L.key[p]);
  if (!sep) return;
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) L.key[at[j]] = (u64)__double_as_longlong(sp[j]);
  __syncthreads();
  for (uint32_t p = t; p < m; p += T) sep[p] = __longlong_as_double((long long)L.key[p]);
}

// n <= PAIR_ORDER_LDS pairs in place, one block: everything is read before
// anything is written.
constexpr uint32_t PO_THREADS_1 = 1024;
// (With cnt the count is taken from there: more than `most` are left alone.)
__global__ __launch_bounds__(PO_THREADS_1) void k_po_block(uint2* pairs, double* sep, uint32_t n, const Counters* cnt,
                                                           u64 most) {
  if (cnt) {
    const u64 found = cnt->n_pairs;
    if (found > most || found < 2ull) return;
    n = (uint32_t)found;
  }
  __shared__ PairLds<PAIR_ORDER_LDS, PO_THREADS_1> L;
  constexpr uint32_t PER = PAIR_ORDER_LDS / PO_THREADS_1;
  u64 key[PER];
  uint32_t src[PER];
  double sp[PER];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    const uint32_t i = threadIdx.x + j * PO_THREADS_1;
    key[j] = i < n ? pair_key(pairs[i]) : 0ull;
    sp[j] = (sep && i < n) ? sep[i] : 0.0;
    src[j] = i;
  }
  order_pairs(L, key, src, sp, n, pairs, sep, [&](uint32_t i) { return sep[i]; });
}

// chunk c's pairs per bucket: counts[c * K + d]
__global__ __launch_bounds__(PO_CHUNK_THREADS) void k_po_count(PairRun run) {
  const PairPlan p = plan_of(run);
  if (blockIdx.x >= p.chunks) return;
  const uint2* __restrict__ pairs = run.pairs;
  uint32_t* __restrict__ counts = run.w.counts;
  const uint32_t n = p.n, K = p.K, chunk = p.chunk;
  const u64 mul = p.mul;
  __shared__ uint32_t s_c[PO_BUCKETS];
  for (uint32_t d = threadIdx.x; d < K; d += PO_CHUNK_THREADS) s_c[d] = 0u;
  __syncthreads();
  const uint32_t b0 = blockIdx.x * chunk, b1 = min(n, b0 + chunk);
#pragma unroll 4
  for (uint32_t i = b0 + threadIdx.x; i < b1; i += PO_CHUNK_THREADS) atomicAdd(&s_c[bucket_of(pairs[i].x, mul, K)], 1u);
  __syncthreads();
  for (uint32_t d = threadIdx.x; d < K; d += PO_CHUNK_THREADS) counts[(size_t)blockIdx.x * K + d] = s_c[d];
}

// Per bucket, the exclusive scan over the chunks (in place) and the total.
// A block takes 64 buckets: 16 rows of threads, each summing a sixteenth of
// the chunks, all loads in flight at once.
// (Two tables' blocks follow each other.)
__device__ inline void scan_tables(const BucketScan& first, const BucketScan& second) {
  constexpr uint32_t ROWS = PO_CHUNK_THREADS / 64, PER = PO_CHUNKS / ROWS;
  __shared__ uint32_t s_sum[ROWS][64];
  const uint32_t l = threadIdx.x & 63u, row = threadIdx.x >> 6;
  const uint32_t nfirst = (first.K + 63u) / 64u;
  const bool other = blockIdx.x >= nfirst;
  uint32_t* const counts = other ? second.counts : first.counts;
  uint32_t* const totals = other ? second.totals : first.totals;
  const uint32_t K = other ? second.K : first.K, nchunks = other ? second.chunks : first.chunks;
  const uint32_t d = (blockIdx.x - (other ? nfirst : 0u)) * 64u + l;
  uint32_t c[PER], sum = 0u;
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) {
    const uint32_t b = row * PER + k;
    c[k] = (d < K && b < nchunks) ? counts[(size_t)b * K + d] : 0u;
  }
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) sum += c[k];
  s_sum[row][l] = sum;
  __syncthreads();
  uint32_t run = 0u;
  for (uint32_t k = 0; k < row; ++k) run += s_sum[k][l];
  if (d >= K) return;
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) {
    const uint32_t b = row * PER + k;
    if (b < nchunks) counts[(size_t)b * K + d] = run;
    run += c[k];
  }
  if (row == ROWS - 1u) totals[d] = run;
}
__global__ __launch_bounds__(PO_CHUNK_THREADS) void k_po_scan(BucketScan first, BucketScan second) {
  scan_tables(first, second);
}
__global__ __launch_bounds__(PO_CHUNK_THREADS) void k_po_scan_ahead(PairRun run) {
  const PairPlan p = plan_of(run);
  if (blockIdx.x * 64u >= p.K) return;
  scan_tables(BucketScan{run.w.counts, p.chunks, p.K, run.w.totals}, BucketScan{});
}

// A chunk's pairs as 16-B records into their buckets, a tile at a time: each
// record's rank in its bucket from an LDS counter, the tile grouped by bucket
// in LDS, runs written out, the next tile's loads in flight meanwhile.
// starts[0..K] are the buckets' first places. *over (in host memory) becomes
// PAIR_ORDER_ROUNDS when a bucket holds more than `cap` pairs, and
// PAIR_ORDER_NONE, nothing being moved, when one holds more than PO_OVER.
__global__ __launch_bounds__(PO_CHUNK_THREADS) void k_po_scatter(PairRun run) {
  const PairPlan plan = plan_of(run);
  u64* const over = run.over;
  if (blockIdx.x >= plan.chunks) {
    if (plan.chunks == 0u && blockIdx.x == 0 && threadIdx.x == 0) *over = PAIR_ORDER_NONE;
    return;
  }
  const uint2* __restrict__ pairs = run.pairs;
  const double* __restrict__ sep = run.sep;
  const uint32_t* __restrict__ counts = run.w.counts;
  const uint32_t* __restrict__ totals = run.w.totals;
  uint32_t* __restrict__ starts = run.w.starts;
  PairRec* __restrict__ rec = run.w.rec;
  const uint32_t n = plan.n, K = plan.K, chunk = plan.chunk, cap = run.cap;
  const u64 mul = plan.mul;
  constexpr uint32_t NW = PO_CHUNK_THREADS / 64, PER = PO_TILE / PO_CHUNK_THREADS;
  constexpr uint32_t BPT = PO_BUCKETS / PO_CHUNK_THREADS;  // buckets per thread
  __shared__ PairRec s_rec[PO_TILE];
  __shared__ uint32_t s_cnt[PO_BUCKETS];
  __shared__ uint32_t s_start[PO_BUCKETS];
  __shared__ uint32_t s_goff[PO_BUCKETS];
  __shared__ uint32_t s_w[NW];
  __shared__ uint32_t s_full;
  const uint32_t t = threadIdx.x;
  if (t == 0) s_full = 0u;
  __syncthreads();
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
  {
    uint32_t c[BPT], st[BPT];
    uint32_t most = 0u;
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) {
      const uint32_t d = t * BPT + u;
      c[u] = d < K ? totals[d] : 0u;
      most = max(most, c[u]);
    }
    scan_buckets(c, st);
    if (most > cap) atomicMax(&s_full, most);
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) {
      const uint32_t d = t * BPT + u;
      if (d < K) {
        s_goff[d] = st[u] + counts[(size_t)blockIdx.x * K + d];
        if (blockIdx.x == 0) starts[d] = st[u];
      }
    }
  }
  __syncthreads();
  if (blockIdx.x == 0 && t == 0) {
    starts[K] = s_full > PO_OVER ? 0xffffffffu : n;
    *over = s_full > PO_OVER ? PAIR_ORDER_NONE : s_full ? PAIR_ORDER_ROUNDS : 0ull;
  }
  if (s_full > PO_OVER) return;
  const uint32_t b0 = blockIdx.x * chunk, b1 = min(n, b0 + chunk);
  uint2 p[PER];
  double sp[PER];
  auto load = [&](uint32_t base) {
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      const uint32_t i = base + k * PO_CHUNK_THREADS + t;
      p[k] = i < b1 ? pairs[i] : make_uint2(0u, 0u);
      sp[k] = (sep && i < b1) ? sep[i] : 0.0;
    }
  };
  if (b0 < b1) load(b0);
  for (uint32_t base = b0; base < b1; base += PO_TILE) {
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) s_cnt[t * BPT + u] = 0u;
    __syncthreads();
    uint32_t bk[PER], rank[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      bk[k] = bucket_of(p[k].x, mul, K);
      rank[k] = base + k * PO_CHUNK_THREADS + t < b1 ? atomicAdd(&s_cnt[bk[k]], 1u) : 0u;
    }
    __syncthreads();
    uint32_t c[BPT], st[BPT];
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) c[u] = s_cnt[t * BPT + u];
    const uint32_t tot = scan_buckets(c, st);
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) s_start[t * BPT + u] = st[u];
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k)
      if (base + k * PO_CHUNK_THREADS + t < b1) s_rec[s_start[bk[k]] + rank[k]] = PairRec{p[k].x, p[k].y, sp[k]};
    if (base + PO_TILE < b1) load(base + PO_TILE);
    __syncthreads();
    for (uint32_t i = t; i < tot; i += PO_CHUNK_THREADS) {
      const PairRec r = s_rec[i];
      const uint32_t d = bucket_of(r.a, mul, K);
      rec[s_goff[d] + (i - s_start[d])] = r;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < BPT; ++u) s_goff[t * BPT + u] += c[u];  // (this thread's buckets only)
  }
}

// Bucket blockIdx.x ordered into its stretch of the caller's buffers, if it
// fits LDS (a kernel of its own: with the rounds below in it the registers of
// both spill: 138 us against 39 us for 4.07M pairs).
template <uint32_t CAP, uint32_t T>
__global__ __launch_bounds__(T, CAP <= PO_CAP_M ? 8 : 4) void k_po_bucket(PairRun run) {
  const uint32_t K = plan_of(run).K;
  if (blockIdx.x >= K) return;
  const PairRec* __restrict__ rec = run.w.rec;
  const uint32_t* __restrict__ starts = run.w.starts;
  uint2* __restrict__ pairs = run.pairs;
  double* __restrict__ sep = run.sep;
  __shared__ PairLds<CAP, T> L;
  if (starts[K] == 0xffffffffu) return;  // nothing was moved
  const uint32_t t = threadIdx.x;
  const uint32_t s0 = starts[blockIdx.x], m = starts[blockIdx.x + 1] - s0;
  if (m == 0u || m > CAP) return;
  const PairRec* r = rec + s0;
  constexpr uint32_t PER = CAP / T;
  u64 key[PER];
  uint32_t src[PER];
  double sp[PER];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    const uint32_t i = t + j * T;
    const PairRec v = i < m ? r[i] : PairRec{0u, 0u, 0.0};
    key[j] = pair_key(make_uint2(v.a, v.b));
    sp[j] = v.sep;
    src[j] = i;
  }
  order_pairs(L, key, src, sp, m, pairs + s0, sep ? sep + s0 : nullptr, [&](uint32_t i) { return r[i].sep; });
}

// The buckets of more than `done_cap` pairs, in rounds: a bucket's keys are
// counted in PO_OUTER bins between the smallest and the largest left, the
// leading bins that fit are gathered and ordered, and so on; a bin that alone
// does not fit is split the same way.
template <uint32_t CAP, uint32_t T>
__global__ __launch_bounds__(T) void k_po_rounds(const PairRec* __restrict__ rec,
                                                 const uint32_t* __restrict__ starts, uint32_t K, uint32_t done_cap,
                                                 uint2* __restrict__ pairs, double* __restrict__ sep) {
  __shared__ PairLds<CAP, T> L;
  __shared__ uint32_t s_n;
  if (starts[K] == 0xffffffffu) return;  // nothing was moved
  const uint32_t t = threadIdx.x;
  const uint32_t s0 = starts[blockIdx.x], m = starts[blockIdx.x + 1] - s0;
  if (m <= done_cap) return;
  const PairRec* r = rec + s0;
  auto key_at = [&](uint32_t i) { return pair_key(make_uint2(r[i].a, r[i].b)); };
  constexpr uint32_t PER = CAP / T;
  u64 lo = ~0ull, top = 0ull;
#pragma unroll 4
  for (uint32_t i = t; i < m; i += T) {
    const u64 k = key_at(i);
    lo = min(lo, k);
    top = max(top, k);
  }
  block_min_max<T>(lo, top, L.red);
  uint32_t* s_outer = L.cnt;  // PO_OUTER + 1 words, done with before a round is ordered
  static_assert(PairLds<CAP, T>::BINS > PO_OUTER, "the splitting bins share the ordering bins' words");
  u64 hi = top;  // the keys in [lo, top] are the m - done that are left
  for (uint32_t done = 0; done < m;) {
    const int sh = shift_to(hi - lo, 10);
    static_assert(PO_OUTER == 1u << 10, "bins of 10 leading bits");
    for (uint32_t i = t; i < PO_OUTER; i += T) s_outer[i] = 0u;
    if (t == 0) s_n = 0u;
    __syncthreads();
#pragma unroll 4
    for (uint32_t i = t; i < m; i += T) {
      const u64 k = key_at(i);
      if (k >= lo && k <= hi) atomicAdd(&s_outer[(uint32_t)((k - lo) >> sh)], 1u);
    }
    __syncthreads();
    {
      constexpr uint32_t PB = PO_OUTER / T;
      uint32_t c[PB], sum = 0u, tot;
#pragma unroll
      for (uint32_t k = 0; k < PB; ++k) {
        c[k] = s_outer[t * PB + k];
        sum += c[k];
      }
      uint32_t run = scan_block<T / 64>(sum, &tot, L.w);
#pragma unroll
      for (uint32_t k = 0; k < PB; ++k) {
        s_outer[t * PB + k] = run;
        run += c[k];
      }
      if (t == 0) s_outer[PO_OUTER] = tot;
    }
    __syncthreads();
    // the leading f bins fit: the largest f with s_outer[f] <= CAP
    uint32_t f = 0, e = PO_OUTER;
    while (f < e) {
      const uint32_t mid = (f + e + 1u) >> 1;
      if (s_outer[mid] <= CAP) f = mid; else e = mid - 1u;
    }
    uint32_t take = s_outer[f];
    if (take == 0u && sh > 0) {
      // bin f alone holds more than CAP keys: its range next
      lo += (u64)f << sh;
      hi = min(hi, lo + ((u64)1 << sh) - 1ull);
      __syncthreads();  // s_outer is cleared next
      continue;
    }
    // (sh == 0 and no bin fits: one key, more than CAP times, goes out as it is)
    const bool same = take == 0u;
    const u64 k0 = same ? lo + f : lo;
    const u64 k1 = same ? k0 : (f == PO_OUTER ? hi : min(hi, lo + ((u64)f << sh) - 1ull));
    if (same) take = s_outer[f + 1u] - s_outer[f];
#pragma unroll 4
    for (uint32_t i = t; i < m; i += T) {
      const u64 k = key_at(i);
      if (k < k0 || k > k1) continue;
      const uint32_t at = atomicAdd(&s_n, 1u);
      if (same) {
        pairs[s0 + done + at] = make_uint2((uint32_t)(k >> 32), (uint32_t)k);
        if (sep) sep[s0 + done + at] = r[i].sep;
      } else {
        L.key[at] = k;
        L.src[at] = (uint16_t)i;
      }
    }
    lo = k1 + 1ull;
    hi = top;
    __syncthreads();
    if (same) {
      done += take;
      continue;
    }
    u64 key[PER];
    uint32_t src[PER];
    double sp[PER];
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      const uint32_t i = t + j * T;
      key[j] = i < take ? L.key[i] : 0ull;
      src[j] = i < take ? L.src[i] : 0u;
      sp[j] = (sep && i < take) ? r[src[j]].sep : 0.0;
    }
    __syncthreads();  // the keys are in registers before LDS is used again
    order_pairs(L, key, src, sp, take, pairs + s0 + done, sep ? sep + s0 + done : nullptr,
                [&](uint32_t i) { return r[i].sep; });
    __syncthreads();
    done += take;
  }
}

// pairs that the ordering blocks of a call take
uint32_t block_cap(uint32_t n, const PairOrderSizes& z) {
  const uint32_t mean = n / z.K;
  return mean <= PO_MEAN_S ? PO_CAP_S : mean <= PO_MEAN_M ? PO_CAP_M : PO_CAP_L;
}

}  // namespace

void launch_bucket_scan(const BucketScan& a, const BucketScan& b, hipStream_t s) {
  k_po_scan<<<(a.K + 63) / 64 + (b.K + 63) / 64, PO_CHUNK_THREADS, 0, s>>>(a, b);
}

PairOrderSizes pair_order_sizes(uint32_t n, uint64_t na) {
  const PairPlan p = pair_plan(n, na);
  return PairOrderSizes{p.K, p.chunks};
}

void launch_pair_order_block(uint2* pairs, double* sep, uint32_t n, hipStream_t s) {
  k_po_block<<<1, PO_THREADS_1, 0, s>>>(pairs, sep, n, nullptr, 0ull);
}

bool pair_order_fits(uint32_t n, const PairOrderSizes& z) { return n / z.K <= 2u * PO_CAP_L - PO_CAP_L / 8u; }

void launch_pair_order(uint2* pairs, double* sep, uint32_t n, uint64_t na, const PairOrderSizes& z,
                       const PairOrderWs& w, unsigned long long* over, hipStream_t s) {
  const PairPlan p = pair_plan(n, na);
  const PairRun run{pairs, sep, na, w, over, block_cap(n, z), p.n, p.K, p.chunks, p.chunk, p.mul, nullptr, 0ull};
  k_po_count<<<z.chunks, PO_CHUNK_THREADS, 0, s>>>(run);
  launch_bucket_scan(BucketScan{w.counts, z.chunks, z.K, w.totals}, BucketScan{}, s);
  k_po_scatter<<<z.chunks, PO_CHUNK_THREADS, 0, s>>>(run);
  switch (run.cap) {
    case PO_CAP_S:
      k_po_bucket<PO_CAP_S, PO_THREADS_S><<<z.K, PO_THREADS_S, 0, s>>>(run);
      break;
    case PO_CAP_M:
      k_po_bucket<PO_CAP_M, PO_THREADS_L><<<z.K, PO_THREADS_L, 0, s>>>(run);
      break;
    default:
      k_po_bucket<PO_CAP_L, PO_THREADS_L><<<z.K, PO_THREADS_L, 0, s>>>(run);
  }
}

void launch_pair_order_ahead(uint2* pairs, double* sep, uint64_t capacity, uint64_t na, const PairOrderAhead& o,
                             const Counters* cnt, hipStream_t s) {
  if (o.block) {
    k_po_block<<<1, PO_THREADS_1, 0, s>>>(pairs, sep, 0u, cnt, std::min<u64>(capacity, PAIR_ORDER_LDS));
    return;
  }
  PairRun run{};
  run.pairs = pairs;
  run.sep = sep;
  run.na = na;
  run.w = o.w;
  run.over = o.over;
  run.cap = PO_CAP_S;
  run.cnt = cnt;
  run.most = std::min<u64>(capacity, o.most);
  const uint32_t chunks = chunk_count((uint32_t)o.most), K = pair_order_ahead_buckets(o.most);
  k_po_count<<<chunks, PO_CHUNK_THREADS, 0, s>>>(run);
  k_po_scan_ahead<<<(K + 63) / 64, PO_CHUNK_THREADS, 0, s>>>(run);
  k_po_scatter<<<chunks, PO_CHUNK_THREADS, 0, s>>>(run);
  k_po_bucket<PO_CAP_S, PO_THREADS_S><<<K, PO_THREADS_S, 0, s>>>(run);
}

uint32_t pair_order_ahead_buckets(uint64_t most) { return bucket_count((uint32_t)most, ~0ull); }
uint32_t pair_order_ahead_chunks(uint64_t most) { return chunk_count((uint32_t)most); }

void launch_pair_order_rounds(uint2* pairs, double* sep, uint32_t n, const PairOrderSizes& z, const PairOrderWs& w,
                              hipStream_t s) {
  k_po_rounds<PO_CAP_L, PO_THREADS_L><<<z.K, PO_THREADS_L, 0, s>>>(w.rec, w.starts, z.K, block_cap(n, z), pairs, sep);
}

}  // namespace hlc
