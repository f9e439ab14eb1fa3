// bucket_order.hpp -- the order of up to a block's worth of 32-bit keys in LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace hlc {

constexpr uint32_t BIN_FULL = 12;  // keys in a bin of an ordering block
// Keys in a bin of the second binning beyond which a network of exchanges takes
// over. A bin of n keys costs each of them n steps: 8,192 sources (of 2,000 to
// match) of one key took 4,066 us a call by ranks and take 301 by the network,
// of 8 keys 620 and 213, of 16 keys 375 and 203; of 32 keys, 254 sources each,
// 248 by ranks.
constexpr uint32_t BIN_RANKED = 256;

// Exclusive scan of one value per thread over a block of NW waves.
template <int NW>
__device__ inline uint32_t scan_block(uint32_t v, uint32_t* total, uint32_t* s_w) {
  const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if (lane >= (uint32_t)off) x += y;
  }
  if (lane == 63u) s_w[w] = x;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const uint32_t s = s_w[k];
    if ((uint32_t)k < w) base += s;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return base + x - v;
}

// The order's working memory: 32 KB for 4,096 keys, so that four blocks of 512
// threads share a CU.
template <uint32_t CAP, uint32_t T>
struct OrderLds {
  static constexpr uint32_t BINS = CAP > 4096 ? 4096 : CAP > 2048 ? 2048 : CAP / 2, NW = T / 64;
  uint32_t key[CAP];
  uint32_t c[BINS + 1 + CAP / 2];  // a word per bin, then 16-bit counts, two a word
  uint32_t red[2][NW];
  uint32_t w[NW];
  uint32_t most;  // 1: a bin holds more than BIN_FULL keys; 2: BIN_RANKED in the second binning
};

// at[j] as order_block's, by a compare-exchange network in LDS: log^2 steps
// whatever the keys. Every exchange puts the smaller key first, so the places
// from m on need not exist.
template <uint32_t CAP, uint32_t T>
__device__ inline void order_network(uint32_t* s_key, uint16_t* s_src, const uint32_t (&key)[CAP / T],
                                     uint32_t (&at)[CAP / T], uint32_t m) {
  constexpr uint32_t PER = CAP / T;
  const uint32_t t = threadIdx.x;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      s_key[t + j * T] = key[j];
      s_src[t + j * T] = (uint16_t)(t + j * T);
    }
  __syncthreads();
  auto exchange = [&](uint32_t x, uint32_t y) {
    if (y >= m) return;
    const uint32_t kx = s_key[x], ky = s_key[y];
    if (kx <= ky) return;
    const uint16_t ix = s_src[x];
    s_key[x] = ky;
    s_key[y] = kx;
    s_src[x] = s_src[y];
    s_src[y] = ix;
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
  // each place's rank, where the keys were
  uint16_t* const s_at = reinterpret_cast<uint16_t*>(s_key);
  for (uint32_t p = t; p < m; p += T) s_at[s_src[p]] = (uint16_t)p;
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) at[j] = s_at[t + j * T];
}

// at[j]: the rank of key[j] (thread t's key of place t + j T) among the m keys.
// The keys are binned in BINS bins evenly between the smallest and the largest;
// where a bin holds more than BIN_FULL, each of those again in as many bins
// evenly as it holds keys, so that a clump, which fills few of the first, is
// spread over the second. A key's rank is its bin's start and the number of
// smaller keys in the bin; where even the second binning leaves more than
// BIN_RANKED keys in a bin (one key many times: no binning splits it), a network
// takes over. Every thread of the block calls it; no thread may still read L.
template <uint32_t CAP, uint32_t T>
__device__ inline void order_block(OrderLds<CAP, T>& L, const uint32_t (&key)[CAP / T], uint32_t (&at)[CAP / T],
                                   uint32_t m) {
  constexpr uint32_t PER = CAP / T, BINS = OrderLds<CAP, T>::BINS, NW = T / 64;
  const uint32_t t = threadIdx.x;
  uint32_t *const c1 = L.c, *const c2 = L.c + BINS + 1;
  if (t == 0) L.most = 0u;
  for (uint32_t i = t; i <= BINS; i += T) c1[i] = 0u;
  for (uint32_t i = t; i < CAP / 2; i += T) c2[i] = 0u;
  uint32_t lo = ~0u, hi = 0u;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      lo = min(lo, key[j]);
      hi = max(hi, key[j]);
    }
  for (int d = 32; d > 0; d >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, d));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d));
  }
  if ((t & 63u) == 0u) {
    L.red[0][t >> 6] = lo;
    L.red[1][t >> 6] = hi;
  }
  __syncthreads();
  for (uint32_t k = 0; k < NW; ++k) {
    lo = min(lo, L.red[0][k]);
    hi = max(hi, L.red[1][k]);
  }
  // (key - lo) scale / 2^32 in [0, BINS): scale rounded down far enough
  const unsigned long long scale =
      (unsigned long long)((double)BINS * 4294967296.0 / ((double)(hi - lo) + 1.0) * (1.0 - 0x1p-40));
  auto first_bin = [&](uint32_t k, uint32_t& frac) {
    const unsigned long long x = (unsigned long long)(k - lo) * scale;
    frac = (uint32_t)x;
    return (uint32_t)(x >> 32);
  };
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      uint32_t f;
      atomicAdd(&c1[first_bin(key[j], f)], 1u);
    }
  __syncthreads();
  {
    constexpr uint32_t PB = BINS / T;
    uint32_t c[PB], sum = 0u, most = 0u, tot;
#pragma unroll
    for (uint32_t k = 0; k < PB; ++k) {
      c[k] = c1[t * PB + k];
      sum += c[k];
      most = max(most, c[k]);
    }
    if (__any(most > BIN_FULL) && (t & 63u) == 0u) L.most = 1u;
    uint32_t run = scan_block<NW>(sum, &tot, L.w);
#pragma unroll
    for (uint32_t k = 0; k < PB; ++k) {
      c1[t * PB + k] = run;
      run += c[k];
    }
    if (t == 0) c1[BINS] = tot;
  }
  __syncthreads();
  uint32_t bin[PER];
  const bool twice = L.most != 0u;
  if (!twice) {
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
      if (t + j * T < m) {
        uint32_t f;
        bin[j] = first_bin(key[j], f);
        at[j] = atomicAdd(&c1[bin[j]], 1u);
        L.key[at[j]] = key[j];
      }
  } else {
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
      if (t + j * T < m) {
        uint32_t f;
        const uint32_t b = first_bin(key[j], f), p = c1[b];
        bin[j] = p + __umulhi(f, c1[b + 1u] - p);
        atomicAdd(&c2[bin[j] >> 1], 1u << ((bin[j] & 1u) * 16u));
      }
    __syncthreads();
    constexpr uint32_t PW = CAP / 2 / T;
    uint32_t c[PW], sum = 0u, most = 0u, tot;
#pragma unroll
    for (uint32_t k = 0; k < PW; ++k) {
      c[k] = c2[t * PW + k];
      sum += (c[k] & 0xffffu) + (c[k] >> 16);
      most = max(most, max(c[k] & 0xffffu, c[k] >> 16));
    }
    if (__any(most > BIN_RANKED) && (t & 63u) == 0u) L.most = 2u;
    uint32_t run = scan_block<NW>(sum, &tot, L.w);
    if (L.most == 2u) {
      order_network<CAP, T>(L.key, reinterpret_cast<uint16_t*>(c2), key, at, m);
      return;
    }
#pragma unroll
    for (uint32_t k = 0; k < PW; ++k) {
      const uint32_t mid = run + (c[k] & 0xffffu);
      c2[t * PW + k] = run | (mid << 16);
      run = mid + (c[k] >> 16);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j)
      if (t + j * T < m) {
        const uint32_t sh = (bin[j] & 1u) * 16u;
        at[j] = (atomicAdd(&c2[bin[j] >> 1], 1u << sh) >> sh) & 0xffffu;
        L.key[at[j]] = key[j];
      }
  }
  __syncthreads();
  // a bin's word is now its end, the start of the next
  auto end_of = [&](uint32_t b) { return twice ? (c2[b >> 1] >> ((b & 1u) * 16u)) & 0xffffu : c1[b]; };
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (t + j * T < m) {
      const uint32_t b0 = bin[j] ? end_of(bin[j] - 1u) : 0u, b1 = end_of(bin[j]);
      uint32_t r = b0;
      for (uint32_t q = b0; q < b1; ++q) {
        const uint32_t o = L.key[q];
        r += (o < key[j] || (o == key[j] && q < at[j])) ? 1u : 0u;
      }
      at[j] = r;
    }
}

}  // namespace hlc
