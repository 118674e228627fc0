// cap.hip -- kernels of the state cap (top-q cut of the selection).
//
// The composite order is (weight descending, tie-break hash ascending,
// canonical key ascending).  Weight keys are the bit patterns of the
// non-negative FP64 weights complemented, so ascending integers are
// descending weights; the hash is the splitmix64 output function (Steele,
// Lea & Flood 2014) chained over the canonical key words, most significant
// first, from 0.  A radix select walks 8-bit digits of (weight key, hash,
// key words) from the top; rows of a realization are decided in bulk once
// their digit differs from the realization's split digit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cap.hpp"
#include "common.hpp"

namespace paces {

namespace {

__device__ __forceinline__ uint64_t splitmix_mix(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Canonical word w (0 = most significant) of an internal key: the last W
// internal words, with the bits at and above B (realization id) cleared.
template <int Wi>
__device__ __forceinline__ uint64_t canon_word(const uint64_t (&k)[Wi], int W,
                                               int B, int w) {
  uint64_t v = k[Wi - W + w];
  if (w == 0) {
    const int top = B - 64 * (W - 1);  // bits held by word 0
    if (top < 64) v &= (uint64_t(1) << top) - 1;
  }
  return v;
}

template <int Wi>
__device__ __forceinline__ int cap_digit(int pass, uint64_t wk, uint64_t hk,
                                         const uint64_t (&k)[Wi], int W,
                                         int B) {
  if (pass < 8) return int((wk >> (56 - 8 * pass)) & 255u);
  if (pass < 16) return int((hk >> (56 - 8 * (pass - 8))) & 255u);
  const int p = pass - 16, w = p >> 3, b = p & 7;
  return int((canon_word<Wi>(k, W, B, w) >> (56 - 8 * b)) & 255u);
}

__global__ void k_cap_zero(uint32_t* ball, int R, const int* err) {
  if (*err) return;
  for (int r = threadIdx.x; r < R; r += blockDim.x) ball[r] = 0;
}

__global__ void __launch_bounds__(kBlock)
    k_cap_count(DevModel m, const StepCtl* ctl, const uint64_t* pay,
                uint32_t* ball, const int* err) {
  __shared__ uint32_t bins[kMaxReal];
  if (*err) return;
  const int64_t n = ctl->n_new;
  for (int r = threadIdx.x; r < m.R; r += blockDim.x) bins[r] = 0;
  __syncthreads();
  for (int64_t i = gtid(); i < n; i += gstride())
    atomicAdd(&bins[pay_real(pay[i])], 1u);
  __syncthreads();
  for (int r = threadIdx.x; r < m.R; r += blockDim.x)
    if (bins[r]) atomicAdd(&ball[r], bins[r]);
}

__global__ void __launch_bounds__(kBlock)
    k_count_real(DevModel m, const uint64_t* pay, const uint32_t* idx,
                 int64_t n, uint32_t* out) {
  __shared__ uint32_t bins[kMaxReal];
  for (int r = threadIdx.x; r < m.R; r += blockDim.x) bins[r] = 0;
  __syncthreads();
  for (int64_t i = gtid(); i < n; i += gstride())
    atomicAdd(&bins[pay_real(pay[idx ? int64_t(idx[i]) : i])], 1u);
  __syncthreads();
  for (int r = threadIdx.x; r < m.R; r += blockDim.x)
    if (bins[r]) atomicAdd(&out[r], bins[r]);
}

__global__ void __launch_bounds__(kBlock)
    k_iota_u32(uint32_t* p, int64_t n) {
  for (int64_t i = gtid(); i < n; i += gstride()) p[i] = uint32_t(i);
}

__global__ void k_cap_over(const uint32_t* ball, int R, int64_t cap,
                            int* err) {
  if (*err) return;
  bool over = false;
  for (int r = threadIdx.x; r < R; r += blockDim.x)
    if (int64_t(ball[r]) > cap) over = true;
  if (over) atomicOr(err, kErrCap);
}

template <int Wi, typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_cap_prepare(DevModel m, int W, const uint32_t* midx, int64_t nM,
                  const uint64_t* keys, const uint64_t* pay, const Amp* psi,
                  const int8_t* capped, uint64_t* wkey, uint64_t* hkey,
                  uint8_t* status) {
  for (int64_t j = gtid(); j < nM; j += gstride()) {
    const int64_t i = midx[j];
    const int r = pay_real(pay[i]);
    if (!capped[r]) {
      status[j] = 1;
      continue;
    }
    status[j] = 0;
    wkey[j] = ~uint64_t(__double_as_longlong(weight(psi[i])));
    uint64_t k[Wi];
    load_key<Wi>(keys, i, k);
    uint64_t h = 0;
    for (int w = 0; w < W; ++w) h = splitmix_mix(h ^ canon_word<Wi>(k, W, m.B, w));
    hkey[j] = h;
  }
}

// Digit histogram of the open rows per realization.  Up to kLdsReal
// realizations the block counts in LDS and adds each nonzero bin once: the
// leading weight digits are shared by almost every row, and global atomics
// on those few bins serialise the whole pass.
constexpr int kLdsReal = 32;  // 32 * 256 counters = 32 KiB of LDS

template <int Wi>
__global__ void __launch_bounds__(kBlock)
    k_cap_hist(DevModel m, int W, int pass, const uint32_t* midx, int64_t nM,
               const uint64_t* keys, const uint64_t* pay,
               const uint64_t* wkey, const uint64_t* hkey,
               const uint8_t* status, uint32_t* hist) {
  __shared__ uint32_t bins[kLdsReal * 256];
  const bool lds = m.R <= kLdsReal;
  if (lds) {
    for (int q = threadIdx.x; q < m.R * 256; q += blockDim.x) bins[q] = 0;
    __syncthreads();
  }
  for (int64_t j = gtid(); j < nM; j += gstride()) {
    if (status[j] != 0) continue;
    const int64_t i = midx[j];
    uint64_t k[Wi] = {};
    if (pass >= 16) load_key<Wi>(keys, i, k);
    const int d = cap_digit<Wi>(pass, wkey[j], hkey[j], k, W, m.B);
    const int b = pay_real(pay[i]) * 256 + d;
    if (lds)
      atomicAdd(&bins[b], 1u);
    else
      atomicAdd(&hist[b], 1u);
  }
  if (lds) {
    __syncthreads();
    for (int q = threadIdx.x; q < m.R * 256; q += blockDim.x)
      if (bins[q]) atomicAdd(&hist[q], bins[q]);
  }
}

template <int Wi>
__global__ void __launch_bounds__(kBlock)
    k_cap_apply(DevModel m, int W, int pass, const uint32_t* midx,
                int64_t nM, const uint64_t* keys, const uint64_t* pay,
                const uint64_t* wkey, const uint64_t* hkey,
                const int32_t* mode, const int32_t* dstar, uint8_t* status) {
  for (int64_t j = gtid(); j < nM; j += gstride()) {
    if (status[j] != 0) continue;
    const int64_t i = midx[j];
    const int r = pay_real(pay[i]);
    const int md = mode[r];
    if (md == kCapSkip) continue;
    if (md == kCapDrop) {
      status[j] = 2;
      continue;
    }
    if (md == kCapKeep) {
      status[j] = 1;
      continue;
    }
    uint64_t k[Wi] = {};
    if (pass >= 16) load_key<Wi>(keys, i, k);
    const int d = cap_digit<Wi>(pass, wkey[j], hkey[j], k, W, m.B);
    const int ds = dstar[r];
    if (d < ds)
      status[j] = 1;
    else if (d > ds)
      status[j] = 2;
    else if (md == kCapCut)
      status[j] = 1;
  }
}

__global__ void __launch_bounds__(kBlock)
    k_cap_clear(uint8_t* keep, int64_t n) {
  for (int64_t i = gtid(); i < n; i += gstride()) keep[i] = 0;
}

__global__ void __launch_bounds__(kBlock)
    k_cap_flags(const uint32_t* midx, int64_t nM, const uint8_t* status,
                uint8_t* keep) {
  for (int64_t j = gtid(); j < nM; j += gstride())
    if (status[j] == 1) keep[midx[j]] = 1;
}

// ---- the cut of one realization -----------------------------------------------
// Radix select over the complemented weight bits (13, 13, 13, 13 and 12 of
// them, most significant first): a pass counts the digit of the rows that
// share the digits decided so far, in LDS (32 KB of bins; the leading digit
// is the exponent and one mantissa bit, which a heavy-tailed state spreads
// over some tens of bins), and the block that arrives last finds the digit
// the cut falls on.  Later passes read 8 bytes per row; a pass that finds
// the cut between two digits ends the search (three passes for distinct
// weights), and the rest return at once.  The search took 6-8 passes of 8
// bits over 21 bytes per row each before, with a host round trip between
// them: 25-site chain, 24 steps at 1.6e7 rows 14.7 ms of kernels.
// Every block adds its bins to the same few counters of the leading digit and
// takes a ticket of one word, a few ns each, so two blocks per CU run with
// eight rows in flight per lane: a pass over 7e6 rows 22.5 -> 16 us on average
// and over 1.6e7 47 -> 35 (1024 blocks, one row in flight; 256 blocks 14 and
// 38).
__device__ __forceinline__ int top_shift(int pass) {
  return pass < 4 ? 51 - 13 * pass : 0;
}

template <typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_top_pass(int pass, const Amp* psi, const uint8_t* dist, int64_t n,
               int all, double th2, TopState* st, uint64_t* w,
               uint32_t* hist) {
  __shared__ uint32_t bins[kTopBins];
  __shared__ uint64_t prefix;
  __shared__ int64_t need;  // read here: the lane that decides writes it
  __shared__ int mode;
  if (threadIdx.x == 0) {
    prefix = st->prefix;
    need = st->need;
    mode = st->mode;
  }
  for (int b = threadIdx.x; b < kTopBins; b += kBlock) bins[b] = 0u;
  __syncthreads();
  if (mode) return;
  const int shift = top_shift(pass), width = pass < 4 ? 13 : 12;
  const uint64_t digit = (uint64_t(1) << width) - 1, pre = prefix;
  constexpr int U = 8;  // rows in flight per lane
  const int64_t step = gstride();
  if (pass == 0) {
    for (int64_t e0 = gtid(); e0 < n; e0 += U * step) {
      Amp a[U];
      uint8_t d[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t e = e0 + u * step < n ? e0 + u * step : e0;
        a[u] = psi[e];
        d[u] = dist[e];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (e0 + u * step >= n) break;
        const double wt = weight(a[u]);
        const bool cand = d[u] != kHole && (all || wt >= th2);
        const uint64_t key =
            cand ? ~uint64_t(__double_as_longlong(wt)) : ~0ull;
        w[e0 + u * step] = key;
        if (cand) atomicAdd(&bins[(key >> shift) & digit], 1u);
      }
    }
  } else {
    for (int64_t e0 = gtid(); e0 < n; e0 += U * step) {
      uint64_t key[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        key[u] = w[e0 + u * step < n ? e0 + u * step : e0];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t e = e0 + u * step;
        if (e >= n) break;
        if ((key[u] >> shift >> width) != pre) continue;
        // the last bin of all also holds the rows that are no candidates
        if (key[u] == ~0ull && (dist[e] == kHole || !(all || th2 <= 0)))
          continue;
        atomicAdd(&bins[(key[u] >> shift) & digit], 1u);
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kTopBins; b += kBlock)
    if (bins[b]) atomicAdd(&hist[b], bins[b]);
  if (!last_block(&st->ticket, gridDim.x)) return;
  constexpr int per = kTopBins / kBlock;
  const int b0 = threadIdx.x * per;
  uint32_t h[per], sum = 0;
#pragma unroll
  for (int q = 0; q < per; ++q) {
    h[q] = hist[b0 + q];
    sum += h[q];
    hist[b0 + q] = 0u;
  }
  uint32_t tot;
  int64_t below = block_excl_scan(sum, &tot);
  if (below < need && need <= below + sum) {
    int d = -1;
    int64_t here = 0;
#pragma unroll
    for (int q = 0; q < per; ++q)
      if (d < 0) {
        if (below + h[q] >= need) {
          d = b0 + q;
          here = h[q];
        } else {
          below += h[q];
        }
      }
    const uint64_t now = (pre << width) | uint64_t(d);
    st->prefix = now;
    st->need = need - below;
    if (need - below == here) {
      st->limit = shift ? ((now + 1) << shift) - 1 : now;
      st->mode = 1;
    } else if (pass == kTopPasses - 1) {
      st->limit = now;
      st->mode = 2;
    }
  }
}

__global__ void k_top_init(TopState* st, int64_t q) {
  st->prefix = 0;
  st->limit = 0;
  st->need = q;
  st->nties = 0;
  st->ticket = 0;
  st->mode = 0;
}

// Bits and sums in the layout of the select kernels; the rows equal to the
// limit in mode 2 are listed.  zeros: a weight of zero can be a candidate's.
__global__ void __launch_bounds__(kBlock)
    k_top_bits(const uint64_t* w, const uint8_t* dist, int64_t n, int zeros,
               TopState* st, uint32_t* ties, uint64_t* bits, uint32_t* sums,
               const int* err) {
  if (*err) return;
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  const uint64_t limit = st->limit;
  const int mode = st->mode;
  uint32_t v = 0;
  for (int64_t t = run.t0; t < run.t1; t += kItems) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      bool keep = false;
      if (e < n) {
        const uint64_t k = w[e];
        const bool cand = k != ~0ull || (zeros && dist[e] != kHole);
        keep = cand && (k < limit || (mode == 1 && k == limit));
        if (mode == 2 && cand && k == limit) {
          const uint32_t at = atomicAdd(&st->nties, 1u);
          if (at < kTopTies) ties[at] = uint32_t(e);
        }
      }
      const uint64_t b = __ballot(keep);
      if ((threadIdx.x & 63) == 0 && e < n) bits[e >> 6] = b;
      v += keep ? 1u : 0u;
    }
  }
  uint32_t tot;
  block_excl_scan(v, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// One block: the first `need` of the listed rows by (key hash, key) join the
// selection.  Equal weights come from orbits of a symmetric lattice, a few to
// a few hundred rows; each is ranked by counting.
template <int Wi>
__global__ void __launch_bounds__(kBlock)
    k_top_ties(DevModel m, int W, const uint64_t* keys, int64_t n, int grid,
               TopState* st, const uint32_t* ties, uint64_t* bits,
               uint32_t* sums, int* err) {
  __shared__ uint64_t hash[kTopTies];
  if (latched(err)) return;
  if (st->mode != 2) return;
  const uint32_t nt = st->nties;
  const int64_t need = st->need;
  __syncthreads();
  if (threadIdx.x == 0) st->nties = 0;
  if (nt > kTopTies) {
    if (threadIdx.x == 0) atomicOr(err, kErrTie);
    return;
  }
  for (uint32_t i = threadIdx.x; i < nt; i += kBlock) {
    uint64_t k[Wi];
    load_key<Wi>(keys, ties[i], k);
    uint64_t h = 0;
    for (int q = 0; q < W; ++q) h = splitmix_mix(h ^ canon_word<Wi>(k, W, m.B, q));
    hash[i] = h;
  }
  __syncthreads();
  const int64_t per = cdiv(cdiv(n, kBlock), grid);
  for (uint32_t i = threadIdx.x; i < nt; i += kBlock) {
    const int64_t row = ties[i];
    int64_t rank = 0;
    for (uint32_t j = 0; j < nt; ++j) {
      bool before = hash[j] < hash[i];
      if (hash[j] == hash[i] && j != i) {
        uint64_t a[Wi], b[Wi];
        load_key<Wi>(keys, ties[j], a);
        load_key<Wi>(keys, row, b);
        for (int q = W - 1; q >= 0; --q) {  // the most significant decides
          const uint64_t x = canon_word<Wi>(a, W, m.B, q);
          const uint64_t y = canon_word<Wi>(b, W, m.B, q);
          if (x != y) before = x < y;
        }
      }
      rank += before ? 1 : 0;
    }
    if (rank >= need) continue;
    atomicOr((unsigned long long*)(bits + (row >> 6)), 1ull << (row & 63));
    atomicAdd(&sums[row / kBlock / per], 1u);
  }
}

}  // namespace

void top_select(int prec, const void* psi, const uint8_t* dist, int64_t n,
                bool all, double th2, int64_t q, const TopBufs& tb,
                hipStream_t s) {
  k_top_init<<<1, 1, 0, s>>>(tb.st, q);
  const int g = std::min(grid_for(cdiv(n, 8)), 512);
  for (int p = 0; p < kTopPasses; ++p) {
    if (prec == 64)
      k_top_pass<double2><<<g, kBlock, 0, s>>>(p, (const double2*)psi, dist, n,
                                               all, th2, tb.st, tb.w, tb.hist);
    else
      k_top_pass<float2><<<g, kBlock, 0, s>>>(p, (const float2*)psi, dist, n,
                                              all, th2, tb.st, tb.w, tb.hist);
  }
}

int top_bits(const DevModel& m, int Wi, int W, const uint64_t* keys,
             const uint8_t* dist, int64_t n, bool zeros, const TopBufs& tb,
             const Sums& sm, int* err, hipStream_t s) {
  const int g = sum_grid(n, kBlock);
  k_top_bits<<<g, kBlock, 0, s>>>(tb.w, dist, n, zeros ? 1 : 0, tb.st, tb.ties,
                                  sm.bits, sm.sel, err);
  PACES_DISPATCH_W(Wi, k_top_ties<WW><<<1, kBlock, 0, s>>>(
                           m, W, keys, n, g, tb.st, tb.ties, sm.bits, sm.sel,
                           err));
  return g;
}

void cap_check(const DevModel& m, const StepCtl* ctl, const uint64_t* pay,
               int64_t est, int64_t cap, uint32_t* ball, int* err,
               hipStream_t s) {
  k_cap_zero<<<1, kBlock, 0, s>>>(ball, m.R, err);
  const int g = std::min(grid_for(est), 2048);
  k_cap_count<<<g, kBlock, 0, s>>>(m, ctl, pay, ball, err);
  k_cap_over<<<1, kBlock, 0, s>>>(ball, m.R, cap, err);
}

void count_per_real(const DevModel& m, const uint64_t* pay, int64_t n,
                    uint32_t* out, hipStream_t s, const uint32_t* idx) {
  (void)hipMemsetAsync(out, 0, size_t(m.R) * 4, s);
  if (n <= 0) return;
  k_count_real<<<std::min(grid_for(n), 2048), kBlock, 0, s>>>(m, pay, idx, n,
                                                              out);
}

void iota_u32(uint32_t* p, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  k_iota_u32<<<grid_for(n), kBlock, 0, s>>>(p, n);
}

void cap_prepare(const DevModel& m, int Wi, int W, int prec,
                 const uint32_t* midx, int64_t nM, const uint64_t* keys,
                 const uint64_t* pay, const void* psi, const int8_t* capped,
                 uint64_t* wkey, uint64_t* hkey, uint8_t* status,
                 hipStream_t s) {
  if (nM <= 0) return;
  const int g = grid_for(nM);
  if (prec == 64) {
    PACES_DISPATCH_W(Wi, k_cap_prepare<WW, double2><<<g, kBlock, 0, s>>>(
                             m, W, midx, nM, keys, pay, (const double2*)psi,
                             capped, wkey, hkey, status));
  } else {
    PACES_DISPATCH_W(Wi, k_cap_prepare<WW, float2><<<g, kBlock, 0, s>>>(
                             m, W, midx, nM, keys, pay, (const float2*)psi,
                             capped, wkey, hkey, status));
  }
}

void cap_hist(const DevModel& m, int Wi, int W, int pass, const uint32_t* midx,
              int64_t nM, const uint64_t* keys, const uint64_t* pay,
              const uint64_t* wkey, const uint64_t* hkey,
              const uint8_t* status, uint32_t* hist, hipStream_t s) {
  if (nM <= 0) return;
  PACES_DISPATCH_W(Wi, k_cap_hist<WW><<<grid_for(nM), kBlock, 0, s>>>(
                           m, W, pass, midx, nM, keys, pay, wkey, hkey,
                           status, hist));
}

void cap_apply(const DevModel& m, int Wi, int W, int pass,
               const uint32_t* midx, int64_t nM, const uint64_t* keys,
               const uint64_t* pay, const uint64_t* wkey,
               const uint64_t* hkey, const int32_t* mode,
               const int32_t* dstar, uint8_t* status, hipStream_t s) {
  if (nM <= 0) return;
  PACES_DISPATCH_W(Wi, k_cap_apply<WW><<<grid_for(nM), kBlock, 0, s>>>(
                           m, W, pass, midx, nM, keys, pay, wkey, hkey, mode,
                           dstar, status));
}

void cap_flags(const uint32_t* midx, int64_t nM, const uint8_t* status,
               uint8_t* keep, int64_t n_old, hipStream_t s) {
  if (n_old > 0) k_cap_clear<<<grid_for(n_old), kBlock, 0, s>>>(keep, n_old);
  if (nM > 0)
    k_cap_flags<<<grid_for(nM), kBlock, 0, s>>>(midx, nM, status, keep);
}

}  // namespace paces
