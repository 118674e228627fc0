// small.hip -- the tail of a step for sets that fit one compute unit's LDS.
//
// A set of a few thousand rows leaves the chip idle whatever the launch: each
// of the thirteen launches after the transfer (bounds, coefficients, nine
// Clenshaw terms, observables, record) takes 4-6 us for well under one
// microsecond of work, most of it the launch itself and the loads' latency.
// One block of 1024 threads does all of it with the three vectors in LDS and
// the rows' columns and matrix values in registers, one barrier per term.
// Beyond three rows per thread, LDS (160 KB) and registers (128 per thread at
// this block size) are full.  At 2500 rows of the 4-site ring the tail takes
// 34 us; its thirteen launches took 66 us and the gaps between them.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "small.hpp"
#include "warm_device.hpp"

namespace paces {

namespace {

constexpr int kNB = 1024, kWaves = kNB / 64, kRows = kSmallRows / kNB;

// Folds of M values over the block at once (two barriers); every lane gets
// the results.
struct Add {
  __device__ double operator()(double a, double b) const { return a + b; }
};
struct Max {
  __device__ double operator()(double a, double b) const { return fmax(a, b); }
};
constexpr int kFoldMax = 6;
template <int M, typename F>
__device__ __forceinline__ void block_fold(double (&v)[M],
                                           double (*red)[kWaves], F f) {
#pragma unroll
  for (int x = 0; x < M; ++x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v[x] = f(v[x], __shfl_xor(v[x], o));
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int x = 0; x < M; ++x) red[x][threadIdx.x >> 6] = v[x];
  }
  __syncthreads();
  // 16 wave results in the 16 lanes of a row of the wave
#pragma unroll
  for (int x = 0; x < M; ++x) {
    double r = red[x][threadIdx.x & (kWaves - 1)];
#pragma unroll
    for (int o = kWaves / 2; o > 0; o >>= 1) r = f(r, __shfl_xor(r, o));
    v[x] = r;
  }
}

template <typename R>
struct SVec;
template <>
struct SVec<double> {
  using T = double2;
};
template <>
struct SVec<float> {
  using T = float2;
};

// The record, the step's commit and the host's mirrors (obs_final with one
// realization).
template <typename Amp>
__device__ __forceinline__ void small_observe(const SmallTail& a, int K,
                                              double emin, double emax,
                                              double energy, int n,
                                              const Amp* psi, double* bins,
                                              double (*red)[kWaves]) {
  const int N = a.m.N;
  StepCtl* ctl = a.ctl;
  for (int j = threadIdx.x; j < N; j += kNB) bins[j] = 0.0;
  __syncthreads();
  double n2 = 0;
  uint32_t rows = 0, kept = 0;
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int i = threadIdx.x + q * kNB;
    bool keep = false;
    if (i < n && !(a.dist && a.dist[i] == kHole)) {
      const double w = weight(psi[i]);
      n2 += w;
      ++rows;
      keep = w >= a.th2;
      atomicAdd(&bins[pay_site(a.pay[i])], w);
    }
    const uint64_t b = __ballot(keep);
    if ((threadIdx.x & 63) == 0 && i < n) a.bits[i >> 6] = b;
    kept += keep ? 1u : 0u;
  }
  double ms = 0, re = 0, im = 0;
  for (int i = threadIdx.x; i < a.n_mass; i += kNB) ms += a.mass_part[i];
  for (int64_t i = threadIdx.x; i < a.n0; i += kNB) {
    const int32_t row = a.p0[i];
    if (row < 0) continue;
    const double2 v = widen(psi[row]);
    const double ar = a.amps0[2 * i], ai = a.amps0[2 * i + 1];
    re += ar * v.x + ai * v.y;  // conj(a0) * v
    im += ar * v.y - ai * v.x;
  }
  double v[6] = {n2, ms, re, im, double(rows), double(kept)};
  block_fold(v, red, Add());
  n2 = v[0];
  ms = v[1];
  const int64_t nrec = ctl->nrec;
  const bool room = nrec + 1 <= a.ring_cap;  // the host keeps it
  double* rec = a.ring + nrec * a.rec_doubles;
  __syncthreads();  // every wave has its record before lane 0 counts it
  if (room) {
    for (int j = threadIdx.x; j < N; j += kNB) rec[kObsFields + j] = bins[j];
    if (threadIdx.x == 0) {
      const double t = ctl->t + a.dt, total = a.mass_tot[0] + ms;
      rec[0] = t;
      rec[1] = n2;
      rec[2] = a.want_energy ? energy : NAN;
      rec[3] = v[2];
      rec[4] = v[3];
      rec[5] = ms;
      rec[6] = total;
      rec[7] = v[4];
      rec[8] = double(a.cnt[0]);
      rec[9] = double(K);
      rec[10] = emin;
      rec[11] = emax;
      a.sel[0] = uint32_t(v[5]);
      if (isfinite(n2)) {
        a.mass_tot[0] = total;
        ctl->t = t;
        ctl->n_old = ctl->n_new;
        ctl->nrec += 1;
      } else {
        atomicOr(a.err, kErrNonFinite);
      }
    }
  }
}

template <typename R, int ND, int NV>
__global__ void __launch_bounds__(kNB) k_small_tail(SmallTail a) {
  using Amp = typename SVec<R>::T;
  constexpr int D = 2 * ND + 2 * NV;
  extern __shared__ double lds[];
  // phi, b_0 and b_1 as offsets into one array (pointers picked at run time
  // would be generic ones, and their loads flat instead of LDS reads)
  Amp* const v = reinterpret_cast<Amp*>(lds);
  __shared__ double J[kMaxTerms + 1], coef[kMaxTerms][2];
  __shared__ double red[kFoldMax][kWaves];
  __shared__ double phase[2];
  __shared__ int latch;
  const DevModel& m = a.m;
  StepCtl* ctl = a.ctl;
  const int n = int(ctl->n_new < uint32_t(kSmallRows + 1) ? ctl->n_new
                                                          : kSmallRows + 1);
  if (threadIdx.x == 0) {
    latch = *a.err;
    if (!latch && n > kSmallRows) {
      latch = kErrBig;
      atomicOr(a.err, kErrBig);
    }
  }
  __syncthreads();
  if (!latch) {
    // rows: columns, diagonal and matrix values stay in registers
    int32_t cols[kRows][D];
    R dv[kRows], gv[kRows][NV][2], jv[3] = {0, 0, 0};
#pragma unroll
    for (int x = 0; x < ND; ++x) jv[x] = R(m.J[x]);
    double lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int i = threadIdx.x + q * kNB;
#pragma unroll
      for (int s = 0; s < D; ++s) cols[q][s] = -1;
      dv[q] = 0;
#pragma unroll
      for (int nu = 0; nu < NV; ++nu) gv[q][nu][0] = gv[q][nu][1] = 0;
      if (i >= n) continue;
      v[i] = static_cast<const Amp*>(a.phi)[i];
      const uint64_t p = a.pay[i];
      load_cols<D>(a.col + int64_t(i) * D, cols[q]);
      const double d = row_diag(m, p, 0);
      dv[q] = R(d);
#pragma unroll
      for (int nu = 0; nu < NV; ++nu) {
        const int occ = pay_occ(p, nu);
        gv[q][nu][0] = R(m.gsq[nu * kGsqStride + occ]);
        gv[q][nu][1] = R(m.gsq[nu * kGsqStride + occ + 1]);
      }
      if (a.dist && a.dist[i] == kHole) continue;
      double rad = 0;
#pragma unroll
      for (int s = 0; s < D; ++s)
        if (cols[q][s] >= 0) rad += fabs(slot_value(m, p, s));
      lo = fmin(lo, d - rad);
      hi = fmax(hi, d + rad);
    }
    {
      double e[2] = {-lo, hi};
      block_fold(e, red, Max());
      lo = -e[0];
      hi = e[1];
    }
    if (lo > hi) lo = hi = 0.0;  // empty set
    // interval, coefficients and term count as in the coefficient kernel
    const double pad = 1e-12 * (fabs(hi) + fabs(lo));
    const double emin = lo - pad, emax = hi + pad;
    double wid = 0.5 * (emax - emin);
    const double b = 0.5 * (emax + emin);
    if (!(wid > 1e-300)) wid = 1e-300;
    const double x = fabs(wid * a.dt);
    const int kcap = a.k_max < kMaxTerms ? a.k_max : kMaxTerms;
    int K = 0;
    if (!(x <= double(kcap))) {
      if (threadIdx.x == 0) latch = isfinite(x) ? kErrTerms : kErrNonFinite;
      __syncthreads();
    } else {
      const double thresh = ldexp(a.tol, -2);
      if (x <= 2.0) {
        for (int k = threadIdx.x; k <= kcap; k += kNB)
          J[k] = bessel_series(x, k, thresh);
      } else if (threadIdx.x == 0) {
        bessel_miller(x, kcap, J);
      }
      if (threadIdx.x == kNB - 1) {
        double sn, cs;
        sincos(b * a.dt, &sn, &cs);
        phase[0] = cs;
        phase[1] = -sn;
      }
      __syncthreads();
      double last = 0;
      for (int k = threadIdx.x; k <= kcap; k += kNB)
        if (fabs(J[k]) > thresh) last = fmax(last, double(k));
      {
        double e[1] = {last};
        block_fold(e, red, Max());
        last = e[0];
      }
      K = int(last) + 1;
      if (K > kcap) {
        K = kcap + 1;
        if (threadIdx.x == 0) latch = kErrTerms;
      }
      for (int k = threadIdx.x; k < K && k < kMaxTerms; k += kNB) {
        const double v =
            (k == 0 ? 1.0 : 2.0) * (a.dt < 0 && (k & 1) ? -J[k] : J[k]);
        const int q = k & 3;  // (-i)^k
        coef[k][0] = (q == 0) ? v : (q == 2 ? -v : 0.0);
        coef[k][1] = (q == 1) ? -v : (q == 3 ? v : 0.0);
        a.cc->c[k][0] = coef[k][0];
        a.cc->c[k][1] = coef[k][1];
      }
      if (threadIdx.x == 0) {
        ctl->kmax = uint32_t(K);
        a.cc->emin = emin;
        a.cc->emax = emax;
        a.cc->a = wid;
        a.cc->b = b;
        a.cc->alpha = 1.0 / wid;
        a.cc->beta = -b / wid;
        a.cc->phase[0] = phase[0];
        a.cc->phase[1] = phase[1];
        a.cc->K = K;
      }
      __syncthreads();
    }
    if (latch) {
      if (threadIdx.x == 0) atomicOr(a.err, latch);
    } else {
      // Clenshaw's recurrence (k_cheb_term's arithmetic, row by row)
      const R alpha = R(1.0 / wid), beta = R(-b / wid);
      double esum = 0;
      for (int kk = K > 1 ? K - 2 : 0; kk >= 0; --kk) {
        const bool first = kk == K - 2 || K == 1, fin = kk == 0;
        const int in = first ? 0 : (((kk + 1) & 1) + 1) * kSmallRows;
        const int out = ((kk & 1) + 1) * kSmallRows;
        const int prev = kk == K - 3 ? 0 : out;
        const R ckr = R(coef[kk][0]), cki = R(coef[kk][1]);
        const double fac = fin ? 1.0 : 2.0;
        R sir = R(fac), sii = 0;
        if (first) {
          sir = K == 1 ? R(0) : R(fac * coef[K - 1][0]);
          sii = K == 1 ? R(0) : R(fac * coef[K - 1][1]);
        }
        R spr = 1, spi = 0;
        if (kk == K - 3) {
          spr = R(coef[K - 1][0]);
          spi = R(coef[K - 1][1]);
        }
        const R phr = fin ? R(phase[0]) : R(1), phm = fin ? R(phase[1]) : R(0);
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
          const int i = threadIdx.x + q * kNB;
          if (i >= n) continue;
          const Amp xi = v[in + i];
          R hr = dv[q] * xi.x, hi2 = dv[q] * xi.y;
#pragma unroll
          for (int s = 0; s < D; ++s) {
            const int32_t c = cols[q][s];
            if (c >= 0) {
              const R w = s < 2 * ND ? jv[s >> 1]
                                     : gv[q][(s - 2 * ND) >> 1][(s - 2 * ND) & 1];
              const Amp xj = v[in + c];
              hr += w * xj.x;
              hi2 += w * xj.y;
            }
          }
          if (first) esum += double(xi.x) * double(hr) + double(xi.y) * double(hi2);
          const R tr = alpha * hr + beta * xi.x, ti = alpha * hi2 + beta * xi.y;
          R yr = sir * tr - sii * ti, yi = sir * ti + sii * tr;
          const Amp f = v[i];
          yr += ckr * f.x - cki * f.y;
          yi += ckr * f.y + cki * f.x;
          if (!first) {
            const Amp z = v[prev + i];
            yr -= spr * z.x - spi * z.y;
            yi -= spr * z.y + spi * z.x;
          }
          Amp o;
          o.x = phr * yr - phm * yi;
          o.y = phr * yi + phm * yr;
          v[out + i] = o;
          if (fin) static_cast<Amp*>(a.psi)[i] = o;
        }
        __syncthreads();
      }
      if (a.ring) {
        double e[1] = {esum};
        block_fold(e, red, Add());
        small_observe(a, K, emin, emax, e[0], n, v + kSmallRows,
                      reinterpret_cast<double*>(v + 2 * kSmallRows), red);
      }
    }
  }
  __syncthreads();
  const int e = latch_now(a.err);
  if (a.ring) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(ctl);
    uint32_t* dst = reinterpret_cast<uint32_t*>(a.h_ctl);
    for (int i = threadIdx.x; i < int(sizeof(StepCtl) / 4); i += kNB)
      dst[i] = src[i];
    if (threadIdx.x == 0) *a.h_err = e;
  } else if (threadIdx.x == 0) {
    a.said[0] = ctl->kmax;
    a.said[1] = uint32_t(e);
  }
  __threadfence_system();
}

// ---- the in-place expansion ---------------------------------------------------
// Exclusive scan over the block of one u32 per lane; total to *tot.
__device__ __forceinline__ uint32_t scan_all(uint32_t v, uint32_t* s,
                                             uint32_t* tot) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) s[wid] = x;
  __syncthreads();
  uint32_t base = 0, all = 0;
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t t = s[w];
    base += w < wid ? t : 0u;
    all += t;
  }
  *tot = all;
  return base + x - v;
}

// One block, thread t holding rows 3t .. 3t+2.  The distance bytes of the old
// range live in LDS until the commit; candidates, table and new rows are the
// launches' own (warm.hip describes the search).  A step of the 4-site ring at
// 2500 rows spends 24 us here; its nineteen launches took 69 us.
template <int W, typename Amp>
__global__ void __launch_bounds__(kNB) k_small_expand(SmallExpand a) {
  __shared__ uint8_t ld[kSmallRows];
  __shared__ uint32_t ws[kWaves];
  __shared__ double red[kFoldMax][kWaves];
  __shared__ uint32_t gs[kMaxRounds + 2];
  __shared__ int latch;
  const DevModel& m = a.m;
  const int D = m.D, k = a.k;
  const Side c = a.c;
  StepCtl* ctl = a.ctl;
  Amp* psi = static_cast<Amp*>(a.psi);
  const uint32_t n_all = ctl->n_old;
  const bool big = n_all > uint32_t(kSmallRows);
  const int n = big ? 0 : int(n_all), e0 = threadIdx.x * kRows;
  // start of the step, selection, holes
  uint32_t sel = 0, hol = 0;
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int e = e0 + q;
    if (e >= n) continue;
    const bool hole = c.dist[e] == kHole;
    const bool in = !hole && weight(psi[e]) >= a.th2;
    ld[e] = hole ? kHole : in ? 0 : kFar;
    sel += in ? 1u : 0u;
    hol += hole ? 1u : 0u;
  }
  uint32_t nM, nfree;
  scan_all(sel, ws, &nM);
  uint32_t at = scan_all(hol, ws, &nfree);
#pragma unroll
  for (int q = 0; q < kRows; ++q)
    if (e0 + q < n && ld[e0 + q] == kHole) a.wb.freel[at++] = uint32_t(e0 + q);
  if (threadIdx.x == 0) {
    a.cnt[0] = nM;
    a.ball[0] = 0;
    *a.err = big ? kErrBig : 0;
    latch = big ? kErrBig : 0;
    ctl->fstart[0] = 0;
    ctl->nM = nM;
    ctl->n_new = 0;
    ctl->kmax = 0;
    ctl->r_need = 0;
    ctl->r_own = 0;
    ctl->c_max = 0;
    ctl->n_staged = 0;
    ctl->gstart[0] = ctl->gstart[1] = 0;
    ctl->nfree = nfree;
    ctl->w_moved = 0;
    ctl->w_tomb = 0;
    ctl->w_drop = 0;
    ctl->ticket = 0;
    gs[0] = gs[1] = 0;
  }
  __syncthreads();
  if (latch) return;
  uint32_t c_max = 0;
  for (int r = 1; r <= k; ++r) {
    // live rows at distance r-1: marks inside the set, slots that leave it
    uint32_t msk[kRows], cnt = 0;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int e = e0 + q;
      msk[q] = 0;
      if (e >= n || ld[e] != uint8_t(r - 1)) continue;
      const uint64_t p = c.pay[e];
      for (int s = 0; s < D; ++s) {
        const int32_t nb = c.col[int64_t(e) * D + s];
        if (nb >= 0) {
          if (ld[nb] > r) ld[nb] = uint8_t(r);
        } else if (slot_live(m, p, s)) {
          msk[q] |= 1u << s;
        }
      }
      cnt += __popc(msk[q]);
    }
    uint32_t noc;
    uint32_t off = scan_all(cnt, ws, &noc);
    const uint32_t f0 = gs[r - 1];
    const uint32_t nc = noc + (gs[r] - f0) * D;
    c_max = nc > c_max ? nc : c_max;
    if (int64_t(nc) > a.rb.cand_cap) {
      if (threadIdx.x == 0) atomicOr(a.err, kErrChunks);
      return;
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      while (msk[q]) {
        const int s = __ffs(msk[q]) - 1;
        msk[q] &= msk[q] - 1;
        a.wb.wlist[off++] = (uint64_t(e0 + q) << 8) | uint64_t(s);
      }
    __syncthreads();
    // insert-if-absent
    for (uint32_t cand = threadIdx.x; cand < nc; cand += kNB) {
      uint64_t key[W];
      int64_t p;
      int s;
      uint32_t ref = kNone;
      if (warm_cand<W>(m, ctl, a.wb.freel, noc, f0, a.wb.wlist, c, cand, key, p,
                       s)) {
        const uint64_t h = key_hash<W>(m, key);
        const uint32_t tag = hash_tag(h);
        const uint64_t mine = (uint64_t(tag) << 32) | uint64_t(kCand | cand);
        uint64_t i = h & a.mask;
        bool done = false;
        for (uint64_t probes = 0; probes <= a.mask && probes < kMaxProbe;
             ++probes) {
          uint64_t e = a.table[i];
          if (e == kEmpty) {
            const uint64_t old = atomicCAS((unsigned long long*)(a.table + i),
                                           (unsigned long long)kEmpty,
                                           (unsigned long long)mine);
            if (old == kEmpty) {
              ref = kOwnerW;
              a.rb.c_slot[cand] = uint32_t(probes);
              done = true;
              break;
            }
            e = old;
          }
          if (uint32_t(e >> 32) == tag) {
            const uint32_t v = uint32_t(e);
            if (v & kCand) {
              uint64_t k2[W];
              int64_t p2;
              int s2;
              warm_cand<W>(m, ctl, a.wb.freel, noc, f0, a.wb.wlist, c,
                           int64_t(v & ~kCand), k2, p2, s2);
              bool same = true;
#pragma unroll
              for (int q = 0; q < W; ++q) same &= (k2[q] == key[q]);
              done = same;
            } else {
              const int64_t row = int64_t(v & ~kStaged);
              if (key_eq<W>(key, c.keys + row * W)) {
                if (!(v & kStaged) && ld[row] > r) ld[row] = uint8_t(r);
                done = true;
              }
            }
            if (done) break;
          }
          i = (i + 1) & a.mask;
        }
        if (!done) atomicOr(&latch, kErrTableFull);
      }
      a.rb.c_ref[cand] = ref;
    }
    __syncthreads();
    // owners take their rows in candidate order
    uint32_t num = gs[r];
    for (uint32_t c0 = 0; c0 < nc; c0 += kNB) {
      const uint32_t cand = c0 + threadIdx.x;
      const bool own = cand < nc && a.rb.c_ref[cand] == kOwnerW;
      uint32_t tot;
      const uint32_t q = num + scan_all(own ? 1u : 0u, ws, &tot);
      num += tot;
      if (!own) continue;
      const int64_t row = found_row(q, ctl, a.wb.freel);
      if (row >= a.cap) {
        atomicOr(&latch, kErrCapacity);
        continue;
      }
      uint64_t key[W];
      int64_t p;
      int s;
      warm_cand<W>(m, ctl, a.wb.freel, noc, f0, a.wb.wlist, c, cand, key, p, s);
      store_key<W>(c.keys, row, key);
      uint64_t np, nt;
      slot_row_info<W>(m, key, c.pay[p], c.tot[p], s, np, nt);
      c.pay[row] = np;
      c.tot[row] = nt;
      if (row < n)
        ld[row] = uint8_t(kNewRow | r);
      else
        c.dist[row] = uint8_t(kNewRow | r);
      const uint64_t h = key_hash<W>(m, key);
      a.table[((h & a.mask) + a.rb.c_slot[cand]) & a.mask] =
          (uint64_t(hash_tag(h)) << 32) | uint64_t(kStaged | uint32_t(row));
      Amp z;
      z.x = 0;
      z.y = 0;
      psi[row] = z;
    }
    if (threadIdx.x == 0) {
      gs[r + 1] = num;
      ctl->gstart[r + 1] = num;
      ctl->n_staged = num;
      if (a.row_limit > 0 && int64_t(nM) + num > a.row_limit)
        atomicOr(&latch, kErrOver);
    }
    __syncthreads();
    // (errors gather in LDS: a barrier does not wait for global adds)
    if (latch) {
      if (threadIdx.x == 0) *a.err = latch;
      return;
    }
  }
  const uint32_t ns = gs[k + 1];
  // state cap: live rows of the new set
  if (a.max_states > 0) {
    uint32_t live = 0, all;
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      if (e0 + q < n && ld[e0 + q] <= k) ++live;
    scan_all(live, ws, &all);
    all += ns;
    if (threadIdx.x == 0) ctl->n_ball = a.ball[0] = all;
    if (int64_t(all) > a.max_states) {
      if (threadIdx.x == 0) atomicOr(a.err, kErrCap);
      return;
    }
  }
  // the commit: rows not reached become holes
  double lost = 0;
  uint32_t tombs = 0, drops = 0;
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int e = e0 + q;
    if (e >= n || ld[e] != kFar) continue;
    ++drops;
    lost += weight(psi[e]);
    Amp z;
    z.x = 0;
    z.y = 0;
    psi[e] = z;
    uint64_t key[W];
    load_key<W>(c.keys, e, key);
    const uint64_t h = key_hash<W>(m, key);
    const int64_t sl =
        warm_slot(a.table, a.mask, h, a.table[h & a.mask], uint32_t(e));
    if (sl >= 0) {
      a.table[sl] = kTomb;
      ++tombs;
    }
    for (int s = 0; s < D; ++s) {
      const int32_t nb = c.col[int64_t(e) * D + s];
      if (nb >= 0 && ld[nb] <= k) c.col[int64_t(nb) * D + (s ^ 1)] = -1;
      c.col[int64_t(e) * D + s] = -1;
    }
  }
  __syncthreads();
  // found states: plain table entries, columns both ways.  (Rows not reached
  // are known by ld, so nothing waits for their holes.)
  for (uint32_t t = threadIdx.x; t < ns * D; t += kNB) {
    const int64_t row = found_row(t / D, ctl, a.wb.freel);
    const int s = int(t % D);
    uint64_t par[W], key[W];
    load_key<W>(c.keys, row, par);
    if (s == 0) {
      const uint64_t h = key_hash<W>(m, par);
      const int64_t sl = warm_slot(a.table, a.mask, h, a.table[h & a.mask],
                                      kStaged | uint32_t(row));
      if (sl >= 0)
        a.table[sl] = (uint64_t(hash_tag(h)) << 32) | uint64_t(row);
    }
    int32_t out = -1;
    if (slot_target<W>(m, par, c.pay[row], s, key)) {
      const int64_t f =
          warm_find<W>(a.table, a.mask, c.keys, key, key_hash<W>(m, key));
      if (f >= 0 && (f >= n || kept(ld[f], k))) {
        out = int32_t(f);
        c.col[f * D + (s ^ 1)] = int32_t(row);
      }
    }
    c.col[row * D + s] = out;
  }
  for (int64_t i = threadIdx.x; i < a.n0; i += kNB) {
    uint64_t key[W];
    load_key<W>(a.keys0, i, key);
    const int64_t f =
        warm_find<W>(a.table, a.mask, c.keys, key, key_hash<W>(m, key));
    a.p0[i] = f >= 0 && (f >= n || kept(ld[f], k)) ? int32_t(f) : -1;
  }
  // distance bytes: holes, and the rounds of the found states
  for (uint32_t t = threadIdx.x; t < ns; t += kNB) {
    const int64_t row = found_row(t, ctl, a.wb.freel);
    if (row >= n) c.dist[row] = uint8_t(c.dist[row] & ~kNewRow);
  }
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int e = e0 + q;
    if (e >= n) continue;
    const uint8_t d = ld[e];
    c.dist[e] = d == kFar || d == kHole ? kHole : uint8_t(d & ~kNewRow);
  }
  double v[3] = {lost, double(tombs), double(drops)};
  block_fold(v, red, Add());
  if (threadIdx.x == 0) {
    a.mass_part[0] = v[0];
    ctl->w_tomb = uint32_t(v[1]);
    ctl->w_drop = uint32_t(v[2]);
    ctl->w_moved = 1;
    ctl->c_max = c_max;
    ctl->n_new = uint32_t(new_range(ctl));
  }
}

template <typename R, int ND, int NV>
bool launch(const SmallTail& a, hipStream_t s) {
  const int bytes = 3 * kSmallRows * int(sizeof(typename SVec<R>::T));
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_tail<R, ND, NV>),
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          bytes) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  k_small_tail<R, ND, NV><<<1, kNB, bytes, s>>>(a);
  return true;
}

}  // namespace

bool small_tail(const SmallTail& a, int prec, hipStream_t s) {
#define PACES_SMALL(ND, NV) \
  case ND * 8 + NV: return prec == 64 ? launch<double, ND, NV>(a, s) \
                                      : launch<float, ND, NV>(a, s)
  switch (a.m.ndim * 8 + a.m.V) {
    PACES_SMALL(1, 1);
    PACES_SMALL(1, 2);
    PACES_SMALL(2, 1);
    PACES_SMALL(2, 2);
    PACES_SMALL(3, 1);
    default: return false;
  }
#undef PACES_SMALL
}

void small_expand(const SmallExpand& a, int Wi, int prec, hipStream_t s) {
  if (prec == 64) {
    PACES_DISPATCH_W(Wi, k_small_expand<WW, double2><<<1, kNB, 0, s>>>(a));
  } else {
    PACES_DISPATCH_W(Wi, k_small_expand<WW, float2><<<1, kNB, 0, s>>>(a));
  }
}

}  // namespace paces
