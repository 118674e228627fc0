// kernels.hip -- HIP kernels of one co-evolving-subspace step on gfx950.
//
// The step is sparse, memory-bound gather/scatter: kernels stream rows with
// one row (or one row slot) per lane, wave64, 256-lane blocks, and no
// matrix cores.  Row counts live in device memory (StepCtl); kernels run on
// grid-stride grids, clamp counts to the allocated capacity and latch
// overflows, and every kernel after a latching one returns at once when the
// latch is set, so a failed step touches nothing out of bounds and leaves
// the previous state intact for a retry.  Sums over rows use a fixed
// lane-to-row mapping, wave shuffles in a fixed order and per-block
// partials summed in block order; population and per-realization bins use
// LDS atomics, whose order within a block is not fixed.
//
// Stages (paper: Sec. "Formal operator representation and notes on
// parallelization"):
//   select     rows of psi with |c|^2 >= theta^2, compacted in row order
//              (Sec. "Truncation & post-adaptation detruncation")
//   expand     k rounds of neighbour generation on packed keys with
//              insert-if-absent into an HBM hash table (Eqs. (def_neighbor_k),
//              (H_eff)); the candidate whose compare-and-swap claims a key
//              owns it, so new rows are numbered in an order that may vary
//              between runs while every amplitude, taken per basis state,
//              is reproduced bit for bit
//   transfer   old amplitudes moved to their rows in the new set, weight of
//              the dropped rows summed (post-adaptation detruncation)
//   build      ELL columns come out of the expansion; values are implied by
//              the slot and the row payload (Sec. "Generating the effective
//              Hamiltonian from the effective Hilbert space")
//   propagate  exp(-i H dt) phi by a Chebyshev series evaluated with
//              Clenshaw's recurrence, one fused SpMV kernel per term
//              (App. "The action of the exponential of a sparse matrix"
//              names series of SpMVs; Chebyshev replaces Taylor here)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "kernels.hpp"

namespace paces {

namespace {

// ---- fills and step control -------------------------------------------------
__global__ void __launch_bounds__(kBlock)
    k_fill_u64(uint64_t* p, int64_t n, uint64_t v) {
  for (int64_t i = gtid(); i < n; i += gstride()) p[i] = v;
}

// A dispatch that does nothing: a marker that kernel traces and counter
// runs show in stream order.
__global__ void k_mark(int tag) { (void)tag; }

__global__ void k_clear_err(int* err, StepCtl* ctl) {
  *err = 0;
  ctl->ticket = 0;
}

// The number of series terms and the error latch into two words (mapped host
// memory or device memory).
__global__ void k_report(const StepCtl* ctl, const int* err, uint32_t* out) {
  out[0] = ctl->kmax;
  out[1] = uint32_t(*err);
  __threadfence_system();
}

// ---- a given set of states (stateless propagation) --------------------------
// Canonical keys of W words to the internal width Wi >= W (leading zero
// words; one realization, so no realization bits).
__global__ void __launch_bounds__(kBlock)
    k_pad_keys(int W, int Wi, const uint64_t* in, uint64_t* out, int64_t n) {
  const int64_t total = n * Wi;
  for (int64_t e = gtid(); e < total; e += gstride()) {
    const int64_t i = e / Wi;
    const int w = int(e % Wi) - (Wi - W);
    out[e] = w >= 0 ? in[i * W + w] : 0ull;
  }
}

// Counts of a step whose set is rows [0, n) in place (frontier 0 is the whole
// set), and its table cleared.
__global__ void __launch_bounds__(kBlock)
    k_set_begin(StepCtl* ctl, int* err, uint32_t n, uint64_t* table,
                int64_t slots) {
  if (gtid() == 0) {
    *err = 0;
    ctl->n_old = n;
    ctl->nM = n;
    ctl->fstart[0] = 0;
    ctl->fstart[1] = n;
    ctl->n_new = n;
    ctl->kmax = 0;
    ctl->r_need = 0;
  }
  for (int64_t i = gtid(); i < slots; i += gstride()) table[i] = kEmpty;
}

// Row i of the set from its key: payload and totals, columns -1, the key into
// the table.  A key that names no basis state (site below N, occupations
// within the cutoffs, no bits above the state's B bits) or that another row
// holds too latches kErrInput.  One pass over the keys where payloads, insert
// and check were three: an equal key is met by the insert's own probe, which
// compares the keys of rows whose tags agree.  1.16e6 rows of a ring of 16: 113
// -> 64 us.
template <int W>
__global__ void __launch_bounds__(kBlock)
    k_set_rows(DevModel m, const uint64_t* keys, int64_t n, uint64_t* pay,
               uint64_t* tot, int32_t* col, uint64_t* table, uint64_t mask,
               int* err) {
  for (int64_t i = gtid(); i < n; i += gstride()) {
    uint64_t k[W];
    load_key<W>(keys, i, k);
    bool ok = true;
#pragma unroll
    for (int q = 0; q < W; ++q) {
      const int lo = 64 * (W - 1 - q);  // bit position of the word's bit 0
      if (lo + 64 <= m.B) continue;
      const uint64_t above = lo >= m.B ? ~0ull : ~((uint64_t(1) << (m.B - lo)) - 1);
      ok &= (k[q] & above) == 0;
    }
    const int j = int(k[W - 1] & ((uint64_t(1) << m.bj) - 1));
    ok &= j < m.N;
    if (!ok) {
      atomicOr(err, kErrInput);
      continue;
    }
    int nj[kMaxV], T[kMaxV];
    for (int nu = 0; nu < m.V; ++nu) {
      nj[nu] = int(get_field<W>(k, field_off(m, j, nu), m.bnu[nu]));
      int sum = 0;
      for (int q = 0; q < m.N; ++q) {
        const int v = int(get_field<W>(k, field_off(m, q, nu), m.bnu[nu]));
        ok &= v <= m.cut[nu];
        sum += v;
      }
      T[nu] = sum;
    }
    pay[i] = make_pay(m.V, j, nj, T, key_real<W>(m, k));
    tot[i] = make_tot(m.V, T);
    for (int s = 0; s < m.D; s += 2)
      *reinterpret_cast<int2*>(col + i * m.D + s) = make_int2(-1, -1);
    const uint64_t h = key_hash<W>(m, k);
    const uint32_t tag = hash_tag(h);
    const uint64_t mine = (uint64_t(tag) << 32) | uint64_t(i);
    uint64_t at = h & mask;
    bool done = false;
    for (uint64_t q = 0; ok && q <= mask && q < kMaxProbe; ++q) {
      uint64_t e = table[at];
      if (e == kEmpty) {
        e = atomicCAS((unsigned long long*)(table + at),
                      (unsigned long long)kEmpty, (unsigned long long)mine);
        done = e == kEmpty;
        if (done) break;
      }
      if (uint32_t(e >> 32) == tag &&
          key_eq<W>(k, keys + int64_t(uint32_t(e)) * W))
        ok = false;
      at = (at + 1) & mask;
    }
    if (!ok)
      atomicOr(err, kErrInput);
    else if (!done)
      atomicOr(err, kErrTableFull);
  }
}

// The columns of a given set.  Slots 2t and 2t + 1 are each other's inverse:
// row i's neighbour f in slot 2t has i in slot 2t + 1, so one lookup per pair
// of slots writes both ends, and an end that nothing writes stays -1 (1.16e6
// rows of a ring of 16: 81 us with every slot looked up, 46 so).
template <int W>
__global__ void __launch_bounds__(kBlock)
    k_set_cols(DevModel m, const uint64_t* keys, const uint64_t* pay,
               int64_t n, const uint64_t* table, uint64_t mask, int32_t* col,
               const int* err) {
  if (*err) return;
  const uint32_t half = uint32_t(m.D) / 2;
  for (int64_t c = gtid(); c < n * half; c += gstride()) {
    const int64_t i = c / half;
    const int s = 2 * int(c - i * half);
    uint64_t par[W], key[W];
    load_key<W>(keys, i, par);
    if (!slot_target<W>(m, par, pay[i], s, key)) continue;
    const int64_t f =
        table_find<W>(table, mask, keys, key, key_hash<W>(m, key));
    if (f < 0) continue;
    col[i * m.D + s] = int32_t(f);
    col[f * m.D + s + 1] = int32_t(i);
  }
}

__global__ void k_begin_step(StepCtl* ctl, int* err, uint32_t* cnt,
                             uint32_t* ball, int R) {
  for (int i = threadIdx.x; i < R; i += blockDim.x) cnt[i] = 0u;
  for (int i = threadIdx.x; i < R; i += blockDim.x) ball[i] = 0u;
  if (threadIdx.x == 0) {
    *err = 0;
    ctl->fstart[0] = 0;
    ctl->nM = 0;
    ctl->n_new = 0;
    ctl->kmax = 0;
    ctl->r_need = 0;
    ctl->r_own = 0;
    ctl->c_max = 0;
    ctl->n_staged = 0;
    ctl->gstart[0] = 0;
    ctl->gstart[1] = 0;
    ctl->nfree = 0;
    ctl->w_moved = 0;  // an in-place step has not committed
    ctl->w_tomb = 0;
    ctl->w_drop = 0;
    ctl->ticket = 0;
  }
}

// ---- select -----------------------------------------------------------------
// A tile is kBlock rows, row t * kBlock + lane of lane `lane`, and a block
// takes kItems of its tiles at a time: every load of the block is one
// contiguous run, and the bits of a wave's 64 rows are one ballot.

// Rows that are holes (dist == kHole, left by dropped rows of in-place
// steps) are never selected; dist may be null (no holes).
__device__ __forceinline__ bool is_hole(const uint8_t* dist, int64_t e) {
  return dist && dist[e] == kHole;
}

// The bits of the wave's 64 rows from e on (lane 0's row a multiple of 64).
__device__ __forceinline__ void put_bits(uint64_t* bits, int64_t e, int64_t n,
                                         bool keep) {
  const uint64_t b = __ballot(keep);
  if ((threadIdx.x & 63) == 0 && e < n) bits[e >> 6] = b;
}

template <typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_select_bits(const Amp* psi, const uint8_t* dist, const StepCtl* ctl,
                  double th2, uint64_t* bits, uint32_t* sums) {
  const int64_t n = ctl->n_old;
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  uint32_t v = 0;
  for (int64_t t = run.t0; t < run.t1; t += kItems) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      const bool keep = e < n && weight(psi[e]) >= th2 && !is_hole(dist, e);
      put_bits(bits, e, n, keep);
      v += keep ? 1u : 0u;
    }
  }
  uint32_t tot;
  block_excl_scan(v, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Selection given as one flag per old row (state cap).
__global__ void __launch_bounds__(kBlock)
    k_flag_bits(const uint8_t* keep, const StepCtl* ctl, uint64_t* bits,
                uint32_t* sums) {
  const int64_t n = ctl->n_old;
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  uint32_t v = 0;
  for (int64_t t = run.t0; t < run.t1; t += kItems) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      const bool k = e < n && keep[e];
      put_bits(bits, e, n, k);
      v += k ? 1u : 0u;
    }
  }
  uint32_t tot;
  block_excl_scan(v, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// The selected rows ascending: the sums of the blocks before, then one block
// scan per run of kBlock rows.  Reads a bit per row where it read the
// amplitude before (16 bytes): 43 us of a step at 1.5e7 rows.
__global__ void __launch_bounds__(kBlock)
    k_select_write(const uint64_t* bits, StepCtl* ctl, const uint32_t* sums,
                   uint32_t* midx, const int* err) {
  if (*err) return;
  const int64_t n = ctl->n_old;
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  uint64_t total;
  uint32_t at = uint32_t(sums_before(sums, gridDim.x, blockIdx.x, &total));
  if (gtid() == 0) {
    ctl->nM = uint32_t(total);
    ctl->fstart[1] = uint32_t(total);
  }
  for (int64_t t = run.t0; t < run.t1; t += kItems) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      const bool k = e < n && ((bits[e >> 6] >> (e & 63)) & 1u);
      uint32_t tot;
      const uint32_t off = block_excl_scan(k ? 1u : 0u, &tot) + at;
      if (k) midx[off] = uint32_t(e);
      at += tot;
    }
  }
}

__global__ void __launch_bounds__(kBlock)
    k_select_all(StepCtl* ctl, uint32_t* midx) {
  const int64_t n = ctl->n_old;
  for (int64_t i = gtid(); i < n; i += gstride()) midx[i] = uint32_t(i);
  if (gtid() == 0) {
    ctl->nM = uint32_t(n);
    ctl->fstart[1] = uint32_t(n);
  }
}

// ---- row metadata from keys -------------------------------------------------
template <int W>
__global__ void __launch_bounds__(kBlock)
    k_row_info(DevModel m, const uint64_t* keys, int64_t n, uint64_t* pay,
               uint64_t* tot) {
  for (int64_t r = gtid(); r < n; r += gstride()) {
    uint64_t k[W];
    load_key<W>(keys, r, k);
    const int j = int(k[W - 1] & ((uint64_t(1) << m.bj) - 1));
    int nj[kMaxV], T[kMaxV];
    for (int nu = 0; nu < m.V; ++nu) {
      nj[nu] = int(get_field<W>(k, field_off(m, j, nu), m.bnu[nu]));
      int s = 0;
      for (int i = 0; i < m.N; ++i)
        s += int(get_field<W>(k, field_off(m, i, nu), m.bnu[nu]));
      T[nu] = s;
    }
    pay[r] = make_pay(m.V, j, nj, T, key_real<W>(m, k));
    tot[r] = make_tot(m.V, T);
  }
}


// ---- insert rows into the cleared table -------------------------------------
// Row i of the new set is row midx[i] of the old one (keys_o given) or is
// already in place (rehash after growth, keys_o null).  With phi given, the
// row's amplitude moves along (the transfer then skips rows of M).  cnt_r: the
// rows per realization, cleared; with one realization that is nM, and no block
// adds to it (16384 of them on one counter: 149 -> 139 us at 1.6e7 rows).
template <int W, typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_insert_rows(DevModel m, const uint64_t* keys_o, const uint64_t* pay_o,
                  const uint64_t* tot_o, const uint32_t* midx,
                  const uint32_t* nptr, int64_t n_fixed, uint64_t* keys_n,
                  uint64_t* pay_n, uint64_t* tot_n, uint8_t* dist_n,
                  uint64_t* table, uint64_t mask, uint32_t* cnt_r, const Amp* psi_o, Amp* phi,
                  int* err) {
  __shared__ uint32_t bins[kMaxReal];
  if (latched(err)) return;
  for (int r = threadIdx.x; r < m.R; r += blockDim.x) bins[r] = 0;
  __syncthreads();
  const int64_t nM = nptr ? int64_t(*nptr) : n_fixed;
  for (int64_t i = gtid(); i < nM; i += gstride()) {
    uint64_t k[W];
    if (keys_o) {
      const int64_t r = midx[i];
      load_key<W>(keys_o, r, k);
      store_key<W>(keys_n, i, k);
      pay_n[i] = pay_o[r];
      tot_n[i] = tot_o[r];
      if (phi) phi[i] = psi_o[r];
      if (cnt_r && m.R > 1) atomicAdd(&bins[pay_real(pay_o[r])], 1u);
    } else {
      load_key<W>(keys_n, i, k);
    }
    if (dist_n) dist_n[i] = 0;
    const uint64_t h = key_hash<W>(m, k);
    const uint64_t mine = (uint64_t(hash_tag(h)) << 32) | uint64_t(i);
    uint64_t s = h & mask;
    bool done = false;
    for (uint64_t p = 0; p <= mask && p < kMaxProbe; ++p) {
      if (table[s] == kEmpty &&
          atomicCAS((unsigned long long*)(table + s), (unsigned long long)kEmpty,
                    (unsigned long long)mine) == kEmpty) {
        done = true;
        break;
      }
      s = (s + 1) & mask;
    }
    if (!done) atomicOr(err, kErrTableFull);
  }
  if (cnt_r && m.R > 1) count_flush(m.R, bins, cnt_r);
  if (cnt_r && m.R == 1 && gtid() == 0) cnt_r[0] = uint32_t(nM);
}

// ---- expansion round --------------------------------------------------------
// Chunk `chunk` of round r: parents [f0, f0 + rows) with f0 = fstart[r-1] +
// chunk * per, per = cand_cap / D, of frontier r-1 = [fstart[r-1],
// fstart[r]).  rows > per: parents are left over for further chunks.
struct Chunk {
  int64_t f0, rows;
};
__device__ __forceinline__ Chunk round_chunk(const StepCtl* ctl, int r,
                                             int chunk, int64_t per) {
  const int64_t f1 = ctl->fstart[r];
  const int64_t start = int64_t(ctl->fstart[r - 1]) + int64_t(chunk) * per;
  return {start < f1 ? start : f1, start < f1 ? f1 - start : 0};
}

// Probe: insert-if-absent of candidate c = (parent f0 + c / D, slot c % D).
// A table slot holds (tag << 32 | ref); ref is a row of the new set or,
// during the round, kCand | candidate id.  The candidate whose
// compare-and-swap fills an empty slot owns that key.  Entries only move
// EMPTY -> CAND(owner) inside this kernel, so a stale read is repaired by
// the compare-and-swap.  Outcomes per candidate:
//   structural zero      col = -1
//   key already a row    col = that row
//   owner                c_ref = kOwner, c_slot = probe distance of the
//                        claimed slot from the key's home, and the owner's
//                        rank in its tile << 16
//   key owned by c2      c_ref = c2 (column linked by the commit)
// A block takes a contiguous run of tiles of kBlock candidates; tile_base
// holds the block's owners before the tile, sums the block's owners, so that
// the commit numbers the new rows without a scan in between (a round was
// eight launches before, two now).
// row_limit > 0 (state cap): once the rows found so far exceed it, kErrOver
// is latched.  A block stops at its next tile once anything is latched, so
// a set that outgrows the table or the cap ends the round there: under a
// binding cap (4x4x4 lattice, ten-word keys, cap 2e6) the uncut ball's
// inserts into an overfull table took 0.6-0.9 s per step before.  A block adds
// its rows to the one counter every fourth tile and at its end: with an add per
// tile the same lattice's probes took 51.4 us on average, 48.8 so.
constexpr uint32_t kOwner = 0xFFFFFFFEu;

template <int W>
__global__ void __launch_bounds__(kBlock)
    k_expand_probe(DevModel m, const uint64_t* keys, const uint64_t* pay,
                   StepCtl* ctl, int r, int chunk, int last, int64_t cand_cap,
                   int64_t row_limit, uint64_t* table, uint64_t mask,
                   uint32_t* c_slot, uint32_t* c_ref, uint32_t* tile_base,
                   uint32_t* sums, int32_t* col, int* err) {
  __shared__ int stop[2];  // latch seen at this tile, by parity of the tile
  if (latched(err)) return;
  const int D = m.D;
  const int64_t per = cand_cap / D;
  const Chunk ch = round_chunk(ctl, r, chunk, per);
  if (ch.rows > per && last) {
    if (gtid() == 0) {
      atomicOr(err, kErrChunks);
      const uint32_t need =
          uint32_t(cdiv(int64_t(ctl->fstart[r]) - ctl->fstart[r - 1], per));
      if (need > ctl->r_need) ctl->r_need = need;
    }
    return;
  }
  const int64_t f0 = ch.f0, nc = (ch.rows < per ? ch.rows : per) * D;
  if (gtid() == 0 && uint32_t(nc) > ctl->c_max) ctl->c_max = uint32_t(nc);
  const int64_t nM = ctl->nM;
  const TileRun run = tile_run(cdiv(nc, kBlock), gridDim.x);
  uint32_t own = 0, pend = 0;  // pend: not yet in r_own
  int par = 0;
  for (int64_t tile = run.t0; tile < run.t1; ++tile, par ^= 1) {
    const int64_t c = tile * kBlock + threadIdx.x;
    if (threadIdx.x == 0) stop[par] = latch_now(err);
    uint32_t owner = 0, dist = 0;
    if (c < nc) {
      const int64_t p = f0 + c / D;
      const int s = int(c % D);
      uint64_t par_k[W], k[W];
      load_key<W>(keys, p, par_k);
      const uint64_t py = pay[p];
      uint32_t rref = kNone;
      if (!slot_target<W>(m, par_k, py, s, k)) {
        col[p * D + s] = -1;
      } else {
        const uint64_t h = key_hash<W>(m, k);
        const uint32_t tag = hash_tag(h);
        const uint64_t mine =
            (uint64_t(tag) << 32) | uint64_t(kCand | uint32_t(c));
        uint64_t i = h & mask;
        bool done = false;
        for (uint64_t probes = 0; probes <= mask && probes < kMaxProbe;
             ++probes) {
          uint64_t e = table[i];
          if (e == kEmpty) {
            const uint64_t old = atomicCAS((unsigned long long*)(table + i),
                                           (unsigned long long)kEmpty,
                                           (unsigned long long)mine);
            if (old == kEmpty) {
              rref = kOwner;
              dist = uint32_t(probes);
              owner = 1;
              done = true;
              break;
            }
            e = old;
          }
          if (uint32_t(e >> 32) == tag) {
            const uint32_t rr = uint32_t(e);
            bool same;
            if (rr & kCand) {
              const int64_t c2 = int64_t(rr & ~kCand);
              uint64_t par2[W], k2[W];
              load_key<W>(keys, f0 + c2 / D, par2);
              slot_target<W>(m, par2, pay[f0 + c2 / D], int(c2 % D), k2);
              same = true;
#pragma unroll
              for (int q = 0; q < W; ++q) same &= (k2[q] == k[q]);
            } else {
              same = key_eq<W>(k, keys + int64_t(rr) * W);
            }
            if (same) {
              if (rr & kCand)
                rref = rr & ~kCand;
              else
                col[p * D + s] = int32_t(rr);
              done = true;
              break;
            }
          }
          i = (i + 1) & mask;
        }
        if (!done) atomicOr(err, kErrTableFull);
      }
      c_ref[c] = rref;
    }
    uint32_t tot;
    const uint32_t rank = block_excl_scan(owner, &tot);
    if (owner) c_slot[c] = dist | (rank << 16);
    if (threadIdx.x == 0) {
      tile_base[tile] = own;
      pend += tot;
      if (row_limit > 0 && pend &&
          (((tile - run.t0) & 3) == 3 || tile + 1 == run.t1)) {
        if (nM + int64_t(atomicAdd(&ctl->r_own, pend)) + pend > row_limit)
          atomicOr(err, kErrOver);
        pend = 0;
      }
    }
    own += tot;
    if (stop[par]) return;  // written before the scan's barriers
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = own;
}

// Owners append their key as a new row: row = rows so far + owners of the
// blocks before + owners of the tiles before + rank in the tile; the table
// slot is pointed at the row.  A candidate whose key another one owns takes
// that one's row.  Same grid as the probe.  Block 0 closes the chunk (after
// the last one, frontier r); more than load_rows rows (0: no limit) latch
// kErrTableFull: the table can still be enlarged, and a round's inserts or
// the last lookups in a table beyond that load cost more than the repeated
// step.
template <int W, typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_expand_commit(DevModel m, Side n, StepCtl* ctl, int r, int chunk,
                    int last, int64_t cand_cap, int64_t cap, int64_t load_rows,
                    uint64_t* table, uint64_t mask, const uint32_t* c_slot,
                    const uint32_t* c_ref, const uint32_t* tile_base,
                    const uint32_t* sums, int32_t* col, Amp* phi, int* err) {
  __shared__ uint32_t pre[kSumBlocks];
  if (latched(err)) return;
  const int D = m.D;
  const int64_t per = cand_cap / D;
  const Chunk ch = round_chunk(ctl, r, chunk, per);
  const int64_t f0 = ch.f0, nc = (ch.rows < per ? ch.rows : per) * D;
  const int64_t n_cur = chunk == 0 ? ctl->fstart[r] : ctl->r_cur[chunk & 1];
  const int64_t ntiles = cdiv(nc, kBlock), tiles_per = cdiv(ntiles, gridDim.x);
  const uint32_t total = sums_scan(sums, gridDim.x, pre);
  if (gtid() == 0) {
    int64_t now = n_cur + total;
    if (load_rows > 0 && now > load_rows) atomicOr(err, kErrTableFull);
    if (now > cap) {
      atomicOr(err, kErrCapacity);
      now = cap;
    }
    ctl->r_cur[(chunk + 1) & 1] = uint32_t(now);
    if (last) ctl->fstart[r + 1] = uint32_t(now);
  }
  const TileRun run = tile_run(ntiles, gridDim.x);
  for (int64_t tile = run.t0; tile < run.t1; ++tile) {
    const int64_t c = tile * kBlock + threadIdx.x;
    if (c >= nc) continue;
    const uint32_t ref = c_ref[c];
    if (ref == kNone) continue;
    const int64_t p = f0 + c / D;
    const int s = int(c % D);
    if (ref != kOwner) {
      const int64_t t2 = int64_t(ref) / kBlock;
      const int64_t row = n_cur + pre[t2 / tiles_per] + tile_base[t2] +
                          (c_slot[ref] >> 16);
      col[p * D + s] = row < cap ? int32_t(row) : -1;
      continue;
    }
    const uint32_t sl = c_slot[c];
    const int64_t row = n_cur + pre[blockIdx.x] + tile_base[tile] + (sl >> 16);
    if (row >= cap) {  // latched by block 0
      col[p * D + s] = -1;
      continue;
    }
    uint64_t par[W], k[W];
    load_key<W>(n.keys, p, par);
    const uint64_t py = n.pay[p];
    slot_target<W>(m, par, py, s, k);
    store_key<W>(n.keys, row, k);
    uint64_t np, nt;
    slot_row_info<W>(m, k, py, n.tot[p], s, np, nt);
    n.pay[row] = np;
    n.tot[row] = nt;
    n.dist[row] = uint8_t(r);
    // the slot holds (tag | candidate); the tag and the home follow from
    // the key, so the entry is rewritten without reading it back
    const uint64_t h = key_hash<W>(m, k);
    table[((h & mask) + (sl & 0xFFFFu)) & mask] =
        (uint64_t(hash_tag(h)) << 32) | uint64_t(row);
    col[p * D + s] = int32_t(row);
    Amp z;
    z.x = 0;
    z.y = 0;
    phi[row] = z;
  }
}

template <int W>
__global__ void __launch_bounds__(kBlock)
    k_lookup_cols(DevModel m, const uint64_t* keys, const uint64_t* pay,
                  StepCtl* ctl, int k, const uint64_t* table, uint64_t mask,
                  int32_t* col, int64_t max_states, uint32_t* ball,
                  const uint64_t* keys0, int64_t n0, int32_t* p0, int* err) {
  if (*err) return;
  const int D = m.D;
  // rows of the initial states in the new set
  for (int64_t i = gtid(); i < n0; i += gstride()) {
    uint64_t key[W];
    load_key<W>(keys0, i, key);
    p0[i] = int32_t(table_find<W>(table, mask, keys, key, key_hash<W>(m, key)));
  }
  const int64_t f0 = ctl->fstart[k];
  const int64_t f1 = ctl->fstart[k + 1];
  const int64_t nc = (f1 - f0) * D;
  if (gtid() == 0) {
    ctl->n_new = uint32_t(f1);
    if (max_states > 0) {
      ctl->n_ball = ball[0] = uint32_t(f1);
      if (f1 > max_states) atomicOr(err, kErrCap);
    }
  }
  for (int64_t c = gtid(); c < nc; c += gstride()) {
    const int64_t p = f0 + c / D;
    const int s = int(c % D);
    uint64_t par[W], key[W];
    load_key<W>(keys, p, par);
    int32_t out = -1;
    if (slot_target<W>(m, par, pay[p], s, key))
      out = int32_t(table_find<W>(table, mask, keys, key, key_hash<W>(m, key)));
    col[p * D + s] = out;
  }
}

// ---- transfer ---------------------------------------------------------------

// Old row i goes to its row of the new set, or counts as discarded weight.
// Rows whose bit is set in sel (M, already placed by the insert) are passed
// over.
template <int W, typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_transfer(DevModel m, const uint64_t* keys_o, const uint8_t* o_dist,
               const Amp* psi_o,
               const StepCtl* ctl, const uint64_t* table, uint64_t mask,
               const uint64_t* keys_n, Amp* phi, double* mass_part,
               int32_t* tmap, const uint64_t* sel, const int* err) {
  __shared__ double bins[kMaxReal];
  if (*err) return;
  const int R = m.R;
  if (R > 1) {
    for (int r = threadIdx.x; r < R; r += blockDim.x) bins[r] = 0.0;
    __syncthreads();
  }
  const int64_t n_old = ctl->n_old;
  double lost = 0;
  for (int64_t i = gtid(); i < n_old; i += gstride()) {
    if (is_hole(o_dist, i)) {
      if (tmap) tmap[i] = -1;
      continue;
    }
    if (sel && ((sel[i >> 6] >> (i & 63)) & 1u)) continue;
    const Amp v = psi_o[i];
    uint64_t k[W];
    load_key<W>(keys_o, i, k);
    const int64_t r = table_find<W>(table, mask, keys_n, k, key_hash<W>(m, k));
    if (tmap) tmap[i] = int32_t(r);
    if (r >= 0)
      phi[r] = v;
    else if (R > 1)
      atomicAdd(&bins[key_real<W>(m, k)], weight(v));
    else
      lost += weight(v);
  }
  if (R > 1) {
    __syncthreads();
    for (int r = threadIdx.x; r < R; r += blockDim.x)
      mass_part[int64_t(blockIdx.x) * R + r] = bins[r];
  } else {
    lost = block_sum(lost);
    if (threadIdx.x == 0) mass_part[blockIdx.x] = lost;
  }
}

// ---- Gershgorin bounds and Chebyshev coefficients ---------------------------
// Order-preserving map of doubles to signed 64-bit integers, so that
// integer min / max (exact, order independent) give the double min / max.
__device__ __forceinline__ long long ord_of(double x) {
  const long long b = __double_as_longlong(x);
  return b >= 0 ? b : (b ^ 0x7FFFFFFFFFFFFFFFll);
}
__device__ __forceinline__ double dbl_of(long long o) {
  return __longlong_as_double(o >= 0 ? o : (o ^ 0x7FFFFFFFFFFFFFFFll));
}

// Gershgorin interval per realization: rows stride over a fixed grid; per
// block the (lo, hi) of each realization go to part[block][r][2].  A lane
// takes two rows at once and forms their slots' values without a branch; with
// each value's load behind a branch of its own a launch waited for one row's
// chain (24 bytes a row: 25-site chain at 1.5e7 rows 85 -> 55 us, ring of 16
// at 0.5 to 2.3 million 18.0 -> 13.8).  A wave whose rows are all of one
// realization folds them first: 64 lanes on one LDS word are served one after
// the other (with it, 64 6x6 lattices 67 -> 46 us).
template <int ND, int NV>
__global__ void __launch_bounds__(kBlock)
    k_bounds(DevModel m, const uint64_t* pay, const uint64_t* tot,
             const uint8_t* dist, const int32_t* col, int64_t cap,
             const StepCtl* ctl, double* part, const int* err) {
  constexpr int D = 2 * ND + 2 * NV, U = 2;
  __shared__ long long blo[kMaxReal], bhi[kMaxReal];
  if (*err) return;
  const int R = m.R;
  if (R > 1) {
    for (int r = threadIdx.x; r < R; r += blockDim.x) {
      blo[r] = ord_of(INFINITY);
      bhi[r] = ord_of(-INFINITY);
    }
    __syncthreads();
  }
  const int64_t n = ctl->n_new;
  double lo = INFINITY, hi = -INFINITY;
  for (int64_t r0 = int64_t(blockIdx.x) * kBlock; r0 < n;
       r0 += U * gstride()) {
    uint64_t p[U], tt[U];
    int32_t cs[U][D];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = r0 + u * gstride() + threadIdx.x;
      ok[u] = r < n && !is_hole(dist, r);
      const int64_t rc = r < n ? r : n - 1;
      p[u] = ld_stream(pay + rc);
      tt[u] = NV > 2 ? tot[rc] : 0;
      load_cols<D>(col + rc * D, cs[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double v[D];
#pragma unroll
      for (int s = 0; s < 2 * ND; ++s) v[s] = fabs(m.J[s >> 1]);
#pragma unroll
      for (int nu = 0; nu < NV; ++nu) {
        const double* g = m.gsq + nu * kGsqStride + (ok[u] ? pay_occ(p[u], nu) : 0);
        v[2 * ND + 2 * nu] = fabs(g[0]);
        v[2 * ND + 2 * nu + 1] = fabs(g[1]);
      }
      double rad = 0;
#pragma unroll
      for (int s = 0; s < D; ++s) rad += cs[u][s] >= 0 ? v[s] : 0.0;
      const double d = ok[u] ? row_diag(m, p[u], tt[u]) : 0.0;
      const double l = ok[u] ? d - rad : INFINITY;
      const double h = ok[u] ? d + rad : -INFINITY;
      if (R > 1) {
        const uint64_t act = __ballot(ok[u]);
        if (act == 0) continue;
        const int q = pay_real(p[u]);
        const int q0 = __shfl(q, __ffsll((unsigned long long)act) - 1);
        if (__ballot(ok[u] && q != q0) == 0) {
          const double wl = wave_min(l), wh = wave_max(h);
          if ((threadIdx.x & 63) == 0) {
            atomicMin(&blo[q0], ord_of(wl));
            atomicMax(&bhi[q0], ord_of(wh));
          }
        } else if (ok[u]) {
          atomicMin(&blo[q], ord_of(l));
          atomicMax(&bhi[q], ord_of(h));
        }
      } else {
        lo = fmin(lo, l);
        hi = fmax(hi, h);
      }
    }
  }
  if (R > 1) {
    __syncthreads();
    for (int r = threadIdx.x; r < R; r += blockDim.x) {
      part[(int64_t(blockIdx.x) * R + r) * 2] = dbl_of(blo[r]);
      part[(int64_t(blockIdx.x) * R + r) * 2 + 1] = dbl_of(bhi[r]);
    }
  } else {
    lo = block_min(lo);
    hi = block_max(hi);
    if (threadIdx.x == 0) {
      part[2 * blockIdx.x] = lo;
      part[2 * blockIdx.x + 1] = hi;
    }
  }
}

// One block per realization: fold the per-block bounds, pad them, and
// compute the Chebyshev coefficients and the number of terms K_r.
__global__ void __launch_bounds__(kBlock)
    k_coef(const double* part, int nparts, int R, double dt, double tol,
           int k_max, int launched, ChebCoef* cc_all, StepCtl* ctl,
           int* err) {
  __shared__ double J[kMaxTerms + 1];
  if (latched(err)) return;
  const int rr = blockIdx.x;
  ChebCoef* cc = cc_all + rr;
  double lo = INFINITY, hi = -INFINITY;
  for (int i = threadIdx.x; i < nparts; i += blockDim.x) {
    lo = fmin(lo, part[(int64_t(i) * R + rr) * 2]);
    hi = fmax(hi, part[(int64_t(i) * R + rr) * 2 + 1]);
  }
  lo = block_min(lo);
  hi = block_max(hi);
  if (lo > hi) lo = hi = 0.0;  // empty set
  // widen by 1e-12 of the magnitude so the interval strictly contains the
  // spectrum
  const double pad = 1e-12 * (fabs(hi) + fabs(lo));
  const double emin = lo - pad, emax = hi + pad;
  double a = 0.5 * (emax - emin);
  const double b = 0.5 * (emax + emin);
  if (!(a > 1e-300)) a = 1e-300;
  const double x = fabs(a * dt);  // dt < 0: J_k(-x) = (-1)^k J_k(x) below
  const int kcap = k_max < kMaxTerms ? k_max : kMaxTerms;
  // the series needs more than x terms: a spectrum too wide for the step
  // (or not finite) is reported before any Bessel recurrence runs
  if (!(x <= double(kcap))) {
    if (threadIdx.x == 0) atomicOr(err, isfinite(x) ? kErrTerms : kErrNonFinite);
    return;
  }
  const double thresh = ldexp(tol, -2);
  if (x <= 2.0) {
    for (int k = threadIdx.x; k <= kcap; k += blockDim.x)
      J[k] = bessel_series(x, k, thresh);
  } else if (threadIdx.x == 0) {
    bessel_miller(x, kcap, J);
  }
  __syncthreads();
  // K = 1 + the last k with |J_k| above tol / 4.  Beyond x each J_k is
  // below half the one before (J_{k+1} / J_k < x / (2k + 2) before the
  // first zero of J_k), so the omitted tail sum_{k>=K} |c_k| =
  // 2 sum |J_k| <= 4 |J_K| stays within tol (|T_k| <= 1 on the interval)
  double last = 0;
  for (int k = threadIdx.x; k <= kcap; k += blockDim.x)
    if (fabs(J[k]) > thresh) last = fmax(last, double(k));
  last = block_max(last);
  int K = int(last) + 1;
  if (K > kcap) K = kcap + 1;
  if (threadIdx.x == 0) {
    if (K > kcap)
      atomicOr(err, kErrTerms);
    else if (K - 1 > launched)  // launch indices K - 2 .. 0 do the work
      atomicOr(err, kErrNeedTerms);
    atomicMax(&ctl->kmax, uint32_t(K));
    cc->emin = emin;
    cc->emax = emax;
    cc->a = a;
    cc->b = b;
    cc->alpha = 1.0 / a;
    cc->beta = -b / a;
    cc->K = K;
  }
  if (threadIdx.x == 64) {  // another wave's lane: beside the stores above
    double sn, cs;
    sincos(b * dt, &sn, &cs);
    cc->phase[0] = cs;
    cc->phase[1] = -sn;
  }
  for (int k = threadIdx.x; k < K && k < kMaxTerms; k += blockDim.x) {
    const double v = (k == 0 ? 1.0 : 2.0) * (dt < 0 && (k & 1) ? -J[k] : J[k]);
    const int q = k & 3;  // (-i)^k
    cc->c[k][0] = (q == 0) ? v : (q == 2 ? -v : 0.0);
    cc->c[k][1] = (q == 1) ? -v : (q == 3 ? v : 0.0);
  }
}

// ---- Clenshaw term ----------------------------------------------------------
// y = sum_{k<K} c_k T_k(H~) phi by Clenshaw's recurrence
//   b_k = c_k phi + 2 H~ b_{k+1} - b_{k+2}   (k = K-1 .. 1),
//   y   = c_0 phi + H~ b_1 - b_2,
// with b_K = b_{K+1} = 0 and b_{K-1} = c_{K-1} phi folded into the first
// launch.  Launch kk computes b_kk into buffer kk & 1, in place over
// b_{kk+2}; launches with kk > K-2 return at once, so the host enqueues a
// fixed number of launches before K is known.  H~ = alpha H + beta; H is
// applied as an ELL SpMV whose values follow from the slot and the row
// payload.  Against the forward three-term recurrence plus an accumulator
// this streams one vector less per term.
template <typename R>
struct VecT;
template <>
struct VecT<double> {
  using T = double2;
};
template <>
struct VecT<float> {
  using T = float2;
};

// The row's off-diagonal part: hr, hi += sum_s v_s in[col_s].  In complex64
// every gather is issued before the first is used, a missing neighbour
// reading the row itself and counting as zero: a middle term of a ring of 16
// at 8.9e6 rows 116 -> 109 us, of 64 6x6 lattices with 4.07e7 rows together
// 756 -> 692 us.  In complex128, where the launch is bound by bytes, those
// reads cost more than they give (ring of 16 at 1.31e7 rows 252 -> 254 us, a
// 25-site chain at 1.63e7 346 -> 353), so there the gathers stay conditional.
template <typename R, int ND, int NV, typename Amp>
__device__ __forceinline__ void gather_row(
    const Amp* __restrict__ in, int64_t i,
    const int32_t (&cols)[2 * ND + 2 * NV], const R (&jv)[3],
    const R (&gv)[NV][2], R& hr, R& hi) {
  constexpr int D = 2 * ND + 2 * NV;
  if constexpr (sizeof(R) == 4) {
    Amp x[D];
#pragma unroll
    for (int s = 0; s < D; ++s) x[s] = in[cols[s] >= 0 ? int64_t(cols[s]) : i];
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const R v =
          s < 2 * ND ? jv[s >> 1] : gv[(s - 2 * ND) >> 1][(s - 2 * ND) & 1];
      // fused by name: without the branch the diagonal's product could be
      // fused instead, and a kernel's rounding would depend on its code
      hr = __builtin_fmaf(v, cols[s] >= 0 ? x[s].x : R(0), hr);
      hi = __builtin_fmaf(v, cols[s] >= 0 ? x[s].y : R(0), hi);
    }
  } else {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int32_t c = cols[s];
      if (c >= 0) {
        const R v =
            s < 2 * ND ? jv[s >> 1] : gv[(s - 2 * ND) >> 1][(s - 2 * ND) & 1];
        const Amp xj = in[c];
        hr += v * xj.x;
        hi += v * xj.y;
      }
    }
  }
}

// MID only names the launches the host expects to be middle terms (neither
// first nor last for the previous step's K), so that profiles can tell them
// apart; the code is the same and still decides its role from the device K.
template <typename R, int ND, int NV, bool MID>
__global__ void __launch_bounds__(kBlock)
    k_cheb_term(DevModel m, int kk, int want_energy,
                const StepCtl* __restrict__ ctl, const int* __restrict__ err,
                const int32_t* __restrict__ col, int64_t cap,
                const uint64_t* __restrict__ pay,
                const uint64_t* __restrict__ tot,
                const ChebCoef* __restrict__ cc,
                const typename VecT<R>::T* __restrict__ phi,
                typename VecT<R>::T* b0, typename VecT<R>::T* b1,
                double* e_part) {
  using Amp = typename VecT<R>::T;
  constexpr int D = 2 * ND + 2 * NV;
  if (*err) return;
  const int K = cc->K;
  if (kk > K - 2 && !(K == 1 && kk == 0)) return;
  const int64_t n = ctl->n_new;
  const bool first = (kk == K - 2) || K == 1;
  const bool fin = kk == 0;
  const bool energy = first && want_energy;
  const Amp* in = first ? phi : (((kk + 1) & 1) ? b1 : b0);
  const Amp* prev = first ? nullptr : (kk == K - 3 ? phi : ((kk & 1) ? b1 : b0));
  Amp* out = (kk & 1) ? b1 : b0;
  const R alpha = R(cc->alpha), beta = R(cc->beta);
  const R ckr = R(cc->c[kk][0]), cki = R(cc->c[kk][1]);
  const double fac = fin ? 1.0 : 2.0;
  R sir = R(fac), sii = 0;
  if (first) {
    sir = K == 1 ? R(0) : R(fac * cc->c[K - 1][0]);
    sii = K == 1 ? R(0) : R(fac * cc->c[K - 1][1]);
  }
  R spr = 1, spi = 0;
  if (kk == K - 3) {
    spr = R(cc->c[K - 1][0]);
    spi = R(cc->c[K - 1][1]);
  }
  // the final launch also applies exp(-i b dt)
  const R phr = fin ? R(cc->phase[0]) : R(1), phim = fin ? R(cc->phase[1]) : R(0);
  R jv[3] = {0, 0, 0};
#pragma unroll
  for (int a = 0; a < ND; ++a) jv[a] = R(m.J[a]);
  double esum = 0;
  for (int64_t i = gtid_xcd(); i < n; i += gstride()) {
    const Amp xi = in[i];
    const uint64_t p = ld_stream(pay + i);
    const R d = R(row_diag(m, p, NV > 2 ? ld_stream(tot + i) : 0));
    R hr = d * xi.x, hi = d * xi.y;
    R gv[NV][2];
#pragma unroll
    for (int nu = 0; nu < NV; ++nu) {
      const int occ = pay_occ(p, nu);
      gv[nu][0] = R(m.gsq[nu * kGsqStride + occ]);
      gv[nu][1] = R(m.gsq[nu * kGsqStride + occ + 1]);
    }
    int32_t cols[D];
    load_cols<D>(col + i * D, cols);
    gather_row<R, ND, NV>(in, i, cols, jv, gv, hr, hi);
    if (energy) esum += double(xi.x) * double(hr) + double(xi.y) * double(hi);
    const R tr = alpha * hr + beta * xi.x, ti = alpha * hi + beta * xi.y;
    R yr = sir * tr - sii * ti, yi = sir * ti + sii * tr;
    const Amp f = ld_stream(phi + i);
    yr += ckr * f.x - cki * f.y;
    yi += ckr * f.y + cki * f.x;
    if (prev) {
      const Amp q = ld_stream(prev + i);
      yr -= spr * q.x - spi * q.y;
      yi -= spr * q.y + spi * q.x;
    }
    Amp o;
    o.x = phr * yr - phim * yi;
    o.y = phr * yi + phim * yr;
    out[i] = o;
  }
  if (energy) {
    esum = block_sum(esum);
    if (threadIdx.x == 0) e_part[blockIdx.x] = esum;
  }
}

// Batched form of the Clenshaw launch: rows of different disorder
// realizations carry their own spectral interval, coefficients and term
// count K_r (cc_all[r]); each row takes its role from its own K_r, so a
// realization's rows do exactly the arithmetic of a single-realization run
// (neighbours of a row always belong to the same realization).  Launches
// beyond a realization's K_r leave its rows untouched.  The energy term
// <phi|H|phi> is left per row in e_row for a segmented reduction.
template <typename R, int ND, int NV>
__global__ void __launch_bounds__(kBlock)
    k_cheb_batch(DevModel m, int kk, int want_energy,
                 const StepCtl* __restrict__ ctl, const int* __restrict__ err,
                 const int32_t* __restrict__ col, int64_t cap,
                 const uint64_t* __restrict__ pay,
                 const uint64_t* __restrict__ tot,
                 const ChebCoef* __restrict__ cc_all,
                 const typename VecT<R>::T* __restrict__ phi,
                 typename VecT<R>::T* b0, typename VecT<R>::T* b1,
                 double* e_row) {
  using Amp = typename VecT<R>::T;
  constexpr int D = 2 * ND + 2 * NV;
  if (*err) return;
  const int64_t n = ctl->n_new;
  R jv[3] = {0, 0, 0};
#pragma unroll
  for (int a = 0; a < ND; ++a) jv[a] = R(m.J[a]);
  for (int64_t i = gtid_xcd(); i < n; i += gstride()) {
    const uint64_t p = ld_stream(pay + i);
    const ChebCoef* cc = cc_all + pay_real(p);
    const int K = cc->K;
    if (kk > K - 2 && !(K == 1 && kk == 0)) continue;
    const bool first = (kk == K - 2) || K == 1;
    const bool fin = kk == 0;
    const Amp* in = first ? phi : (((kk + 1) & 1) ? b1 : b0);
    const Amp* prev = first ? nullptr : (kk == K - 3 ? phi : ((kk & 1) ? b1 : b0));
    Amp* out = (kk & 1) ? b1 : b0;
    const R alpha = R(cc->alpha), beta = R(cc->beta);
    const R ckr = R(cc->c[kk][0]), cki = R(cc->c[kk][1]);
    const double fac = fin ? 1.0 : 2.0;
    R sir = R(fac), sii = 0;
    if (first) {
      sir = K == 1 ? R(0) : R(fac * cc->c[K - 1][0]);
      sii = K == 1 ? R(0) : R(fac * cc->c[K - 1][1]);
    }
    R spr = 1, spi = 0;
    if (kk == K - 3) {
      spr = R(cc->c[K - 1][0]);
      spi = R(cc->c[K - 1][1]);
    }
    const R phr = fin ? R(cc->phase[0]) : R(1), phim = fin ? R(cc->phase[1]) : R(0);
    const Amp xi = in[i];
    const R d = R(row_diag(m, p, NV > 2 ? ld_stream(tot + i) : 0));
    R hr = d * xi.x, hi = d * xi.y;
    R gv[NV][2];
#pragma unroll
    for (int nu = 0; nu < NV; ++nu) {
      const int occ = pay_occ(p, nu);
      gv[nu][0] = R(m.gsq[nu * kGsqStride + occ]);
      gv[nu][1] = R(m.gsq[nu * kGsqStride + occ + 1]);
    }
    int32_t cols[D];
    load_cols<D>(col + i * D, cols);
    gather_row<R, ND, NV>(in, i, cols, jv, gv, hr, hi);
    if (first && want_energy)
      e_row[i] = double(xi.x) * double(hr) + double(xi.y) * double(hi);
    const R tr = alpha * hr + beta * xi.x, ti = alpha * hi + beta * xi.y;
    R yr = sir * tr - sii * ti, yi = sir * ti + sii * tr;
    const Amp f = ld_stream(phi + i);
    yr += ckr * f.x - cki * f.y;
    yi += ckr * f.y + cki * f.x;
    if (prev) {
      const Amp q = ld_stream(prev + i);
      yr -= spr * q.x - spi * q.y;
      yi -= spr * q.y + spi * q.x;
    }
    Amp o;
    o.x = phr * yr - phim * yi;
    o.y = phr * yi + phim * yr;
    out[i] = o;
  }
}

// Population bins in LDS: with one realization and up to kPrivBins sites
// every lane of a wave owns a column (bin j, lane l at j*64 + l), so the
// four waves of a block meet on an address at most four at a time; other
// shapes share one bin per (realization, site).
constexpr int kPrivBins = 120;  // N * 64 + 3 doubles fit in 64 KiB
constexpr int kRegBins = 16;

// Norm, exciton populations, row counts and (batched) energy of psi per
// realization as per-block partials.  Rows are visited in the select
// kernels' tile layout, so the same pass also leaves the next step's
// selection (bits and per-block sums).  A lane reads four rows before it uses
// the first (25-site chain at 1.5e7 rows 81 -> 73 us).  Batched, a
// realization's norm is the sum of its populations, and its count and energy
// are folded by the wave where all its rows are of one realization: 64 6x6
// lattices 101 -> 53 us, most of which went to lanes waiting for their turn on
// the same LDS words.  Row counts are left per block like the norms: one
// counter that 1024 blocks add to is served at about 4 ns each (ring of 16
// 23.0 -> 19.1 us, in complex64 18.6 -> 14.3).
template <typename R>
__global__ void __launch_bounds__(kBlock)
    k_pop_norm(int N, int Rn, double th2, const StepCtl* ctl,
               const typename VecT<R>::T* psi, const uint64_t* pay,
               const uint8_t* dist,
               const double* e_row, double* n2_part, double* en_part,
               double* pop_part, uint64_t* sel_bits, uint32_t* sel_sums,
               const int* err) {
  extern __shared__ double lds[];
  if (*err) return;
  const int64_t n = ctl->n_new;
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  const bool priv = Rn == 1 && N <= kPrivBins;
  // up to kRegBins sites: each thread sums its rows' weights per site in
  // registers and adds them to its lane's LDS bins once at the end
  const bool regs = priv && N <= kRegBins;
  double acc[kRegBins];
#pragma unroll
  for (int q = 0; q < kRegBins; ++q) acc[q] = 0.0;
  const int npop = priv ? N * 64 : Rn * N;
  double* pop_lds = lds;
  double* en_lds = lds + npop;  // Rn (batched only)
  uint32_t* cnt_lds = reinterpret_cast<uint32_t*>(en_lds + Rn);  // Rn
  for (int j = threadIdx.x; j < npop; j += blockDim.x) pop_lds[j] = 0.0;
  for (int j = threadIdx.x; j < Rn; j += blockDim.x) {
    en_lds[j] = 0.0;
    cnt_lds[j] = 0u;
  }
  __syncthreads();
  double n2 = 0;
  uint32_t rows = 0, kept = 0;
  constexpr int G = 4;
  for (int64_t t = run.t0; t < run.t1; t += G) {
    typename VecT<R>::T a[G];
    uint64_t pq[G];
    double er[G];
    bool ok[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      const int64_t ec = e < n ? e : n - 1;
      a[q] = psi[ec];
      pq[q] = pay[ec];
      er[q] = e_row ? e_row[ec] : 0.0;
      ok[q] = t + q < run.t1 && e < n && !is_hole(dist, ec);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      bool keep = false;
      const uint64_t p = pq[q];
      const double w = weight(a[q]);
      if (Rn > 1) {
        const uint64_t act = __ballot(ok[q]);
        const int r = pay_real(p);
        if (ok[q]) atomicAdd(&pop_lds[r * N + pay_site(p)], w);
        if (act != 0) {
          const int r0 = __shfl(r, __ffsll((unsigned long long)act) - 1);
          if (__ballot(ok[q] && r != r0) == 0) {
            const double ew = e_row ? wave_sum(ok[q] ? er[q] : 0.0) : 0.0;
            if ((threadIdx.x & 63) == 0) {
              atomicAdd(&cnt_lds[r0], uint32_t(__popcll(act)));
              if (e_row) atomicAdd(&en_lds[r0], ew);
            }
          } else if (ok[q]) {
            atomicAdd(&cnt_lds[r], 1u);
            if (e_row) atomicAdd(&en_lds[r], er[q]);
          }
        }
      }
      if (ok[q]) {
        keep = w >= th2;
        if (Rn == 1) {
          n2 += w;
          ++rows;
          if (regs) {
            const int j = pay_site(p);
#pragma unroll
            for (int q = 0; q < kRegBins; ++q) acc[q] += q == j ? w : 0.0;
          } else if (priv) {
            atomicAdd(&pop_lds[pay_site(p) * 64 + (threadIdx.x & 63)], w);
          } else {
            atomicAdd(&pop_lds[pay_site(p)], w);
          }
        }
      }
      put_bits(sel_bits, e, n, keep);
      kept += keep ? 1u : 0u;
    }
  }
  {
    uint32_t tot;
    block_excl_scan(kept, &tot);
    if (threadIdx.x == 0) sel_sums[blockIdx.x] = tot;
  }
  if (regs) {
#pragma unroll
    for (int q = 0; q < kRegBins; ++q)
      if (q < N) atomicAdd(&pop_lds[q * 64 + (threadIdx.x & 63)], acc[q]);
  }
  if (Rn == 1) {
    n2 = block_sum(n2);
    uint32_t all;
    block_excl_scan(rows, &all);
    if (threadIdx.x == 0) {
      n2_part[blockIdx.x] = n2;
      n2_part[kPopBlocks + blockIdx.x] = double(all);
    }
    __syncthreads();
    if (priv) {
      for (int j = threadIdx.x >> 6; j < N; j += kBlock / 64) {
        const double v = wave_sum(pop_lds[j * 64 + (threadIdx.x & 63)]);
        if ((threadIdx.x & 63) == 0) pop_part[int64_t(blockIdx.x) * N + j] = v;
      }
    } else {
      for (int j = threadIdx.x; j < N; j += blockDim.x)
        pop_part[int64_t(blockIdx.x) * N + j] = pop_lds[j];
    }
  } else {
    __syncthreads();
    for (int r = threadIdx.x; r < Rn; r += blockDim.x) {
      double n2r = 0;
      for (int j = 0; j < N; ++j) n2r += pop_lds[r * N + j];
      n2_part[int64_t(blockIdx.x) * Rn + r] = n2r;
      en_part[int64_t(blockIdx.x) * Rn + r] = en_lds[r];
      n2_part[int64_t(kPopBlocks + blockIdx.x) * Rn + r] = double(cnt_lds[r]);
    }
    for (int j = threadIdx.x; j < Rn * N; j += blockDim.x)
      pop_part[int64_t(blockIdx.x) * Rn * N + j] = pop_lds[j];
  }
}

// ---- observation record -----------------------------------------------------
// Commit of a step on the device: time, cumulative discarded weight per
// realization, record count and the row count of the current set.  The
// counts and the error latch are mirrored into mapped pinned host memory, so
// the host reads them after one stream synchronisation without copy
// dispatches.
__device__ __forceinline__ void close_step(StepCtl* ctl, int Rn,
                                           const double* ring, int rec_doubles,
                                           double* mass_tot, int e,
                                           uint32_t* h_ctl, int* h_err) {
  if (!e) {
    const double* rec = ring + int64_t(ctl->nrec) * Rn * rec_doubles;
    for (int r = threadIdx.x; r < Rn; r += blockDim.x)
      mass_tot[r] = rec[int64_t(r) * rec_doubles + 6];
    __syncthreads();
    if (threadIdx.x == 0) {
      ctl->t = rec[0];
      ctl->n_old = ctl->n_new;
      ctl->nrec += 1;
    }
  }
  __syncthreads();
  const uint32_t* src = reinterpret_cast<const uint32_t*>(ctl);
  for (int i = threadIdx.x; i < int(sizeof(StepCtl) / 4); i += blockDim.x)
    h_ctl[i] = src[i];
  if (threadIdx.x == 0) *h_err = e;
  __threadfence_system();
}

// Sum of n partials at a stride, up to 32 loads in flight per lane: the block
// that adds up the Clenshaw launch's up to 16384 of them waits for memory
// twice (with eight in flight 8 times: a record of the 25-site chain 25 -> 9
// us, of a ring of 16 at 0.5 to 1e7 rows 14.3 -> 8.1).
__device__ __forceinline__ double sum_partials(const double* p, int n,
                                               int64_t stride) {
  double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int i = threadIdx.x;
  for (; i + 31 * kBlock < n; i += 32 * kBlock) {
    double v[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) v[q] = p[int64_t(i + q * kBlock) * stride];
#pragma unroll
    for (int q = 0; q < 32; ++q) a[q & 7] += v[q];
  }
  for (; i < n; i += 8 * kBlock) {
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = i + q * kBlock;
      v[q] = p[int64_t(j < n ? j : i) * stride];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] += i + q * kBlock < n ? v[q] : 0.0;
  }
  return block_sum(((a[0] + a[1]) + (a[2] + a[3])) +
                   ((a[4] + a[5]) + (a[6] + a[7])));
}

// Blocks of the record per realization beside its N populations: norm and
// row counts, energy, discarded weight, <psi0|psi(t)>.
constexpr int kObsBlocks = 4;

// Share of block (x, r) in the records: x < N reduces population (r, x), the
// others a scalar each of realization r (<psi0|psi(t)> over its n0 initial
// states, rows p0); each folds the per-block partials with a fixed lane
// mapping.  Records of one step are stored realization after realization.
template <typename Amp>
__device__ __forceinline__ void obs_block(
    int N, int Rn, int want_energy, double dt, int n_mass, int n_e, int n_pop,
    const double* mass_part, const double* n2_part, const double* e_part,
    const double* en_part, const double* pop_part, const double* amps0,
    int64_t n0, const int32_t* p0, const Amp* psi, const ChebCoef* cc,
    const StepCtl* ctl, const uint32_t* cnt, const double* mass_tot,
    double* ring, int rec_doubles, int* err) {
  const int r = blockIdx.y, what = int(blockIdx.x) - N;
  double* rec = ring + (int64_t(ctl->nrec) * Rn + r) * rec_doubles;
  if (what < 0) {
    const double s = sum_partials(pop_part + int64_t(r) * N + blockIdx.x,
                                  n_pop, int64_t(Rn) * N);
    if (threadIdx.x == 0) rec[kObsFields + blockIdx.x] = s;
  } else if (what == 0) {
    const double n2 = sum_partials(n2_part + r, n_pop, Rn);
    const double rows =
        sum_partials(n2_part + int64_t(kPopBlocks) * Rn + r, n_pop, Rn);
    if (threadIdx.x == 0) {
      rec[0] = ctl->t + dt;
      rec[1] = n2;
      rec[7] = rows;
      rec[8] = double(cnt[r]);
      rec[9] = double(cc[r].K);
      rec[10] = cc[r].emin;
      rec[11] = cc[r].emax;
      if (!isfinite(n2)) atomicOr(err, kErrNonFinite);
    }
  } else if (what == 1) {
    double en = NAN;
    if (want_energy)
      en = Rn == 1 ? sum_partials(e_part, n_e, 1)
                   : sum_partials(en_part + r, n_pop, Rn);
    if (threadIdx.x == 0) rec[2] = en;
  } else if (what == 2) {
    const double ms = sum_partials(mass_part + r, n_mass, Rn);
    if (threadIdx.x == 0) {
      rec[5] = ms;
      rec[6] = mass_tot[r] + ms;
    }
  } else {
    double re = 0, im = 0;
    const int64_t base = int64_t(r) * n0;
    for (int64_t i = base + threadIdx.x; i < base + n0; i += blockDim.x) {
      const int32_t row = p0[i];
      if (row < 0) continue;
      const double2 v = widen(psi[row]);
      const double ar = amps0[2 * i], ai = amps0[2 * i + 1];
      re += ar * v.x + ai * v.y;  // conj(a0) * v
      im += ar * v.y - ai * v.x;
    }
    re = block_sum(re);
    im = block_sum(im);
    if (threadIdx.x == 0) {
      rec[3] = re;
      rec[4] = im;
    }
  }
}

// h_ctl given (one realization): the block that arrives last closes the
// step.  The sums of the weight and energy partials, <psi0|psi> and the close
// were four launches of their own before, 3-5 us each.
template <typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_obs_final(int N, int Rn, int want_energy, double dt, int n_mass, int n_e,
                int n_pop, const double* mass_part, const double* n2_part,
                const double* e_part, const double* en_part,
                const double* pop_part, const double* amps0, int64_t n0,
                const int32_t* p0, const Amp* psi, const ChebCoef* cc,
                StepCtl* ctl, const uint32_t* cnt, double* mass_tot,
                double* ring, int rec_doubles, int64_t ring_cap,
                uint32_t* h_ctl, int* h_err, int* err) {
  __shared__ int latch;
  if (threadIdx.x == 0) latch = *err;
  __syncthreads();
  if (!latch && int64_t(ctl->nrec) + 1 <= ring_cap)  // the host keeps room
    obs_block(N, Rn, want_energy, dt, n_mass, n_e, n_pop, mass_part, n2_part,
              e_part, en_part, pop_part, amps0, n0, p0, psi, cc, ctl, cnt,
              mass_tot, ring, rec_doubles, err);
  // every block arrives, also when something is latched
  if (h_ctl && last_block(&ctl->ticket, gridDim.x * gridDim.y)) {
    if (threadIdx.x == 0) latch = latch_now(err);
    __syncthreads();
    close_step(ctl, Rn, ring, rec_doubles, mass_tot, latch, h_ctl, h_err);
  }
}

__global__ void __launch_bounds__(kBlock)
    k_end_step(StepCtl* ctl, int Rn, const double* ring, int rec_doubles,
               double* mass_tot, const int* err, uint32_t* h_ctl, int* h_err) {
  close_step(ctl, Rn, ring, rec_doubles, mass_tot, *err, h_ctl, h_err);
}

// ---- precision conversion ---------------------------------------------------
__global__ void __launch_bounds__(kBlock)
    k_f32_to_f64(const float2* src, double* dst, int64_t n) {
  for (int64_t i = gtid(); i < n; i += gstride()) {
    dst[2 * i] = src[i].x;
    dst[2 * i + 1] = src[i].y;
  }
}
__global__ void __launch_bounds__(kBlock)
    k_f64_to_f32(const double* src, float2* dst, int64_t n) {
  for (int64_t i = gtid(); i < n; i += gstride())
    dst[i] = make_float2(float(src[2 * i]), float(src[2 * i + 1]));
}

}  // namespace

// ============================================================================
// host wrappers
// ============================================================================
int supported_words(int W) {
  static const int ws[] = {1, 2, 3, 4, 6, 8, 10, 16};
  for (int w : ws)
    if (w >= W) return w;
  return 0;
}

int64_t sel_bit_words(int64_t n) { return cdiv(n, 64) + 1; }

void fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s) {
  if (n <= 0) return;
  k_fill_u64<<<grid_for(n), kBlock, 0, s>>>(p, n, v);
}

void mark(int tag, hipStream_t s) { k_mark<<<1, 64, 0, s>>>(tag); }

void clear_latch(StepCtl* ctl, int* err, hipStream_t s) {
  k_clear_err<<<1, 1, 0, s>>>(err, ctl);
}

void report(const StepCtl* ctl, const int* err, uint32_t* out,
            hipStream_t s) {
  k_report<<<1, 1, 0, s>>>(ctl, err, out);
}

void pad_keys(int W, int Wi, const uint64_t* in, uint64_t* out, int64_t n,
              hipStream_t s) {
  if (n <= 0) return;
  k_pad_keys<<<grid_for(n * Wi), kBlock, 0, s>>>(W, Wi, in, out, n);
}

void build_set(const DevModel& m, int Wi, const Side& n, int64_t rows,
               StepCtl* ctl, uint64_t* table, uint64_t mask, int32_t* col,
               int* err, hipStream_t s) {
  const int64_t slots = int64_t(mask) + 1;
  k_set_begin<<<grid_for(slots), kBlock, 0, s>>>(ctl, err, uint32_t(rows),
                                                 table, slots);
  PACES_DISPATCH_W(Wi, k_set_rows<WW><<<grid_for(rows), kBlock, 0, s>>>(
                           m, n.keys, rows, n.pay, n.tot, col, table, mask,
                           err));
  PACES_DISPATCH_W(
      Wi, k_set_cols<WW><<<grid_for(rows * m.D / 2), kBlock, 0, s>>>(
              m, n.keys, n.pay, rows, table, mask, col, err));
}

void begin_step(StepCtl* ctl, int* err, uint32_t* cnt, uint32_t* ball, int R,
                hipStream_t s) {
  k_begin_step<<<1, kBlock, 0, s>>>(ctl, err, cnt, ball, R);
}

int select_bits(int prec, const void* psi, const uint8_t* dist, double th2,
                const StepCtl* ctl, const Sums& sm, int64_t n, hipStream_t s) {
  const int g = sum_grid(n, kBlock);
  if (prec == 64)
    k_select_bits<double2><<<g, kBlock, 0, s>>>((const double2*)psi, dist, ctl,
                                                th2, sm.bits, sm.sel);
  else
    k_select_bits<float2><<<g, kBlock, 0, s>>>((const float2*)psi, dist, ctl,
                                               th2, sm.bits, sm.sel);
  return g;
}

int flag_bits(const uint8_t* keep, const StepCtl* ctl, const Sums& sm,
              int64_t n, hipStream_t s) {
  const int g = sum_grid(n, kBlock);
  k_flag_bits<<<g, kBlock, 0, s>>>(keep, ctl, sm.bits, sm.sel);
  return g;
}

void select_write(StepCtl* ctl, const Sums& sm, int grid, uint32_t* midx,
                  const int* err, hipStream_t s) {
  k_select_write<<<grid, kBlock, 0, s>>>(sm.bits, ctl, sm.sel, midx, err);
}

void select_all(StepCtl* ctl, uint32_t* midx, int64_t n, hipStream_t s) {
  k_select_all<<<grid_for(n), kBlock, 0, s>>>(ctl, midx);
}

void insert_rows(const DevModel& m, int Wi, int prec, const Side& o,
                 const Side& n, const uint32_t* midx, const StepCtl* ctl,
                 int64_t bound, uint64_t* table, uint64_t mask,
                 uint32_t* cnt_m, const void* psi_o, void* phi, int* err,
                 hipStream_t s) {
  const int g = grid_for(bound);
  if (prec == 64) {
    PACES_DISPATCH_W(Wi, k_insert_rows<WW, double2><<<g, kBlock, 0, s>>>(
                             m, o.keys, o.pay, o.tot, midx, &ctl->nM, 0,
                             n.keys, n.pay, n.tot, n.dist, table, mask, cnt_m,
                             (const double2*)psi_o, (double2*)phi, err));
  } else {
    PACES_DISPATCH_W(Wi, k_insert_rows<WW, float2><<<g, kBlock, 0, s>>>(
                             m, o.keys, o.pay, o.tot, midx, &ctl->nM, 0,
                             n.keys, n.pay, n.tot, n.dist, table, mask, cnt_m,
                             (const float2*)psi_o, (float2*)phi, err));
  }
}

void rehash_rows(const DevModel& m, int Wi, const Side& n, int64_t rows,
                 uint64_t* table, uint64_t mask, int* err, hipStream_t s) {
  if (rows <= 0) return;
  PACES_DISPATCH_W(Wi, k_insert_rows<WW, double2><<<grid_for(rows), kBlock, 0, s>>>(
                           m, nullptr, nullptr, nullptr, nullptr, nullptr,
                           rows, n.keys, n.pay, n.tot, n.dist, table, mask,
                           nullptr, nullptr, nullptr, err));
}

void expand_round(const DevModel& m, int Wi, int prec, const Side& n, int r,
                  StepCtl* ctl, int64_t cap, int64_t est, uint64_t* table,
                  uint64_t mask, const RoundBufs& rb, const Sums& sm,
                  int32_t* col, void* phi, int chunks, int64_t row_limit,
                  int64_t load_rows, int* err, hipStream_t s) {
  const int g = sum_grid(std::min<int64_t>(rb.cand_cap, est * m.D), kBlock);
  for (int q = 0; q < chunks; ++q) {
    const int last = q == chunks - 1 ? 1 : 0;
    PACES_DISPATCH_W(Wi, k_expand_probe<WW><<<g, kBlock, 0, s>>>(
                             m, n.keys, n.pay, ctl, r, q, last, rb.cand_cap,
                             row_limit, table, mask, rb.c_slot, rb.c_ref,
                             rb.tile_base, sm.own, col, err));
    if (prec == 64) {
      PACES_DISPATCH_W(Wi, k_expand_commit<WW, double2><<<g, kBlock, 0, s>>>(
                               m, n, ctl, r, q, last, rb.cand_cap, cap,
                               load_rows, table, mask, rb.c_slot, rb.c_ref,
                               rb.tile_base, sm.own, col, (double2*)phi, err));
    } else {
      PACES_DISPATCH_W(Wi, k_expand_commit<WW, float2><<<g, kBlock, 0, s>>>(
                               m, n, ctl, r, q, last, rb.cand_cap, cap,
                               load_rows, table, mask, rb.c_slot, rb.c_ref,
                               rb.tile_base, sm.own, col, (float2*)phi, err));
    }
  }
}

void lookup_last(const DevModel& m, int Wi, const Side& n, int k,
                 StepCtl* ctl, int64_t est, const uint64_t* table,
                 uint64_t mask, int32_t* col, int64_t max_states,
                 uint32_t* ball, const uint64_t* keys0, int64_t n0,
                 int32_t* p0, int* err, hipStream_t s) {
  PACES_DISPATCH_W(Wi, k_lookup_cols<WW><<<grid_for(est * m.D), kBlock, 0, s>>>(
                           m, n.keys, n.pay, ctl, k, table, mask, col,
                           max_states, ball, keys0, n0, p0, err));
}

int part_grid(int64_t rows) { return grid_for(rows); }

int transfer(const DevModel& m, int Wi, int prec, const Side& o,
             const void* psi_o, int64_t n_old, const StepCtl* ctl,
             const uint64_t* table, uint64_t mask, const uint64_t* keys_n,
             void* phi, double* mass_part, int32_t* tmap, const uint64_t* sel,
             int* err, hipStream_t s) {
  const int g = m.R > 1 ? std::min(grid_for(n_old), kPartBlocks) : grid_for(n_old);
  if (prec == 64) {
    PACES_DISPATCH_W(Wi, k_transfer<WW, double2><<<g, kBlock, 0, s>>>(
                             m, o.keys, o.dist, (const double2*)psi_o, ctl, table, mask,
                             keys_n, (double2*)phi, mass_part, tmap, sel, err));
  } else {
    PACES_DISPATCH_W(Wi, k_transfer<WW, float2><<<g, kBlock, 0, s>>>(
                             m, o.keys, o.dist, (const float2*)psi_o, ctl, table, mask,
                             keys_n, (float2*)phi, mass_part, tmap, sel, err));
  }
  return g;
}

namespace {
void launch_bounds_kernel(const DevModel& m, const Side& n, const int32_t* col,
                          int64_t cap, int g, const StepCtl* ctl, double* part,
                          const int* err, hipStream_t s) {
  PACES_DISPATCH_SHAPE(m.ndim, m.V, k_bounds<A, B><<<g, kBlock, 0, s>>>(
      m, n.pay, n.tot, n.dist, col, cap, ctl, part, err));
}
}  // namespace

int bounds_part(const DevModel& m, const Side& n, const int32_t* col,
                int64_t cap, int64_t est, const StepCtl* ctl, double* part,
                const int* err, hipStream_t s) {
  const int g = std::min(grid_for(est), kPartBlocks);
  launch_bounds_kernel(m, n, col, cap, g, ctl, part, err, s);
  return g;
}

void bounds_and_coef(const DevModel& m, const Side& n, const int32_t* col,
                     int64_t cap, int64_t est, StepCtl* ctl, double dt,
                     double tol, int k_max, int launched, double* part,
                     ChebCoef* cc, int* err, hipStream_t s) {
  // a bounded grid: each block reduces many rows, and k_coef folds few
  // partials
  const int g = std::min(grid_for(est), kPartBlocks);
  launch_bounds_kernel(m, n, col, cap, g, ctl, part, err, s);
  k_coef<<<m.R, kBlock, 0, s>>>(part, g, m.R, dt, tol, k_max, launched, cc,
                                ctl, err);
}

int cheb_term(const DevModel& m, int prec, int kk, bool energy, bool mid,
              int64_t est, const StepCtl* ctl, const int32_t* col, int64_t cap,
              const Side& n, const ChebCoef* cc, const void* phi, void* b0,
              void* b1, double* e_part, double* e_row, int* err,
              hipEvent_t ev_a, hipEvent_t ev_b, hipStream_t s) {
  const int e = energy ? 1 : 0;
  const int g = grid_for(est);
  if (m.R > 1) {
    if (prec == 64) {
      PACES_DISPATCH_SHAPE(m.ndim, m.V,
          launch_ev(k_cheb_batch<double, A, B>, g, s, ev_a, ev_b,
                    m, kk, e, ctl, err, col, cap, n.pay, n.tot, cc,
                    (const double2*)phi, (double2*)b0, (double2*)b1, e_row));
    } else {
      PACES_DISPATCH_SHAPE(m.ndim, m.V,
          launch_ev(k_cheb_batch<float, A, B>, g, s, ev_a, ev_b,
                    m, kk, e, ctl, err, col, cap, n.pay, n.tot, cc,
                    (const float2*)phi, (float2*)b0, (float2*)b1, e_row));
    }
    return g;
  }
#define PACES_TERM(R, AMP, MIDV)                                              \
  PACES_DISPATCH_SHAPE(m.ndim, m.V,                                           \
      launch_ev(k_cheb_term<R, A, B, MIDV>, g, s, ev_a, ev_b,                 \
                m, kk, e, ctl, err, col, cap, n.pay, n.tot, cc,               \
                (const AMP*)phi, (AMP*)b0, (AMP*)b1, e_part))
  if (prec == 64) {
    if (mid) { PACES_TERM(double, double2, true); } else { PACES_TERM(double, double2, false); }
  } else {
    if (mid) { PACES_TERM(float, float2, true); } else { PACES_TERM(float, float2, false); }
  }
#undef PACES_TERM
  return g;
}

int pop_norm(int prec, int N, int R, double th2, int64_t est,
             const StepCtl* ctl, const void* psi, const uint64_t* pay,
             const uint8_t* dist,
             const double* e_row, double* n2_part, double* en_part,
             double* pop_part, const Sums& sm, int* err, hipStream_t s) {
  const bool priv = R == 1 && N <= kPrivBins;
  const size_t lds = sizeof(double) * ((priv ? N * 64 : R * N) + 2 * R);
  // a bounded grid: blocks stride over the tiles, so the per-block work (bins
  // cleared and folded, R * N partials written) is amortised
  const int g = std::min(sum_grid(est, kBlock), kPopBlocks);
  if (prec == 64)
    k_pop_norm<double><<<g, kBlock, lds, s>>>(
        N, R, th2, ctl, (const double2*)psi, pay, dist, e_row, n2_part, en_part,
        pop_part, sm.bits, sm.sel, err);
  else
    k_pop_norm<float><<<g, kBlock, lds, s>>>(
        N, R, th2, ctl, (const float2*)psi, pay, dist, e_row, n2_part, en_part,
        pop_part, sm.bits, sm.sel, err);
  return g;
}

void end_step(StepCtl* ctl, int R, const double* ring, int rec_doubles,
              double* mass_tot, int* err, StepCtl* h_ctl_dev, int* h_err_dev,
              hipStream_t s) {
  static_assert(sizeof(StepCtl) % 4 == 0, "StepCtl is copied as 32-bit words");
  k_end_step<<<1, kBlock, 0, s>>>(ctl, R, ring, rec_doubles, mass_tot, err,
                                  reinterpret_cast<uint32_t*>(h_ctl_dev),
                                  h_err_dev);
}

void obs_final(int prec, int N, int R, int want_energy, double dt, int n_mass,
               int n_e, int n_pop, const double* mass_part,
               const double* n2_part, const double* e_part,
               const double* en_part, const double* pop_part,
               const double* amps0, int64_t n0, const int32_t* p0,
               const void* psi, const ChebCoef* cc, StepCtl* ctl,
               const uint32_t* cnt, double* mass_tot, double* ring,
               int rec_doubles, int64_t ring_cap, StepCtl* h_ctl_dev,
               int* h_err_dev, int* err, hipStream_t s) {
#define PACES_OBS(AMP)                                                        \
  k_obs_final<AMP><<<dim3(N + kObsBlocks, R), kBlock, 0, s>>>(                \
      N, R, want_energy, dt, n_mass, n_e, n_pop, mass_part, n2_part, e_part,  \
      en_part, pop_part, amps0, n0, p0, (const AMP*)psi, cc, ctl, cnt,        \
      mass_tot, ring, rec_doubles, ring_cap,                                  \
      reinterpret_cast<uint32_t*>(h_ctl_dev), h_err_dev, err)
  if (prec == 64)
    PACES_OBS(double2);
  else
    PACES_OBS(float2);
#undef PACES_OBS
}

void row_info(const DevModel& m, int Wi, const uint64_t* keys, int64_t n,
              uint64_t* pay, uint64_t* tot, hipStream_t s) {
  if (n <= 0) return;
  PACES_DISPATCH_W(Wi, k_row_info<WW><<<grid_for(n), kBlock, 0, s>>>(
                           m, keys, n, pay, tot));
}

void amps_to_f64(int prec, const void* src, double* dst, int64_t n,
                 hipStream_t s) {
  if (n <= 0) return;
  if (prec == 64)
    (void)hipMemcpyAsync(dst, src, size_t(n) * 16, hipMemcpyDeviceToDevice, s);
  else
    k_f32_to_f64<<<grid_for(n), kBlock, 0, s>>>((const float2*)src, dst, n);
}
void amps_from_f64(int prec, const double* src, void* dst, int64_t n,
                   hipStream_t s) {
  if (n <= 0) return;
  if (prec == 64)
    (void)hipMemcpyAsync(dst, src, size_t(n) * 16, hipMemcpyDeviceToDevice, s);
  else
    k_f64_to_f32<<<grid_for(n), kBlock, 0, s>>>(src, (float2*)dst, n);
}

}  // namespace paces
