// warm.hip -- the in-place step from the previous step's graph on gfx950
// (the method and its invariants are described in warm.hpp).
//
// The search inside the set streams the rows' distance bytes and the
// columns of the frontier rows; only slots that leave the set, and the slots
// of states new to it, reach the hash table.  Found states are numbered in
// the order of their candidates.  A round is three launches, and one more
// before the first; its counts stay per block between them (common.hpp), and
// every block adds up what it needs.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "warm.hpp"
#include "warm_device.hpp"

namespace paces {

namespace {

// ---- rows by distance byte --------------------------------------------------
// The search finds its rows by their distance bytes.  A block takes tiles of
// kBlock * vb rows, vb bytes per lane in one load, and collects the matching
// rows of a tile in LDS in ascending order; then every lane works on a listed
// row.  With one row per lane and iteration (one byte load each, most of them
// not matching) the four rounds of a ring16 step at 1.5e7 rows took 340 us.
constexpr int kMaxVb = 16;

// Bit 8b+7 of the result is set where byte b of x equals d.
__device__ __forceinline__ uint32_t match4(uint32_t x, uint8_t d) {
  x ^= uint32_t(d) * 0x01010101u;
  x = ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);
  x >>= 7;
  return (x & 1u) | ((x >> 7) & 2u) | ((x >> 14) & 4u) | ((x >> 21) & 8u);
}

// Which of the rows [e0, e0 + vb), e0 a multiple of vb, below n have
// distance byte d.
__device__ __forceinline__ uint32_t match_rows(const uint8_t* dist, int64_t e0,
                                               int64_t n, int vb, uint8_t d) {
  if (e0 >= n) return 0u;
  uint32_t hit;
  if (vb == 16) {
    const uint4 v = *reinterpret_cast<const uint4*>(dist + e0);
    hit = match4(v.x, d) | (match4(v.y, d) << 4) | (match4(v.z, d) << 8) |
          (match4(v.w, d) << 12);
  } else if (vb == 4) {
    hit = match4(*reinterpret_cast<const uint32_t*>(dist + e0), d);
  } else {
    hit = dist[e0] == d ? 1u : 0u;
  }
  const int64_t left = n - e0;
  return left < vb ? hit & ((1u << left) - 1u) : hit;
}

// The tile's rows (from row t * kBlock * vb on) with distance byte d, as
// offsets in the tile, ascending, into list (LDS); returns their number.
// Ends with a barrier.
__device__ __forceinline__ uint32_t list_rows(const uint8_t* dist, int64_t t,
                                              int64_t n, int vb, uint8_t d,
                                              uint16_t* list) {
  uint32_t hit = match_rows(dist, (t * kBlock + threadIdx.x) * vb, n, vb, d);
  uint32_t tot;
  uint32_t off = block_excl_scan(__popc(hit), &tot);
  while (hit) {
    const int b = __ffs(hit) - 1;
    hit &= hit - 1;
    list[off++] = uint16_t(threadIdx.x * vb + b);
  }
  __syncthreads();
  return tot;
}

// vb 16 for sets that put four tiles of 4096 rows on every CU, 4 and 1 below:
// what a lane does with a listed row is a chain of two or three dependent
// loads, so the work is spread over as many waves as the chip holds.  (With 16
// from one tile per CU on, the search of a ring16 step at 1e6..4e6 rows ran on
// two waves per SIMD.)
inline int rows_per_lane(int64_t n) {
  return n >= int64_t(kBlock) * 16 * 1024 ? 16 : n >= kBlock * 4 * 128 ? 4 : 1;
}

// ---- start ------------------------------------------------------------------
// Distance bytes of the step from the selection's bits: 0 on M, kFar on the
// other live rows, kHole kept; 16 rows per lane.  (Bytes past n_old of the
// last group belong to rows past the range, which a step writes before
// reading.)  |M| from the selection's sums, per realization by counting; the
// holes of each block into hole_sums (null: the set has none).  This took
// three launches before (fill, index list, mark).
__global__ void __launch_bounds__(kBlock)
    k_warm_select(DevModel m, StepCtl* ctl, const uint64_t* bits,
                  const uint32_t* sel_sums, int sel_grid, const uint64_t* pay,
                  uint8_t* dist, uint32_t* cnt_m, uint32_t* hole_sums,
                  const int* err) {
  __shared__ uint32_t bins[kMaxReal];
  if (*err) return;
  if (m.R > 1) {
    for (int r = threadIdx.x; r < m.R; r += blockDim.x) bins[r] = 0;
    __syncthreads();
  }
  const int64_t n = ctl->n_old;
  const TileRun run = tile_run(cdiv(n, kBlock * 16), gridDim.x);
  uint32_t holes = 0;
  for (int64_t t = run.t0; t < run.t1; ++t) {
    const int64_t e0 = (t * kBlock + threadIdx.x) * 16;
    if (e0 >= n) continue;
    const uint4 v = *reinterpret_cast<const uint4*>(dist + e0);
    uint32_t sel = reinterpret_cast<const uint16_t*>(bits)[e0 >> 4];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4], hmask = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t hole = match4(w[q], kHole);
      hmask |= hole << (4 * q);
      uint32_t x = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t byte = (hole >> b) & 1u             ? kHole
                              : (sel >> (4 * q + b)) & 1u ? 0u
                                                          : uint32_t(kFar);
        x |= byte << (8 * b);
      }
      o[q] = x;
    }
    *reinterpret_cast<uint4*>(dist + e0) = make_uint4(o[0], o[1], o[2], o[3]);
    const int64_t left = n - e0;
    holes += __popc(left < 16 ? hmask & ((1u << left) - 1u) : hmask);
    if (m.R > 1)
      while (sel) {
        const int b = __ffs(sel) - 1;
        sel &= sel - 1;
        atomicAdd(&bins[pay_real(pay[e0 + b])], 1u);
      }
  }
  if (hole_sums) {
    uint32_t tot;
    block_excl_scan(holes, &tot);
    if (threadIdx.x == 0) hole_sums[blockIdx.x] = tot;
  }
  if (blockIdx.x == 0) {
    uint64_t total;
    sums_before(sel_sums, sel_grid, 0, &total);
    if (threadIdx.x == 0) {
      ctl->nM = uint32_t(total);
      if (m.R == 1) cnt_m[0] = uint32_t(total);
    }
  }
  if (m.R > 1) count_flush(m.R, bins, cnt_m);
}

// The holes ascending (same grid as k_warm_select).
__global__ void __launch_bounds__(kBlock)
    k_warm_holes(StepCtl* ctl, const uint8_t* dist, const uint32_t* sums,
                 uint32_t* freel, const int* err) {
  __shared__ uint16_t list[kBlock * kMaxVb];
  if (*err) return;
  const int64_t n = ctl->n_old;
  const TileRun run = tile_run(cdiv(n, kBlock * 16), gridDim.x);
  uint64_t total;
  uint64_t at = sums_before(sums, gridDim.x, blockIdx.x, &total);
  if (gtid() == 0) ctl->nfree = uint32_t(total);
  for (int64_t t = run.t0; t < run.t1; ++t) {
    const uint32_t tot = list_rows(dist, t, n, 16, kHole, list);
    for (uint32_t i = threadIdx.x; i < tot; i += kBlock)
      freel[at + i] = uint32_t(t * kBlock * 16 + list[i]);
    at += tot;
  }
}

// Rows of [0, n) with a given distance byte (d >= 0) or live (d < 0),
// counted per block in the select layout, then written in row order.
__device__ __forceinline__ bool dist_hit(uint8_t v, int d) {
  return d < 0 ? v != kHole : v == uint8_t(d);
}

__global__ void __launch_bounds__(kBlock)
    k_dist_count(const uint8_t* dist, int64_t n, int d, uint32_t* sums) {
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  uint32_t v = 0;
  for (int64_t t = run.t0; t < run.t1; t += kItems) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      if (e < n && dist_hit(dist[e], d)) ++v;
    }
  }
  uint32_t tot;
  block_excl_scan(v, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kBlock)
    k_dist_write(int Wi, const uint64_t* keys, const uint8_t* dist, int64_t n,
                 int d, const uint32_t* sums, uint32_t* count, uint64_t* out,
                 uint32_t* rows) {
  const TileRun run = tile_run(cdiv(n, kBlock), gridDim.x);
  uint64_t total;
  uint64_t at = sums_before(sums, gridDim.x, blockIdx.x, &total);
  if (gtid() == 0) *count = uint32_t(total);
  for (int64_t t = run.t0; t < run.t1; t += kItems) {
#pragma unroll 1
    for (int q = 0; q < kItems; ++q) {
      if (t + q >= run.t1) break;
      const int64_t e = (t + q) * kBlock + threadIdx.x;
      const bool hit = e < n && dist_hit(dist[e], d);
      uint32_t tot;
      const uint64_t off = block_excl_scan(hit ? 1u : 0u, &tot) + at;
      at += tot;
      if (!hit) continue;
      if (rows) rows[off] = uint32_t(e);
      if (out)
        for (int w = 0; w < Wi; ++w) out[off * Wi + w] = keys[e * Wi + w];
    }
  }
}

// ---- a round ----------------------------------------------------------------
// Live rows at distance r-1.  Count pass: columns mark their rows at
// distance r (unless nearer; every writer writes r, and no row at distance
// r-1 is written in round r), the slots whose neighbour lies outside the set
// go to wmask and are counted per block.  Holes and found states never match
// r-1.  Bound by the latency of a row's chain (listed offset, columns,
// neighbours' distances): a lane takes U rows at once, and the distances of
// all their neighbours are asked for before one is looked at (a missing
// neighbour reads the row itself).  Together with rows_per_lane this took 604
// of these launches on a ring of 16 (0.5 to 2.3 million rows) from 13.4 to 6.9
// ms, on 64 6x6 lattices (D = 6) from 58 to 33 us each, on the aggregate (D =
// 8) from 62 to 33.
template <int D>
__device__ __forceinline__ void count_part(
    const DevModel& m, int r, int vb, int block, int grid, const StepCtl* ctl,
    const uint64_t* pay, const int32_t* col, uint8_t* dist, uint16_t* wmask,
    uint32_t* sums) {
  constexpr int U = D <= 4 ? 4 : D <= 8 ? 2 : 1;
  __shared__ uint16_t list[kBlock * kMaxVb];
  const int64_t n = ctl->n_old, tile = int64_t(kBlock) * vb;
  const TileRun run = tile_run(cdiv(n, tile), grid, block);
  uint32_t cnt = 0;
  for (int64_t t = run.t0; t < run.t1; ++t) {
    const uint32_t tot = list_rows(dist, t, n, vb, uint8_t(r - 1), list);
    for (uint32_t i = threadIdx.x; i < tot; i += U * kBlock) {
      int64_t e[U];
      uint64_t p[U];
      int32_t cs[U][D];
      uint8_t ds[U][D];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t x = i + u * kBlock;
        e[u] = t * tile + list[x < tot ? x : i];
        p[u] = pay[e[u]];
        load_cols<D>(col + e[u] * D, cs[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int s = 0; s < D; ++s)
          ds[u][s] = dist[cs[u][s] >= 0 ? int64_t(cs[u][s]) : e[u]];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i + u * kBlock >= tot) continue;
        uint32_t msk = 0;
#pragma unroll
        for (int s = 0; s < D; ++s) {
          const int32_t c = cs[u][s];
          if (c >= 0) {
            if (ds[u][s] > r) dist[c] = uint8_t(r);
          } else if (slot_live(m, p[u], s)) {
            msk |= 1u << s;
          }
        }
        wmask[e[u]] = uint16_t(msk);
        cnt += __popc(msk);
      }
    }
  }
  uint32_t tot;
  block_excl_scan(cnt, &tot);
  if (threadIdx.x == 0) sums[block] = tot;
}

template <int D>
__global__ void __launch_bounds__(kBlock)
    k_warm_count(DevModel m, int r, int vb, const StepCtl* ctl,
                 const uint64_t* pay, const int32_t* col, uint8_t* dist,
                 uint16_t* wmask, uint32_t* sums, const int* err) {
  if (*err) return;
  count_part<D>(m, r, vb, blockIdx.x, gridDim.x, ctl, pay, col, dist, wmask,
                sums);
}

// Write pass (same grid): those slots as candidates, in row order.
__global__ void __launch_bounds__(kBlock)
    k_warm_list(int r, int vb, const StepCtl* ctl, const uint8_t* dist,
                const uint16_t* wmask, const uint32_t* sums, uint64_t* wlist,
                int64_t cand_cap, int* err) {
  __shared__ uint16_t list[kBlock * kMaxVb];
  if (latched(err)) return;
  const int64_t n = ctl->n_old, tile = int64_t(kBlock) * vb;
  const TileRun run = tile_run(cdiv(n, tile), gridDim.x);
  uint64_t total;
  uint64_t at = sums_before(sums, gridDim.x, blockIdx.x, &total);
  if (sums[blockIdx.x] == 0) return;
  for (int64_t t = run.t0; t < run.t1; ++t) {
    const uint32_t tot = list_rows(dist, t, n, vb, uint8_t(r - 1), list);
    for (uint32_t i0 = 0; i0 < tot; i0 += kBlock) {
      const uint32_t i = i0 + threadIdx.x;
      const int64_t e = i < tot ? t * tile + list[i] : 0;
      uint32_t msk = i < tot ? wmask[e] : 0u;
      uint32_t c;
      uint64_t off = at + block_excl_scan(__popc(msk), &c);
      at += c;
      while (msk) {
        const int s = __ffs(msk) - 1;
        msk &= msk - 1;
        if (int64_t(off) < cand_cap)
          wlist[off] = (uint64_t(e) << 8) | uint64_t(s);
        else
          atomicOr(err, kErrChunks);
        ++off;
      }
    }
  }
}

// Insert-if-absent of each candidate's key.  Table values: a live row, a
// found state's row (kStaged | row) or, during the round, kCand |
// candidate.  A key found as a live row marks it at distance r; a key
// found staged or claimed by another candidate needs nothing; the
// candidate whose compare-and-swap fills an empty slot owns the key (probe
// distance into c_slot), counted per block.  Candidates of round r: w_noc
// from live rows (the count pass's sums), then every slot of the states
// found in round r-1.  Tombstones are
// passed over and never claimed, so removing the staged entries restores
// the table.  row_limit > 0 (state cap): M and the states found so far
// exceeding it latch kErrOver; a block stops at its next tile once anything
// is latched (as in the rounds of an expansion from scratch).
template <int W>
__global__ void __launch_bounds__(kBlock)
    k_warm_probe(DevModel m, int r, StepCtl* ctl, int64_t row_limit, Side c,
                 const uint32_t* freel, const uint64_t* wlist,
                 const uint32_t* old_sums, int old_grid, int64_t cand_cap,
                 uint64_t* table, uint64_t mask, uint32_t* c_slot,
                 uint32_t* c_ref, uint32_t* sums, int* err) {
  __shared__ int stop[2];  // latch seen at this tile, by parity of the tile
  if (latched(err)) return;
  uint64_t total;
  sums_before(old_sums, old_grid, 0, &total);
  const int64_t noc = int64_t(total), f0 = ctl->gstart[r - 1], nM = ctl->nM;
  const int64_t nc = noc + (int64_t(ctl->gstart[r]) - f0) * m.D;
  if (nc > cand_cap) {
    if (gtid() == 0) atomicOr(err, kErrChunks);
    return;
  }
  if (gtid() == 0) {
    ctl->w_noc = uint32_t(noc);
    ctl->r_ncand = uint32_t(nc);
    if (uint32_t(nc) > ctl->c_max) ctl->c_max = uint32_t(nc);
  }
  const TileRun run = tile_run(cdiv(nc, kBlock), gridDim.x);
  uint32_t own = 0, pend = 0;  // pend: not yet in r_own
  int par = 0;
  for (int64_t tile = run.t0; tile < run.t1; ++tile, par ^= 1) {
    const int64_t cand = tile * kBlock + threadIdx.x;
    if (threadIdx.x == 0) stop[par] = latch_now(err);
    uint32_t owner = 0;
    if (cand < nc) {
      uint64_t k[W];
      int64_t p;
      int s;
      uint32_t ref = kNone;
      if (warm_cand<W>(m, ctl, freel, noc, f0, wlist, c, cand, k, p, s)) {
        const uint64_t h = key_hash<W>(m, k);
        const uint32_t tag = hash_tag(h);
        const uint64_t mine =
            (uint64_t(tag) << 32) | uint64_t(kCand | uint32_t(cand));
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
              ref = kOwnerW;
              c_slot[cand] = uint32_t(probes);
              owner = 1;
              done = true;
              break;
            }
            e = old;
          }
          if (uint32_t(e >> 32) == tag) {
            const uint32_t v = uint32_t(e);
            if (v & kCand) {
              const int64_t c2 = int64_t(v & ~kCand);
              uint64_t k2[W];
              int64_t p2;
              int s2;
              warm_cand<W>(m, ctl, freel, noc, f0, wlist, c, c2, k2, p2, s2);
              bool same = true;
#pragma unroll
              for (int q = 0; q < W; ++q) same &= (k2[q] == k[q]);
              done = same;
            } else {
              const int64_t row = int64_t(v & ~kStaged);
              if (key_eq<W>(k, c.keys + row * W)) {
                // a live row is within distance r; a staged one is nearer
                if (!(v & kStaged) && c.dist[row] > r)
                  c.dist[row] = uint8_t(r);
                done = true;
              }
            }
            if (done) break;
          }
          i = (i + 1) & mask;
        }
        if (!done) atomicOr(err, kErrTableFull);
      }
      c_ref[cand] = ref;
    }
    uint32_t tot;
    block_excl_scan(owner, &tot);
    own += tot;
    pend += tot;
    if (threadIdx.x == 0 && row_limit > 0 && pend &&
        (((tile - run.t0) & 3) == 3 || tile + 1 == run.t1)) {
      if (nM + int64_t(atomicAdd(&ctl->r_own, pend)) + pend > row_limit)
        atomicOr(err, kErrOver);
      pend = 0;
    }
    if (stop[par]) return;  // written before the scan's barriers
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = own;
}

// Owners take their rows, numbered by the owners of the blocks before and
// a scan per tile (same grid as the probe): key, payload, totals, distance
// kNewRow | r, amplitude 0; their table slot points at the row, staged.
template <int W>
__device__ __forceinline__ void commit_part(
    const DevModel& m, int r, int block, int grid, StepCtl* ctl, int64_t cap,
    const Side& c, const uint32_t* freel, const uint64_t* wlist,
    uint64_t* table, uint64_t mask, const uint32_t* c_slot,
    const uint32_t* c_ref, const uint32_t* sums, uint64_t* psi, int A8,
    int* err) {
  const int64_t nc = ctl->r_ncand, noc = ctl->w_noc, f0 = ctl->gstart[r - 1];
  const TileRun run = tile_run(cdiv(nc, kBlock), grid, block);
  uint64_t total;
  int64_t at = ctl->gstart[r] +
               int64_t(sums_before(sums, grid, block, &total));
  if (block == 0 && threadIdx.x == 0) {
    ctl->n_staged = uint32_t(ctl->gstart[r] + total);
    ctl->gstart[r + 1] = ctl->n_staged;
  }
  if (sums[block] == 0) return;
  for (int64_t tile = run.t0; tile < run.t1; ++tile) {
    const int64_t cand = tile * kBlock + threadIdx.x;
    const bool own = cand < nc && c_ref[cand] == kOwnerW;
    uint32_t tot_in_tile;
    const int64_t num = at + block_excl_scan(own ? 1u : 0u, &tot_in_tile);
    at += tot_in_tile;
    if (!own) continue;
    const int64_t row = found_row(num, ctl, freel);
    if (row >= cap) {
      atomicOr(err, kErrCapacity);
      continue;
    }
    uint64_t k[W];
    int64_t p;
    int s;
    warm_cand<W>(m, ctl, freel, noc, f0, wlist, c, cand, k, p, s);
    store_key<W>(c.keys, row, k);
    uint64_t np, nt;
    slot_row_info<W>(m, k, c.pay[p], c.tot[p], s, np, nt);
    c.pay[row] = np;
    c.tot[row] = nt;
    c.dist[row] = uint8_t(kNewRow | r);
    const uint64_t h = key_hash<W>(m, k);
    table[((h & mask) + c_slot[cand]) & mask] =
        (uint64_t(hash_tag(h)) << 32) | uint64_t(kStaged | uint32_t(row));
    for (int w = 0; w < A8; ++w) psi[row * A8 + w] = 0ull;
  }
}

template <int W>
__global__ void __launch_bounds__(kBlock)
    k_warm_commit(DevModel m, int r, StepCtl* ctl, int64_t cap, Side c,
                  const uint32_t* freel, const uint64_t* wlist,
                  uint64_t* table, uint64_t mask, const uint32_t* c_slot,
                  const uint32_t* c_ref, const uint32_t* sums, uint64_t* psi,
                  int A8, int* err) {
  if (latched(err)) return;
  commit_part<W>(m, r, blockIdx.x, gridDim.x, ctl, cap, c, freel, wlist, table,
                 mask, c_slot, c_ref, sums, psi, A8, err);
}

// The commit of round r by blocks [0, grid) beside the count pass of round r +
// 1 by the others.  The two need nothing of each other: the commit takes rows
// that no live row's column names, at distances that the count does not
// match, and the count marks live rows and writes wmask and its own sums, last
// read by round r's probe.  A launch less per round, and two kernels that wait
// for memory share the chip: a ring of 16 at 1e3 to 4e5 rows 4.7 + 6.3 us ->
// 7.0, in complex64 at up to 8e6 5.1 + 9.4 -> 10.8; 64 6x6 lattices 34 + 33 ->
// 51.
template <int W, int D>
__global__ void __launch_bounds__(kBlock)
    k_warm_turn(DevModel m, int r, int grid, int vb, StepCtl* ctl, int64_t cap,
                Side c, const uint32_t* freel, const uint64_t* wlist,
                uint64_t* table, uint64_t mask, const uint32_t* c_slot,
                const uint32_t* c_ref, const uint32_t* sums, uint64_t* psi,
                int A8, uint16_t* wmask, uint32_t* old_sums, int* err) {
  if (latched(err)) return;
  if (int(blockIdx.x) < grid)
    commit_part<W>(m, r, blockIdx.x, grid, ctl, cap, c, freel, wlist, table,
                   mask, c_slot, c_ref, sums, psi, A8, err);
  else
    count_part<D>(m, r + 1, vb, int(blockIdx.x) - grid,
                  int(gridDim.x) - grid, ctl, c.pay, c.col, c.dist, wmask,
                  old_sums);
}

// ---- sizes (state cap) --------------------------------------------------------
// Live rows of the new set per realization.  A thread reads the distances
// of 16 rows at once (the array's allocation is a multiple of 256 bytes, so
// the last group stays inside it).
__global__ void __launch_bounds__(kBlock)
    k_warm_live(DevModel m, int k, const StepCtl* ctl, const uint8_t* dist,
                const uint64_t* pay, uint32_t* ball, const int* err) {
  __shared__ uint32_t bins[kMaxReal];
  if (*err) return;
  for (int r = threadIdx.x; r < m.R; r += blockDim.x) bins[r] = 0;
  __syncthreads();
  const int64_t n = new_range(ctl), n16 = cdiv(n, 16);
  const uint4* d16 = reinterpret_cast<const uint4*>(dist);
  uint32_t live = 0;
  for (int64_t g = gtid(); g < n16; g += gstride()) {
    const uint4 v = d16[g];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int64_t e = g * 16 + q;
      if (e >= n || !kept(uint8_t(w[q >> 2] >> (8 * (q & 3))), k)) continue;
      ++live;
      if (m.R > 1) atomicAdd(&bins[pay_real(pay[e])], 1u);
    }
  }
  if (m.R == 1) {
    uint32_t tot;
    block_excl_scan(live, &tot);
    if (threadIdx.x == 0) bins[0] = tot;
  }
  count_flush(m.R, bins, ball);
}

__global__ void k_warm_cap_over(StepCtl* ctl, int R, int64_t max_states,
                                 const uint32_t* ball, int* err) {
  if (*err) return;
  ctl->n_ball = ball[0];
  for (int r = 0; r < R; ++r)
    if (int64_t(ball[r]) > max_states) atomicOr(err, kErrCap);
}

// ---- the commit -------------------------------------------------------------
// First every block's share of the old rows: those the search did not reach
// become holes (weight into the partials, amplitude 0, table entry a
// tombstone, columns of the row and of its neighbours toward it -1, distance
// kHole).  Then its share of the found states' slots: distance r, table
// entry plain (lane of slot 0), columns by lookup.  An edge is seen from
// both ends as slots s and s ^ 1, so a found state also sets the column of a
// live row toward it (that row had -1 there: the state was outside the old
// set); between two found states both ends write the same values.  The two
// parts need no order between blocks: a lookup may still find a row that is
// being dropped, whose distance byte (kFar or kHole) says so, and they write
// different columns.  Bound by random access (a table line per dropped and
// found state, one per slot of a found state) and by the latency of the chains
// to it: rows and their slots are separate loops, so that a lane's chain is
// one row's table walk or one slot's neighbour, and a lane keeps U rows or
// four slots in flight.  On a ring of 16 at about 1e5 rows 17.0 -> 12.0 us, at
// 0.5 to 2.3 million 23.3 -> 19.3, 64 6x6 lattices 273 -> 246, a 25-site chain
// 239 -> 222.
template <int W, typename Amp>
__global__ void __launch_bounds__(kBlock)
    k_warm_settle(DevModel m, int k, int vb, StepCtl* ctl, Side c,
                  const uint32_t* freel, uint64_t* table, uint64_t mask,
                  Amp* psi, double* mass_part, const uint64_t* keys0,
                  int64_t n0, int32_t* p0, const int* err) {
  __shared__ double bins[kMaxReal];
  __shared__ uint16_t list[kBlock * kMaxVb];
  if (*err) return;
  if (gtid() == 0) {
    ctl->w_moved = 1;
    ctl->n_new = uint32_t(new_range(ctl));
  }
  constexpr int U = W <= 4 ? 2 : 1;
  const int R = m.R;
  const uint32_t D = uint32_t(m.D);
  if (R > 1) {
    for (int r = threadIdx.x; r < R; r += blockDim.x) bins[r] = 0.0;
    __syncthreads();
  }
  const int64_t nold = ctl->n_old;
  const int64_t tile = int64_t(kBlock) * vb;
  const TileRun run = tile_run(cdiv(nold, tile), gridDim.x);
  double lost = 0;
  uint32_t tombs = 0, drops = 0;
  for (int64_t t = run.t0; t < run.t1; ++t) {
    const uint32_t tot = list_rows(c.dist, t, nold, vb, kFar, list);
    drops += tot;
    for (uint32_t i = threadIdx.x; i < tot; i += U * kBlock) {
      int64_t e[U];
      Amp v[U];
      uint64_t key[U][W], ent[U];
      int real[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t x = i + u * kBlock;
        e[u] = t * tile + list[x < tot ? x : i];
        v[u] = psi[e[u]];
        load_key<W>(c.keys, e[u], key[u]);
        real[u] = R > 1 ? pay_real(c.pay[e[u]]) : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        ent[u] = table[key_hash<W>(m, key[u]) & mask];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i + u * kBlock >= tot) continue;
        if (R > 1)
          atomicAdd(&bins[real[u]], weight(v[u]));
        else
          lost += weight(v[u]);
        Amp z;
        z.x = 0;
        z.y = 0;
        psi[e[u]] = z;
        const int64_t sl = warm_slot(table, mask, key_hash<W>(m, key[u]),
                                     ent[u], uint32_t(e[u]));
        if (sl >= 0) {
          table[sl] = kTomb;
          ++tombs;
        }
        c.dist[e[u]] = kHole;
      }
    }
    for (uint32_t i = threadIdx.x; i < tot * D; i += 4 * kBlock) {
      int64_t e[4];
      uint32_t sl[4];
      int32_t nb[4];
      uint8_t dn[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t x = i + u * kBlock < tot * D ? i + u * kBlock : i;
        const uint32_t q = x / D;
        e[u] = t * tile + list[q];
        sl[u] = x - q * D;
        nb[u] = c.col[e[u] * D + sl[u]];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        dn[u] = c.dist[nb[u] >= 0 ? int64_t(nb[u]) : e[u]];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i + u * kBlock >= tot * D) continue;
        // a neighbour that stays (within k) loses its column toward e; one
        // dropped too clears its own
        if (nb[u] >= 0 && dn[u] <= k)
          c.col[int64_t(nb[u]) * D + (sl[u] ^ 1u)] = -1;
        c.col[e[u] * D + sl[u]] = -1;
      }
    }
  }
  const int64_t ns = ctl->n_staged;
  for (int64_t q = gtid(); q < ns; q += gstride()) {
    const int64_t row = found_row(q, ctl, freel);
    uint64_t key[W];
    load_key<W>(c.keys, row, key);
    const uint64_t h = key_hash<W>(m, key);
    const int64_t sl =
        warm_slot(table, mask, h, table[h & mask], kStaged | uint32_t(row));
    if (sl >= 0) table[sl] = (uint64_t(hash_tag(h)) << 32) | uint64_t(row);
    c.dist[row] = uint8_t(c.dist[row] & ~kNewRow);
  }
  for (int64_t t0 = int64_t(blockIdx.x) * kBlock; t0 < ns * D;
       t0 += gstride()) {
    if (t0 + threadIdx.x >= ns * D) break;
    const uint32_t x = uint32_t(t0 % D) + threadIdx.x;
    const int64_t q = t0 / D + x / D;
    const int s = int(x % D);
    const int64_t row = found_row(q, ctl, freel);
    uint64_t par[W], kk[W];
    load_key<W>(c.keys, row, par);
    int32_t out = -1;
    if (slot_target<W>(m, par, c.pay[row], s, kk)) {
      const int64_t f = warm_find<W>(table, mask, c.keys, kk, key_hash<W>(m, kk));
      if (f >= 0 && kept(c.dist[f], k)) {
        out = int32_t(f);
        c.col[f * D + (s ^ 1)] = int32_t(row);
      }
    }
    c.col[row * D + s] = out;
  }
  // rows of the initial states in the new set
  for (int64_t i = gtid(); i < n0; i += gstride()) {
    uint64_t kk[W];
    load_key<W>(keys0, i, kk);
    const int64_t f = warm_find<W>(table, mask, c.keys, kk, key_hash<W>(m, kk));
    p0[i] = f >= 0 && kept(c.dist[f], k) ? int32_t(f) : -1;
  }
  if (R > 1) {
    __syncthreads();
    for (int r = threadIdx.x; r < R; r += blockDim.x)
      mass_part[int64_t(blockIdx.x) * R + r] = bins[r];
  } else {
    lost = block_sum(lost);
    if (threadIdx.x == 0) mass_part[blockIdx.x] = lost;
  }
  uint32_t tot;
  block_excl_scan(tombs, &tot);
  if (threadIdx.x == 0 && drops) {
    atomicAdd(&ctl->w_tomb, tot);
    atomicAdd(&ctl->w_drop, drops);
  }
}

// ---- repeat and bookkeeping ---------------------------------------------------
__global__ void __launch_bounds__(kBlock)
    k_warm_unstage_table(uint64_t* table, uint64_t mask) {
  const int64_t P = int64_t(mask) + 1;
  for (int64_t i = gtid(); i < P; i += gstride()) {
    const uint64_t e = table[i];
    if (e == kEmpty || uint32_t(e >> 32) == 0xFFFFFFFFu) continue;
    if (uint32_t(e) & (kCand | kStaged)) table[i] = kEmpty;
  }
}

// Holes that took a found state become holes again (bytes past the range
// need nothing).
__global__ void __launch_bounds__(kBlock)
    k_warm_unstage_rows(uint8_t* dist, int64_t n) {
  for (int64_t e = gtid(); e < n; e += gstride()) {
    const uint8_t d = dist[e];
    if (d >= kNewRow && d < kHole) dist[e] = kHole;
  }
}

__global__ void __launch_bounds__(kBlock)
    k_dist_fill(uint8_t* dist, int64_t n, uint8_t v) {
  for (int64_t e = gtid(); e < n; e += gstride()) dist[e] = v;
}

__global__ void k_u32_set(uint32_t* out, int64_t v) { *out = uint32_t(v); }

__global__ void __launch_bounds__(kBlock)
    k_gather_rows(int Wi, int A8, const uint64_t* keys, const uint64_t* pay,
                  const uint64_t* tot, const uint64_t* psi,
                  const uint32_t* idx, int64_t n, uint64_t* okeys,
                  uint64_t* opay, uint64_t* otot, uint64_t* oamps) {
  for (int64_t i = gtid(); i < n; i += gstride()) {
    const int64_t r = idx[i];
    if (okeys)
      for (int w = 0; w < Wi; ++w) okeys[i * Wi + w] = keys[r * Wi + w];
    if (opay) opay[i] = pay[r];
    if (otot) otot[i] = tot[r];
    if (oamps)
      for (int w = 0; w < A8; ++w) oamps[i * A8 + w] = psi[r * A8 + w];
  }
}

__global__ void __launch_bounds__(kBlock)
    k_rank_rows(const uint32_t* idx, int64_t n, const int32_t* rows,
                int32_t* out, int64_t n0) {
  for (int64_t i = gtid(); i < n0; i += gstride()) {
    const int64_t r = rows[i];
    int64_t lo = 0, hi = r < 0 ? 0 : n;  // first listed row >= r
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      if (int64_t(idx[mid]) < r)
        lo = mid + 1;
      else
        hi = mid;
    }
    out[i] = r >= 0 && lo < n && int64_t(idx[lo]) == r ? int32_t(lo) : -1;
  }
}

}  // namespace

// ---- host wrappers ----------------------------------------------------------

void warm_begin(const DevModel& m, StepCtl* ctl, const Sums& sm, int sel_grid,
                const Side& c, const WarmBufs& wb, uint32_t* cnt_m,
                int64_t n_old, bool holes, int* err, hipStream_t s) {
  const int g = sum_grid(n_old, kBlock * 16);
  k_warm_select<<<g, kBlock, 0, s>>>(m, ctl, sm.bits, sm.sel, sel_grid, c.pay,
                                     c.dist, cnt_m, holes ? sm.hole : nullptr,
                                     err);
  if (holes)
    k_warm_holes<<<g, kBlock, 0, s>>>(ctl, c.dist, sm.hole, wb.freel, err);
}

void warm_round(const DevModel& m, int Wi, int prec, const Side& c, int r,
                int k,
                StepCtl* ctl, int64_t cap, int64_t n_old, int64_t n_cand,
                uint64_t* table, uint64_t mask, const RoundBufs& rb,
                const WarmBufs& wb, const Sums& sm, void* psi,
                int64_t row_limit, int* err, hipStream_t s) {
  const int vb = rows_per_lane(n_old);
  const int go = sum_grid(n_old, int64_t(kBlock) * vb);
#define PACES_DISPATCH_D(...)                              \
  switch (m.D) {                                           \
    case 4: { constexpr int DD = 4; __VA_ARGS__; } break;   \
    case 6: { constexpr int DD = 6; __VA_ARGS__; } break;   \
    case 8: { constexpr int DD = 8; __VA_ARGS__; } break;   \
    case 10: { constexpr int DD = 10; __VA_ARGS__; } break; \
    case 12: { constexpr int DD = 12; __VA_ARGS__; } break; \
    case 14: { constexpr int DD = 14; __VA_ARGS__; } break; \
    default: break;                                        \
  }
  if (r == 1)
    PACES_DISPATCH_D(k_warm_count<DD><<<go, kBlock, 0, s>>>(
        m, r, vb, ctl, c.pay, c.col, c.dist, wb.wmask, sm.old_, err));
  k_warm_list<<<go, kBlock, 0, s>>>(r, vb, ctl, c.dist, wb.wmask, sm.old_,
                                    wb.wlist, rb.cand_cap, err);
  const int g = sum_grid(std::min(rb.cand_cap, n_cand), kBlock);
  PACES_DISPATCH_W(Wi, k_warm_probe<WW><<<g, kBlock, 0, s>>>(
                           m, r, ctl, row_limit, c, wb.freel, wb.wlist,
                           sm.old_, go, rb.cand_cap, table, mask, rb.c_slot,
                           rb.c_ref, sm.own, err));
  uint64_t* const psi8 = static_cast<uint64_t*>(psi);
  const int A8 = prec == 64 ? 2 : 1;
  if (r == k) {
    PACES_DISPATCH_W(Wi, k_warm_commit<WW><<<g, kBlock, 0, s>>>(
                             m, r, ctl, cap, c, wb.freel, wb.wlist, table,
                             mask, rb.c_slot, rb.c_ref, sm.own, psi8, A8,
                             err));
  } else {
    PACES_DISPATCH_W(Wi, PACES_DISPATCH_D(
        k_warm_turn<WW, DD><<<g + go, kBlock, 0, s>>>(
            m, r, g, vb, ctl, cap, c, wb.freel, wb.wlist, table, mask,
            rb.c_slot, rb.c_ref, sm.own, psi8, A8, wb.wmask, sm.old_, err)));
  }
#undef PACES_DISPATCH_D
}

void warm_cap_check(const DevModel& m, const Side& c, int k, StepCtl* ctl,
                    int64_t est, int64_t max_states, uint32_t* ball, int* err,
                    hipStream_t s) {
  // 16 rows per thread and one count added to the total per block
  k_warm_live<<<std::min(grid_for(cdiv(est, 16)), 512), kBlock, 0, s>>>(
      m, k, ctl, c.dist, c.pay, ball, err);
  k_warm_cap_over<<<1, 1, 0, s>>>(ctl, m.R, max_states, ball, err);
}

int warm_commit(const DevModel& m, int Wi, int prec, const Side& c, int k,
                StepCtl* ctl, int64_t n_old, int64_t n_found, uint64_t* table,
                uint64_t mask, const WarmBufs& wb, void* psi,
                double* mass_part, const uint64_t* keys0, int64_t n0,
                int32_t* p0, int* err, hipStream_t s) {
  const int vb = rows_per_lane(n_old);
  const int g = std::min(std::max(sum_grid(n_old, int64_t(kBlock) * vb),
                                  grid_for(n_found * m.D)), kPartBlocks);
  if (prec == 64) {
    PACES_DISPATCH_W(Wi, k_warm_settle<WW, double2><<<g, kBlock, 0, s>>>(
                             m, k, vb, ctl, c, wb.freel, table, mask,
                             (double2*)psi, mass_part, keys0, n0, p0, err));
  } else {
    PACES_DISPATCH_W(Wi, k_warm_settle<WW, float2><<<g, kBlock, 0, s>>>(
                             m, k, vb, ctl, c, wb.freel, table, mask,
                             (float2*)psi, mass_part, keys0, n0, p0, err));
  }
  return g;
}

void warm_unstage(const StepCtl* ctl, const Side& c, const WarmBufs& wb,
                  uint64_t* table, uint64_t mask, int64_t n_old,
                  hipStream_t s) {
  (void)ctl;
  (void)wb;
  k_warm_unstage_table<<<grid_for(int64_t(mask) + 1), kBlock, 0, s>>>(table,
                                                                      mask);
  if (n_old > 0)
    k_warm_unstage_rows<<<grid_for(n_old), kBlock, 0, s>>>(c.dist, n_old);
}

void dist_fill(uint8_t* dist, int64_t n, uint8_t v, hipStream_t s) {
  if (n > 0) k_dist_fill<<<grid_for(n), kBlock, 0, s>>>(dist, n, v);
}

void rows_at_distance(int Wi, const uint64_t* keys, const uint8_t* dist,
                      int64_t n, int d, uint64_t* out, uint32_t* rows,
                      uint32_t* count, uint32_t* sums, hipStream_t s) {
  if (n <= 0) {
    k_u32_set<<<1, 1, 0, s>>>(count, 0);
    return;
  }
  const int g = sum_grid(n, kBlock);
  k_dist_count<<<g, kBlock, 0, s>>>(dist, n, d, sums);
  k_dist_write<<<g, kBlock, 0, s>>>(Wi, keys, dist, n, d, sums, count, out,
                                    rows);
}

void gather_rows(int Wi, size_t A, const Side& c, const void* psi,
                 const uint32_t* idx, int64_t n, uint64_t* keys,
                 uint64_t* pay, uint64_t* tot, void* amps, hipStream_t s) {
  if (n <= 0) return;
  k_gather_rows<<<grid_for(n), kBlock, 0, s>>>(
      Wi, int(A / 8), c.keys, c.pay, c.tot, static_cast<const uint64_t*>(psi),
      idx, n, keys, pay, tot, static_cast<uint64_t*>(amps));
}

void rank_rows(const uint32_t* idx, int64_t n, const int32_t* rows,
               int32_t* out, int64_t n0, hipStream_t s) {
  if (n0 <= 0) return;
  k_rank_rows<<<grid_for(n0), kBlock, 0, s>>>(idx, n, rows, out, n0);
}

}  // namespace paces
