// warm_device.hpp -- device helpers of the in-place step (warm.hpp), shared by
// its launches (warm.hip) and the one-block form for small sets (small.hip).
#pragma once
#include "common.hpp"
#include "warm.hpp"

namespace paces {

namespace {

constexpr uint64_t kTomb = 0xFFFFFFFF00000000ull;  // entry of a dropped row
constexpr uint32_t kOwnerW = 0xFFFFFFFEu;           // candidate owns its key

// Whether slot s of a row with payload pay is structurally nonzero (the
// test of slot_target without forming the key).
__device__ __forceinline__ bool slot_live(const DevModel& m, uint64_t pay,
                                          int s) {
  const int j = pay_site(pay);
  if (s < 2 * m.ndim) {
    if (!((m.hop_mask >> (s >> 1)) & 1u)) return false;
    return m.nbr[j * 2 * m.ndim + s] >= 0;
  }
  const int e = s - 2 * m.ndim, nu = e >> 1;
  if (!((m.eph_mask >> nu) & 1u)) return false;
  const int n = pay_occ(pay, nu);
  return (e & 1) == 0 ? n > 0 : n < m.cut[nu];
}

// Whether a distance byte marks a row of the new set: a live row within k,
// or a state found this step (kNewRow | r, below kHole).
__device__ __forceinline__ bool kept(uint8_t d, int k) {
  return d <= k || (d >= kNewRow && d < kHole);
}

// Row of the q-th state found this step: the q-th hole, else the next row
// past the set's range.
__device__ __forceinline__ int64_t found_row(int64_t q, const StepCtl* ctl,
                                             const uint32_t* freel) {
  const int64_t nf = ctl->nfree;
  return q < nf ? int64_t(freel[q]) : int64_t(ctl->n_old) + (q - nf);
}

// Row range of the set after the found states took their rows.
__device__ __forceinline__ int64_t new_range(const StepCtl* ctl) {
  const int64_t extra = int64_t(ctl->n_staged) - ctl->nfree;
  return int64_t(ctl->n_old) + (extra > 0 ? extra : 0);
}

// Row of key k in the table (plain or staged entry; tombstones and
// candidates passed over), or -1.
template <int W>
__device__ __forceinline__ int64_t warm_find(const uint64_t* table,
                                             uint64_t mask,
                                             const uint64_t* keys,
                                             const uint64_t (&k)[W],
                                             uint64_t h) {
  const uint32_t tag = hash_tag(h);
  uint64_t i = h & mask;
  for (uint64_t probes = 0; probes <= mask && probes < kMaxProbe; ++probes) {
    const uint64_t e = table[i];
    if (e == kEmpty) break;
    if (uint32_t(e >> 32) == tag) {
      const uint32_t v = uint32_t(e);
      if (!(v & kCand)) {
        const int64_t row = int64_t(v & ~kStaged);
        if (key_eq<W>(k, keys + row * W)) return row;
      }
    }
    i = (i + 1) & mask;
  }
  return -1;
}

// Slot of the table entry with hash h whose value is `value`, or -1; e0: the
// entry at the hash's own slot, loaded by the caller.
__device__ __forceinline__ int64_t warm_slot(const uint64_t* table,
                                             uint64_t mask, uint64_t h,
                                             uint64_t e0, uint32_t value) {
  const uint64_t want = (uint64_t(hash_tag(h)) << 32) | value;
  uint64_t i = h & mask, e = e0;
  for (uint64_t probes = 0; probes <= mask && probes < kMaxProbe; ++probes) {
    if (e == want) return int64_t(i);
    if (e == kEmpty) break;
    i = (i + 1) & mask;
    e = table[i];
  }
  return -1;
}

// Key of candidate c and its parent's row: a live row (from wlist) or the
// row of a state found in the round before.  False for a structurally
// zero slot.
template <int W>
__device__ __forceinline__ bool warm_cand(const DevModel& m,
                                          const StepCtl* ctl,
                                          const uint32_t* freel, int64_t noc,
                                          int64_t f0, const uint64_t* wlist,
                                          const Side& c, int64_t cand,
                                          uint64_t (&k)[W], int64_t& p,
                                          int& s) {
  if (cand < noc) {
    const uint64_t e = wlist[cand];
    p = int64_t(e >> 8);
    s = int(e & 0xFFu);
  } else {
    const int64_t d = cand - noc;
    p = found_row(f0 + d / m.D, ctl, freel);
    s = int(d % m.D);
  }
  uint64_t par[W];
  load_key<W>(c.keys, p, par);
  return slot_target<W>(m, par, c.pay[p], s, k);
}

}  // namespace

}  // namespace paces
