// small.hpp -- the part of a step after the transfer, in one launch, for sets
// that fit the LDS of one compute unit (small.hip).
#pragma once
#include "warm.hpp"

namespace paces {

// Rows that one block propagates: three per thread of 1024, their three
// vectors in LDS (144 KiB in complex128).
constexpr int kSmallRows = 3072;
constexpr int kSmallSites = 2048;  // population bins reuse a vector's LDS
constexpr int kSmallSlots = 8;     // columns per row held in registers

inline bool small_shape(const DevModel& m) {
  return m.R == 1 && m.D <= kSmallSlots && m.V <= 2 && m.N <= kSmallSites;
}

// Spectral bounds, Chebyshev coefficients, psi = exp(-i H dt) phi and, with a
// record ring, the observables, the next step's selection and the close of
// the step (what bounds_and_coef, the cheb_term launches, pop_norm and
// obs_final do).  More than kSmallRows rows latch kErrBig.
struct SmallTail {
  DevModel m;
  StepCtl* ctl;
  int* err;
  const uint64_t* pay;
  const uint8_t* dist;  // may be null (no holes)
  const int32_t* col;
  const void* phi;
  void* psi;
  ChebCoef* cc;
  double dt, tol;
  int k_max;
  // observables (ring null: none; then K and the latch go to said[2])
  int want_energy;
  double th2;
  const double* mass_part;
  int n_mass;
  const double* amps0;
  int64_t n0;
  const int32_t* p0;
  const uint32_t* cnt;
  double* mass_tot;
  double* ring;
  int rec_doubles;
  int64_t ring_cap;
  uint64_t* bits;
  uint32_t* sel;
  StepCtl* h_ctl;  // device addresses of the host's mirrors
  int* h_err;
  uint32_t* said;
};
// False where the launch cannot be made (then nothing is enqueued).
bool small_tail(const SmallTail& a, int prec, hipStream_t s);

// The in-place step up to its transfer in one launch, for sets of at most
// kSmallRows rows (range included) selected by threshold: what begin_step,
// warm_begin, the k rounds, the state-cap check and warm_commit do, with the
// same results.  Writes one partial of the dropped weight.  Latches as those
// do (kErrChunks where a round's candidates are too many) and kErrBig for a
// larger set, and until its commit changes nothing of the set but what
// warm_unstage restores.
struct SmallExpand {
  DevModel m;
  int k;
  StepCtl* ctl;
  int* err;
  uint32_t *cnt, *ball;
  Side c;
  WarmBufs wb;
  RoundBufs rb;
  uint64_t* table;
  uint64_t mask;
  void* psi;
  double th2;
  int64_t cap, row_limit, max_states;
  double* mass_part;
  const uint64_t* keys0;
  int64_t n0;
  int32_t* p0;
};
void small_expand(const SmallExpand& a, int Wi, int prec, hipStream_t s);

}  // namespace paces
