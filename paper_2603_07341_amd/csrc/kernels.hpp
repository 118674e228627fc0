// kernels.hpp -- host-side launch wrappers of the step's HIP kernels.
//
// Row counts of a step live in device memory (StepCtl) and every kernel
// reads them there, so a whole step is enqueued without the host waiting on
// the GPU.  Kernels run on fixed grid-stride grids and clamp every count to
// the allocated capacity; an overflow is latched and the host repeats the
// step with larger buffers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.hpp"

namespace paces {

constexpr int kMaxTerms = 128;   // Chebyshev terms per step, hard limit
constexpr int kMaxRounds = 30;   // neighbour order per step, hard limit
constexpr int kPartBlocks = 2048;  // largest grid that leaves partials
// Blocks of the record pass: n2_part holds their norms, and from row
// kPopBlocks on their row counts.
constexpr int kPopBlocks = 1024;
constexpr int kMaxPartials = 1 << 18;  // per-block partials of row kernels
constexpr int kObsFields = 12;
constexpr int kMaxReal = 256;      // disorder realizations per sim
constexpr int kMaxSums = 2048;     // blocks of a kernel that leaves sums

// Chebyshev expansion of exp(-i H dt) on [E_min, E_max], computed on the
// device from the Gershgorin bounds of the step.
struct ChebCoef {
  double emin, emax;   // padded Gershgorin interval
  double a, b;         // half width and centre
  double alpha, beta;  // H~ = alpha H + beta: alpha = 1/a, beta = -b/a
  double phase[2];     // exp(-i b dt)
  int K;               // number of terms used
  int pad_;
  double c[kMaxTerms][2];  // c_k = (2 - delta_k0) (-i)^k J_k(a dt)
};

// Device-resident counts of one step.
struct StepCtl {
  uint32_t n_old;                     // rows of the set the step starts from
  uint32_t nM;                        // selected rows
  uint32_t fstart[kMaxRounds + 2];    // frontier r: [fstart[r], fstart[r+1])
  uint32_t n_new;                     // rows of the new set
  // expansion from scratch: rows of the set before chunk q of a round
  // (q > 0) in r_cur[q & 1]; chunks the largest round needs
  uint32_t r_cur[2], r_need;
  uint32_t r_own;                     // states found so far, counted while a
                                      // round runs (state cap of one
                                      // realization only)
  uint32_t c_max;                     // candidates of the largest round
  uint32_t n_ball;                    // rows of the new set counted against
                                      // the state cap (one realization)
  uint32_t kmax;                      // largest K over realizations
  uint32_t nrec;                      // steps recorded (R records each)
  // expansion from the previous step's graph (warm.hpp): states found in
  // round r are numbers [gstart[r], gstart[r+1]) of the n_staged found in
  // all; the current round has r_ncand candidates, the first w_noc of them
  // from old rows; w_moved is set once the step has committed; w_tomb
  // counts the table entries of dropped rows turned into tombstones by this
  // step, w_drop the rows dropped
  uint32_t gstart[kMaxRounds + 2];
  uint32_t n_staged, r_ncand, w_noc, w_moved, w_tomb, w_drop;
  // in-place steps: holes of the set at the step's start (the free list's
  // length); n_new is the set's row range
  uint32_t nfree;
  uint32_t ticket;                    // blocks of the running kernel that
                                      // have arrived at its end
  double t;                           // time after the last completed step
};

// Buffers of one expansion round.
struct RoundBufs {
  uint32_t* c_slot;     // [cand] of an owning candidate: probe distance from
                        // the key's home slot (below kMaxProbe); from
                        // scratch also its rank in its tile << 16
  uint32_t* c_ref;      // [cand] outcome of the probe
  uint32_t* tile_base;  // [cand / 256] owners of the block before the tile
  int64_t cand_cap;     // candidates the buffers hold
};

// Per-block sums of the counting kernels (kSumBlocks words each), kept
// apart where two are in use at a time, and one bit per row: the next
// step's selection.
struct Sums {
  uint32_t *sel, *hole, *old_, *own, *rows;
  uint64_t* bits;
};

// Row arrays of one set.  col (ELL columns, D per row) and dist (distance
// of the row from the step's selection, 0..k) describe the set a step
// built; dist is written by steps that expand from the previous graph.
struct Side {
  uint64_t* keys;
  uint64_t* pay;
  uint64_t* tot;
  int32_t* col;
  uint8_t* dist;
};

int supported_words(int W);  // internal word count >= W, or 0
// Words of the selection's bits for n rows.
int64_t sel_bit_words(int64_t n);

void fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s);
// One empty dispatch (kernel k_mark) on the stream.
void mark(int tag, hipStream_t s);
// The error latch (and the arrival counter) cleared on the stream.
void clear_latch(StepCtl* ctl, int* err, hipStream_t s);
// ctl->kmax and the latch into out[0] and out[1].
void report(const StepCtl* ctl, const int* err, uint32_t* out, hipStream_t s);
// Keys of a given set of n states padded from W to Wi words.
void pad_keys(int W, int Wi, const uint64_t* in, uint64_t* out, int64_t n,
              hipStream_t s);
// Counts, payloads, totals, table (mask + 1 slots) and columns of the set given
// as rows [0, rows) of n.keys; a key out of range or repeated latches
// kErrInput.
void build_set(const DevModel& m, int Wi, const Side& n, int64_t rows,
               StepCtl* ctl, uint64_t* table, uint64_t mask, int32_t* col,
               int* err, hipStream_t s);

// Start of a step: clear the latch, reset the counters (cnt: |M_r| of the R
// realizations; ball: R).
void begin_step(StepCtl* ctl, int* err, uint32_t* cnt, uint32_t* ball, int R,
                hipStream_t s);
// The selection over rows [0, ctl->n_old) as bits and per-block sums
// (pop_norm leaves the same for the next step): rows with weight >= th2
// that are not holes (dist may be null), or rows with keep[row] != 0.
// n: bound of the row count for the grid, which is returned.
int select_bits(int prec, const void* psi, const uint8_t* dist, double th2,
                const StepCtl* ctl, const Sums& sm, int64_t n, hipStream_t s);
int flag_bits(const uint8_t* keep, const StepCtl* ctl, const Sums& sm,
              int64_t n, hipStream_t s);
// The selected rows ascending into midx, their number into ctl->nM; grid:
// that of the kernel that left the bits.  select_all: every row.
void select_write(StepCtl* ctl, const Sums& sm, int grid, uint32_t* midx,
                  const int* err, hipStream_t s);
void select_all(StepCtl* ctl, uint32_t* midx, int64_t n, hipStream_t s);
// Rows 0..nM-1 of the new side are M; inserted into the cleared table.
// phi (may be null) receives their amplitudes from psi_o.  Their distance
// bytes become 0.  bound: of nM, for the grid.
void insert_rows(const DevModel& m, int Wi, int prec, const Side& o,
                 const Side& n, const uint32_t* midx, const StepCtl* ctl,
                 int64_t bound, uint64_t* table, uint64_t mask,
                 uint32_t* cnt_m, const void* psi_o, void* phi, int* err,
                 hipStream_t s);
// Rows [0, rows) of a side into the cleared table, their distance bytes 0
// (dist may be null).
void rehash_rows(const DevModel& m, int Wi, const Side& n, int64_t rows,
                 uint64_t* table, uint64_t mask, int* err, hipStream_t s);
// Expansion round r (1..k): frontier r-1 emits its slots; new rows are
// appended and become frontier r.  Writes the parents' ELL columns, zeroes
// phi of the new rows and sets their distance bytes to r.  The frontier is taken in `chunks` chunks of
// at most cand_cap / D parents each (one after another, each sees the rows
// the previous ones added); a frontier larger than that latches kErrChunks
// with the chunk count it needs in ctl->r_need.
// est: host estimate of the new set's rows, used only to size grids.
// row_limit: rows beyond which the round latches kErrOver; load_rows: rows
// beyond which it latches kErrTableFull (0: no such limit).
void expand_round(const DevModel& m, int Wi, int prec, const Side& n, int r,
                  StepCtl* ctl, int64_t cap, int64_t est, uint64_t* table,
                  uint64_t mask, const RoundBufs& rb, const Sums& sm,
                  int32_t* col, void* phi, int chunks, int64_t row_limit,
                  int64_t load_rows, int* err, hipStream_t s);
// Columns of frontier k (lookup only); sets ctl->n_new.  max_states > 0
// (one realization): the row count into ball[0], kErrCap beyond it.  p0[i]:
// row of keys0[i], i < n0, or -1.
void lookup_last(const DevModel& m, int Wi, const Side& n, int k,
                 StepCtl* ctl, int64_t est, const uint64_t* table,
                 uint64_t mask, int32_t* col, int64_t max_states,
                 uint32_t* ball, const uint64_t* keys0, int64_t n0,
                 int32_t* p0, int* err, hipStream_t s);
// Number of per-block partials written by a kernel over `rows` rows.
int part_grid(int64_t rows);
// Returns the number of mass partials written.  tmap (may be null) gets
// the new row of every old row, -1 if dropped (then sel must be null).
// sel (may be null): the selection's bits; those rows, placed by insert_rows,
// are passed over.
int transfer(const DevModel& m, int Wi, int prec, const Side& o,
             const void* psi_o, int64_t n_old, const StepCtl* ctl,
             const uint64_t* table, uint64_t mask, const uint64_t* keys_n,
             void* phi, double* mass_part, int32_t* tmap, const uint64_t* sel,
             int* err, hipStream_t s);
// Gershgorin bounds + Chebyshev coefficients per realization (cc[R]);
// latches if some K_r exceeds the launches enqueued.
void bounds_and_coef(const DevModel& m, const Side& n, const int32_t* col,
                     int64_t cap, int64_t est, StepCtl* ctl, double dt,
                     double tol, int k_max, int launched, double* part,
                     ChebCoef* cc, int* err, hipStream_t s);
// Gershgorin bounds only: per-block (lo, hi) per realization into
// part[block][R][2]; returns the number of blocks.
int bounds_part(const DevModel& m, const Side& n, const int32_t* col,
                int64_t cap, int64_t est, const StepCtl* ctl, double* part,
                const int* err, hipStream_t s);
// Clenshaw launch for index kk (see kernels.hip); buffers b[0], b[1].
// Returns the number of energy partials (written by the first launch).
// mid: the launch is expected to be a middle term (selects a kernel name).
// Batched sims (R > 1) leave the energy per row in e_row.  ev_a / ev_b
// (may be null): events the dispatch records at its start and stop.
int cheb_term(const DevModel& m, int prec, int kk, bool energy, bool mid,
              int64_t est, const StepCtl* ctl, const int32_t* col, int64_t cap,
              const Side& n, const ChebCoef* cc, const void* phi, void* b0,
              void* b1, double* e_part, double* e_row, int* err,
              hipEvent_t ev_a, hipEvent_t ev_b, hipStream_t s);
// |psi|^2 and exciton populations as per-block partials (returns their
// count, at most kPartBlocks), plus the next step's selection as bits and
// per-block sums (that count is the grid select_write needs).
int pop_norm(int prec, int N, int R, double th2, int64_t est,
             const StepCtl* ctl, const void* psi, const uint64_t* pay,
             const uint8_t* dist,
             const double* e_row, double* n2_part, double* en_part,
             double* pop_part, const Sums& sm, int* err,
             hipStream_t s);
// Commit a successful step on the device: time, discarded weight per
// realization, record count and the row count of the current set; then
// mirror *ctl and *err into mapped pinned host memory (device addresses
// h_ctl_dev, h_err_dev), also when an error is latched.
void end_step(StepCtl* ctl, int R, const double* ring, int rec_doubles,
              double* mass_tot, int* err, StepCtl* h_ctl_dev, int* h_err_dev,
              hipStream_t s);
// Reduce partials into observation record ctl->nrec (skipped when an error
// is latched, so a repeated step records once); <psi0|psi> per realization
// from its n0 initial amplitudes and their rows p0 (-1: not in the set).
// With one realization it then does what end_step does.
void obs_final(int prec, int N, int R, int want_energy, double dt, int n_mass,
               int n_e, int n_pop, const double* mass_part,
               const double* n2_part, const double* e_part,
               const double* en_part, const double* pop_part,
               const double* amps0, int64_t n0, const int32_t* p0,
               const void* psi, const ChebCoef* cc, StepCtl* ctl,
               const uint32_t* cnt, double* mass_tot, double* ring,
               int rec_doubles, int64_t ring_cap, StepCtl* h_ctl_dev,
               int* h_err_dev, int* err, hipStream_t s);

void row_info(const DevModel& m, int Wi, const uint64_t* keys, int64_t n,
              uint64_t* pay, uint64_t* tot, hipStream_t s);
void amps_to_f64(int prec, const void* src, double* dst, int64_t n,
                 hipStream_t s);
void amps_from_f64(int prec, const double* src, void* dst, int64_t n,
                   hipStream_t s);

}  // namespace paces
