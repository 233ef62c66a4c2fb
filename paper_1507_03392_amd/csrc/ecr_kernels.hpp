// ecr_kernels.hpp -- launch entry points of the gfx950 kernels (host side).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "ecr_device.hpp"
#include "ecrpic.h"

namespace ecr {

// Coulomb chunking: a workgroup owns the cells whose first sorted slot falls
// in [b*kCoulCap, (b+1)*kCoulCap); it orders up to kCoulMaxE pool members
// (ions; atoms take no room) in LDS.
constexpr int kCoulCap = 256;
constexpr int kCoulMaxE = 1024;
static_assert(kBirthNone == ECR_BIRTH_NONE, "birth sentinel");

// a launch whose error is its own (hipGetLastError could name an earlier
// call's) and is left to no later call: what a read hands back rests on it
template <typename... A, typename... B>
hipError_t launch_checked(void (*kernel)(A...), dim3 grid, dim3 block, hipStream_t st, B &&...arg) {
  return [&](A... a) {
    void *p[] = {(void *)&a...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, p, 0, st);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
  }(std::forward<B>(arg)...);
}

// Error bits raised by kernels (read back with the tallies).
enum : uint32_t { ERR_COUL_OVERFLOW = 1, ERR_PARTNER_OVERFLOW = 2 };

struct DevAccum {
  ecr_tallies t;           // steps field unused on the device
  uint32_t err;            // ERR_* bits
  uint32_t pad[63];
};

// one Coulomb work item of a chunk: chunk-relative slots a, b (and c for an
// odd pool's triplet), the pool size m and the id of a; a chunk owns
// kCoulItems items
struct CoulItem {
  uint16_t a, b, c, m;
  uint32_t id;
};
constexpr int kCoulItems = kCoulMaxE / 2;

template <typename R>
void launch_init(const KParams &P, Soa<R> S, hipStream_t st);

// push + wall/aperture + MCC; also deposits when dens != nullptr; with
// chg_cur, ionisation uses the cell's ion charge (self-consistent n_e) and
// the updated charges are summed per cell into chg_next (zeroed before)
template <typename R>
void launch_push(const KParams &P, const Tables *T, Soa<R> S, const double *ef, uint8_t *evlog,
                 DevAccum *acc, StepArg step, const uint32_t *chg_cur, uint32_t *chg_next, hipStream_t st);

// exchange partners (ECR_FLAG_CX_PARTNER): per Coulomb chunk, the atoms of
// each requesting collision cell become ions in (key, id) order; chg is the
// next step's cell grids, updated for the new charges; the requests are
// cleared, and clear_n words at clear (this step's cell grids, or none) set to
// zero
template <typename R>
void launch_cx_partner(const KParams &P, Soa<R> S, const uint32_t *chunk_lo, uint32_t *chg, uint32_t *clear,
                       int64_t clear_n, uint8_t *evlog, DevAccum *acc, StepArg step, hipStream_t st);

// |B| at every cell centre times hx, into bden[ncell] (once, at create)
void launch_cell_bden(const KParams &P, double *bden, hipStream_t st);

// ion charge per cell of the current state, added into chg (zeroed before)
template <typename R>
void launch_charge_grid(const KParams &P, Soa<R> S, uint32_t *chg, hipStream_t st);

template <typename R>
void launch_deposit(const KParams &P, Soa<R> S, double *dens, hipStream_t st);

// optional ion pressure moment (field ECR_F_ION_P)
template <typename R>
void launch_deposit_pressure(const KParams &P, Soa<R> S, double *dens, hipStream_t st);

// Coulomb chunk table: chunk b covers slots [chunk_lo[b], chunk_lo[b+1]),
// nchunks+1 entries, rebuilt after every sort
int64_t coul_nchunks(int64_t n);
void launch_coul_chunks(const uint32_t *cellid, const uint32_t *cell_off, int64_t n, uint32_t *chunk_lo, int64_t cap,
                        hipStream_t st);

// pairing (k_coul_order) then collisions (k_coul_pairs); items holds
// kCoulItems entries per chunk, counts one (pairs, triplets) per chunk
// moments: coul_moment_slots(n) x 5 doubles of per-wavefront momentum /
// energy sums, reduced into the tallies by launch_sum_moments.  The ordering
// kernel also clears zero[0..zero_n) (the next step's cell grids) when zero
// is given; it does nothing at all for n <= 1
template <typename R>
void launch_coul_order(const KParams &P, Soa<R> S, const uint32_t *cellid, const uint32_t *chunk_lo, DevAccum *acc,
                       CoulItem *items, uint2 *counts, StepArg step, uint32_t *zero, int64_t zero_n,
                       hipStream_t st);
template <typename R>
void launch_coul_pairs(const KParams &P, const Tables *T, Soa<R> S, const uint32_t *chunk_lo, const CoulItem *items,
                       const uint2 *counts, double *moments, StepArg step, hipStream_t st);
int64_t coul_moment_slots(int64_t n);
// (the tallies then to out as well, memory of the host, or null)
hipError_t launch_sum_moments(const double *moments, int64_t nslots, DevAccum *acc, DevAccum *out, hipStream_t st);

// The fused step kernels (ecr_fused.hpp): the whole step in one kernel
// (Coulomb pairing and collisions, push, wall/aperture loss, MCC, deposit),
// for one or several runs in a launch.  A run's arguments sit in its job in
// device memory (written by launch_set_job, passed by value); the launch's
// list names each job, its step and its first workgroup (run j owns
// step_wgs(n_j) workgroups from wg0[j] in launch_period, step_wgs_one(n_j) in
// launch_step).

// The chunk table, rebuilt at every sort by launch_step_prep.  The slots are
// cut into windows of kWinChunks chunks' slots; window w has its chunks at
// chunk[w kWinList] in order of slot, where a workgroup of a fixed number
// finds them: what a workgroup sums is the same from run to run.  win[w]: how
// many chunks, and << 16 how many groups, at group[w kWinGroups], a single step
// takes instead of them.  cnt[0] cells of more than kPSlots slots (first slot,
// end; in any order), and a word per slot (bk_*): the buckets of its cell in
// the ordering (2^floor(log2 m) for a cell of m slots, numbered from the
// chunk's first), its cell's number in the chunk and whether it is the cell's
// first slot.
// launch_step_units, before the first single step after a sort, puts them in a
// row without gaps: units, the chunks (of windows without groups) at flat and
// the groups at gflat, dealt out so that neighbours in space are apart
struct ChunkEntry {
  uint32_t lo, end;  // slots [lo, end)
  uint32_t x, y, z;  // the box of its cells: the lowest index along each axis,
  uint32_t wxy, wz;  // and highest - lowest, x | y << 16 and z (at most 65535: no wider box has a brick)
  uint32_t nn;       // buckets | cells << 16
  __host__ __device__ uint32_t buckets() const { return nn & 0xffffu; }
  __host__ __device__ uint32_t cells() const { return nn >> 16; }
};
// up to three chunks in a row, at most 2 kPSlots slots: all of them as one
// entry, and where the second and the third begin (or kNoPlace), counted from
// the first slot, with the buckets and cells of the chunk before them
struct GroupEntry {
  ChunkEntry all;
  uint32_t s[2], a[2];
};
constexpr uint32_t kNoPlace = 1u << 20;
// what a single step's workgroups take: the first 2 pairs chunks two at a time
// (the last of them may be missing), the others one at a time, the groups
struct StepUnits {
  uint32_t pairs, singles, groups, chunks;
};
struct ChunkTable {
  uint32_t *cnt, *win;
  ChunkEntry *chunk, *flat;
  GroupEntry *group, *gflat;
  StepUnits *units;
  uint32_t *big, *bkinfo;
};
__host__ __device__ constexpr uint32_t bk_pack(uint32_t first, uint32_t lg, uint32_t cell, bool head) {
  return first | (lg << 10) | (cell << 16) | ((uint32_t)head << 31);
}
__host__ __device__ constexpr uint32_t bk_first(uint32_t w) { return w & 0x3ffu; }
__host__ __device__ constexpr uint32_t bk_lg(uint32_t w) { return (w >> 10) & 15u; }
__host__ __device__ constexpr uint32_t bk_cell(uint32_t w) { return (w >> 16) & 0x3ffu; }
__host__ __device__ constexpr bool bk_head(uint32_t w) { return (w >> 31) != 0u; }
constexpr int kPSlots = 512;  // most slots of a chunk
constexpr int kWinChunks = 8;
// most chunks of a window: a chunk ends half a chunk size or more from its
// start, or the cell that would take it there begins the next one, so two in
// a row hold half a chunk size
constexpr int kWinList = 4 * kWinChunks + 2;
constexpr int kWinGroups = kWinList / 2;  // fewer groups than pairs
constexpr int kPlaces = 1024;  // workgroups of the step kernels that the chip holds at a time
// workgroups at the front of a run's that take cells beyond a chunk only
constexpr int kBigWG = 16;
int64_t step_fill(int64_t n);  // slots a chunk is filled up to
int64_t step_windows(int64_t n);
int64_t step_max_big(int64_t n);
uint32_t step_win_wgs(int64_t n);  // workgroups to a window's chunks
uint32_t step_wgs(int64_t n);      // workgroups of launch_period
uint32_t step_wgs_one(int64_t n);  // of launch_step, no more than those
// From here a workgroup of a single step takes two chunks: 600k ions 46 us a
// step with one, 39 with two, 1M 64 and 54, 2M 112 and 89; below, half the
// workgroups no longer fill the chip (300k 28 us with one, 33 with two; 450k
// 32 and 34).
constexpr int64_t kPairMin = 450000;
__host__ __device__ constexpr bool step_pairs(int64_t n) { return n >= kPairMin; }
void launch_step_prep(const KParams &P, ChunkTable C, hipStream_t st);
void launch_step_units(int64_t n, ChunkTable C, hipStream_t st);

// moments: slots of 5 doubles (momentum and energy sums of the collisions),
// one for each of step_wgs(n) workgroups' chunks, then one for every kPSlots +
// 1 slots, of the cell beyond kPSlots that starts there; scratch64: n 64-bit
// words of sort space for pools beyond the LDS
inline int64_t step_moment_slots(int64_t n) { return (int64_t)step_wgs(n) + step_max_big(n); }
template <typename R>
struct StepJob {
  KParams P;
  const Tables *T;
  Soa<R> S;
  ChunkTable C;
  const double *ef;  // electric node grid, or null
  uint8_t *evlog;
  DevAccum *acc;
  double *dens, *moments;
  uint64_t *scratch64;
  uint32_t windows, win_wgs;  // step_windows, step_win_wgs
};
constexpr int kMaxBatch = 32;
template <typename R>
struct StepBatch {
  const StepJob<R> *job[kMaxBatch];
  const uint32_t *stepw[kMaxBatch];  // step = *stepw + step, or step alone when stepw is null
  uint32_t step[kMaxBatch];
  uint32_t wg0[kMaxBatch + 1];
  int n;
};
// a few 32-bit words set from the launch's arguments (the step counters
// read by captured graphs)
struct SetWords {
  uint32_t *ptr[kMaxBatch];
  uint32_t val[kMaxBatch];
  int n;
};
// the cell grids of a run that has them (the only one of its launch): the
// step reads cur and adds to next, zeroed before, and sets n words at clear
// (or none) to zero
struct CellGrids {
  const uint32_t *cur;
  uint32_t *next, *clear;
  int64_t n;
};
// cur's n words to home, then zero to clear (which may be cur)
void launch_grids_home(const uint32_t *cur, uint32_t *home, uint32_t *clear, int64_t n, hipStream_t st);

// ext: optional physics (step_ext); fields: node grids of E or B.
// One step; nq: exactly the ion number and charge are deposited
bool step_ext(const KParams &P);
template <typename R>
void launch_step(const StepBatch<R> &B, bool nq, bool ext, bool fields, const CellGrids &grids, hipStream_t st);
// nsteps steps in one launch, the state on chip from the first to the last;
// for runs without cell grids (nothing then couples two chunks between
// sorts).  pressure: with the ion pressure field
template <typename R>
void launch_period(const StepBatch<R> &B, uint32_t nsteps, bool ext, bool fields, bool pressure, hipStream_t st);
template <typename R>
void launch_set_job(const StepJob<R> &J, StepJob<R> *dst, hipStream_t st);
void launch_set_words(const SetWords &w, hipStream_t st);

// sort by cell: keys either from positions or (given != nullptr) from
// given[pid].  count is zero before and after; clear[0] and clear[1] (or
// null) are zero after
template <typename R>
void launch_sort(const KParams &P, Soa<R> A, Soa<R> B, const uint32_t *given, uint32_t *key, uint32_t *rank,
                 uint32_t *count, uint32_t *cell_off, uint32_t *blocksums, uint32_t *cellid_out, int64_t ncell,
                 uint32_t *clear, hipStream_t st);

// the state by particle id into another set of arrays: q and species as bytes
// of their own, cells from cellid.  bad: set when an id is out of range
template <typename R>
hipError_t launch_state_out(const Soa<R> &A, const uint32_t *cellid, int64_t n, const Soa<R> &out, uint8_t *species,
                            uint32_t *cell, uint32_t *bad, hipStream_t st);
// a state given in order of id: charge states q (and birth, where there is a
// step for an ion) to packed charges, ids and birth steps
struct SpeciesEnds {
  int64_t end[kMaxS];
  int n;
};
void launch_state_in(const uint8_t *q, const uint32_t *birth, int64_t n, SpeciesEnds sp, uint8_t *qs, uint32_t *pid,
                     uint32_t *birth_out, hipStream_t st);

size_t scan_blocksums_len(int64_t ncell);

void launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st);
void launch_fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t st);
void launch_fill_f64(double *p, double v, int64_t n, hipStream_t st);

void launch_selftest_philox(uint64_t seed, uint32_t ctr0, uint32_t c1, uint32_t c2, uint32_t c3, int64_t n,
                            uint32_t *out, hipStream_t st);
void launch_selftest_divsqrt(const double *a, const double *b, int64_t n, double *q, double *r, hipStream_t st);

}  // namespace ecr
