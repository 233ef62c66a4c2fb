// ecr_single.hpp -- the whole ion step of the model (Mironov et al., Sec. II)
// in one launch per step: what runs with cell grids take (they couple the
// chunks at every step) and calls of a single step.
//
// A workgroup takes one chunk of whole cells, or in large runs two of them, or
// up to three in a row, kORounds rounds of kNT slots.  The parts of a step are
// those of ecr_fused.hpp, with two differences from ecr_period.hpp: all
// wavefronts make the order, whose arrays lie where the velocities go after
// it, and the deposit adds within the step, through a brick over everything
// that the pushed chunk no longer needs.
//
// What bounds it, 2M binary64 ions: 91 us a step, of which its 1006 vector
// instructions per particle take 51 to issue and the state's 212 MB 41 at the
// rate of a large copy.
#pragma once

#include "ecr_fused.hpp"

namespace ecr {

namespace {

constexpr int kOSlots = 2 * kPSlots;
constexpr int kORounds = kOSlots / kNT;
constexpr int kCRounds = kPSlots / kNT;  // rounds of a chunk

template <typename R>
struct OneShared {
  union {
    R v[3 * kOSlots];     // velocities, then the offsets in the base cell
    Ordering<kOSlots> o;  // before them
  };
  uint32_t sid[kOSlots];
  union {
    WorkList<kOSlots> item;
    uint64_t base[kOSlots];  // after the push: base cell (pack_cell) | charge << 32, 255 for none
  };
  uint8_t sqs[kOSlots];
  double cacc[5 * 64];  // the collisions' momentum and energy sums, an entry per lane number
  // the density brick takes everything but the collisions' sums
  static constexpr int kBrick = (int)(sizeof(R[3 * kOSlots]) > sizeof(Ordering<kOSlots>) ? sizeof(R[3 * kOSlots])
                                                                                         : sizeof(Ordering<kOSlots>)) /
                                    8 +
                                (4 * kOSlots + 8 * kOSlots + kOSlots) / 8;
};

// a chunk's entry through scalar loads: the table was made before the launch
using EntryPtr = const __attribute__((address_space(4))) ChunkEntry *;
__device__ __forceinline__ ChunkEntry entry(EntryPtr p, uint32_t e) { return ((const ChunkEntry *)p)[e]; }

// one step of the chunks E[0] and, two of them, E[1]; ROW: of the group (or
// cell) E[0], its slots past kPSlots in the second half of the workgroup's
// places, whose chunks begin at G.s; the cell grids chg_cur and chg_next (or
// null) are read and summed.  NQ: exactly the ion number and charge are
// deposited.
template <typename R, int FLD, bool EXT, bool NQ, bool ROW>
__device__ __forceinline__ void chunk_step(const JobPtr<R> job, const ChunkEntry (&E)[2], const bool two,
                                           const GroupEntry &G, double *__restrict__ mslot, const uint32_t step, OneShared<R> &sh,
                                           uint32_t *wsum, uint32_t *tot, const int turn,
                                           const uint32_t *__restrict__ chg_cur, uint32_t *__restrict__ chg_next) {
  const int tid = threadIdx.x;
  const int64_t lo[2] = {E[0].lo, ROW ? E[0].lo + kPSlots : two ? E[1].lo : 0u};
  const int n0 = (int)(E[0].end - E[0].lo);
  const int n[2] = {ROW ? min(n0, kPSlots) : n0, ROW ? max(n0 - kPSlots, 0) : two ? (int)(E[1].end - E[1].lo) : 0};
  const int nb0 = ROW ? 0 : (int)E[0].buckets(), nh0 = ROW ? 0 : (int)E[0].cells();
  const int nb = ROW ? (int)E[0].buckets() : nb0 + (two ? (int)E[1].buckets() : 0);
  const int nh = ROW ? (int)E[0].cells() : nh0 + (two ? (int)E[1].cells() : 0);
  const bool coul = (job->P.pmask & P_COULOMB) != 0 && n[0] + n[1] >= 2;
  const bool mcc = needs_mcc_uniform(fresh<R>(job).P);
  const uint32_t dm = job->dens ? (NQ ? 3u : job->P.dmask & 7u) : 0u;
  const bool dep = dm != 0u;

  // 1-2. the STEP draws and the pools' order.  The velocities stay in
  // registers until then, so that the draws wait for the ids only (the
  // memory counter drains in the order of the loads)
  R v0[kORounds][3];
  uint32_t w0[kORounds], key[kORounds], bk[kORounds], id[kORounds];
  uint8_t qs[kORounds];
  {
    const StepJob<R> &J = fresh<R>(job);
    const Soa<R> S = J.S;
    const uint32_t *bkinfo = J.C.bkinfo;
    rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      w0[k] = key[k] = bk[k] = id[k] = 0u;
      qs[k] = 0;
      v0[k][0] = v0[k][1] = v0[k][2] = (R)0;
    });
    rounds<2>([&](auto cc) __attribute__((always_inline)) {
      constexpr int c = decltype(cc)::value;
      if (n[c] == 0) return;  // uniform
      int64_t t[kCRounds];
#pragma unroll
      for (int k = 0; k < kCRounds; ++k) t[k] = lo[c] + min(tid + k * kNT, n[c] - 1);
#pragma unroll
      for (int k = 0; k < kCRounds; ++k) id[c * kCRounds + k] = S.pid[t[k]];
#pragma unroll
      for (int k = 0; k < kCRounds; ++k) {
        qs[c * kCRounds + k] = S.qs[t[k]];
        bk[c * kCRounds + k] = bkinfo[t[k]];
        if (ROW) {
          const uint32_t q = (uint32_t)(tid + (c * kCRounds + k) * kNT);
          bk[c * kCRounds + k] += (q >= G.s[0] ? G.a[0] : 0u) + (q >= G.s[1] ? G.a[1] : 0u);
        }
      }
#pragma unroll
      for (int k = 0; k < kCRounds; ++k) {
        v0[c * kCRounds + k][0] = S.vx[t[k]];
        v0[c * kCRounds + k][1] = S.vy[t[k]];
        v0[c * kCRounds + k][2] = S.vz[t[k]];
      }
    });
  }
  if (coul) {
    for (int i = tid; i < kOSlots; i += kNT) sh.o.hist[i] = 0u;
    if (tid == 0) sh.o.cellb[nh] = (uint16_t)nb;
  }
  rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value, c = k / kCRounds;
    const int q = tid + k * kNT;
    if (tid + (k % kCRounds) * kNT < n[c]) {
      sh.sid[q] = id[k];
      sh.sqs[q] = qs[k];
      if (coul && bk_head(bk[k])) sh.o.cellb[bk_cell(bk[k]) + (c ? nh0 : 0)] = (uint16_t)(bk_first(bk[k]) + (c ? nb0 : 0));
    }
  });
  for (int i = tid; i < 5 * 64; i += kNT) sh.cacc[i] = 0.0;
  {
    const KParams &P = fresh<R>(job).P;
    if (mcc || coul)
      rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value, c = k / kCRounds;
        if (n[c] > 0) {
          const uint4 W = draw(P, id[k], step, S_STEP, 0);
          w0[k] = W.x;
          key[k] = W.z;
        }
      });
  }
  if (coul) {
    uint32_t arr[kORounds];
    const auto pool = [&](int k) { return tid + (k % kCRounds) * kNT < n[k / kCRounds] && q_of(qs[k]) >= 1; };
    __syncthreads();
    rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value, c = k / kCRounds;
      // the bucket and the cell of both chunks together
      const uint32_t b = (uint32_t)bucket_of(bk[k], key[k]) + (c ? (uint32_t)nb0 : 0u);
      bk[k] = b | ((bk_cell(bk[k]) + (c ? (uint32_t)nh0 : 0u)) << 16);
      arr[k] = 0u;
      if (pool(k)) arr[k] = atomicAdd(&sh.o.hist[b], 1u);
    });
    __syncthreads();
    (void)wg_exscan<kNT>(sh.o.hist, nb, wsum, true);  // hist[nb] = members in all
    rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      if (pool(k)) sh.o.bkey[sh.o.hist[bk[k] & 0xffffu] + arr[k]] = ((uint64_t)key[k] << 32) | id[k];
    });
    if (tid < 64) number_items(sh.o, nh, nb, tot);
    __syncthreads();
    rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      if (pool(k)) list_member(sh.o, sh.item, (int)(bk[k] & 0xffffu), bk[k] >> 16, key[k], id[k], tid + k * kNT);
    });
    __syncthreads();
  }
  rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value, c = k / kCRounds;
    const int q = tid + k * kNT;
    if (tid + (k % kCRounds) * kNT < n[c]) {
      sh.v[q] = v0[k][0];
      sh.v[kOSlots + q] = v0[k][1];
      sh.v[2 * kOSlots + q] = v0[k][2];
    }
  });
  // 3. the collisions
  if (coul) {
    __syncthreads();
    collide_list<R, kNT, kOSlots>(job, LdsAcc<R, kOSlots>{sh.v, sh.sqs}, sh.sid, sh.item, sh.cacc, (int)tot[0],
                                  (int)tot[1], (tid + turn) & (kNT - 1), step);
  }
  // 4. push, losses, Monte Carlo collisions (positions on their way while the
  // wavefronts wait for each other)
  R x[kORounds], y[kORounds], z[kORounds];
  {
    const Soa<R> S = fresh<R>(job).S;
    rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      x[k] = y[k] = z[k] = (R)0;
    });
    rounds<2>([&](auto cc) __attribute__((always_inline)) {
      constexpr int c = decltype(cc)::value;
      if (n[c] == 0) return;
#pragma unroll
      for (int k = 0; k < kCRounds; ++k) {
        const int64_t t = lo[c] + min(tid + k * kNT, n[c] - 1);
        x[c * kCRounds + k] = S.x[t];
        y[c * kCRounds + k] = S.y[t];
        z[c * kCRounds + k] = S.z[t];
      }
    });
  }
  if (coul) {
    __syncthreads();
    add_moments(sh.cacc, mslot);
  }
  rounds<kORounds>([&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value, c = k / kCRounds;
    if (n[c] == 0) return;  // uniform
    const int j = tid + (k % kCRounds) * kNT, q = tid + k * kNT;
    uint32_t ccell = 0xffffffffu, cq = 0u;
    if (j < n[c]) {
      const StepJob<R> &J = fresh<R>(job);
      const KParams &P = J.P;
      const Soa<R> S = soa_at(J.S, lo[c]);
      R vx = sh.v[q], vy = sh.v[kOSlots + q], vz = sh.v[2 * kOSlots + q];
      const int s = sp_of(qs[k]);
      int Q = q_of(qs[k]);
      const uint8_t ev = advance<R, FLD, EXT>(P, J.T, J.ef, J.acc, step, id[k], s, Q, x[k], y[k], z[k], vx, vy, vz,
                                              S.birth, j, lo[c] + j, chg_cur, w0[k]);
      S.x[j] = x[k];
      S.y[j] = y[k];
      S.z[j] = z[k];
      S.vx[j] = vx;
      S.vy[j] = vy;
      S.vz[j] = vz;
      S.qs[j] = make_qs(Q, s);
      if (EXT && chg_next) {
        // the next step's cell grids: ion charge in channel 0, atoms of
        // species s in channel 1 + s
        const uint32_t cell = cell_of<R>(P, x[k], y[k], z[k]);
        ccell = Q >= 1 ? cell : (uint32_t)(1 + s) * P.ncell + cell;
        cq = Q >= 1 ? (uint32_t)Q : 1u;
      }
      if (J.evlog) J.evlog[lo[c] + j] = ev;
      if (dep) {
        int ix, iy, iz;
        R tx, ty, tz;
        cic_axis<R>(x[k], (R)P.R0, (R)P.idx, P.nx, ix, tx);
        cic_axis<R>(y[k], (R)P.R0, (R)P.idy, P.ny, iy, ty);
        cic_axis<R>(z[k], (R)P.hL, (R)P.idz, P.nz, iz, tz);
        const bool on = Q >= 1 ? (dm & 3u) != 0u : (dm & 4u) != 0u;
        // staged for the brick: the offsets over the slot's velocity, which
        // only its own lane still reads
        sh.v[q] = tx;
        sh.v[kOSlots + q] = ty;
        sh.v[2 * kOSlots + q] = tz;
        sh.base[q] = pack_cell(P, ix, iy, iz) | ((uint64_t)(uint32_t)(on ? Q : 255) << 32);
      }
    }
    if (EXT && chg_next) add_charge(chg_next, ccell, cq);  // all lanes: the run sums use lane moves
  });
  if (!dep) return;

  // 5. the deposit through a brick over both chunks' cells, or one for each
  // where that is smaller (the two need not be neighbours)
  const int nf = 2 + ((dm & 4u) ? 1 : 0);
  double *const brick = reinterpret_cast<double *>(&sh);
  Box box[2];
  int at0[2] = {0, 0};  // their first doubles
  bool one_box = false;
  {
    const KParams &P = fresh<R>(job).P;
    const int cap = OneShared<R>::kBrick / nf;
    int ba[6], bb[6], u[6];
    cell_box(E[0], ba);
    box[0] = make_box(P, ba, two && !ROW ? cap / 2 : cap);
    box[1] = Box{0, 0, 0, 1, 1, 0};
    if (ROW) {
      box[1] = box[0];
      one_box = true;
    } else if (two) {
      cell_box(E[1], bb);
      box[1] = make_box(P, bb, cap / 2);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        u[d] = min(ba[d], bb[d]);
        u[3 + d] = max(ba[3 + d], bb[3 + d]);
      }
      const Box both = make_box(P, u, cap);
      if (both.nodes && (box[0].nodes == 0 || box[1].nodes == 0 || both.nodes <= box[0].nodes + box[1].nodes)) {
        box[0] = both;
        box[1] = both;
        one_box = true;
      } else {
        at0[1] = nf * box[0].nodes;
      }
    }
  }
  const int nbrick = one_box ? nf * box[0].nodes : nf * (box[0].nodes + box[1].nodes);
  const StepJob<R> &J = fresh<R>(job);
  const int nx1 = J.P.nx1, nxy1 = J.P.nx1 * J.P.ny1;
  // a base cell's place in its chunk's brick, or kOut + its node outside
  constexpr int64_t kOut = 1ll << 32;
  const auto place = [&](const Box &b, int ix, int iy, int iz) -> int64_t {
    const int i = b.at(ix, iy, iz);
    return i >= 0 ? (int64_t)i : kOut + (ix + nx1 * iy + nxy1 * iz);
  };
  const auto add = [&](const Box &b, int first, int64_t at, int f, int c, double v) {
    if (at < kOut) {
      atomicAdd(&brick[first + f * b.nodes + (int)at + ((c & 1) + ((c & 2) ? b.bx : 0) + ((c & 4) ? b.bx * b.by : 0))], v);
    } else {
      unsafeAtomicAdd(&J.dens[(int64_t)f * J.P.nnode + (at - kOut) + ((c & 1) + ((c & 2) ? nx1 : 0) + ((c & 4) ? nxy1 : 0))],
                      v);
    }
  };
  __syncthreads();
  // a lane takes four consecutive slots and sums its runs of equal cells;
  // the lanes' last runs are summed over groups of four lanes (every slot's
  // weights straight to the brick, for chunks of fewer than six slots a
  // cell, took 77 us where this takes 63: one step of push and deposit of a
  // settled 2M run; no gain at one slot a cell either)
  DepIn<R> D;
  constexpr int kLanes = kPSlots / 4;  // of a chunk, whole wavefronts
  const int c = tid / kLanes, j0 = 4 * (tid % kLanes), q0 = 4 * tid;
  static_assert(kOSlots == 4 * kNT, "four slots per lane");
#pragma unroll
  for (int p = 0; p < 4; ++p) D.on[p] = false;
  if (j0 < (c ? n[1] : n[0])) {
    lds_load4(&sh.v[q0], D.tx);
    lds_load4(&sh.v[kOSlots + q0], D.ty);
    lds_load4(&sh.v[2 * kOSlots + q0], D.tz);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint64_t b = sh.base[q0 + p];
      unpack_cell(J.P, (uint32_t)b, D.ix[p], D.iy[p], D.iz[p]);
      D.q[p] = (int)(b >> 32);
      D.on[p] = j0 + p < (c ? n[1] : n[0]) && D.q[p] != 255;
    }
  }
  __syncthreads();
  for (int i = tid; i < nbrick; i += kNT) brick[i] = 0.0;
  __syncthreads();
  const int cu = __builtin_amdgcn_readfirstlane(c);  // uniform over a wavefront
  const Box bx = cu ? box[1] : box[0];
  const int first = cu ? at0[1] : 0;
  const auto add1 = [&](int64_t at, int f, int cc, double v) { add(bx, first, at, f, cc, v); };
  DepRun L;
  run_accumulate<R, true>(
      D, dm, [&](int ix, int iy, int iz) { return place(bx, ix, iy, iz); }, add1, L);
  int seg;
  bool tail;
  wave_runs(L.node, seg, tail);
  const GroupSteps<4> st = group_steps<4>(seg);
  const bool out = (tail || (tid & 3) == 3) && L.node >= 0;
  for (int cc = 0; cc < 8; ++cc) {
    if (dm & 1u) {
      const double v = group_scan<4>(st, L.a[cc]);
      if (out && v != 0.0) add1(L.node, 0, cc, v);
    }
    if (dm & 2u) {
      const double v = group_scan<4>(st, L.b[cc]);
      if (out && v != 0.0) add1(L.node, 1, cc, v);
    }
    if (dm & 4u) {
      const double v = group_scan<4>(st, L.c[cc]);
      if (out && v != 0.0) add1(L.node, 2, cc, v);
    }
  }
  __syncthreads();
  flush_brick<R>(job, brick, box[0], nf, false);
  if (two && !one_box) flush_brick<R>(job, brick + at0[1], box[1], nf, false);
}

// one step (four workgroups per CU, by the LDS and by the registers)
template <typename R, int FLD, bool EXT, bool NQ>
__global__ void __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_step(StepBatch<R> B, CellGrids grids) {
  __shared__ __align__(16) OneShared<R> sh;
  __shared__ uint32_t wsum[kNW], tot[2];
  static_assert(sizeof(sh) + 64 <= 40 * 1024, "four workgroups share a CU's 160 KB");
  __shared__ uint32_t red[kNW], gcount;
  const RunWG own = run_of(B);
  const JobPtr<R> job = (JobPtr<R>)B.job[own.run];
  const uint32_t step = StepArg{B.stepw[own.run], B.step[own.run]}.get();
  const ChunkTable C = fresh<R>(job).C;
  const EntryPtr table = (EntryPtr)C.flat;
  const uint32_t per = step_pairs(job->P.n) ? 2u : 1u;
  uint32_t u = own.wg - kBigWG;  // (the first kBigWG: none)
  // the table has room for these two whatever it holds; their loads do not
  // wait for the number of chunks
  const uint32_t at = own.wg >= (uint32_t)kBigWG ? per * u : 0u;
  ChunkEntry E[2] = {entry(table, at), entry(table, at + 1)};
  const StepUnits N = *(const StepUnits *)(const __attribute__((address_space(4))) StepUnits *)C.units;
  const uint32_t nbig = *(const __attribute__((address_space(4))) uint32_t *)C.cnt;
  const uint32_t chunked = N.pairs + N.singles, units = chunked + N.groups;
  if (own.wg >= (uint32_t)kBigWG)
    for (; u < chunked; u += own.nwg - kBigWG) {
      const bool pair = u < N.pairs;
      const uint32_t a = pair ? 2u * u : u + N.pairs, b = min(a + 1u, N.chunks - 1u);
      if (a != at) {
        E[0] = entry(table, a);
        E[1] = entry(table, b);
      }
      chunk_step<R, FLD, EXT, NQ, false>(job, E, pair && a + 1u < N.chunks, GroupEntry{}, job->moments + 5 * (int64_t)own.wg,
                                         step, sh, wsum, tot, 64 * (int)(own.wg % kNW), grids.cur, grids.next);
      __syncthreads();  // the next ones reuse the LDS
    }
  else
    u = units;
  // the groups, after the chunks; the cells beyond a chunk, by all of the run's
  // workgroups in turn
  for (uint32_t e = own.wg; u < units || e < nbig;) {
    GroupEntry G;
    double *mslot;
    bool row = true;
    if (u < units) {
      G = ((const GroupEntry *)(const __attribute__((address_space(4))) GroupEntry *)C.gflat)[u - chunked];
      mslot = job->moments + 5 * (int64_t)own.wg;
      u += own.nwg - kBigWG;
    } else {
      const uint32_t lo = C.big[2 * e], end = C.big[2 * e + 1];
      row = end - lo <= 2u * kPSlots;
      G = cell_entry(fresh<R>(job).P, lo, end);
      mslot = cell_moments<R>(job, lo);
      e += own.nwg;
    }
    if (row) {
      const ChunkEntry M[2] = {G.all, G.all};
      chunk_step<R, FLD, EXT, NQ, true>(job, M, G.all.end - G.all.lo > (uint32_t)kPSlots, G, mslot, step, sh, wsum, tot,
                                        64 * (int)(own.wg % kNW), grids.cur, grids.next);
      __syncthreads();
    } else {
      const StepJob<R> &J = fresh<R>(job);
      big_cell<R, FLD, EXT, false, kNT, (int)sizeof(sh)>(J.P, J.T, J.S, J.ef, G.all.lo, G.all.end, J.evlog, J.acc, J.dens,
                                                         mslot, J.scratch64, step, grids.cur, grids.next,
                                                         (unsigned char *)&sh, red, &gcount);
    }
  }
  if (EXT) clear_grid(grids_arg<R>());
}

}  // namespace

template <typename R, int FLD, bool EXT>
static void launch_step_e(const StepBatch<R> &B, bool nq, const CellGrids &grids, hipStream_t st) {
  const dim3 g(B.wg0[B.n]), b(kNT);
  if (nq) hipLaunchKernelGGL((k_step<R, FLD, EXT, true>), g, b, 0, st, B, grids);
  else hipLaunchKernelGGL((k_step<R, FLD, EXT, false>), g, b, 0, st, B, grids);
}

template <typename R>
void launch_step(const StepBatch<R> &B, bool nq, bool ext, bool fields, const CellGrids &grids, hipStream_t st) {
  if (B.n <= 0 || B.wg0[B.n] == 0) return;
  if (fields) launch_step_e<R, 7, true>(B, nq, grids, st);
  else if (ext || grids.cur) launch_step_e<R, 0, true>(B, nq, grids, st);
  else launch_step_e<R, 0, false>(B, nq, CellGrids{}, st);
}

}  // namespace ecr
