// ecr_period.hpp -- the whole ion step of the model (Mironov et al., Sec. II)
// over several steps in one launch, and what it shares with the kernel of a
// single step (ecr_single.hpp).  Between two sorts by cell a chunk of whole
// collision cells is coupled to no other one except through sums (densities,
// tallies), so its workgroup runs all the steps up to the next sort with its
// particles on the chip: velocities, ids and charges in LDS, positions in
// registers, read from HBM once and written once per launch instead of once
// per step.
//
// Per step:
//  1. lane = slot: one STEP draw per particle (words 0-1 its Monte-Carlo
//     uniform, word 2 its pairing key);
//  2. the pool of each cell ordered by (key, id) in LDS: an LDS histogram of
//     the keys' top bits over the cell's buckets (tabulated at the sort), its
//     scan, the (key, id) listed by bucket, and a member's rank from its
//     bucket mates; the cells' pairs and triplets are numbered, so a member
//     writes its slot straight to its place in the work list;
//  3. the collisions in LDS, one binary collision per lane and iteration (a
//     triplet is three in a row in its lane);
//  4. lane = slot, kRounds rounds of kNT: push, walls and aperture, Monte
//     Carlo collisions;
//  5. the deposit, summed over time instead of over space: a slot keeps the
//     eight corner weights of its current cell and charge and adds the
//     step's weights to them; only when the particle leaves its cell or
//     changes its charge (a few in a thousand per step) do the sums go out,
//     to an LDS brick over the chunk's cells and their neighbours or,
//     outside it, to HBM.  The charge field is charge times the same sums.
// One wavefront does 1-2 of step n + 1 while the other three do 3 of step n:
// the order needs the ids and charges only, and an event that makes an ion
// an atom or an atom an ion has it made again.  At the end the slots' last
// sums are added over the runs of equal cells of each wavefront, the brick
// goes to HBM with one FP64 atomic per touched node, the state is stored.
//
// What bounds it, 2M binary64 ions, 50 steps a launch: 75 us a step (a launch
// per step, ecr_single.hpp: 91).  Its 748 vector instructions per
// particle-step take 38 us of them to issue; the rest is the latency of the
// collisions' chains, of LDS and of scratch memory that four wavefronts per
// SIMD do not hide.  The sums over time and the registers that do not fit
// (256 bytes a lane) go through scratch memory, 180 MB a step at 2.4 TB/s.
// 10M ions in binary32-mixed: 352 us a step, 821 instructions, 209 us.
#pragma once

#include "ecr_single.hpp"

namespace ecr {

namespace {

constexpr int kRounds = kPSlots / kNT;  // rounds of kNT slots
// four workgroups share a CU's 160 KB
constexpr int kLds = 40 * 1024 - 80;

template <typename R>
struct FusedShared {
  R v[3 * kPSlots];  // velocities
  Ordering<kPSlots> o;
  uint32_t sid[kPSlots];
  uint16_t w16[2][kPSlots];   // the leading 16 bits of a slot's Monte-Carlo uniform in the current and the next step
  WorkList<kPSlots> item[2];  // of the current and the next step
  uint8_t sqs[kPSlots];
  double cacc[5 * 64];        // the collisions' momentum and energy sums, an entry per lane number
};
template <typename R>
struct FusedLds {
  static constexpr int kBrick = (kLds - (int)sizeof(FusedShared<R>)) / 8;
  FusedShared<R> s;
  double brick[kBrick];  // of the densities
};

// The STEP draws and (order) the pools' order of a whole chunk for one step
// by one wavefront, into work list and uniforms number buf.  The wavefront's
// LDS operations execute in order, so it needs no barrier; the fences keep
// the compiler's order.
template <typename R>
__device__ __forceinline__ void order_wave(const JobPtr<R> job, const ChunkEntry &E, uint32_t step,
                                           FusedShared<R> &sh, uint32_t *tot, bool order, int buf) {
  constexpr int kG = 4;  // draws interleaved
  constexpr int kN = kPSlots / 64;
  const int lane = threadIdx.x & 63;
  const int nsl = (int)(E.end - E.lo), nb = (int)E.buckets();
  const StepJob<R> &J = fresh<R>(job);
  const KParams &P = J.P;
  Ordering<kPSlots> &o = sh.o;
  const uint32_t *bkinfo = J.C.bkinfo + E.lo;
  const auto fence = []() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  // per slot: key; bucket | place in it << 10 | cell << 20 | member << 31
  uint32_t key[kN], at[kN];
  static_assert(kPSlots <= 512, "bucket, place and cell fit their bits");
  uint4 *h4 = reinterpret_cast<uint4 *>(&o.hist[8 * lane]);
  h4[0] = make_uint4(0u, 0u, 0u, 0u);
  h4[1] = make_uint4(0u, 0u, 0u, 0u);
  fence();
  rounds<kN / kG>([&](auto gc) __attribute__((always_inline)) {
    constexpr int g = decltype(gc)::value * kG;
    if (64 * g >= nsl) return;  // uniform
    rounds<kG>([&](auto rc) __attribute__((always_inline)) {
      constexpr int r = g + decltype(rc)::value;
      const int j = min(lane + 64 * r, nsl - 1);  // lanes past the end repeat the last slot, as no member
      const uint32_t w = order ? bkinfo[j] : 0u;
      const uint4 W = draw(P, sh.sid[j], step, S_STEP, 0);
      sh.w16[buf][j] = (uint16_t)(W.x >> 16);
      key[r] = W.z;
      const bool pool = order & (lane + 64 * r < nsl) & (q_of(sh.sqs[j]) >= 1);
      at[r] = (uint32_t)bucket_of(w, W.z) | (bk_cell(w) << 20) | ((uint32_t)pool << 31);
    });
    rounds<kG>([&](auto rc) __attribute__((always_inline)) {
      constexpr int r = g + decltype(rc)::value;
      if (at[r] >> 31) at[r] |= atomicAdd(&o.hist[at[r] & 0x3ffu], 1u) << 10;
    });
  });
  if (!order) return;
  fence();
  {
    const uint4 a = h4[0], b = h4[1];
    uint32_t s[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}, sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t v = s[k];
      s[k] = sum;
      sum += v;
    }
    const uint32_t incl = wave_incl_scan(sum), ex = incl - sum;
    h4[0] = make_uint4(ex + s[0], ex + s[1], ex + s[2], ex + s[3]);
    h4[1] = make_uint4(ex + s[4], ex + s[5], ex + s[6], ex + s[7]);
    if (lane == 63) o.hist[kPSlots] = incl;
  }
  fence();
  rounds<kN>([&](auto rc) __attribute__((always_inline)) {
    constexpr int r = decltype(rc)::value;
    if (64 * (r / kG * kG) >= nsl) return;
    if (at[r] >> 31)
      o.bkey[o.hist[at[r] & 0x3ffu] + ((at[r] >> 10) & 0x3ffu)] =
          ((uint64_t)key[r] << 32) | sh.sid[lane + 64 * r];
  });
  number_items(o, (int)E.cells(), nb, tot + 2 * buf);
  fence();
  rounds<kN>([&](auto rc) __attribute__((always_inline)) {
    constexpr int r = decltype(rc)::value;
    if (64 * (r / kG * kG) >= nsl) return;
    if (at[r] >> 31)
      list_member(o, sh.item[buf], (int)(at[r] & 0x3ffu), (at[r] >> 20) & 0x3ffu, key[r], sh.sid[lane + 64 * r],
                  lane + 64 * r);
  });
}

// nsteps steps of the chunk E; PR: the ion pressure field is deposited as well
template <typename R, int FLD, bool EXT, bool PR>
__device__ __forceinline__ void chunk_steps(const JobPtr<R> job, const ChunkEntry &E,
                                            double *__restrict__ mslot, const uint32_t step0, const uint32_t nsteps,
                                            FusedLds<R> &lds, uint32_t *tot, const int turn) {
  FusedShared<R> &sh = lds.s;
  const int tid = threadIdx.x;
  const int64_t lo = E.lo;
  const int nsl = (int)(E.end - E.lo);
  const bool coul = (job->P.pmask & P_COULOMB) != 0 && nsl >= 2;
  const uint32_t dm = job->dens ? job->P.dmask & 7u : 0u;
  const bool dep = PR || dm != 0u;

  // the state into registers and LDS (indices clamped to the chunk)
  R x[kRounds], y[kRounds], z[kRounds];
  {
    const StepJob<R> &J = fresh<R>(job);
    const Soa<R> S = soa_at(J.S, lo);
    const uint32_t *bkinfo = J.C.bkinfo + lo;
    R v0[kRounds][3];
    uint32_t bk[kRounds], id[kRounds];
    uint8_t qs[kRounds];
    int j[kRounds];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) j[k] = min(tid + k * kNT, nsl - 1);
#pragma unroll
    for (int k = 0; k < kRounds; ++k) id[k] = S.pid[j[k]];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) qs[k] = S.qs[j[k]];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) bk[k] = bkinfo[j[k]];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
      v0[k][0] = S.vx[j[k]];
      v0[k][1] = S.vy[j[k]];
      v0[k][2] = S.vz[j[k]];
    }
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
      x[k] = S.x[j[k]];
      y[k] = S.y[j[k]];
      z[k] = S.z[j[k]];
    }
    if (tid == 0) sh.o.cellb[E.cells()] = (uint16_t)E.buckets();
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
      if (tid + k * kNT < nsl) {
        sh.sid[j[k]] = id[k];
        sh.sqs[j[k]] = qs[k];
        if (bk_head(bk[k])) sh.o.cellb[bk_cell(bk[k])] = (uint16_t)bk_first(bk[k]);
        sh.v[j[k]] = v0[k][0];
        sh.v[kPSlots + j[k]] = v0[k][1];
        sh.v[2 * kPSlots + j[k]] = v0[k][2];
      }
    }
  }
  double *const brick = lds.brick;
  const int nf = 2 + ((dm & 4u) ? 1 : 0) + (PR ? 1 : 0);
  Box box{0, 0, 0, 1, 1, 0};
  if (dep) {
    int bb[6];
    cell_box(E, bb);
    box = make_box(fresh<R>(job).P, bb, FusedLds<R>::kBrick / nf);
    for (int i = tid; i < nf * box.nodes; i += kNT) brick[i] = 0.0;
  }
  // the deposit sums of each slot: base node (-1: none) and weights; the
  // charge they are for is the slot's
  double a[kRounds][8], ap[kRounds][8];  // ap: pressure (PR)
  int cn[kRounds];
#pragma unroll
  for (int k = 0; k < kRounds; ++k) {
    cn[k] = -1;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      a[k][c] = 0.0;
      if (PR) ap[k][c] = 0.0;
    }
  }
  // corner sums s (of weights), sq (of charge times weight) and sp (pressure)
  // of base node `node` go out; ion: number, charge and pressure, else atoms
  const auto put = [&](int node, bool ion, const double *s, const double *sq, const double *sp) {
    const StepJob<R> &J = fresh<R>(job);
    const int nx1 = J.P.nx1, ny1 = J.P.ny1, nxy1 = nx1 * ny1;
    const int r = (int)((uint32_t)node / (uint32_t)nx1), iz = (int)((uint32_t)r / (uint32_t)ny1);
    const int li = box.at(node - r * nx1, r - iz * ny1, iz);
    if (li >= 0) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int o = li + (c & 1) + ((c & 2) ? box.bx : 0) + ((c & 4) ? box.bx * box.by : 0);
        if (ion) {
          if (dm & 1u) atomicAdd(&brick[o], s[c]);
          if (dm & 2u) atomicAdd(&brick[box.nodes + o], sq[c]);
          if (PR) atomicAdd(&brick[(nf - 1) * box.nodes + o], sp[c]);
        } else {
          atomicAdd(&brick[2 * box.nodes + o], s[c]);
        }
      }
    } else {
      const int64_t nnode = J.P.nnode;
      double *d0 = J.dens + node;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        double *d = d0 + ((c & 1) + ((c & 2) ? nx1 : 0) + ((c & 4) ? nxy1 : 0));
        if (ion) {
          if (dm & 1u) unsafeAtomicAdd(d, s[c]);
          if (dm & 2u) unsafeAtomicAdd(d + nnode, sq[c]);
          if (PR) unsafeAtomicAdd(d + 3 * nnode, sp[c]);
        } else {
          unsafeAtomicAdd(d + 2 * nnode, s[c]);
        }
      }
    }
  };
  if (tid == 0) tot[4] = 0u;
  for (int i = tid; i < 5 * 64; i += kNT) sh.cacc[i] = 0.0;
  __syncthreads();

  const int ct = (tid + turn) & (kNT - 1);  // the lane counted from the chunk's first wavefront
  if (ct >= kNT - 64) order_wave<R>(job, E, step0, sh, tot, coul, 0);
  __syncthreads();
  for (uint32_t it = 0; it < nsteps; ++it) {
    const uint32_t step = step0 + it;
    const int cur = (int)(it & 1u);
    // 1-2. the next step's draws and order, by the chunk's last wavefront
    // beside the collisions of this one
    if (ct >= kNT - 64 && it + 1 < nsteps) order_wave<R>(job, E, step + 1, sh, tot, coul, cur ^ 1);
    // 3. the collisions
    if (coul)
      collide_list<R, kNT - 64, kPSlots>(job, LdsAcc<R, kPSlots>{sh.v, sh.sqs}, sh.sid, sh.item[cur], sh.cacc,
                                         (int)tot[2 * cur], (int)tot[2 * cur + 1], ct, step);
    __syncthreads();
    // 4-5. push, losses, Monte Carlo collisions, deposit
    rounds<kRounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      const int j = tid + k * kNT;
      if (j < nsl) {
        const StepJob<R> &J = fresh<R>(job);
        const KParams &P = J.P;
        R vx = sh.v[j], vy = sh.v[kPSlots + j], vz = sh.v[2 * kPSlots + j];
        const uint8_t qs = sh.sqs[j];
        const int Q0 = q_of(qs), s = sp_of(qs);
        int Q = Q0;
        const uint8_t ev = advance<R, FLD, EXT>(P, J.T, J.ef, J.acc, step, sh.sid[j], s, Q, x[k], y[k], z[k], vx, vy,
                                                vz, J.S.birth + lo, j, lo + j, nullptr,
                                                (uint32_t)sh.w16[cur][j] << 16);
        sh.v[j] = vx;
        sh.v[kPSlots + j] = vy;
        sh.v[2 * kPSlots + j] = vz;
        if (ev != EV_NONE) [[unlikely]] {
          sh.sqs[j] = make_qs(Q, s);
          if ((Q >= 1) != (Q0 >= 1)) tot[4] = 1u;  // a pool gained or lost a member
        }
        if (J.evlog && it + 1 == nsteps) J.evlog[lo + j] = ev;
        if (dep) {
          int ix, iy, iz;
          R tx, ty, tz;
          cic_axis<R>(x[k], (R)P.R0, (R)P.idx, P.nx, ix, tx);
          cic_axis<R>(y[k], (R)P.R0, (R)P.idy, P.ny, iy, ty);
          cic_axis<R>(z[k], (R)P.hL, (R)P.idz, P.nz, iz, tz);
          const bool on = Q >= 1 ? PR || (dm & 3u) != 0u : (dm & 4u) != 0u;
          const int node = on ? ix + P.nx1 * (iy + P.ny1 * iz) : -1;
          if (node != cn[k] || Q != Q0) [[unlikely]] {
            if (cn[k] >= 0) {
              double aq[8];
#pragma unroll
              for (int c = 0; c < 8; ++c) aq[c] = (double)Q0 * a[k][c];
              put(cn[k], Q0 >= 1, a[k], aq, ap[k]);
            }
            cn[k] = node;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              a[k][c] = 0.0;
              if (PR) ap[k][c] = 0.0;
            }
          }
          if (on) {
            double w[8];
            cic_weights<R>(tx, ty, tz, w);
            double e = 0.0;
            if (PR) e = (P.mass[s] * (double)((vx * vx + vy * vy) + vz * vz)) / 3.0;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              a[k][c] += w[c];
              if (PR) ap[k][c] += w[c] * e;
            }
          }
        }
      }
    });
    __syncthreads();
    if (coul && tot[4] != 0u) [[unlikely]] {
      // the next step's order was made with the pools as they were
      __syncthreads();
      if (tid == 0) tot[4] = 0u;
      if (ct >= kNT - 64 && it + 1 < nsteps) order_wave<R>(job, E, step + 1, sh, tot, true, cur ^ 1);
      __syncthreads();
    }
  }
  if (coul) add_moments(sh.cacc, mslot);
  if (dep) {
    // the sums out: runs of equal cells of each wavefront first
    rounds<kRounds>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      if (k * kNT >= nsl) return;  // uniform
      const int Q = cn[k] < 0 ? 0 : q_of(sh.sqs[tid + k * kNT]);
      const int64_t rk = cn[k] < 0 ? -1 : 2 * (int64_t)cn[k] + (Q >= 1 ? 0 : 1);
      int seg;
      bool tail;
      wave_runs(rk, seg, tail);
      const SegSteps st = seg_steps(seg);
      double s[8], sq[8], sp[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        s[c] = seg_scan(st, a[k][c]);
        sq[c] = seg_scan(st, (double)Q * a[k][c]);
        if (PR) sp[c] = seg_scan(st, ap[k][c]);
      }
      if (tail && rk >= 0) put(cn[k], Q >= 1, s, sq, sp);
    });
    __syncthreads();
    flush_brick<R>(job, brick, box, nf, PR);
  }
  // the state back
  const Soa<R> S = soa_at(fresh<R>(job).S, lo);
#pragma unroll
  for (int k = 0; k < kRounds; ++k) {
    const int j = tid + k * kNT;
    if (j < nsl) {
      S.x[j] = x[k];
      S.y[j] = y[k];
      S.z[j] = z[k];
      S.vx[j] = sh.v[j];
      S.vy[j] = sh.v[kPSlots + j];
      S.vz[j] = sh.v[2 * kPSlots + j];
      S.qs[j] = sh.sqs[j];
    }
  }
}

// several steps (four workgroups per CU, by the LDS and by the registers;
// with the pressure sums three, by the registers)
template <typename R, int FLD, bool EXT, bool PR>
__global__ void __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(PR ? 3 : 4, PR ? 3 : 4)))
k_period(StepBatch<R> B, uint32_t nsteps) {
  __shared__ __align__(16) FusedLds<R> lds;
  // pairs and triplets of the two work lists, and whether a pool changed
  __shared__ uint32_t tot[5 + kNW];
  static_assert(sizeof(OneShared<R>) <= sizeof(lds), "a medium cell's step fits");
  __shared__ uint32_t red[kNW], gcount;
  const RunWG own = run_of(B);
  const JobPtr<R> job = (JobPtr<R>)B.job[own.run];
  const uint32_t step0 = StepArg{B.stepw[own.run], B.step[own.run]}.get();
  if (own.wg >= (uint32_t)kBigWG) {
    // the windows' first chunks, then their second ones, ...: the workgroups
    // that find none come last
    const uint32_t e = own.wg - kBigWG, nw = job->windows, i0 = e / nw, w = e - i0 * nw;
    const uint32_t nchunk = ((const __attribute__((address_space(4))) uint32_t *)job->C.win)[w] & 0xffffu;
    const ChunkEntry *chunk = job->C.chunk + (size_t)w * kWinList;
    double *mslot = job->moments + 5 * (int64_t)own.wg;
    const int turn = 64 * (int)(e % kNW);
    for (uint32_t i = i0; i < nchunk; i += job->win_wgs) {
      chunk_steps<R, FLD, EXT, PR>(job, chunk[i], mslot, step0, nsteps, lds, tot, turn);
      __syncthreads();  // the next one reuses the LDS
    }
  }
  // the cells beyond a chunk, by all of the run's workgroups in turn
  const ChunkTable C = fresh<R>(job).C;
  const uint32_t nbig = *(const __attribute__((address_space(4))) uint32_t *)C.cnt;
  for (uint32_t e = own.wg; e < nbig; e += own.nwg) {
    const uint32_t lo = C.big[2 * e], end = C.big[2 * e + 1];
    double *mslot = cell_moments<R>(job, lo);
    if (!PR && end - lo <= 2u * kPSlots) {
      const GroupEntry G = cell_entry(fresh<R>(job).P, lo, end);
      const ChunkEntry M[2] = {G.all, G.all};
      for (uint32_t it = 0; it < nsteps; ++it) {
        chunk_step<R, FLD, EXT, false, true>(job, M, true, G, mslot, step0 + it, *(OneShared<R> *)&lds, tot + 5, tot, 0,
                                             nullptr, nullptr);
        __syncthreads();
      }
      continue;
    }
    for (uint32_t it = 0; it < nsteps; ++it) {
      const StepJob<R> &J = fresh<R>(job);
      big_cell<R, FLD, EXT, PR, kNT, (int)sizeof(lds)>(J.P, J.T, J.S, J.ef, lo, end,
                                                       it + 1 == nsteps ? J.evlog : nullptr, J.acc, J.dens, mslot,
                                                       J.scratch64, step0 + it, nullptr, nullptr, (unsigned char *)&lds,
                                                       red, &gcount);
    }
  }
}

}  // namespace

template <typename R>
void launch_period(const StepBatch<R> &B, uint32_t nsteps, bool ext, bool fields, bool pressure, hipStream_t st) {
  if (B.n <= 0 || B.wg0[B.n] == 0 || nsteps == 0u) return;
  const dim3 g(B.wg0[B.n]), b(kNT);
  if (pressure) hipLaunchKernelGGL((k_period<R, 7, true, true>), g, b, 0, st, B, nsteps);
  else if (fields) hipLaunchKernelGGL((k_period<R, 7, true, false>), g, b, 0, st, B, nsteps);
  else if (ext) hipLaunchKernelGGL((k_period<R, 0, true, false>), g, b, 0, st, B, nsteps);
  else hipLaunchKernelGGL((k_period<R, 0, false, false>), g, b, 0, st, B, nsteps);
}

}  // namespace ecr
