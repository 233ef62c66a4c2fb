// ecr_fused.hpp -- what the kernels of the whole ion step share: the order of
// the pools (Takizuka-Abe) in LDS, the collisions of a work list, the density
// brick, the workgroup's way through its run's chunks and large cells.
#pragma once

#include <stddef.h>

#include <utility>

#include "ecr_step.hpp"

namespace ecr {

namespace {

constexpr int kNT = 256;             // lanes per workgroup
constexpr int kNW = kNT / 64;

// the work list of M slots: two slots per pair, three per triplet, their
// pools' sizes
template <int M>
struct WorkList {
  uint16_t pair[M], tri[M + 2], pair_pool[M / 2], tri_pool[M / 3 + 2];
};

// what orders the pools of M slots
template <int M>
struct Ordering {
  uint64_t bkey[M + 4];               // (key, id) by bucket; read in batches of four
  uint64_t cinfo[M];                  // per cell: pool start, size, first pair, first triplet (16 bits each)
  alignas(16) uint32_t hist[M + 4];   // members per bucket, then before it
  uint16_t cellb[M + 2];              // first bucket of each cell
};

template <typename R>
__device__ __forceinline__ Soa<R> soa_at(const Soa<R> &S, int64_t lo) {
  return {S.x + lo, S.y + lo, S.z + lo, S.vx + lo, S.vy + lo, S.vz + lo, S.qs + lo, S.pid + lo, S.birth + lo};
}

// f(0), f(1), ... f(N-1) with constant arguments: a loop over the rounds of a
// lane's register arrays that is unrolled whatever its body's size
template <typename F, int... K>
__device__ __forceinline__ void rounds_of(F &&f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void rounds(F &&f) {
  rounds_of(f, std::make_integer_sequence<int, N>{});
}

// A run's arguments sit in its job in device memory and are read through
// scalar loads where they are used.  fresh() hides from the compiler that
// they are the same from one phase to the next: kept over the whole loop,
// the parameter block's two hundred scalars do not fit the scalar registers
// and come back through lane reads, vector instructions in every phase.
template <typename R>
using JobPtr = const __attribute__((address_space(4))) StepJob<R> *;
template <typename R>
__device__ __forceinline__ const StepJob<R> &fresh(JobPtr<R> p) {
  asm volatile("" : "+s"(p));
  return *(const StepJob<R> *)p;
}

// a member's bucket: its cell's first plus the key's top bits (written so
// that a shift by 32 is none)
__device__ __forceinline__ int bucket_of(uint32_t w, uint32_t key) {
  return (int)(bk_first(w) + ((key >> 1) >> (31u - bk_lg(w))));
}

// the cells' pools and the numbers of their first pair and triplet, from the
// scanned histogram (all lanes of one wavefront call it): a pool of m has
// m/2 pairs, or for odd m >= 3 one triplet and (m-3)/2 pairs; a pool of one
// has none.  tot: the pairs and triplets in all
template <int M>
__device__ __forceinline__ void number_items(Ordering<M> &sh, int nh, int nb, uint32_t *tot) {
  const int lane = threadIdx.x & 63;
  uint32_t run = 0;  // triplets | pools of one << 16 before
  for (int h0 = 0; h0 < nh; h0 += 64) {
    const int h = h0 + lane;
    uint32_t ps = 0, m = 0;
    if (h < nh) {
      ps = sh.hist[sh.cellb[h]];
      m = sh.hist[sh.cellb[h + 1]] - ps;
    }
    const uint32_t f = ((m & 1u) && m >= 3u ? 1u : 0u) | (m == 1u ? 0x10000u : 0u);
    const uint32_t incl = wave_incl_scan(f), ex = run + incl - f;
    const uint32_t tb = ex & 0xffffu, ob = ex >> 16;
    if (h < nh)
      sh.cinfo[h] = (uint64_t)(ps | (m << 16)) | ((uint64_t)(((ps - 3u * tb - ob) >> 1) | (tb << 16)) << 32);
    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  }
  if (lane == 0) {
    const uint32_t nt = run & 0xffffu;
    tot[0] = (sh.hist[nb] - 3u * nt - (run >> 16)) >> 1;
    tot[1] = nt;
  }
}

// a member's rank in its cell's pool, from its bucket mates of smaller (key,
// id), and its slot to its place in the work list
template <int M>
__device__ __forceinline__ void list_member(const Ordering<M> &sh, WorkList<M> &item, int bk, uint32_t cell,
                                            uint32_t key, uint32_t id, int slot) {
  const uint64_t me = ((uint64_t)key << 32) | id;
  const int b0 = (int)sh.hist[bk], b1 = (int)sh.hist[bk + 1];
  // the bucket's first four entries in one batch of loads (a bucket holds one
  // or two members mostly; entries past its end are masked), the rest one by
  // one
  const uint64_t q0 = sh.bkey[b0], q1 = sh.bkey[b0 + 1], q2 = sh.bkey[b0 + 2], q3 = sh.bkey[b0 + 3];
  const uint64_t ci = sh.cinfo[cell];
  int rib = (q0 < me ? 1 : 0) + (b0 + 1 < b1 && q1 < me ? 1 : 0) + (b0 + 2 < b1 && q2 < me ? 1 : 0) +
            (b0 + 3 < b1 && q3 < me ? 1 : 0);
  for (int t = b0 + 4; t < b1; ++t) rib += sh.bkey[t] < me ? 1 : 0;
  const int r = b0 + rib - (int)(ci & 0xffffu);
  const uint32_t m = (uint32_t)(ci >> 16) & 0xffffu;
  const bool odd = (m & 1u) != 0u;
  if (m >= 2u) {
    if (odd && r < 3) {
      const uint32_t t = (uint32_t)(ci >> 48);
      item.tri[3 * t + r] = (uint16_t)slot;
      if (r == 0) item.tri_pool[t] = (uint16_t)m;
    } else {
      const uint32_t i = 2u * ((uint32_t)(ci >> 32) & 0xffffu) + (uint32_t)(odd ? r - 3 : r);
      item.pair[i] = (uint16_t)slot;
      if (!(i & 1u)) item.pair_pool[i >> 1] = (uint16_t)m;
    }
  }
}

// The collisions of a work list by NC lanes, lane ct of them (ct takes turns
// over the chunks, as the first wavefront is the busiest and wavefronts of
// one number share a SIMD; lanes past NC do none): triplets one to a lane in
// the first wavefronts, whose spare lanes take pairs three at a time, and the
// other lanes the rest.
template <typename R, int NC, int M>
__device__ __forceinline__ void collide_list(const JobPtr<R> job, const LdsAcc<R, M> V, const uint32_t *sid,
                                             const WorkList<M> &item, double *cacc_sum, const int np,
                                             const int ntri, const int ct, const uint32_t step) {
  const int lane = threadIdx.x & 63;
  int first, count, stride;
  if (ntri > NC - 64) {
    const int nitems = np + ntri;
    first = ct;
    stride = NC;
    count = ct < nitems ? (nitems - 1 - ct) / NC + 1 : 0;
  } else {
    const int l3 = (ntri + 63) & ~63;         // lanes of the triplet wavefronts
    const int n3 = min(np, 3 * (l3 - ntri));  // pairs taken three to a lane
    if (ct < ntri) {
      first = ct;
      count = 1;
      stride = 1;
    } else if (ct < l3) {
      const int q = 3 * (ct - ntri);
      first = ntri + q;
      count = max(0, min(3, n3 - q));
      stride = 1;
    } else {
      const int q = ct - l3;
      stride = NC - l3;
      first = ntri + n3 + q;
      count = q < np - n3 ? (np - n3 - 1 - q) / stride + 1 : 0;
    }
  }
  if (ct >= NC) count = 0;
  const StepJob<R> &J = fresh<R>(job);
  const double *lnA = J.T->lnA;
  // the list as one array of slots: a triplet's start at tri, a pair's at pair
  const uint16_t *list = item.pair;
  constexpr int kTri = (int)(offsetof(WorkList<M>, tri) / 2), kPairPool = (int)(offsetof(WorkList<M>, pair_pool) / 2),
                kTriPool = (int)(offsetof(WorkList<M>, tri_pool) / 2);
  // sixteen entries of each sum are this wavefront's own, so that what goes
  // into an entry, and in what order, does not depend on the others' pace
  const int own = (threadIdx.x >> 6) * 16 + (lane & 15);
  int i = first, sub = 0;
  while (count > 0) {
    // a triplet's collisions (a, b), (b, c), (c, a) are at dt/2
    const bool tri = i < ntri;
    const int p = i - ntri;
    const int oa = tri ? kTri + 3 * i + sub : 2 * p;
    const int ob = tri && sub == 2 ? kTri + 3 * i : oa + 1;
    const uint32_t ia = list[oa], ib = list[ob], m = list[tri ? kTriPool + i : kPairPool + p];
    // the energy of the pool before counts each member once
    double cacc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    collide_acc<R>(J.P, lnA, V, ia, ib, sid[ia], (double)m * J.P.nfac, tri ? 0.5 * J.P.dt : J.P.dt, step, cacc,
                   sub == 0, sub < 2);
#pragma unroll
    for (int c = 0; c < 5; ++c) atomicAdd(&cacc_sum[64 * c + own], cacc[c]);
    if (tri && sub < 2) {
      ++sub;
    } else {
      sub = 0;
      i += stride;
      --count;
    }
  }
}

// the box of nodes of a brick over cells [bb[0..2], bb[3..5]]: those and
// their neighbours, without those along z, or without any, whichever has at
// most cap nodes; else one that holds no cell
struct Box {
  int x0, y0, z0, bx, by, nodes;
  // a base node's place, or -1 (the last node planes belong to no base cell)
  __device__ __forceinline__ int at(int ix, int iy, int iz) const {
    const int lx = ix - x0, ly = iy - y0, lz = iz - z0, cyz = bx * by;
    return (unsigned)lx < (unsigned)(bx - 1) && (unsigned)ly < (unsigned)(by - 1) && lz >= 0 && (lz + 2) * cyz <= nodes
               ? lx + bx * ly + cyz * lz
               : -1;
  }
};
__device__ __forceinline__ Box make_box(const KParams &P, const int bb[6], int cap) {
  Box b{0, 0, 0, 1, 1, 0};
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int g = t < 2 ? 1 : 0, gz = t < 1 ? 1 : 0;  // cells around the box
    const int ax = max(bb[0] - g, 0), ay = max(bb[1] - g, 0), az = max(bb[2] - gz, 0);
    const int wx = min(bb[3] + g, P.nx - 1) - ax + 2, wy = min(bb[4] + g, P.ny - 1) - ay + 2;
    const int wz = min(bb[5] + gz, P.nz - 1) - az + 2;
    if (b.nodes == 0 && (int64_t)wx * wy * wz <= cap) b = {ax, ay, az, wx, wy, wx * wy * wz};
  }
  return b;
}
__device__ __forceinline__ void cell_box(const ChunkEntry &E, int bb[6]) {
  bb[0] = (int)E.x;
  bb[1] = (int)E.y;
  bb[2] = (int)E.z;
  bb[3] = (int)(E.x + (E.wxy & 0xffffu));
  bb[4] = (int)(E.y + (E.wxy >> 16));
  bb[5] = (int)(E.z + E.wz);
}

// a brick's nf fields to HBM (field f of it to field f of the densities, the
// last to the pressure's if last3)
template <typename R>
__device__ __forceinline__ void flush_brick(const JobPtr<R> job, const double *brick, const Box &b, int nf, bool last3) {
  const StepJob<R> &J = fresh<R>(job);
  const int nx1 = J.P.nx1, ny1 = J.P.ny1;
  const int64_t nnode = J.P.nnode;
  double *dens = J.dens;
  const float rbx = 1.0f / (float)b.bx, rby = 1.0f / (float)b.by;
  for (int i = threadIdx.x; i < b.nodes; i += kNT) {
    const int t = small_div(i, b.bx, rbx), lx = i - t * b.bx;
    const int lz = small_div(t, b.by, rby), ly = t - lz * b.by;
    const int64_t node = (int64_t)(b.x0 + lx) + (int64_t)nx1 * ((b.y0 + ly) + (int64_t)ny1 * (b.z0 + lz));
    for (int f = 0; f < nf; ++f) {
      const double v = brick[f * b.nodes + i];
      if (v != 0.0) unsafeAtomicAdd(&dens[(last3 && f == nf - 1 ? 3 : f) * nnode + node], v);
    }
  }
}

// the collisions' sums into the workgroup's moment slot: wavefront c sums
// moment c, wavefront 0 the fifth as well (a barrier lies between the last
// collision and this)
__device__ __forceinline__ void add_moments(const double *cacc, double *__restrict__ mslot) {
  const int lane = threadIdx.x & 63;
  for (int c = threadIdx.x >> 6; c < 5; c += kNW) {
    const double v = wave_sum_last(cacc[64 * c + lane]);
    if (lane == 63) mslot[c] += v;
  }
}

// a cell [lo, end) of more than kPSlots slots, up to 2 kPSlots, as one entry
__device__ __forceinline__ GroupEntry cell_entry(const KParams &P, uint32_t lo, uint32_t end) {
  const uint32_t c = P.cellid[lo], r = c / (uint32_t)P.nx, lg = 31u - (uint32_t)__clz((int)(end - lo));
  return {{lo, end, c - r * (uint32_t)P.nx, r % (uint32_t)P.ny, r / (uint32_t)P.ny, 0u, 0u, (1u << lg) | (1u << 16)},
          {kNoPlace, kNoPlace},
          {0u, 0u}};
}
// its moment slot, after the workgroups'
template <typename R>
__device__ __forceinline__ double *cell_moments(JobPtr<R> job, uint32_t lo) {
  return job->moments + 5 * (int64_t)(kBigWG + job->windows * job->win_wgs + lo / (uint32_t)(kPSlots + 1));
}

// several runs in one launch: run j owns workgroups [wg0[j], wg0[j+1])
struct RunWG {
  int run;
  uint32_t wg, nwg;
};
template <typename R>
__device__ __forceinline__ RunWG run_of(const StepBatch<R> &B) {
  int run = 0;
  for (int t = 1; t < B.n; ++t) run = blockIdx.x >= B.wg0[t] ? t : run;
  return {run, blockIdx.x - B.wg0[run], B.wg0[run + 1] - B.wg0[run]};
}

// The cell grids among the kernel's own arguments, which follow its StepBatch:
// read again where the step clears, not kept in scalar registers (as lanes of
// a vector register, mostly) from the kernel's start to its end.  A settled
// run of 2M with a self-consistent n_e 110.0 -> 109.2 us a step, with the
// heating kick 146.1 -> 144.4.
template <typename R>
__device__ __forceinline__ CellGrids grids_arg() {
  static_assert(sizeof(StepBatch<R>) % alignof(CellGrids) == 0, "the second argument follows the first");
  auto p = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(StepBatch<R>);
  asm volatile("" : "+s"(p));
  return *(const CellGrids *)p;
}

// clear the grid that the step before read
__device__ __forceinline__ void clear_grid(const CellGrids &grids) {
  // the grid that the step before read, for the step to come to add to: a
  // fill of its own between two steps took 4-5 us of 61 at 600k ions, and
  // these stores, after everything that waits for a load, cost next to none
  if (!grids.clear) return;
  uint4 *c = reinterpret_cast<uint4 *>(grids.clear);
  const int64_t n4 = grids.n / 4, i0 = (int64_t)blockIdx.x * kNT + threadIdx.x;
  for (int64_t i = i0; i < n4; i += (int64_t)gridDim.x * kNT) c[i] = make_uint4(0u, 0u, 0u, 0u);
  if (i0 < grids.n - 4 * n4) grids.clear[4 * n4 + i0] = 0u;
}

}  // namespace

}  // namespace ecr
