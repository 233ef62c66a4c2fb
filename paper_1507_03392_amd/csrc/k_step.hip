// k_step.hip -- the binary64 instances of the fused step kernels
// (ecr_period.hpp, ecr_single.hpp), and what both precisions share: the chunk
// table made at every sort, the units of a single step, the size of a launch,
// and the small kernels that write a run's job and its step word.
#include "ecr_period.hpp"

namespace ecr {

namespace {

// ---------------------------------------------------------------------------
// The chunk table, once per sort.  A workgroup takes a window of kWinChunks
// chunks' slots (the cells whose first slot lies in it), marks the cells'
// first slots in LDS, and one wavefront spreads the cells over as few chunks
// of at most the chunk size as hold them, evenly; a cell beyond that size is a
// chunk of its own, beyond kPSlots a big cell.  Filling them cell by cell
// leaves half a cell of a chunk empty on average, where chunks of fixed first
// slots need a whole large cell's room.
// A chunk at least half full ends with its plane of cells: the box of one
// that spans two planes is a whole plane wide, too wide for the deposit's
// brick.
// ---------------------------------------------------------------------------
constexpr int kWinMax = kWinChunks * kPSlots;  // a window's slots, its last cell's overhang left out
constexpr int kWinWords = kWinMax / 64;

constexpr int kPrepNT = 1024;

__global__ void __launch_bounds__(kPrepNT) k_step_prep(KParams P, int fill, ChunkTable C) {
  const uint32_t *__restrict__ cellid = P.cellid, *__restrict__ cell_off = P.cell_off;
  const int64_t n = P.n;
  const uint32_t plane = (uint32_t)(P.nx * P.ny);
  __shared__ uint64_t head[kWinWords], phead[kWinWords];  // first slots of the cells, and of the planes
  __shared__ uint32_t wpre[kWinWords + 1], nbs[kWinMax + 1], wsum[kPrepNT / 64];
  __shared__ uint16_t cs[kWinMax + 1];
  __shared__ int8_t ck[kWinMax];  // a cell's chunk, -1 for a big cell
  __shared__ int ncb, nbg, bbase, ngr;
  __shared__ uint8_t gr[kWinList + 1];  // the groups' first chunks
  __shared__ int cb[kWinList], ce[kWinList], box[kWinList][6], bc[kWinChunks + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t win = (int64_t)kWinChunks * fill;
  // the first cell that starts at or after slot t
  const auto first_cell = [&](int64_t t) -> int64_t {
    if (t >= n) return n;
    const uint32_t c = cellid[t], st = cell_off[c];
    return st == (uint32_t)t ? t : (int64_t)cell_off[c + 1];
  };
  const int64_t lo = first_cell(blockIdx.x * win), hi = first_cell((blockIdx.x + 1) * win);
  if (hi <= lo) {
    if (tid == 0) C.win[blockIdx.x] = 0u;
    return;
  }
  const int total = (int)(hi - lo);
  // heads among the window's own slots (a cell starts before the window's end)
  const int len = (int)min(hi - lo, win);
#pragma unroll
  for (int k = 0; k < kWinMax / kPrepNT; ++k) {
    const int i = tid + k * kPrepNT;
    uint32_t c = 0, p = 0;
    if (i < len) {
      c = cellid[lo + i];
      p = i > 0 ? cellid[lo + i - 1] : c + 1u;
    }
    const uint64_t b = __ballot(c != p), q = __ballot(c != p && i > 0 && c / plane != p / plane);
    if (lane == 0) {
      head[i >> 6] = b;
      phead[i >> 6] = q;
      wpre[i >> 6] = (uint32_t)__popcll(b);
    }
  }
  __syncthreads();
  const int nh = (int)wg_exscan<kPrepNT>(wpre, kWinWords, wsum);
  for (int i = tid; i < len; i += kPrepNT) {
    const uint64_t b = head[i >> 6];
    if ((b >> (i & 63)) & 1ull) cs[wpre[i >> 6] + __popcll(b & ((1ull << (i & 63)) - 1ull))] = (uint16_t)i;
  }
  __syncthreads();
  const auto cell_end = [&](int h) -> int { return h + 1 < nh ? (int)cs[h + 1] : total; };
  for (int h = tid; h < nh; h += kPrepNT) {
    const int m = cell_end(h) - (int)cs[h];
    nbs[h] = m > kPSlots ? 0u : 1u << (31 - __clz(m));
  }
  __syncthreads();
  (void)wg_exscan<kPrepNT>(nbs, nh, wsum, true);
  if (tid < 64) {
    // the chunks, by one wavefront with the bit words in its lanes: the
    // window's slots are spread over as few chunks as hold them, evenly
    static_assert(kWinMax <= 64 * 64, "a word per lane");
    const uint64_t hw = head[lane], pw = phead[lane];
    const uint32_t pre = wpre[lane];
    const auto lane64 = [](uint64_t v, int l) -> uint64_t {
      return (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l) |
             ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32);
    };
    // the bits of w at or before position i
    const auto upto = [&](uint64_t w, int i) -> uint64_t {
      return lane < (i >> 6) ? w : (lane == (i >> 6) ? w & (~0ull >> (63 - (i & 63))) : 0ull);
    };
    // the last bit of w at or before position i, or -1; all lanes agree
    const auto last_at = [&](uint64_t w, int i) -> int {
      const uint64_t m = upto(w, i), any = __ballot(m != 0ull);
      if (!any) return -1;
      const int l = 63 - __clzll((long long)any);
      return 64 * l + 63 - __clzll((long long)lane64(m, l));
    };
    // the first head after position i, or the end
    const auto next_head = [&](int i) -> int {
      const uint64_t m = hw & ~upto(~0ull, i), any = __ballot(m != 0ull);
      if (!any) return total;
      const int l = __ffsll((unsigned long long)any) - 1;
      return 64 * l + __ffsll((unsigned long long)lane64(m, l)) - 1;
    };
    // the number of the cell whose head is at position i
    const auto number = [&](int i) -> int {
      return __builtin_amdgcn_readlane((int)pre, i >> 6) +
             __popcll(lane64(hw, i >> 6) & ((1ull << (i & 63)) - 1ull));
    };
    int k = 0, g = 0, st = 0, h = 0;
    while (st < total) {
      const int ce1 = next_head(st);
      if (ce1 - st > kPSlots) {
        if (lane == 0) bc[g] = h;
        ++g;
        ++h;
        st = ce1;
        continue;
      }
      const int rest = total - st;
      int e = ce1;  // the first slot past the chunk
      if (rest <= fill) {
        e = total;
      } else {
        const int m = (rest + fill - 1) / fill;
        const int want = min(st + min(fill, (rest + m - 1) / m + (ce1 - st) / 2), len - 1);
        // the cell that starts last at or before `want`: the chunk ends there
        const int i = last_at(hw, want);
        if (i > st) e = i;
        // or where a plane of cells starts that leaves half a chunk
        const int pp = last_at(pw, want);
        if (pp > st && 2 * (pp - st) >= fill) e = pp;
      }
      const int he = e < len ? number(e) : nh;
      if (lane == 0) {
        cb[k] = h;
        ce[k] = he;
      }
      ++k;
      h = he;
      st = e;
    }
    if (lane == 0) {
      ncb = k;
      nbg = g;
      if (g) bbase = (int)atomicAdd(&C.cnt[0], (uint32_t)g);
      // Cells of a third of a chunk and more leave the chunks short: a
      // workgroup of a single step then takes up to three in a row, as its room
      // holds, instead of two (5M ions, 290 a cell: 248 us a step with pairs,
      // 223 with groups)
      int m = 0;
      if (step_pairs(n)) {
        for (int j = 0; j < k; ++m) {
          gr[m] = (uint8_t)j;
          const int f = j, s0 = cs[cb[j]];
          do ++j;
          while (j < k && j - f < 3 && cb[j] == ce[j - 1] && cell_end(ce[j] - 1) - s0 <= 2 * kPSlots);
        }
        gr[m] = (uint8_t)k;
        if (m >= (k + 1) / 2) m = 0;
      }
      ngr = m;
      C.win[blockIdx.x] = (uint32_t)(k | (m << 16));
    }
  }
  __syncthreads();
  if (tid < nbg) {
    const int h = bc[tid];
    ck[h] = -1;
    C.big[2 * (bbase + tid)] = (uint32_t)(lo + cs[h]);
    C.big[2 * (bbase + tid) + 1] = (uint32_t)(lo + cell_end(h));
  }
  // the chunks' boxes, a wavefront to a chunk
  for (int k = tid >> 6; k < ncb; k += kPrepNT / 64) {
    int b[6] = {0x7fffffff, 0x7fffffff, 0x7fffffff, -1, -1, -1};
    for (int h = cb[k] + lane; h < ce[k]; h += 64) {
      ck[h] = (int8_t)k;
      const uint32_t c = cellid[lo + cs[h]], r = c / (uint32_t)P.nx;
      const int i[3] = {(int)(c - r * (uint32_t)P.nx), (int)(r % (uint32_t)P.ny), (int)(r / (uint32_t)P.ny)};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        b[d] = min(b[d], i[d]);
        b[3 + d] = max(b[3 + d], i[d]);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        b[d] = min(b[d], __shfl_xor(b[d], o, 64));
        b[3 + d] = max(b[3 + d], __shfl_xor(b[3 + d], o, 64));
      }
    if (lane < 6) box[k][lane] = lane == 0 ? b[0] : lane == 1 ? b[1] : lane == 2 ? b[2] : lane == 3 ? b[3] : lane == 4 ? b[4] : b[5];
  }
  __syncthreads();
  // chunks t0 up to t1 in one entry
  const auto entry_of = [&](int t0, int t1) -> ChunkEntry {
    int b[6];
    for (int d = 0; d < 6; ++d) b[d] = box[t0][d];
    for (int t = t0 + 1; t < t1; ++t)
      for (int d = 0; d < 3; ++d) {
        b[d] = min(b[d], box[t][d]);
        b[3 + d] = max(b[3 + d], box[t][3 + d]);
      }
    const int h0 = cb[t0], h1 = ce[t1 - 1];
    return {(uint32_t)(lo + cs[h0]),
            (uint32_t)(lo + cell_end(h1 - 1)),
            (uint32_t)b[0],
            (uint32_t)b[1],
            (uint32_t)b[2],
            (uint32_t)(min(b[3] - b[0], 0xffff) | (min(b[4] - b[1], 0xffff) << 16)),
            (uint32_t)min(b[5] - b[2], 0xffff),
            (nbs[h1] - nbs[h0]) | ((uint32_t)(h1 - h0) << 16)};
  };
  if (tid < ncb) C.chunk[(int64_t)blockIdx.x * kWinList + tid] = entry_of(tid, tid + 1);
  if (tid < ngr) {
    const int t0 = gr[tid], t1 = gr[tid + 1];
    GroupEntry g{entry_of(t0, t1), {kNoPlace, kNoPlace}, {0u, 0u}};
    for (int t = t0 + 1; t < t1; ++t) {
      g.s[t - t0 - 1] = (uint32_t)((int)cs[cb[t]] - (int)cs[cb[t0]]);
      g.a[t - t0 - 1] = (nbs[cb[t]] - nbs[cb[t - 1]]) | ((uint32_t)(cb[t] - cb[t - 1]) << 16);
    }
    C.group[(int64_t)blockIdx.x * kWinGroups + tid] = g;
  }
  for (int i = tid; i < total; i += kPrepNT) {
    // the slot's cell: the last head at or before it
    int h = nh - 1;
    if (i < len) h = (int)wpre[i >> 6] + (int)__popcll(head[i >> 6] << (63 - (i & 63))) - 1;
    // (a cell of two chunks' slots at most counts from itself; the larger
    // ones do not use theirs)
    const int k = ck[h];
    const int lg = 31 - __clz(cell_end(h) - (int)cs[h]);
    C.bkinfo[lo + i] = bk_pack(k < 0 ? 0u : nbs[h] - nbs[cb[k]], (uint32_t)(lg & 15), k < 0 ? 0u : (uint32_t)(h - cb[k]),
                               i == (int)cs[h]);
  }
}

}  // namespace

// Runs from 128 full chunks up fill their chunks; a smaller run gets about
// 128 chunks of a power-of-two size (at least 64 slots), so that it still
// spreads over the CUs.  The line is that of a kernel of one step; other sizes
// have not been timed with k_period.
int64_t step_fill(int64_t n) {
  int64_t p = 64;
  while (2 * p <= n / 128 && 2 * p <= kPSlots) p *= 2;
  return p;
}

int64_t step_windows(int64_t n) {
  const int64_t w = kWinChunks * step_fill(n);
  return (n + w - 1) / w;
}

int64_t step_max_big(int64_t n) { return n / kPSlots + 1; }

// Nine chunks to a window mostly, up to sixteen where the cells are just over
// half a chunk.  A workgroup that finds none ends at once, so runs that leave
// the chip's 1024 places idle take as many as they may need: two chunks in a
// row in one workgroup cost such a launch twice the time (75k ions in cells of
// 285, one step: 34 us with 183 workgroups for 263 chunks, 21 with enough)
uint32_t step_win_wgs(int64_t n) {
  const int64_t w = step_windows(n), idle = w > 0 ? (kPlaces - kBigWG) / w : 0;
  return (uint32_t)(idle < 11 ? 11 : (idle > 2 * kWinChunks + 1 ? 2 * kWinChunks + 1 : idle));
}
uint32_t step_wgs(int64_t n) { return (uint32_t)(kBigWG + step_windows(n) * step_win_wgs(n)); }
uint32_t step_wgs_one(int64_t n) {
  return step_pairs(n) ? (uint32_t)(kBigWG + (step_windows(n) * 11 + 1) / 2) : step_wgs(n);
}

// ---------------------------------------------------------------------------
// The single step's units.  Each workgroup adds up the counts of all windows
// and of those before its own (489 of them at 2M ions), and moves its windows'
// entries to their places.  Neighbours share nodes of the density, and
// workgroups that add to the same nodes at the same time wait for each other:
// the row is dealt out in nine turns, so that neighbours are a ninth of it
// apart (a settled 2M run, one step: 104 us in order of slot, 98 dealt out).
// ---------------------------------------------------------------------------
constexpr int kUnitWins = 16;  // windows to a workgroup
__device__ __forceinline__ uint32_t dealt(uint32_t i, uint32_t n) {
  const uint32_t t = i % 9u;
  return t * (n / 9u) + min(t, n % 9u) + i / 9u;
}

__global__ void __launch_bounds__(256) k_step_units(uint32_t windows, bool pairs, ChunkTable C) {
  __shared__ uint32_t part[4][4], c0[kUnitWins + 1], g0[kUnitWins + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t w0 = blockIdx.x * kUnitWins;
  const auto count = [&](uint32_t w, uint32_t &wc, uint32_t &wg) {
    const uint32_t v = C.win[w];
    wg = v >> 16;
    wc = wg ? 0u : v & 0xffffu;
  };
  uint32_t sum[4] = {0u, 0u, 0u, 0u};  // chunks and groups before, in all
  for (uint32_t w = tid; w < windows; w += 256) {
    uint32_t wc, wg;
    count(w, wc, wg);
    sum[2] += wc;
    sum[3] += wg;
    if (w < w0) {
      sum[0] += wc;
      sum[1] += wg;
    }
  }
  for (int k = 0; k < 4; ++k) {
    const uint32_t v = wave_incl_scan(sum[k]);
    if (lane == 63) part[k][tid >> 6] = v;
  }
  __syncthreads();
  for (int k = 0; k < 4; ++k) sum[k] = part[k][0] + part[k][1] + part[k][2] + part[k][3];
  const uint32_t nc = sum[2], ng = sum[3];
  if (tid == 0) {
    for (int k = 0; k <= kUnitWins; ++k) {
      c0[k] = sum[0];
      g0[k] = sum[1];
      uint32_t wc = 0, wg = 0;
      if (w0 + k < windows) count(w0 + k, wc, wg);
      sum[0] += wc;
      sum[1] += wg;
    }
    if (blockIdx.x == 0) {
      // pairs fill the chip's places so many times over; a small rest ends
      // sooner in single chunks (1M ions, one step: 59 us with 76 pairs left
      // over after one time, 54 with their chunks; 4M, 300 after four: 163
      // and 170)
      const uint32_t p = pairs ? (nc + 1u) / 2u : 0u, turns = (p + ng) / kPlaces, rest = (p + ng) % kPlaces;
      const uint32_t np = turns >= 1u && turns < 8u && rest * turns * turns * turns < 480u ? p - min(p, rest) : p;
      *C.units = {np, nc > 2u * np ? nc - 2u * np : 0u, ng, nc};
    }
  }
  __syncthreads();
  for (int i = tid; i < kUnitWins * kWinList; i += 256) {
    const int k = i / kWinList, j = i - k * kWinList;
    const int64_t w = w0 + k;
    const uint32_t c = c0[k] + j, g = g0[k] + j, whole = nc / 2u;
    if (c < c0[k + 1]) {
      const uint32_t to = !pairs ? dealt(c, nc) : c / 2u < whole ? 2u * dealt(c / 2u, whole) + (c & 1u) : c;
      C.flat[to] = C.chunk[w * kWinList + j];
    }
    if (j < kWinGroups && g < g0[k + 1]) C.gflat[dealt(g, ng)] = C.group[w * kWinGroups + j];
  }
}

void launch_step_units(int64_t n, ChunkTable C, hipStream_t st) {
  const uint32_t w = (uint32_t)step_windows(n);
  if (w > 0)
    hipLaunchKernelGGL(k_step_units, dim3((w + kUnitWins - 1) / kUnitWins), dim3(256), 0, st, w, step_pairs(n), C);
}

void launch_step_prep(const KParams &P, ChunkTable C, hipStream_t st) {
  if (P.n <= 0) return;
  hipLaunchKernelGGL(k_step_prep, dim3((unsigned)step_windows(P.n)), dim3(kPrepNT), 0, st, P, (int)step_fill(P.n), C);
}

bool step_ext(const KParams &P) { return (P.pmask & (P_HEAT | P_ELASTIC)) || P.nion > 1; }

// a run's job, passed by value, into device memory (one lane writes it)
template <typename R>
__global__ void k_set_job(StepJob<R> J, StepJob<R> *__restrict__ dst) {
  if (threadIdx.x == 0) *dst = J;
}

__global__ void k_set_words(SetWords w) {
  if ((int)threadIdx.x < w.n) *w.ptr[threadIdx.x] = w.val[threadIdx.x];
}

template <typename R>
void launch_set_job(const StepJob<R> &J, StepJob<R> *dst, hipStream_t st) {
  hipLaunchKernelGGL((k_set_job<R>), dim3(1), dim3(64), 0, st, J, dst);
}

__global__ void __launch_bounds__(256) k_grids_home(const uint32_t *cur, uint32_t *home, uint32_t *clear, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    home[i] = cur[i];
    clear[i] = 0u;
  }
}

void launch_grids_home(const uint32_t *cur, uint32_t *home, uint32_t *clear, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_grids_home, dim3((unsigned)(n < 1048576 ? (n + 255) / 256 : 4096)), dim3(256), 0, st, cur, home,
                     clear, n);
}

void launch_set_words(const SetWords &w, hipStream_t st) {
  if (w.n > 0) hipLaunchKernelGGL(k_set_words, dim3(1), dim3(64), 0, st, w);
}

template void launch_set_job<double>(const StepJob<double> &, StepJob<double> *, hipStream_t);
template void launch_set_job<float>(const StepJob<float> &, StepJob<float> *, hipStream_t);
template void launch_period<double>(const StepBatch<double> &, uint32_t, bool, bool, bool, hipStream_t);
template void launch_step<double>(const StepBatch<double> &, bool, bool, bool, const CellGrids &, hipStream_t);

}  // namespace ecr
