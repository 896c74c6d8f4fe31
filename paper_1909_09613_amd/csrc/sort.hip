// Counting sort of the particles by (tile, species), run only when a tile's
// particles have outgrown the staging margin of the gather-push-deposit
// kernel (a device-side request flag; all kernels exit at once otherwise).
//
// count    key = 2 * tile + species per particle; wave-aggregated counts;
//          the last block to finish scans the counts into segment offsets
//          and clears them
// scatter  each particle to its segment of the other store (the counts again
//          count what each segment holds), every tile's box to its rectangle
// arrange  one block per segment: order the segment back into the current
//          store by (rank within its cell, cell): first every cell's first
//          particle, cells in tile order, then every cell's second particle,
//          and so on, ranked by their place in the cell.  The lanes of a
//          wave then hold particles of 64 nearby cells, one each, so that the
//          gather reads and the current atomics of a wave touch distinct, nearly
//          consecutive LDS addresses.  Ranks beyond `kcap` (dense cells) follow in cell order.
//          The last arrange block to finish clears the request and counts
//          the sort.  Between sorts the counts are zero, so a sort needs no
//          clearing pass, and each of the three kernels reads
//          the request flag itself (only the particle kernel sets it, and it
//          does not run during a sort).
#include "common.hpp"
#include "launch.hpp"

namespace wtpic {

namespace {

template <class Real>
__device__ int find_run(const RunDev<Real>* runs, int nruns, long long p) {
  int lo = 0, hi = nruns - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (runs[mid].p0 <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The valid lanes of the wave that share this lane's key.
__device__ __forceinline__ unsigned long long same_key(int key, bool valid) {
  unsigned long long todo = __ballot(valid), mine = 0;
  while (todo) {
    const int k = __builtin_amdgcn_readlane(key, __ffsll((long long)todo) - 1);
    const unsigned long long m = __ballot(valid && key == k);
    if (key == k) mine = m;
    todo &= ~m;
  }
  return valid ? mine : 0;
}

// Quotient of a cell index by a tile edge (inv = 1 / edge): the half step
// keeps the approximate product off the integers, whose distance shrinks with
// the edge as the quotient's error does.
__device__ __forceinline__ int tile_of(int m, float inv) { return (int)(((float)m + 0.5f) * inv); }

}  // namespace

// Exclusive scan of the counts into segment offsets by one block, which leaves
// the counts zero for the scatter.  The counts were added with device-scope
// atomics; they are read the same way, several per thread in flight (one after
// the other, the 4700 of 24 runs took a tenth of the whole pass).
template <class Real>
__device__ void scan_counts(const SortArgs<Real>& A, int* part) {
  constexpr int K = 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int done = 0;
  for (int i0 = 0; i0 < A.nkeys; i0 += K * kSortBlock) {
    const int lo = i0 + K * tid;
    int c[K], s = 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
      c[k] = lo + k < A.nkeys ? __hip_atomic_load(&A.counts[lo + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
#pragma unroll
    for (int k = 0; k < K; ++k) s += c[k];
    int incl = s;
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(incl, off);
      if (lane >= off) incl += t;
    }
    if (lane == 63) part[wave] = incl;
    __syncthreads();
    int base = done + incl - s;
#pragma unroll
    for (int w = 0; w < kSortBlock / 64; ++w) {
      if (w < wave) base += part[w];
      done += part[w];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (lo + k >= A.nkeys) break;
      A.seg[lo + k] = base;
      base += c[k];
      A.counts[lo + k] = 0;
    }
    __syncthreads();
  }
  if (tid == 0) A.seg[A.nkeys] = done;
}

// Count and scatter take kSortItems particles per thread at once, so that a
// wave waits once for four particles' loads.  The lanes of equal keys are found by
// scalar reads, and there is one atomic per distinct key of the wave, all keys in
// one instruction; the count's return nothing, the scatter waits for its own once
// per key set.  (One particle per thread, the keys matched through the LDS and the
// scatter's atomics one key after the other: 19M particles in mixed precision 311 and
// 404 us, 0.87M in FP64 56 and 48 us; now 140 to 180 and 320, 19 to 23 and 18 to 20 us.)
template <class P, int DIM>
__global__ void __launch_bounds__(kSortBlock) sort_count(SortArgs<typename P::Real> A) {
  using Real = typename P::Real;
  if (!A.st->sort_request) return;
  constexpr int V = kSortItems;
  const PBuf<Real> B = A.buf[0];
  const long long stride = (long long)gridDim.x * kSortBlock * V;
  float inv[3];
  for (int d = 0; d < 3; ++d) inv[d] = 1.0f / (float)A.tile[d];
  // (every lane of a wave iterates the same number of times)
  for (long long b0 = (long long)blockIdx.x * kSortBlock * V; b0 < A.np_total; b0 += stride) {
    int pc[V], tag[V];
    Real x[V][3];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const long long p = min(b0 + v * kSortBlock + threadIdx.x, A.np_total - 1);
      tag[v] = B.tag[p];
      if (P::kAbs) {
#pragma unroll
        for (int d = 0; d < DIM; ++d) x[v][d] = B.pos[d][p];
      } else {
        pc[v] = B.cell[p];
      }
    }
    // the group's particles lie in one run but at a run's end
    const int r0 = A.nruns == 1 ? 0 : find_run(A.runs, A.nruns, b0);
    const bool one = r0 == A.nruns - 1 || b0 + kSortBlock * V <= A.runs[r0 + 1].p0;
    auto count_in = [&](int v, const RunDev<Real>& R) {
      const long long p = b0 + v * kSortBlock + threadIdx.x;
      const bool valid = p < A.np_total;
      int key = 0;
      if (valid) {
        int c[3] = {0, 0, 0};
        if (P::kAbs) {
#pragma unroll
          for (int d = 0; d < DIM; ++d) c[d] = (int)floor(x[v][d]);
        } else {
          unpack_cell<DIM>(pc[v], c[0], c[1], c[2]);
        }
        int t[3] = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
          int m = c[d];
          if (m < 0 || m >= R.n[d]) {  // never for a valid store; keep the index in range
            atomicAdd(&A.st->n_out_of_range, 1ull);
            m = wrapi(m, R.n[d]);
          }
          t[d] = tile_of(m, inv[d]);
        }
        const int g = R.tile0 + t[0] + R.ntile[0] * (t[1] + R.ntile[1] * t[2]);
        key = 2 * g + ((tag[v] >> kSpeciesShift) & 1);
        A.keys[p] = key;
      }
      const unsigned long long m = same_key(key, valid);
      if (m && __ffsll((long long)m) - 1 == (int)(threadIdx.x & 63)) atomicAdd(A.counts + key, __popcll(m));
    };
    if (one) {
#pragma unroll
      for (int v = 0; v < V; ++v) count_in(v, A.runs[r0]);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        count_in(v, A.runs[find_run(A.runs, A.nruns, min(b0 + v * kSortBlock + threadIdx.x, A.np_total - 1))]);
    }
  }
  // the last block to finish turns the counts into segment offsets.  Every wave
  // waits for its own counts to land before its group takes the ticket: the adds
  // return nothing, so the barrier does not wait for them, and a fence of thread 0
  // waits for those of its wave alone.  The counts are touched by device-scope
  // atomics only, so that having landed is all they need (a fence in every
  // wave also writes the L2s back: 19M particles in mixed precision 263 us, 118 with
  // the wait; 7.3M in FP64 205 and 61 us).
  __shared__ int part[kSortBlock / 64];
  __shared__ int last;
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), the other counters at their maxima
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(&A.st->count_done, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  __threadfence();
  scan_counts(A, part);
  if (threadIdx.x == 0) A.st->count_done = 0;
}

template <class P, int DIM>
__global__ void __launch_bounds__(kSortBlock) sort_scatter(SortArgs<typename P::Real> A) {
  using Real = typename P::Real;
  if (!A.st->sort_request) return;
  constexpr int V = kSortItems;
  const PBuf<Real> S = A.buf[0];
  const PBuf<Real> D = A.buf[1];
  const int lane = threadIdx.x & 63;
  const long long stride = (long long)gridDim.x * kSortBlock * V;
  // every tile's particles now lie in its rectangle; its current bounds are
  // rebuilt by the arrange pass
  for (int g = blockIdx.x * kSortBlock + threadIdx.x; g < A.G; g += gridDim.x * kSortBlock) {
    const int4 where = A.tiles[g];
    const int org[3] = {where.x, where.y, where.z};
    const RunDev<Real>& R = A.runs[where.w];
    for (int d = 0; d < 3; ++d) {
      A.bbox[g * 6 + 2 * d] = 0;
      A.bbox[g * 6 + 2 * d + 1] = min(A.tile[d], R.n[d] - org[d]) - 1;
    }
    for (int c = 0; c < 4; ++c) A.jb[4 * g + c] = 0.0f;
  }
  for (long long b0 = (long long)blockIdx.x * kSortBlock * V; b0 < A.np_total; b0 += stride) {
    int key[V], pc[V], tag[V], to[V];
    Real x[V][3], u[V][3];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const long long p = min(b0 + v * kSortBlock + threadIdx.x, A.np_total - 1);
      key[v] = A.keys[p];
      pc[v] = P::kAbs ? 0 : S.cell[p];
#pragma unroll
      for (int d = 0; d < DIM; ++d) x[v][d] = S.pos[d][p];
#pragma unroll
      for (int d = 0; d < 3; ++d) u[v][d] = S.u[d][p];
      tag[v] = S.tag[p];
    }
    unsigned long long m[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      m[v] = same_key(key[v], b0 + v * kSortBlock + threadIdx.x < A.np_total);
      to[v] = 0;
      if (m[v] && __ffsll((long long)m[v]) - 1 == lane)
        to[v] = A.seg[key[v]] + atomicAdd(A.counts + key[v], __popcll(m[v]));
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int base = __shfl(to[v], m[v] ? __ffsll((long long)m[v]) - 1 : lane);
      if (!m[v]) continue;
      const int q = base + __popcll(m[v] & ((1ull << lane) - 1ull));
      if (!P::kAbs) D.cell[q] = pc[v];
#pragma unroll
      for (int d = 0; d < DIM; ++d) D.pos[d][q] = x[v][d];
#pragma unroll
      for (int d = 0; d < 3; ++d) D.u[d][q] = u[v][d];
      D.tag[q] = tag[v];
    }
  }
}

// Index of a particle's cell in the order the arrange pass lays cells out: x
// first, then y, then z; in 3D mixed precision with an even number of rows
// every second row of a plane before the others, so that the 32 lanes that
// the LDS serves at once are two rows apart (their current atomics do not meet
// where particles of one row start a row further than those of the other; with
// the row pitches of FixedPitch they also lie on different banks).  With ranks
// in the order of the offset, other orders are slower: cells of even x
// before those of odd x (which kept neighbours' atomics apart when ranks were
// in arrival order) 616 -> 631 us at 96x64x64 FP64 and 32.3 -> 37.5 us at 256x128
// cubic mixed; 3D mixed at 128x128x64, with the pitches of that time: plain
// order 740 us, every second row 719, every second plane 780, even x 733, even x
// and rows 898 us.
template <class P, int DIM>
__device__ __forceinline__ int cell_index(const int c[3], const int org[3], const int tile[3]) {
  int m[3] = {0, 0, 0};
  for (int d = 0; d < DIM; ++d) m[d] = min(max(c[d] - org[d], 0), tile[d] - 1);
  if (!P::kAbs && DIM == 3 && (tile[1] & 1) == 0) {
    const int h = tile[1] >> 1;
    return m[0] + tile[0] * ((m[1] >> 1) + h * (m[2] + tile[2] * (m[1] & 1)));
  }
  int cl = 0, stride = 1;
  for (int d = 0; d < DIM; ++d) {
    cl += m[d] * stride;
    stride *= tile[d];
  }
  return cl;
}

template <class P, int DIM>
__device__ __forceinline__ int cell_in_tile(const PBuf<typename P::Real>& S, long long q, const int org[3],
                                            const int tile[3]) {
  int c[3] = {0, 0, 0};
  if (P::kAbs) {
    for (int d = 0; d < DIM; ++d) c[d] = (int)floor(S.pos[d][q]);
  } else {
    unpack_cell<DIM>(S.cell[q], c[0], c[1], c[2]);
  }
  return cell_index<P, DIM>(c, org, tile);
}

// Order of a particle among those of its cell, as a 16-bit key: its offset
// along x1, in 3D FP64 first the half of the cell along x2 that it lies in (a
// group of 16 lanes then holds four rows).  The lanes of a wave hold one
// particle each of consecutive cells along x1, all of the same rank, so with
// ranks in the order of the offset they lie at about the same place in their
// cells.  Their stencils then mostly start at the same node of their cell, and
// the lanes' LDS addresses stay distinct and consecutive; where some lanes start
// one node further than others, the reads conflict and the atomics of
// neighbouring cells meet at one address (LDS cycles per 64-lane access at
// rows of 32 cells, with every lane's start random: reads 3.4 against 2.7,
// 32-bit adds 6.5 against 4.5, FP64 adds 20.8 against 8.6).  A drift moves all
// particles of the wave alike and keeps the order.  Particle kernel, against
// ranks in arrival order: 2D cubic 1024x512 mixed precision 347 -> 326 us, 777x389
// FP64 334 -> 310 us.  3D, offset alone / half and offset: 128x128x64 mixed 670 /
// 682 us, 96x64x64 FP64 576 / 557 us.
template <class P, int DIM>
__device__ __forceinline__ unsigned order_key(typename P::Real fx, typename P::Real fy) {
  using Real = typename P::Real;
  if (DIM == 2 || !P::kAbs) return (unsigned)((float)fx * 65535.0f);
  return (fy >= Real(0.5) ? 32768u : 0u) + (unsigned)((float)fx * 32767.0f);
}

// Each particle's slot is found first; the slots' sources then lie in LDS, in
// the keys' place, and every array is read through them and written in slot
// order, one array after the other: the reads of one array stay within the L1,
// and the writes are whole lines.  (The particles written to their slots
// from registers, all arrays at once, filled lines of all arrays piecemeal, and
// more groups per CU only drove them out of the L2 earlier, 638 -> 888 us.)
// Two groups of 16 waves fill a CU within 64 registers per thread: cell
// and rank share one, two keys another, and the batches are as large as still
// fits without scratch, whose allocation a stream's first launch pays with some
// 200 us (in groups of 512 the items' 32 registers do not fit).
// 19M particles in mixed precision 638 -> 477 us, 0.87M in FP64 48 -> 44 us.
//
// DENSE: most particles lie in segments of more than kArrangeCap, or in cells of
// more than kArrangeOrderCount.  All segments take the arrival order, and the keys' place holds as many levels more, since
// ranks beyond the levels lie cell by cell, whole waves in one cell, whose atomics
// all meet at one address (a longer chain than the levels' random starts).
// Particle kernel, without -> with the levels in the keys' place (0.45 dx, particles
// per cell and species): 512x512 cubic FP64 at 40 1153 -> 820 us, quadratic 750 ->
// 628, cubic at 70 3860 -> 1573; 40^3 linear FP64 at 150 1198 -> 488; 1024x512 cubic
// mixed at 40 2660 -> 1023; 64^3 quadratic mixed at 70 2500 -> 1266; for the cells alone
// (smaller segments) 40^3 quadratic FP64 at 100 1336 -> 1098, 32^3 cubic mixed 1305 -> 646.  (The even
// cells of a row before the odd ones, which pays in arrival order while ranks lie
// beyond the levels, 1153 -> 1085, does not with them, 628 -> 737.)
template <class P, int DIM, bool DENSE>
__global__ void __launch_bounds__(kArrangeBlock, 8) sort_arrange(SortArgs<typename P::Real> A) {
  using Real = typename P::Real;
  if (!A.st->sort_request) return;
  extern __shared__ __align__(16) int sm[];
  __shared__ int cmax_s;
  const int TC = A.tc, KC = A.kcap;
  int* cnt = sm;                                                // TC: particles per cell
  int* xpre = cnt + TC;                                         // TC + 1: prefix of ranks >= KC
  int* base = xpre + TC + 1;                                    // KC + 1: slots below level k
  unsigned short* pre = reinterpret_cast<unsigned short*>(base + KC + 1);  // KC x TC
  unsigned short* first = pre + KC * TC;                        // TC: first key of a cell in keys
  unsigned short* keys = first + TC;                            // kArrangeCap: keys by cell
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int nwave = kArrangeBlock / 64;
  constexpr unsigned kCellBits = 11, kCellMask = (1u << kCellBits) - 1u;
  static_assert(kArrangeOrderCells <= (1 << kCellBits) && (long long)kArrangeCap << kCellBits <= 1ll << 32);
  // items in flight: in the ranking pass, in the moves
  constexpr int U = kArrangeItems, V = P::kAbs ? 1 : 2, W = (P::kAbs || DIM == 2) ? 4 : 2;
  const PBuf<Real> S = A.buf[1];
  const PBuf<Real> D = A.buf[0];
  const unsigned long long below = (1ull << lane) - 1ull;
  // the scatter is done with the counts: clear them for the next sort
  for (int i = blockIdx.x * kArrangeBlock + tid; i < A.nkeys; i += gridDim.x * kArrangeBlock) A.counts[i] = 0;
  for (int key = blockIdx.x; key < A.nkeys; key += gridDim.x) {
    // (the group's values in scalar registers: the kernel has no vector one left)
    const int s0 = __builtin_amdgcn_readfirstlane(A.seg[key]);
    const int n = __builtin_amdgcn_readfirstlane(A.seg[key + 1]) - s0;
    if (n == 0) continue;
    const int g = key >> 1;
    const int4 where = A.tiles[g];
    const RunDev<Real>& R = A.runs[__builtin_amdgcn_readfirstlane(where.w)];
    const int org[3] = {__builtin_amdgcn_readfirstlane(where.x), __builtin_amdgcn_readfirstlane(where.y),
                        __builtin_amdgcn_readfirstlane(where.z)};
    // a segment of up to kArrangeCap particles keeps each particle's cell and
    // rank in registers and orders the cells; a larger one (dense cells, many
    // particles per cell) takes the arrival order, its ranks through global
    // memory
    const bool ordered = !DENSE && TC <= kArrangeOrderCells && n <= kArrangeCap;
    for (int i = tid; i < TC; i += kArrangeBlock) cnt[i] = 0;
    if (tid == 0) cmax_s = 0;
    __syncthreads();
    // rank of each particle within its cell, in arrival order
    unsigned place[U];      // cell | rank << kCellBits
    unsigned key2[U / 2];   // the keys of two particles
    if (ordered) {
#pragma unroll
      for (int u0 = 0; u0 < U; u0 += V) {
        if (u0 * kArrangeBlock >= n) break;
        Real x[V][3];
        int pc[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const int q = s0 + min(tid + (u0 + v) * kArrangeBlock, n - 1);
          pc[v] = P::kAbs ? 0 : S.cell[q];
#pragma unroll
          for (int d = 0; d < DIM; ++d)
            if (P::kAbs || d < 1) x[v][d] = S.pos[d][q];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
          int c[3] = {0, 0, 0};
          if (P::kAbs) {
#pragma unroll
            for (int d = 0; d < DIM; ++d) {
              const Real fl = floor(x[v][d]);
              c[d] = (int)fl;
              x[v][d] -= fl;
            }
          } else {
            unpack_cell<DIM>(pc[v], c[0], c[1], c[2]);
          }
          const int cl = cell_index<P, DIM>(c, org, A.tile);
          const unsigned k = order_key<P, DIM>(x[v][0], x[v][1]);
          unsigned r = 0;
          if (tid + (u0 + v) * kArrangeBlock < n) r = (unsigned)atomicAdd(&cnt[cl], 1);
          place[u0 + v] = (unsigned)cl | (r << kCellBits);
          if (((u0 + v) & 1) == 0) key2[(u0 + v) / 2] = k;
          else key2[(u0 + v) / 2] |= k << 16;
        }
      }
    } else {
      for (int i = tid; i < n; i += kArrangeBlock) {
        const int q = s0 + i;
        A.keys[q] = atomicAdd(&cnt[cell_in_tile<P, DIM>(S, q, org, A.tile)], 1);
      }
    }
    __syncthreads();
    // level k < KC: cells holding more than k particles, numbered in cell order
    for (int k = wave; k < KC; k += nwave) {
      int run = 0;
      for (int c0 = 0; c0 < TC; c0 += 64) {
        const int c = c0 + lane;
        const bool f = c < TC && cnt[c] > k;
        const unsigned long long b = __ballot(f);
        if (c < TC) pre[k * TC + c] = (unsigned short)(run + __popcll(b & below));
        run += __popcll(b);
      }
      if (lane == 0) base[k + 1] = run;
    }
    // exclusive prefixes over cells: of max(0, count - KC) for the ranks
    // beyond the levels, and of the counts for the keys by cell
    if (wave == 0 || (wave == 1 && ordered)) {
      int run = 0;
      for (int c0 = 0; c0 < TC; c0 += 64) {
        const int c = c0 + lane;
        const int v = c < TC ? (wave == 0 ? max(0, cnt[c] - KC) : cnt[c]) : 0;
        int incl = v;
        for (int off = 1; off < 64; off <<= 1) {
          const int t = __shfl_up(incl, off);
          if (lane >= off) incl += t;
        }
        if (c < TC) {
          if (wave == 0) xpre[c] = run + incl - v;
          else first[c] = (unsigned short)(run + incl - v);
        }
        run += __shfl(incl, 63);
      }
      if (wave == 0 && lane == 0) xpre[TC] = run;
    }
    __syncthreads();
    if (tid == 0) {
      base[0] = 0;
      for (int k = 0; k < KC; ++k) base[k + 1] += base[k];
    }
    if (ordered) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (tid + u * kArrangeBlock < n)
          keys[first[place[u] & kCellMask] + (place[u] >> kCellBits)] = (unsigned short)(key2[u / 2] >> (16 * (u & 1)));
    }
    __syncthreads();
    float mb[3] = {0.0f, 0.0f, 0.0f};
    // slot of a particle of cell cl at rank k
    auto slot_of = [&](int cl, int k) { return (k < KC) ? base[k] + (int)pre[k * TC + cl] : base[KC] + xpre[cl] + (k - KC); };
    // bounds of the next step's current contributions (see gpd.hip): |step|
    // per axis, and |v3| for the out-of-plane current in 2D
    auto bound = [&](float u0, float u1, float u2) {
      const float ig = 1.0f / sqrtf(1.0f + u0 * u0 + u1 * u1 + u2 * u2);
      mb[0] = fmaxf(mb[0], (float)R.a[0] * fabsf(u0) * ig);
      mb[1] = fmaxf(mb[1], (float)R.a[1] * fabsf(u1) * ig);
      mb[2] = fmaxf(mb[2], (DIM == 2 ? 1.0f : (float)R.a[2]) * fabsf(u2) * ig);
    };
    // slots o0, o0 + kArrangeBlock, .. from their sources, array by array
    auto fill = [&](int o0, const int* src) {
      auto move = [&](const auto* from, auto* to, auto* v) {
#pragma unroll
        for (int u = 0; u < W; ++u) v[u] = from[src[u]];
#pragma unroll
        for (int u = 0; u < W; ++u)
          if (o0 + u * kArrangeBlock < n) to[s0 + o0 + u * kArrangeBlock] = v[u];
      };
      int iv[W];
      Real rv[W], uv[3][W];
      if (!P::kAbs) move(S.cell, D.cell, iv);
      move(S.tag, D.tag, iv);
#pragma unroll
      for (int d = 0; d < DIM; ++d) move(S.pos[d], D.pos[d], rv);
#pragma unroll
      for (int d = 0; d < 3; ++d) move(S.u[d], D.u[d], uv[d]);
      if (!P::kAbs) {
#pragma unroll
        for (int u = 0; u < W; ++u)
          if (o0 + u * kArrangeBlock < n) bound((float)uv[0][u], (float)uv[1][u], (float)uv[2][u]);
      }
    };
    if (ordered) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u * kArrangeBlock >= n) break;
        if (tid + u * kArrangeBlock >= n) continue;
        // the rank in the order of the keys (equal keys in arrival order);
        // a cell too dense for a look at all its keys keeps the arrival order
        const int cl = (int)(place[u] & kCellMask), m = cnt[cl], f0 = first[cl];
        int k = (int)(place[u] >> kCellBits);
        if (m <= kArrangeOrderCount) {
          const int r = k, kv = keys[f0 + r];
          k = 0;
          for (int j = 0; j < m; ++j) {
            const int o = keys[f0 + j];
            k += (o < kv || (o == kv && j < r)) ? 1 : 0;
          }
        }
        place[u] = (unsigned)slot_of(cl, k);
      }
      // the source of every slot, in the keys' place
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (tid + u * kArrangeBlock < n) keys[place[u]] = (unsigned short)(tid + u * kArrangeBlock);
      __syncthreads();
#pragma unroll 1
      for (int u0 = 0; u0 < U; u0 += W) {
        if (u0 * kArrangeBlock >= n) break;
        int src[W];
        const int o0 = tid + u0 * kArrangeBlock;
#pragma unroll
        for (int u = 0; u < W; ++u) src[u] = s0 + keys[min(o0 + u * kArrangeBlock, n - 1)];
        fill(o0, src);
      }
    } else if (DENSE) {
      // the sources through the tags' place of the current store, which holds
      // nothing yet: 4 bytes of a particle are scattered there, not all of it
      // (42M particles in mixed precision 2.76 -> 1.57 ms, 21M in FP64 1.40 -> 1.10)
      for (int i = tid; i < n; i += kArrangeBlock)
        D.tag[s0 + slot_of(cell_in_tile<P, DIM>(S, s0 + i, org, A.tile), A.keys[s0 + i])] = i;
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): written before any other wave reads them
      __syncthreads();
      for (int o0 = tid; o0 < n; o0 += W * kArrangeBlock) {
        int src[W];
#pragma unroll
        for (int u = 0; u < W; ++u) {
          const int o = o0 + u * kArrangeBlock;
          src[u] = s0 + (o < n ? D.tag[s0 + o] : 0);
        }
        fill(o0, src);
      }
    } else {
      for (int i = tid; i < n; i += kArrangeBlock) {
        const int q = s0 + i;
        const int cl = cell_in_tile<P, DIM>(S, q, org, A.tile);
        if (!P::kAbs) bound((float)S.u[0][q], (float)S.u[1][q], (float)S.u[2][q]);
        const int o = s0 + slot_of(cl, A.keys[q]);
        if (!P::kAbs) D.cell[o] = S.cell[q];
        for (int d = 0; d < DIM; ++d) D.pos[d][o] = S.pos[d][q];
        D.u[0][o] = S.u[0][q];
        D.u[1][o] = S.u[1][q];
        D.u[2][o] = S.u[2][q];
        D.tag[o] = S.tag[q];
      }
    }
    if (!P::kAbs) {
      for (int c = 0; c < 3; ++c) {
        float m = mb[c];
        for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
        if (lane == 0) atomicMax(reinterpret_cast<int*>(A.jb) + 4 * g + c, __float_as_int(m));
      }
      // largest particle count of one cell; the two species' maxima add
      int cm = 0;
      for (int i = tid; i < TC; i += kArrangeBlock) cm = max(cm, cnt[i]);
      for (int off = 32; off >= 1; off >>= 1) cm = max(cm, __shfl_xor(cm, off));
      if (lane == 0) atomicMax(&cmax_s, cm);
      __syncthreads();
      if (tid == 0) atomicAdd(A.jb + 4 * g + 3, (float)cmax_s);
    }
    __syncthreads();
  }
  // the last group to finish ends the sort.  Every wave of a group has read the
  // request before the group is counted: a group whose segments are all empty
  // has met no other barrier, and a wave that found the request cleared would
  // leave its part of the counts to the next sort.
  __syncthreads();
  if (tid == 0 && atomicAdd(&A.st->arrange_done, 1u) == gridDim.x - 1) {
    A.st->arrange_done = 0;
    A.st->n_sorts += 1;
    A.st->sort_request = 0;
  }
}

template <class P>
hipError_t launch_sort(const SortArgs<typename P::Real>& a, int ndim, hipStream_t s) {
  constexpr long long per = (long long)kSortBlock * kSortItems;
  const long long blocks = (a.np_total + per - 1) / per;
  // grid-stride kernels: enough groups to fill the chip when a sort runs,
  // few enough that the launches between sorts (all exit at once) are cheap
  const int grid = (int)(blocks < kSortGrid ? (blocks > 0 ? blocks : 1) : kSortGrid);
  if (ndim == 2)
    hipLaunchKernelGGL((sort_count<P, 2>), dim3(grid), dim3(kSortBlock), 0, s, a);
  else
    hipLaunchKernelGGL((sort_count<P, 3>), dim3(grid), dim3(kSortBlock), 0, s, a);
  if (ndim == 2)
    hipLaunchKernelGGL((sort_scatter<P, 2>), dim3(grid), dim3(kSortBlock), 0, s, a);
  else
    hipLaunchKernelGGL((sort_scatter<P, 3>), dim3(grid), dim3(kSortBlock), 0, s, a);
  const int agrid = a.nkeys < 1024 ? a.nkeys : 1024;
  const size_t lds = arrange_lds(a.tc, a.kcap, a.dense);
  if (ndim == 2) {
    if (a.dense) hipLaunchKernelGGL((sort_arrange<P, 2, true>), dim3(agrid), dim3(kArrangeBlock), lds, s, a);
    else hipLaunchKernelGGL((sort_arrange<P, 2, false>), dim3(agrid), dim3(kArrangeBlock), lds, s, a);
  } else {
    if (a.dense) hipLaunchKernelGGL((sort_arrange<P, 3, true>), dim3(agrid), dim3(kArrangeBlock), lds, s, a);
    else hipLaunchKernelGGL((sort_arrange<P, 3, false>), dim3(agrid), dim3(kArrangeBlock), lds, s, a);
  }
  return hipGetLastError();
}

template hipError_t launch_sort<F32>(const SortArgs<float>&, int, hipStream_t);
template hipError_t launch_sort<F64>(const SortArgs<double>&, int, hipStream_t);

}  // namespace wtpic
