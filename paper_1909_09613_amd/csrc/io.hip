// Particles between the caller's FP64 arrays and the device layout.  The host
// copies its arrays as they are (x and u, [n][3] doubles) into the second
// particle store, which holds nothing between sorts, and the device converts:
// a pass over one particle's 48 bytes and its 28 to 52 bytes of state, bound by
// HBM and far below the copy itself.  (Converted on one host core, with the
// stores of both species read back for each: 1.05M particles in FP64, loaded,
// stepped eight times and read back, 24 to 39 ms, now 10 ms, mostly
// the copies and the first touch of the caller's result arrays.)
#include "common.hpp"
#include "launch.hpp"

namespace wtpic {

// Bit 0: some position is not finite, bit 1: some momentum.
template <int DIM>
__global__ void __launch_bounds__(256) io_check_kernel(const double* x, const double* u, long long n, int* flag) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  int bad = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
#pragma unroll
    for (int k = 0; k < DIM; ++k) bad |= isfinite(x[3 * i + k]) ? 0 : 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) bad |= isfinite(u[3 * i + k]) ? 0 : 2;
  }
  if (bad) atomicOr(flag, bad);
}

// One species of one run into its place in the current store, positions
// wrapped into [0, n), a mixed-precision offset that rounds to 1 carried into
// the next cell.
template <class P, int DIM>
__global__ void __launch_bounds__(256) io_load_kernel(IoArgs<typename P::Real> A) {
  using Real = typename P::Real;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < A.n; i += stride) {
    const long long p = A.base + i;
    int cc[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      const double nd = A.cells[k];
      double v = fmod(A.x[3 * i + k], nd);
      while (v < 0.0) v += nd;
      while (v >= nd) v -= nd;
      if (P::kAbs) {
        A.buf.pos[k][p] = Real(v);
      } else {
        double fl = floor(v);
        float f = (float)(v - fl);
        if (f >= 1.0f) {
          f = 0.0f;
          fl += 1.0;
          if (fl >= nd) fl = 0.0;
        }
        cc[k] = (int)fl;
        A.buf.pos[k][p] = Real(f);
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) A.buf.u[k][p] = Real(A.u[3 * i + k]);
    if (!P::kAbs) A.buf.cell[p] = pack_cell<DIM>(cc[0], cc[1], cc[2]);
    A.buf.tag[p] = (A.species << kSpeciesShift) | (int)i;
  }
}

// One species of one run from the current store (the run's particles of both
// species, in any order) in identity order; *found counts them.
template <class P, int DIM>
__global__ void __launch_bounds__(256) io_store_kernel(IoArgs<typename P::Real> A, int* found) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  int mine = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < 2 * A.n; i += stride) {
    const long long p = A.base + i;
    const int tag = A.buf.tag[p];
    const long long id = tag & ((1 << kSpeciesShift) - 1);
    if (((tag >> kSpeciesShift) & 1) != A.species || id >= A.n) continue;
    ++mine;
    int cc[3] = {0, 0, 0};
    if (!P::kAbs) unpack_cell<DIM>(A.buf.cell[p], cc[0], cc[1], cc[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      A.x[3 * id + k] = k < DIM ? (P::kAbs ? (double)A.buf.pos[k][p] : (double)cc[k] + (double)A.buf.pos[k][p]) : 0.0;
      A.u[3 * id + k] = (double)A.buf.u[k][p];
    }
  }
  for (int off = 32; off >= 1; off >>= 1) mine += __shfl_xor(mine, off);
  if ((threadIdx.x & 63) == 0 && mine) atomicAdd(found, mine);
}

namespace {
unsigned io_grid(long long n) {
  const long long b = (n + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}
}  // namespace

template <class P>
hipError_t launch_io_check(const IoArgs<typename P::Real>& a, int ndim, int* flag, hipStream_t s) {
  if (ndim == 2)
    hipLaunchKernelGGL(io_check_kernel<2>, dim3(io_grid(a.n)), dim3(256), 0, s, a.x, a.u, a.n, flag);
  else
    hipLaunchKernelGGL(io_check_kernel<3>, dim3(io_grid(a.n)), dim3(256), 0, s, a.x, a.u, a.n, flag);
  return hipGetLastError();
}

template <class P>
hipError_t launch_io_load(const IoArgs<typename P::Real>& a, int ndim, hipStream_t s) {
  if (ndim == 2)
    hipLaunchKernelGGL((io_load_kernel<P, 2>), dim3(io_grid(a.n)), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((io_load_kernel<P, 3>), dim3(io_grid(a.n)), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <class P>
hipError_t launch_io_store(const IoArgs<typename P::Real>& a, int ndim, int* found, hipStream_t s) {
  if (ndim == 2)
    hipLaunchKernelGGL((io_store_kernel<P, 2>), dim3(io_grid(2 * a.n)), dim3(256), 0, s, a, found);
  else
    hipLaunchKernelGGL((io_store_kernel<P, 3>), dim3(io_grid(2 * a.n)), dim3(256), 0, s, a, found);
  return hipGetLastError();
}

template hipError_t launch_io_check<F32>(const IoArgs<float>&, int, int*, hipStream_t);
template hipError_t launch_io_check<F64>(const IoArgs<double>&, int, int*, hipStream_t);
template hipError_t launch_io_load<F32>(const IoArgs<float>&, int, hipStream_t);
template hipError_t launch_io_load<F64>(const IoArgs<double>&, int, hipStream_t);
template hipError_t launch_io_store<F32>(const IoArgs<float>&, int, int*, hipStream_t);
template hipError_t launch_io_store<F64>(const IoArgs<double>&, int, int*, hipStream_t);

}  // namespace wtpic
