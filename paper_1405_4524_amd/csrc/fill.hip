// fill.hip -- the outer-product fill of the all-to-all propagator (Sec. 7, eq. Sfill) on the
// FP64 matrix cores, and the contraction sum_{z,x} tr[S1 S2^dag] built on it (the "S_s fill",
// "S_s^dag fill" and "sum_x sum_z tr S_s S_s^dag" operations of the paper's timing study).
//
//   S(t, z; t_src, x)_{ab} = (1/N) sum_i X_i(t, z)_a conj(eta_i(t_src, x)_b)
//
// is, for one sink timeslice t, the complex matrix product C = P Q^H of the (12 L^3) x N block
// P of solutions at t and the (12 L^3) x N block Q of sources at t_src; in the canonical
// [src][t][z][y][x][spin][colour] arrays each (source, timeslice) column is contiguous.  The
// kernel is generic in the K strides: C(m, n) = scale sum_k P(m, k) conj(Q(n, k)) with
// P(m, k) = P[m + k pk], Q(n, k) = Q[n + k qk] (complex elements); the contraction makes one product
// per grid.y index z (P offset by pz per z).
//
// A wave owns a 32 x 32 tile of C (M = 12 X Y Z is a multiple of 96: no tile is ragged) as 2 x 2 tiles of
// 16 x 16 on v_mfma_f64_16x16x4_f64, four real products per complex tile and K step of 4 (Re += Pr Qr +
// Pi Qi, Im += Pi Qr - Pr Qi).  Each lane loads its operands straight from memory in fragment layout (one
// 16-byte complex per operand tile and K step; 16 lanes read 256 contiguous bytes of a column), the next K
// step's before the products of this one, in two register sets that alternate.  Bound by the FP64 matrix
// rate.  8^3x16, 1024 sources: 5.7 ms with the loads right before their products (54 TFLOP/s), 4.7 now (66;
// the library's FP64 products reach 71-74 here).  Two waves per SIMD are asked for so that everything stays in
// vector registers: given more, the compiler moves operands between register files (5.1 ms; 3 x 3 tiles
// 5.2 and up).
// Elements past K are zeroed.  Blocks are in row-major tile order, so that an XCD's waves share a few rows
// and columns of tiles in its L2.
//
// Fill mode stores C, or the spin-colour dagger of its 12 x 12 blocks.  Contract mode multiplies two
// products (S1 from the first operand pair, S2 from the second) tile by tile and accumulates sum C1 conj(C2)
// without storing either: a wave takes several tiles in turn, and a block's FP64 partial is summed in block
// order by a second launch.
#include "a2a_contract.h"
#include "a2a_kernels.h"

namespace a2a {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
// global loads / stores through address-space-1 pointers (the arrays are device memory)
__device__ __forceinline__ double2 ldc(const double* base, long long idx) {
  const d2v v = *(const __attribute__((address_space(1))) d2v*)(base + 2 * idx);
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ void stc(double* p, double re, double im) {
  d2v v;
  v.x = re;
  v.y = im;
  *(__attribute__((address_space(1))) d2v*)p = v;
}

__device__ __forceinline__ d4v mfma(double a, double b, const d4v& c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

}  // namespace

// products of the operand pairs: NT x NT tiles of 16 x 16 each, from this lane's row and K offset
template <int NP, int NT>
__device__ __forceinline__ void fill_tile(const FillArgs& a, int kr, const double* const (&P)[NP],
                                          const double* const (&Q)[NP], d4v (&cr)[NP][NT][NT],
                                          d4v (&ci)[NP][NT][NT]) {
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) cr[p][i][j] = ci[p][i][j] = d4v{0.0, 0.0, 0.0, 0.0};

  struct Step {
    double2 A[NP][NT], B[NP][NT];
  } s0, s1;
  auto load = [&](Step& s, int k0) {
    long long k = k0;                                  // wave-uniform, but for the last step,
    if (k0 + 4 > a.K) k = min(k0 + kr, a.K - 1) - kr;  // whose lanes past K read K - 1
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        s.A[p][i] = ldc(P[p], k * a.pk + 16 * i);
        s.B[p][i] = ldc(Q[p], k * a.qk + 16 * i);
      }
  };
  auto step = [&](Step& s, int k0) {
    if (k0 + 4 > a.K) {
      if (k0 + kr >= a.K)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int i = 0; i < NT; ++i) s.A[p][i] = s.B[p][i] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) cr[p][i][j] = mfma(s.A[p][i].x, s.B[p][j].x, cr[p][i][j]);
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) ci[p][i][j] = mfma(s.A[p][i].y, s.B[p][j].x, ci[p][i][j]);
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) cr[p][i][j] = mfma(s.A[p][i].y, s.B[p][j].y, cr[p][i][j]);
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) ci[p][i][j] = mfma(-s.A[p][i].x, s.B[p][j].y, ci[p][i][j]);
    }
  };
  load(s0, 0);
  for (int k0 = 0; k0 < a.K; k0 += 8) {  // two steps' operands alternate
    load(s1, k0 + 4);
    step(s0, k0);
    if (k0 + 4 >= a.K) break;
    load(s0, k0 + 8);
    step(s1, k0 + 4);
  }
}

// DAG: store the product's spin-colour dagger; NT: 16-wide tiles along an edge of the wave's tile
template <bool DAG, int NT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_fill(FillArgs a) {
  constexpr int E = 16 * NT;
  const int lane = threadIdx.x, idx = lane & 15, kr = lane >> 4;
  const int tiles_n = a.N / E;
  const int m0 = (int)(blockIdx.x / tiles_n) * E, n0 = (int)(blockIdx.x % tiles_n) * E;
  const double* const P[1] = {a.P[0] + 2 * (m0 + idx + kr * a.pk)};
  const double* const Q[1] = {a.Q[0] + 2 * (n0 + idx + kr * a.qk)};
  d4v cr[1][NT][NT], ci[1][NT][NT];
  fill_tile<1, NT>(a, kr, P, Q, cr, ci);
  // element q of a 16 x 16 accumulator tile is row 4 q + lane / 16, column lane % 16
  if constexpr (!DAG) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          stc(a.out + 2 * ((m0 + 16 * i + 4 * q + kr) * a.om + n0 + 16 * j + idx),
              a.scale * cr[0][i][j][q], a.scale * ci[0][i][j][q]);
  } else {
    // (12 u + s, 12 v + s2) -> (12 u + s2, 12 v + s), conjugated
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = m0 + 16 * i + 4 * q + kr, n = n0 + 16 * j + idx, d = n % 12 - m % 12;
          stc(a.out + 2 * ((m + d) * a.om + n - d), a.scale * cr[0][i][j][q], -a.scale * ci[0][i][j][q]);
        }
  }
}

// sum C1 conj(C2) over 16 x 16 tiles (whose two products hold twice the operands of a stored one: 8^3x16 with
// 256 sources 41.5 ms, 60 TFLOP/s; 2 x 2 tiles, where operands move between register files, took 12% longer).  A wave
// takes every 4 gridDim.x-th tile in row-major order, so that the waves at work share rows and columns in the
// L2s, and keeps its sum in registers.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_fill_contract(FillArgs a) {
  const int lane = threadIdx.x & 63, idx = lane & 15, kr = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tm = a.M / 16, tn = a.N / 16, stride = 4 * (int)gridDim.x;
  const long long z = blockIdx.y;
  int row = (4 * (int)blockIdx.x + w) / tn, col = (4 * (int)blockIdx.x + w) % tn;
  double v[2] = {0.0, 0.0};
  while (row < tm) {
    const double *P[2], *Q[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      P[p] = a.P[p] + 2 * (z * a.pz + 16 * row + idx + kr * a.pk);
      Q[p] = a.Q[p] + 2 * (16 * col + idx + kr * a.qk);
    }
    d4v cr[2][1][1], ci[2][1][1];
    fill_tile<2, 1>(a, kr, P, Q, cr, ci);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double r1 = cr[0][0][0][q], i1 = ci[0][0][0][q], r2 = cr[1][0][0][q], i2 = ci[1][0][0][q];
      v[0] += r1 * r2 + i1 * i2;
      v[1] += i1 * r2 - r1 * i2;
    }
    row += stride / tn;
    col += stride % tn;
    if (col >= tn) {
      col -= tn;
      ++row;
    }
  }
  v[0] *= a.scale * a.scale;
  v[1] *= a.scale * a.scale;
  block_sum_n<2, 256>(v);
  if (threadIdx.x < 2) a.partial[2 * (z * gridDim.x + blockIdx.x) + threadIdx.x] = threadIdx.x == 0 ? v[0] : v[1];
}

// corr[z] = sum of the block partials of z, in block order
__global__ __launch_bounds__(64) void k_fill_sum(int nblk, const double* partial, double* corr) {
  const long long z = blockIdx.x;
  double r = 0.0, im = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 64) {
    r += partial[2 * (z * nblk + b)];
    im += partial[2 * (z * nblk + b) + 1];
  }
  r = wave_sum(r);
  im = wave_sum(im);
  if (threadIdx.x == 0) {
    corr[2 * z] = r;
    corr[2 * z + 1] = im;
  }
}

// Blocks of four waves: one per 64 x 64 entries (four tiles a wave), up to 32 times the 512 that the chip
// holds, from where on the waves take more tiles each instead.  With one wave and one partial per tile
// 24^3x48 asked for 83 GB of partials and for more threads than a launch can have, and their sum was a good
// part of the time: 16^3x2 with 8 sources 72.6 ms, now 12.6; 8^3x16 with 256 47.0, now 41.5; only the
// smallest lose (2^3x4 with 64 27 us, now 39, three tiles in turn).
int fill_blocks(int M, int N) {
  return (int)std::min(16384LL, (long long)((M + 63) / 64) * ((N + 63) / 64));
}

template <int NT>
static void launch_fill_t(const FillArgs& a, hipStream_t s) {
  const dim3 g((unsigned)((long long)(a.M / (16 * NT)) * (a.N / (16 * NT))));
  if (a.dagger)
    hipLaunchKernelGGL((k_fill<true, NT>), g, dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((k_fill<false, NT>), g, dim3(64), 0, s, a);
}

// 2 x 2 tiles from 1024 rows on; below, four times the waves fill more of the chip (768 rows, 128 sources: 36
// us in 2 x 2 tiles, 34 in single ones; 6144 rows, 1024 sources: 4.7 ms and 5.5)
void launch_fill(const FillArgs& a, hipStream_t s) {
  if (a.M >= 1024)
    launch_fill_t<2>(a, s);
  else
    launch_fill_t<1>(a, s);
}

void launch_fill_contract(const FillArgs& a, int nz, double* corr, hipStream_t s) {
  const int nb = fill_blocks(a.M, a.N);
  hipLaunchKernelGGL(k_fill_contract, dim3((unsigned)nb, (unsigned)nz), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_fill_sum, dim3((unsigned)nz), dim3(64), 0, s, nb, a.partial, corr);
}

}  // namespace a2a
