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
// P(m, k) = P[m + k pk], Q(n, k) = Q[n + k qk] (complex elements), one product per
// grid.y index z (operand offsets pz, qz per z).
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
// without storing either: per-block FP64 partials, summed in block order by a second launch.
#include "a2a_contract.h"
#include "a2a_kernels.h"

namespace a2a {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));
// tiles along an edge in the contraction, whose two products hold twice the operands: 8^3x16 with 256
// sources 42 ms (58 TFLOP/s), 47 with 2 x 2 tiles (operands move between register files), 62 before
constexpr int FTC = 1;

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

// MODE 0: store the product, 1: its spin-colour dagger, 2: contract two products; NT: 16-wide tiles along
// an edge of the wave's tile
template <int MODE, int NT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_fill(FillArgs a) {
  constexpr int NP = MODE == 2 ? 2 : 1, E = 16 * NT;
  const int lane = threadIdx.x, idx = lane & 15, kr = lane >> 4;
  const int tiles_n = a.N / E;
  const int m0 = (int)(blockIdx.x / tiles_n) * E, n0 = (int)(blockIdx.x % tiles_n) * E;
  const long long z = blockIdx.y;
  const double* P[NP];  // this lane's row and K offset
  const double* Q[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    P[p] = a.P[p] + 2 * (z * a.pz + m0 + idx + kr * a.pk);
    Q[p] = a.Q[p] + 2 * (z * a.qz + n0 + idx + kr * a.qk);
  }
  d4v cr[NP][NT][NT], ci[NP][NT][NT];
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
    long long k = k0;                                           // wave-uniform, but for the last step,
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

  // element q of a 16 x 16 accumulator tile is row 4 q + lane / 16, column lane % 16
  if constexpr (MODE == 0) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          stc(a.out + 2 * (z * a.oz + (m0 + 16 * i + 4 * q + kr) * a.om + n0 + 16 * j + idx),
              a.scale * cr[0][i][j][q], a.scale * ci[0][i][j][q]);
  } else if constexpr (MODE == 1) {
    // (12 u + s, 12 v + s2) -> (12 u + s2, 12 v + s), conjugated
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = m0 + 16 * i + 4 * q + kr, n = n0 + 16 * j + idx, d = n % 12 - m % 12;
          stc(a.out + 2 * (z * a.oz + (m + d) * a.om + n - d), a.scale * cr[0][i][j][q], -a.scale * ci[0][i][j][q]);
        }
  } else {
    double vr = 0.0, vi = 0.0;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // C1 conj(C2)
          const double r1 = cr[0][i][j][q], i1 = ci[0][i][j][q], r2 = cr[NP - 1][i][j][q], i2 = ci[NP - 1][i][j][q];
          vr += r1 * r2 + i1 * i2;
          vi += i1 * r2 - r1 * i2;
        }
    vr = wave_sum(vr * a.scale * a.scale);
    vi = wave_sum(vi * a.scale * a.scale);
    if (lane == 0) {
      a.partial[2 * (z * gridDim.x + blockIdx.x)] = vr;
      a.partial[2 * (z * gridDim.x + blockIdx.x) + 1] = vi;
    }
  }
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

long long fill_blocks(int M, int N) { return (long long)(M / (16 * FTC)) * (N / (16 * FTC)); }

template <int NT>
static void launch_fill_t(const FillArgs& a, int nz, hipStream_t s) {
  const dim3 g((unsigned)((long long)(a.M / (16 * NT)) * (a.N / (16 * NT))), (unsigned)nz);
  if (a.dagger)
    hipLaunchKernelGGL((k_fill<1, NT>), g, dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((k_fill<0, NT>), g, dim3(64), 0, s, a);
}

// 2 x 2 tiles from 1024 rows on; below, four times the waves fill more of the chip (768 rows, 128 sources: 36
// us in 2 x 2 tiles, 34 in single ones; 6144 rows, 1024 sources: 4.7 ms and 5.5)
void launch_fill(const FillArgs& a, int nz, hipStream_t s) {
  if (a.M >= 1024)
    launch_fill_t<2>(a, nz, s);
  else
    launch_fill_t<1>(a, nz, s);
}

void launch_fill_contract(const FillArgs& a, int nz, double* corr, hipStream_t s) {
  const int nb = (int)fill_blocks(a.M, a.N);
  hipLaunchKernelGGL((k_fill<2, FTC>), dim3((unsigned)nb, (unsigned)nz), dim3(64), 0, s, a);
  hipLaunchKernelGGL(k_fill_sum, dim3((unsigned)nz), dim3(64), 0, s, nb, a.partial, corr);
}

}  // namespace a2a
