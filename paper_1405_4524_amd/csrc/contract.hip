// contract.hip -- the stochastic-operator contraction (Sec. 7, eq. stoop) and the
// zero-momentum pion / pi-pi correlators built from it (Sec. 7; Sec. 5 and 8 diagrams).
//
//   O_ab(t) = sum_{y in timeslice t} eta_a(y)^dag gamma_5 X_b(y)
//
// is, per timeslice, a complex matrix product E_t^dag (gamma_5 X_t) with inner dimension
// K = 12 L^3 taken straight from the canonical [src][t][z][y][x][spin][colour] arrays, where
// each (source, timeslice) column is contiguous.
#include "a2a_contract.h"
#include "a2a_kernels.h"

namespace a2a {

typedef double d4v __attribute__((ext_vector_type(4)));

// One wave computes a tile of 16 NA x 16 NB entries over a chunk of sites on the FP64 matrix cores,
// its operands loaded from memory in fragment layout: v_mfma_f64_16x16x4 takes A[l % 16][l / 16] from
// lane l, and with the K step's four elements taken as component c of the four spins of one site, lane
// (row, spin) reads its row's 48 contiguous bytes of that spin and gamma_5 is a sign per lane.  Every
// element is read once per tile, no LDS and no barrier are used, and the next sites' operands load
// during the products of the current ones (9 tiles of a 48-source block: 108 products a site, ~7000
// cycles).  Rows and columns past na and n read the last one; their entries are not stored.  Chunk
// partials are summed in fixed order.
//   The largest tile that n allows (up to 4 x 4) reads the operands the fewest times.  Memory bounds it up
// to 48 sources: rows are a power of two apart, and what counts is how long a row is read before the next
// one (sites per iteration: one 9.3 ms, two 8.05 ms for 32^3x64 with 48 sources, where 64 x 64 block tiles
// staged through LDS between barriers took 13.3 ms, 33 TFLOP/s and 2.9 TB/s; now 58 TFLOP/s and
// 4.8 TB/s); from 64 sources on the FP64 matrix rate does (57 TFLOP/s at 128 and 256).
// Virtual rows: row r < na is source r % ns (or rows[t ns + r % ns]) times phase r / ns of the phases
// [na / ns][V3], so that all momenta of a call share one pass over X.
struct StochArgs {
  int n, na, ns;         // columns, virtual rows, rows per phase
  int nchunk, spc;       // chunks of a timeslice, sites per chunk
  int nta, ntb;          // row and column tiles
  int nt, t_first, g5;
  long V;
  int V3;
  const double* eta;
  const double* X;
  const double* phase;
  const int* rows;
  double* partial;
};

// sites per iteration: as many as the registers of one wave per SIMD hold twice (they divide X Y Z)
constexpr int stoch_sites(int na, int nb) {
  return 16 * na * nb + 96 * (na + nb) <= 450 ? 4 : 16 * na * nb + 48 * (na + nb) <= 450 ? 2 : 1;
}

template <int NA, int NB>
__global__ __launch_bounds__(64) void k_stoch_partial(StochArgs a) {
  constexpr int SN = stoch_sites(NA, NB);
  // blocks: the tiles of one (timeslice, chunk) share its rows through the L2 of one XCD
  const int ntile = a.nta * a.ntb, units = a.nt * a.nchunk;
  const int g = blockIdx.x / (8 * ntile), r = blockIdx.x % (8 * ntile);
  const int unit = g * 8 + r % 8, tile = r / 8;
  if (unit >= units) return;
  const int tl = unit % a.nt, chunk = unit / a.nt, t = a.t_first + tl;
  const int a0 = tile / a.ntb * 16 * NA, b0 = tile % a.ntb * 16 * NB;
  const int lane = threadIdx.x, li = lane & 15, q = lane >> 4;
  const int s0 = chunk * a.spc, s1 = min(a.V3, s0 + a.spc);
  const double sg = a.g5 && q >= 2 ? -1.0 : 1.0;  // gamma_5 = diag(1,1,-1,-1)
  const double *pe[NA], *px[NB], *pf[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int ra = min(a0 + 16 * i + li, a.na - 1), ph = ra / a.ns, rr = ra - ph * a.ns;
    const int ar = a.rows ? a.rows[(size_t)t * a.ns + rr] : rr;
    pe[i] = a.eta + 2 * ((size_t)ar * 12 * a.V + (size_t)t * 12 * a.V3 + 3 * q);
    pf[i] = a.phase ? a.phase + 2 * (size_t)ph * a.V3 : nullptr;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int rb = min(b0 + 16 * j + li, a.n - 1);
    px[j] = a.X + 2 * ((size_t)rb * 12 * a.V + (size_t)t * 12 * a.V3 + 3 * q);
  }
  d4v cr[NA][NB], ci[NA][NB];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) cr[i][j] = ci[i][j] = d4v{0.0, 0.0, 0.0, 0.0};
  double2 ne[NA][SN][3], nx[NB][SN][3], nf[NA][SN];
  auto load = [&](int s) {
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int u = 0; u < SN; ++u) {
        const double2* p = (const double2*)(pe[i] + (size_t)24 * (s + u));
#pragma unroll
        for (int c = 0; c < 3; ++c) ne[i][u][c] = p[c];
        if (a.phase) nf[i][u] = *(const double2*)(pf[i] + (size_t)2 * (s + u));
      }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int u = 0; u < SN; ++u) {
        const double2* p = (const double2*)(px[j] + (size_t)24 * (s + u));
#pragma unroll
        for (int c = 0; c < 3; ++c) nx[j][u][c] = p[c];
      }
  };
  if (s0 < s1) load(s0);
  for (int s = s0; s < s1; s += SN) {
    double2 e[NA][SN][3], x[NB][SN][3];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int u = 0; u < SN; ++u)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          e[i][u][c] = ne[i][u][c];
          if (a.phase)  // eta conj(f) with f = exp(-i p.y): the product below takes conj(eta) f
            e[i][u][c] = make_double2(ne[i][u][c].x * nf[i][u].x + ne[i][u][c].y * nf[i][u].y,
                                      ne[i][u][c].y * nf[i][u].x - ne[i][u][c].x * nf[i][u].y);
        }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int u = 0; u < SN; ++u)
#pragma unroll
        for (int c = 0; c < 3; ++c) x[j][u][c] = make_double2(sg * nx[j][u][c].x, sg * nx[j][u][c].y);
    load(min(s + SN, s1 - SN));
    // four real products per complex K step: Re += er xr + ei xi, Im += er xi - ei xr, tile-interleaved
    // so that consecutive products accumulate into different registers
#pragma unroll
    for (int u = 0; u < SN; ++u)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[i][u][c].x, x[j][u][c].x, cr[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[i][u][c].x, x[j][u][c].y, ci[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[i][u][c].y, x[j][u][c].y, cr[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-e[i][u][c].y, x[j][u][c].x, ci[i][j], 0, 0, 0);
      }
  }
  // element k of a 16 x 16 accumulator tile is row 4 k + lane / 16, column lane % 16
  double* out = a.partial + ((size_t)tl * a.nchunk + chunk) * a.na * a.n * 2;
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ra = a0 + 16 * i + 4 * k + q, rb = b0 + 16 * j + li;
        if (ra < a.na && rb < a.n)
          *(double2*)(out + 2 * ((size_t)ra * a.n + rb)) = make_double2(cr[i][j][k], ci[i][j][k]);
      }
}

// chunk sums; blockDim.y splits the chunks, in a fixed order
__global__ __launch_bounds__(256) void k_stoch_sum(long per, int T, int nchunk, const double* partial, double* O) {
  __shared__ double2 part[256];
  const int nx = blockDim.x, ny = blockDim.y;
  const long i = (long)blockIdx.x * nx + threadIdx.x;  // over T * per complex
  double2 s = make_double2(0.0, 0.0);
  if (i < (long)T * per) {
    const long t = i / per, ab = i % per;
    for (int c = threadIdx.y; c < nchunk; c += ny) {
      const double2 p = ((const double2*)partial)[((size_t)t * nchunk + c) * per + ab];
      s.x += p.x;
      s.y += p.y;
    }
  }
  if (ny > 1) {
    part[threadIdx.y * nx + threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.y) return;
    for (int y = 1; y < ny; ++y) {
      s.x += part[y * nx + threadIdx.x].x;
      s.y += part[y * nx + threadIdx.x].y;
    }
  }
  if (i < (long)T * per) ((double2*)O)[i] = s;
}

// tiles of 16 a wave takes along a dimension of n entries: the blocks of at most four tiles that waste least
static int stoch_tiles(int n) {
  const int tiles = (n + 15) / 16, blocks = (tiles + 3) / 4;
  return (tiles + blocks - 1) / blocks;
}

// Chunks of a timeslice: one wave per SIMD (more of them read from more places at once and were slower,
// 32^3x64 with 32 sources 6.1 ms at one and 7.2 ms at two per SIMD); twice as many where a wave reads few
// distinct rows.
int stoch_chunks(const Geo& g, int na, int n, int nt) {
  const int V3 = g.X * g.Y * g.Z, ta = stoch_tiles(na), tb = stoch_tiles(n);
  const long waves = std::min(na, n) <= 8 ? 2048 : 1024;
  const long tiles = (long)nt * ((na + 16 * ta - 1) / (16 * ta)) * ((n + 16 * tb - 1) / (16 * tb));
  return (int)std::max(1L, std::min(waves / std::max(1L, tiles), (long)V3 / stoch_sites(ta, tb)));
}

template <int NA>
static void launch_stoch_na(int nb, const StochArgs& a, dim3 grid, hipStream_t s) {
  switch (nb) {
    case 1: hipLaunchKernelGGL((k_stoch_partial<NA, 1>), grid, dim3(64), 0, s, a); break;
    case 2: hipLaunchKernelGGL((k_stoch_partial<NA, 2>), grid, dim3(64), 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_stoch_partial<NA, 3>), grid, dim3(64), 0, s, a); break;
    default: hipLaunchKernelGGL((k_stoch_partial<NA, 4>), grid, dim3(64), 0, s, a); break;
  }
}

static void launch_stoch_sum(long per, int nt, int nchunk, const double* partial, double* O, hipStream_t s) {
  const long tot = (long)nt * per;
  // few outputs: split the chunks of an output over threads too
  const int ny = tot >= 65536 || nchunk < 16 ? 1 : 16, nx = 256 / ny;
  hipLaunchKernelGGL(k_stoch_sum, dim3((unsigned)((tot + nx - 1) / nx)), dim3(nx, ny), 0, s, per, nt, nchunk, partial, O);
}

void launch_stoch_ops(const Geo& g, int n, const double* eta, const double* X, double* partial, int nchunk,
                      double* O, hipStream_t s, int g5, int t_first, int nt, const double* phase, const int* rows,
                      int na, int ns) {
  StochArgs a{};
  a.V3 = g.X * g.Y * g.Z;
  a.V = (long)a.V3 * g.T;
  if (nt < 0) nt = g.T;
  if (na <= 0) na = n;  // rows == null: eta rows 0 .. na - 1
  a.n = n;
  a.na = na;
  a.ns = ns > 0 ? ns : na;
  a.nchunk = nchunk;
  const int ta = stoch_tiles(na), tb = stoch_tiles(n), sn = stoch_sites(ta, tb);
  a.spc = ((a.V3 + nchunk - 1) / nchunk + sn - 1) / sn * sn;
  a.nt = nt;
  a.t_first = t_first;
  a.g5 = g5;
  a.eta = eta;
  a.X = X;
  a.phase = phase;
  a.rows = rows;
  a.partial = nchunk > 1 ? partial : O;  // a single chunk needs no sum
  a.nta = (na + 16 * ta - 1) / (16 * ta);
  a.ntb = (n + 16 * tb - 1) / (16 * tb);
  const dim3 grid((unsigned)(((long)nt * nchunk + 7) / 8 * 8 * a.nta * a.ntb));
  switch (ta) {
    case 1: launch_stoch_na<1>(tb, a, grid, s); break;
    case 2: launch_stoch_na<2>(tb, a, grid, s); break;
    case 3: launch_stoch_na<3>(tb, a, grid, s); break;
    default: launch_stoch_na<4>(tb, a, grid, s); break;
  }
  if (nchunk > 1) launch_stoch_sum((long)na * n, nt, nchunk, partial, O, s);
}

// Gram form of sum_{z,x} tr[S1 S2^dag]: corr[t] = (1/n^2) sum_ij E[i][j] F[t][j][i] with
// E = <eta1_i, eta2_j> on the source timeslice and F[t] = <X2_j, X1_i> on timeslice t.
__global__ __launch_bounds__(256) void k_gram_corr(int n, const double* E, const double* F, double* corr) {
  const int t = blockIdx.x;
  const long per = (long)n * n;
  const double* Ft = F + 2 * (size_t)t * per;
  double v[2] = {0.0, 0.0};
  for (long e = threadIdx.x; e < per; e += 256) {
    const long i = e / n, j = e % n;
    const double er = E[2 * (i * n + j)], ei = E[2 * (i * n + j) + 1];
    const double fr = Ft[2 * (j * n + i)], fi = Ft[2 * (j * n + i) + 1];
    v[0] += er * fr - ei * fi;
    v[1] += er * fi + ei * fr;
  }
  block_sum_n<2, 256>(v);
  const double inv = 1.0 / ((double)n * n);
  if (threadIdx.x < 2) corr[2 * t + threadIdx.x] = (threadIdx.x == 0 ? v[0] : v[1]) * inv;
}

void launch_gram_corr(int T, int n, const double* E, const double* F, double* corr, hipStream_t s) {
  hipLaunchKernelGGL(k_gram_corr, dim3((unsigned)T), dim3(256), 0, s, n, E, F, corr);
}

// pi-pi diagrams from point propagators S_p (the 12 solutions of the point sources at
// (t0, x0)) and stochastic propagators of two noise sets (Sec. 8), in factorised form, from the
// timeslice Gram matrices
//   G[t][i][j] = <eta1_i, eta2_j>_t   Fp[t][i][j] = <X1_i, X2_j>_t   Pn[t][k][l] = <Sp_k, Sp_l>_t
//   A[k][i] = <Sp_k, X1_i>_t0          B[t][j][k] = <X2_j, Sp_k>_t
// with, for t = t0 + dt:
//   Cs(dt) = sum_ij G[t0]_ij conj(Fp[t]_ij) / (n1 n2)       L(dt) = sum_ij G[t]_ij conj(Fp[t]_ij) / (n1 n2)
//   D2(dt) = sum_ij G[t]_ij sum_k B[t]_jk A_ki / (n1 n2)    Cp(dt) = sum_k Pn[t]_kk
// The partial kernel sums a chunk of rows i per block (grid: chunks x T); the final kernel sums
// the chunks in order and forms D0 = Cp Cs, D1 = L Cp(0), D2, D3 = conj(D2).
__global__ __launch_bounds__(256) void k_pipi_mixed_partial(int T, int t0, int n1, int n2, int rows,
                                                            const double* G, const double* Fp, const double* A,
                                                            const double* B, double* partial) {
  const int c = blockIdx.x, dt = blockIdx.y, t = (t0 + dt) % T;
  const int i0 = c * rows, i1 = min(n1, i0 + rows);
  const size_t per = (size_t)n1 * n2;
  const double* G0 = G + 2 * (size_t)t0 * per;
  const double* Gt = G + 2 * (size_t)t * per;
  const double* Ft = Fp + 2 * (size_t)t * per;
  const double* Bt = B + 2 * (size_t)t * n2 * 12;
  double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // Cs, L, D2 (re, im)
  const long cnt = (long)(i1 - i0) * n2;
  for (long e = threadIdx.x; e < cnt; e += 256) {
    const int i = i0 + (int)(e / n2), j = (int)(e % n2);
    const size_t ij = 2 * ((size_t)i * n2 + j);
    const double fr = Ft[ij], fi = -Ft[ij + 1];  // F_ji = conj(Fp_ij)
    const double g0r = G0[ij], g0i = G0[ij + 1], gr = Gt[ij], gi = Gt[ij + 1];
    v[0] += g0r * fr - g0i * fi;
    v[1] += g0r * fi + g0i * fr;
    v[2] += gr * fr - gi * fi;
    v[3] += gr * fi + gi * fr;
    double br = 0.0, bi = 0.0;  // (B A)_ji
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double* b = Bt + 2 * ((size_t)j * 12 + k);
      const double* a = A + 2 * ((size_t)k * n1 + i);
      br += b[0] * a[0] - b[1] * a[1];
      bi += b[0] * a[1] + b[1] * a[0];
    }
    v[4] += gr * br - gi * bi;
    v[5] += gr * bi + gi * br;
  }
  block_sum_n<6, 256>(v);
  if (threadIdx.x < 6) {
    double r = 0.0;
#pragma unroll
    for (int q = 0; q < 6; ++q)
      if (q == (int)threadIdx.x) r = v[q];
    partial[((size_t)dt * gridDim.x + c) * 6 + threadIdx.x] = r;
  }
}

__global__ __launch_bounds__(64) void k_pipi_mixed_final(int T, int t0, int nchunk, double norm, const double* Pn,
                                                         const double* partial, double* diag, double* pieces) {
  const int dt = blockIdx.x, t = (t0 + dt) % T;
  double v[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    double s = 0.0;
    for (int c = threadIdx.x; c < nchunk; c += 64) s += partial[((size_t)dt * nchunk + c) * 6 + q];
    v[q] = wave_sum(s) * norm;
  }
  if (threadIdx.x != 0) return;
  double cpr = 0.0, cpi = 0.0, c0r = 0.0, c0i = 0.0;  // traces of the point Gram matrices at t, t0
  for (int k = 0; k < 12; ++k) {
    cpr += Pn[2 * (((size_t)t * 12 + k) * 12 + k)];
    cpi += Pn[2 * (((size_t)t * 12 + k) * 12 + k) + 1];
    c0r += Pn[2 * (((size_t)t0 * 12 + k) * 12 + k)];
    c0i += Pn[2 * (((size_t)t0 * 12 + k) * 12 + k) + 1];
  }
  double* d = diag + 2 * dt;
  d[0] = cpr * v[0] - cpi * v[1];  // D0 = Cp Cs
  d[1] = cpr * v[1] + cpi * v[0];
  d[2 * T] = v[2] * c0r - v[3] * c0i;  // D1 = L Cp(0)
  d[2 * T + 1] = v[2] * c0i + v[3] * c0r;
  d[4 * T] = v[4];  // D2
  d[4 * T + 1] = v[5];
  d[6 * T] = v[4];  // D3 = conj(D2)
  d[6 * T + 1] = -v[5];
  if (pieces) {
    double* p = pieces + 2 * dt;
    p[0] = cpr;
    p[1] = cpi;
    p[2 * T] = v[0];
    p[2 * T + 1] = v[1];
    p[4 * T] = v[2];
    p[4 * T + 1] = v[3];
  }
}

int pipi_mixed_chunks(int n1) { return std::max(1, std::min(n1, 64)); }

void launch_pipi_mixed(int T, int t0, int n1, int n2, const double* Pn, const double* G, const double* Fp,
                       const double* A, const double* B, double* partial, double* diag, double* pieces,
                       hipStream_t s) {
  const int nchunk = pipi_mixed_chunks(n1), rows = (n1 + nchunk - 1) / nchunk;
  hipLaunchKernelGGL(k_pipi_mixed_partial, dim3((unsigned)nchunk, (unsigned)T), dim3(256), 0, s, T, t0, n1, n2, rows,
                     G, Fp, A, B, partial);
  hipLaunchKernelGGL(k_pipi_mixed_final, dim3((unsigned)T), dim3(64), 0, s, T, t0, nchunk,
                     1.0 / ((double)n1 * (double)n2), Pn, partial, diag, pieces);
}

// ------------------------------------------------------------------------------------
// momentum phases and spin-colour diluted operators
// ------------------------------------------------------------------------------------
// off[block] = 1 if the block met an element outside its source's own component that is not zero: of source
// (i, c) over the whole lattice, or with time over the piece's own timeslice.
constexpr int SC_CHECK_SPAN = 1024;  // elements a block takes at a time

__device__ void sc_check_block(const ScCheck& k, int block, int T, int V3) {
  const long V = (long)V3 * T, len = 12L * (k.time ? V3 : V), spans = (len + SC_CHECK_SPAN - 1) / SC_CHECK_SPAN;
  const int runs = 12 * k.nv * (k.time ? T : 1);
  int bad = 0;
  for (long u = block; u < runs * spans; u += SC_CHECK_BLOCKS) {
    const int run = (int)(u / spans), c = run % 12, t = k.time ? run / 12 % T : 0, i = run / (k.time ? 12 * T : 12);
    const long e0 = u % spans * SC_CHECK_SPAN;
    const double2* p = (const double2*)k.eta + ((size_t)i * k.group + 12 * t + c) * 12 * V + (size_t)t * 12 * V3 + e0;
    const int r0 = (int)(e0 % 12), left = (int)min((long)SC_CHECK_SPAN, len - e0);
#pragma unroll
    for (int q = 0; q < SC_CHECK_SPAN / 256; ++q) {
      const int e = 256 * q + threadIdx.x;
      const double2 v = p[min(e, left - 1)];
      bad |= e < left && (r0 + e) % 12 != c && !(v.x == 0.0 && v.y == 0.0);
    }
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) k.off[block] = bad != 0;
}

// f[k][y] = exp(-i p_k.y) on the spatial sites of a timeslice (x fastest), the angle reduced exactly; the
// blocks after those check the sources' support (at the memory rate: 75 MB for 8^3x16 with 768
// time-spin-colour pieces, 15 us of 760; a launch of its own would cost short calls as much again)
__global__ __launch_bounds__(256) void k_phases(int X, int Y, int V3, int T, MomBatch m, double* f, ScCheck check) {
  const int per = (V3 + 255) / 256, b = blockIdx.x;
  if (b >= per * m.nph) return sc_check_block(check, b - per * m.nph, T, V3);
  const int s = b % per * 256 + threadIdx.x, k = b / per;
  if (s >= V3) return;
  const int x = s % X, y = s / X % Y, z = s / (X * Y), Z = V3 / (X * Y);
  const long long* p = m.p[k];
  const double g = (double)(p[0] * x % X) / X + (double)(p[1] * y % Y) / Y + (double)(p[2] * z % Z) / Z;
  double sn, cs;
  sincospi(2.0 * g, &sn, &cs);
  ((double2*)f)[(size_t)k * V3 + s] = make_double2(cs, -sn);
}

void launch_phases(const Geo& g, const MomBatch& m, double* f, const ScCheck& check, hipStream_t s) {
  const int V3 = g.X * g.Y * g.Z, blocks = (V3 + 255) / 256 * m.nph + (check.off ? SC_CHECK_BLOCKS : 0);
  hipLaunchKernelGGL(k_phases, dim3((unsigned)blocks), dim3(256), 0, s, g.X, g.Y, V3, g.T, m, f, check);
}

// Stochastic operators of spin-colour diluted sources (schemes SC and TSC): the source (i, c) is zero
// but for component c, so row (ph, i, c) of O(t) sums over the sites only, with column elements
// X_b(y)_c: a twelfth of the dense products, and of the X rows only one read for all momenta.  One
// wave per component (12 per block), 16 NA virtual rows (phase, noise vector) x 32 columns; the block
// stages 4 sites of its columns in LDS (768-byte runs), every wave takes its component from
// there as the K step's four sites.  8^3x16, 768 sources, 11 phases: the dense products over zeros took
// 13.9 ms, this 0.72 (40 TFLOP/s of matrix products, padding counted).  Neither memory (1.6 GB fetched) nor the
// matrix cores (53% busy) bound it: a CU holds one block, whose waves stage, meet at a barrier and multiply
// in turn, and 384 blocks are one and a half rounds (more, shorter ones cost as much in repeated rows or
// partial sums).
constexpr int SC_SITES = 4;                 // sites per stage (one K step)
constexpr int SC_COLS = 2;                  // column tiles of a block
constexpr int SC_ROW = SC_SITES * 12 + 1;   // complex per staged column (padded: 16 columns, distinct banks)

struct ScArgs {
  int n, nv, nph, group, time;  // columns, noise vectors, phases, pieces per noise vector, time-diluted
  int nchunk, spc, V3;          // chunks of a timeslice, sites per chunk (a multiple of SC_SITES)
  long V;
  const double* eta;
  const double* X;
  const double* phase;
  double* partial;
};

template <int NA>
__global__ __launch_bounds__(768) void k_stoch_sc(ScArgs a) {
  constexpr int NB = SC_COLS;
  __shared__ double2 xs[2][16 * NB * SC_ROW];
  const int c = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
  const int b0 = blockIdx.x * 16 * NB, t = blockIdx.y;
  const int chunk = blockIdx.z % a.nchunk, v0 = blockIdx.z / a.nchunk * 16 * NA, vr = a.nph * a.nv;
  const int s0 = chunk * a.spc, s1 = min(a.V3, s0 + a.spc);
  const double sg = c >= 6 ? -1.0 : 1.0;  // gamma_5
  const double *pe[NA], *pf[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int v = min(v0 + 16 * i + li, vr - 1), ph = v / a.nv, nz = v - ph * a.nv;
    const size_t src = (size_t)nz * a.group + (a.time ? 12 * t : 0) + c;
    pe[i] = a.eta + 2 * (src * 12 * a.V + (size_t)t * 12 * a.V3 + c);
    pf[i] = a.phase + 2 * (size_t)ph * a.V3;
  }
  // staging: 48 lanes load the 768 bytes of four sites of one column; a thread takes two columns
  const int sr = threadIdx.x / 48, sc = threadIdx.x % 48;
  const double2* px = (const double2*)a.X + (size_t)t * 12 * a.V3;
  const double2* px0 = px + (size_t)min(b0 + sr, a.n - 1) * 12 * a.V;
  const double2* px1 = px + (size_t)min(b0 + sr + 16, a.n - 1) * 12 * a.V;
  double2 st0, st1;
  auto fetch = [&](int s) {  // past the timeslice: its last element
    const int e = min(12 * s + sc, 12 * a.V3 - 1);
    st0 = px0[e];
    st1 = px1[e];
  };
  auto put = [&](int buf) {
    xs[buf][sr * SC_ROW + sc] = st0;
    xs[buf][(sr + 16) * SC_ROW + sc] = st1;
  };
  double2 ne[NA], nf[NA];
  auto load = [&](int s) {
    const int y = min(s + q, a.V3 - 1);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      ne[i] = *(const double2*)(pe[i] + (size_t)24 * y);
      nf[i] = *(const double2*)(pf[i] + (size_t)2 * y);
    }
  };
  d4v cr[NA][NB], ci[NA][NB];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) cr[i][j] = ci[i][j] = d4v{0.0, 0.0, 0.0, 0.0};
  fetch(s0);
  load(s0);
  put(0);
  __syncthreads();
  for (int s = s0, buf = 0; s < s1; s += SC_SITES, buf ^= 1) {
    double2 e[NA], x[NB];
    const bool in = s + q < s1;  // sites past the chunk count nothing
#pragma unroll
    for (int i = 0; i < NA; ++i) {  // eta conj(f) g5, as in the dense kernel
      e[i].x = in ? sg * (ne[i].x * nf[i].x + ne[i].y * nf[i].y) : 0.0;
      e[i].y = in ? sg * (ne[i].y * nf[i].x - ne[i].x * nf[i].y) : 0.0;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      x[j] = xs[buf][(16 * j + li) * SC_ROW + 12 * q + c];
      if (!in) x[j] = make_double2(0.0, 0.0);
    }
    fetch(s + SC_SITES);
    load(s + SC_SITES);
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[i].x, x[j].x, cr[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[i].x, x[j].y, ci[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[i].y, x[j].y, cr[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-e[i].y, x[j].x, ci[i][j], 0, 0, 0);
    put(buf ^ 1);
    __syncthreads();
  }
  const int na = 12 * a.nv;
  double2* out = (double2*)a.partial + ((size_t)t * a.nchunk + chunk) * a.nph * na * a.n;
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int v = v0 + 16 * i + 4 * k + q, b = b0 + 16 * j + li;
        if (v < vr && b < a.n) {
          const int ph = v / a.nv, nz = v - ph * a.nv;
          out[((size_t)ph * na + 12 * nz + c) * a.n + b] = make_double2(cr[i][j][k], ci[i][j][k]);
        }
      }
}

static int sc_tiles(int vr) { return std::min(3, (vr + 15) / 16); }
// chunks of a timeslice: a block per CU, at least four stages each
int stoch_sc_chunks(const Geo& g, int nv, int nph, int n) {
  const int V3 = g.X * g.Y * g.Z, vr = nv * nph, ra = 16 * sc_tiles(vr);
  const long blocks = (long)((n + 16 * SC_COLS - 1) / (16 * SC_COLS)) * g.T * ((vr + ra - 1) / ra);
  return (int)std::max(1L, std::min(256 / std::max(1L, blocks), (long)V3 / (4 * SC_SITES)));
}

void launch_stoch_sc(const Geo& g, int n, int nv, int nph, int group, int time, const double* eta, const double* X,
                     const double* phase, double* partial, int nchunk, double* O, hipStream_t s) {
  ScArgs a{};
  a.n = n;
  a.nv = nv;
  a.nph = nph;
  a.group = group;
  a.time = time;
  a.V3 = g.X * g.Y * g.Z;
  a.V = (long)a.V3 * g.T;
  a.nchunk = nchunk;
  a.spc = ((a.V3 + nchunk - 1) / nchunk + SC_SITES - 1) / SC_SITES * SC_SITES;
  a.eta = eta;
  a.X = X;
  a.phase = phase;
  a.partial = nchunk > 1 ? partial : O;
  const int vr = nv * nph, na = sc_tiles(vr);
  const dim3 grid((unsigned)((n + 16 * SC_COLS - 1) / (16 * SC_COLS)), (unsigned)g.T,
                  (unsigned)(nchunk * ((vr + 16 * na - 1) / (16 * na)))), blk(768);
  if (na == 1) hipLaunchKernelGGL(k_stoch_sc<1>, grid, blk, 0, s, a);
  if (na == 2) hipLaunchKernelGGL(k_stoch_sc<2>, grid, blk, 0, s, a);
  if (na == 3) hipLaunchKernelGGL(k_stoch_sc<3>, grid, blk, 0, s, a);
  if (nchunk > 1) launch_stoch_sum((long)nph * 12 * nv * n, g.T, nchunk, partial, O, s);
}

// ------------------------------------------------------------------------------------
// pair correlators: corr[m][dt] = sum_t0 sum_ab keep_ab O[t0 + dt][ip_m][a][b] O[t0][im_m][b][a]
// with O [T][nph][n][n]; keep drops pairs of one noise vector (a / group == b / group) when skip is set
// (group 1: the diagonal).
// ------------------------------------------------------------------------------------
// For one (a, b) the sum is a circular correlation over time, so a block takes an EB x EB patch of
// (a, b) and all timeslices: O is read once per dt tile, and the T^2 products per entry come from LDS
// (one block per dt reading every O(t) took 285 us for T = 64 and 48 sources, this 17).
// A thread owns one of DT separations and a part of the t0 tile; block partials are summed in block order.
template <int DT, int EB>
__global__ __launch_bounds__(256) void k_pair_corr(int T, int n, int nph, int group, int skip, MomPairs mp,
                                                   const double* O, double* partial) {
  constexpr int E = EB * EB, PARTS = 256 / DT, PER = DT / PARTS;  // PER t0 per part and tile of DT
  __shared__ double2 xs[2 * DT - 1][E + 1], ys[DT][E + 1];
  const int nb = (n + EB - 1) / EB;
  const int d0 = blockIdx.y * DT, m = blockIdx.z;
  const int ip = mp.ip[m], im = mp.im[m];
  const double2* Oc = (const double2*)O;
  const int dt = threadIdx.x % DT, part = threadIdx.x / DT;
  double vr = 0.0, vi = 0.0;
  for (int u = blockIdx.x; u < nb * nb; u += gridDim.x) {  // the block's patches
    const int a0 = u / nb * EB, b0 = u % nb * EB;
    for (int t0 = 0; t0 < T; t0 += DT) {
      for (int k = threadIdx.x; k < (2 * DT - 1) * E; k += 256) {  // rows t0 + d0 + 0 .. 2 DT - 2 (mod T)
        const int r = k / E, e = k % E, a = a0 + e / EB, b = b0 + e % EB;
        const bool on = a < n && b < n && !(skip && a / group == b / group);
        const int t1 = (t0 + d0 + r) % T;
        xs[r][e] = on ? Oc[(((size_t)t1 * nph + ip) * n + a) * n + b] : make_double2(0.0, 0.0);
      }
      for (int k = threadIdx.x; k < DT * E; k += 256) {
        const int r = k / E, e = k % E, b = b0 + e / EB, a = a0 + e % EB;  // consecutive a: O[b][a] in runs
        const bool on = t0 + r < T && a < n && b < n && !(skip && a / group == b / group);
        ys[r][(e % EB) * EB + e / EB] = on ? Oc[(((size_t)(t0 + r) * nph + im) * n + b) * n + a] : make_double2(0.0, 0.0);
      }
      __syncthreads();
      // a dropped pair or timeslice must not meet the other factor, which may be infinite: both factors of a
      // pair are zero, and rows past T are left out
      for (int k = 0; k < PER && t0 + part * PER + k < T; ++k) {
        const int r = part * PER + k;
#pragma unroll 8
        for (int e = 0; e < E; ++e) {
          const double2 x = xs[r + dt][e], y = ys[r][e];
          vr += x.x * y.x - x.y * y.y;
          vi += x.x * y.y + x.y * y.x;
        }
      }
      __syncthreads();
    }
  }
  double2* red = &xs[0][0];  // [PARTS][DT]
  red[part * DT + dt] = make_double2(vr, vi);
  __syncthreads();
  if (part == 0 && d0 + dt < T) {
    for (int k = 1; k < PARTS; ++k) {
      vr += red[k * DT + dt].x;
      vi += red[k * DT + dt].y;
    }
    ((double2*)partial)[((size_t)m * T + d0 + dt) * gridDim.x + blockIdx.x] = make_double2(vr, vi);
  }
}

// corr[i] = sum of its nblk partials, in a fixed order, divided by norm
__global__ __launch_bounds__(256) void k_corr_sum(int nblk, double norm, const double* partial, double* corr) {
  const double2* p = (const double2*)partial + (size_t)blockIdx.x * nblk;
  double v[2] = {0.0, 0.0};
  for (int k = threadIdx.x; k < nblk; k += 256) {
    v[0] += p[k].x;
    v[1] += p[k].y;
  }
  block_sum_n<2, 256>(v);
  if (threadIdx.x < 2) corr[2 * blockIdx.x + threadIdx.x] = (threadIdx.x == 0 ? v[0] : v[1]) / norm;
}

// time-diluted sources: O [T][nph][na][n] holds the na sources rows[t][r] supported on timeslice t; a
// source contributes to O(t) only at its own timeslice.  One block per (t0, dt, m).
__global__ __launch_bounds__(256) void k_pair_corr_rows(int T, int N, int na, int nph, const int* rows, int group,
                                                        int skip, MomPairs mp, const double* O, double* partial) {
  const int t0 = blockIdx.x, dt = blockIdx.y, m = blockIdx.z, t1 = (t0 + dt) % T;
  const double2* Op = (const double2*)O + ((size_t)t1 * nph + mp.ip[m]) * na * N;
  const double2* Om = (const double2*)O + ((size_t)t0 * nph + mp.im[m]) * na * N;
  double v[2] = {0.0, 0.0};
  for (long e = threadIdx.x; e < (long)na * na; e += 256) {
    const int r1 = (int)(e / na), r0 = (int)(e % na);
    const int a = rows[(size_t)t1 * na + r1], b = rows[(size_t)t0 * na + r0];
    if (skip && a / group == b / group) continue;
    const double2 x = Op[(size_t)r1 * N + b], y = Om[(size_t)r0 * N + a];
    v[0] += x.x * y.x - x.y * y.y;
    v[1] += x.x * y.y + x.y * y.x;
  }
  block_sum_n<2, 256>(v);
  if (threadIdx.x < 2)
    partial[2 * (((size_t)m * T + dt) * T + t0) + threadIdx.x] = threadIdx.x == 0 ? v[0] : v[1];
}

// few timeslices: 16 separations x 16 parts on 8 x 8 patches; else 64 x 4 on 4 x 4
static int pair_edge(int T) { return T <= 16 ? 8 : 4; }
// Blocks: one per patch, up to many times what the chip holds, from where on they take more patches (one
// each would be more threads than a launch can have from 32768 sources on, 16384 with many timeslices)
static int pair_blocks(int T, int n) {
  const int nb = (n + pair_edge(T) - 1) / pair_edge(T);
  return std::min(nb * nb, 1 << 16);
}
size_t pair_corr_partials(int T, int n, int nm) { return (size_t)nm * T * pair_blocks(T, n); }

static void launch_pair_corr(int T, int n, int nph, int group, int skip, const MomPairs& mp, double norm, const double* O,
                             double* partial, double* corr, hipStream_t s) {
  const int nblk = pair_blocks(T, n);
  if (T <= 16)
    hipLaunchKernelGGL((k_pair_corr<16, 8>), dim3((unsigned)nblk, 1, mp.nm), dim3(256), 0, s, T, n, nph, group, skip, mp,
                       O, partial);
  else
    hipLaunchKernelGGL((k_pair_corr<64, 4>), dim3((unsigned)nblk, (unsigned)((T + 63) / 64), mp.nm), dim3(256), 0, s, T, n,
                       nph, group, skip, mp, O, partial);
  hipLaunchKernelGGL(k_corr_sum, dim3((unsigned)(mp.nm * T)), dim3(256), 0, s, nblk, norm, partial, corr);
}

// Momentum-projected pions over pairs of sources from different noise vectors, normalised by
// 1 / (T n (n - 1)) with n = N / group noise vectors (mode 0), or over all pairs without normalisation
// (mode 3).
void launch_pion_mom(int T, int N, int nph, int group, int mode, const MomPairs& mp, const double* O, double* partial,
                     double* corr, hipStream_t s) {
  const double nv = (double)(N / group);
  launch_pair_corr(T, N, nph, group, mode == 0, mp, mode == 0 ? (double)T * nv * (nv - 1.0) : 1.0, O, partial, corr, s);
}

void launch_pion_mom_rows(int T, int N, int na, int nph, const int* rows, int group, int mode, const MomPairs& mp,
                          const double* O, double* partial, double* corr, hipStream_t s) {
  hipLaunchKernelGGL(k_pair_corr_rows, dim3((unsigned)T, (unsigned)T, mp.nm), dim3(256), 0, s, T, N, na, nph, rows, group,
                     mode == 0, mp, O, partial);
  const double nv = (double)(N / group);
  hipLaunchKernelGGL(k_corr_sum, dim3((unsigned)(mp.nm * T)), dim3(256), 0, s, T,
                     mode == 0 ? (double)T * nv * (nv - 1.0) : 1.0, partial, corr);
}

// pion correlator from O.  mode 0: unbiased a != b, 1/(T N (N-1)); 1: all pairs 1/(T N^2)
// (the form printed with eq. stoop).  partial: pair_corr_partials(T, n, 1) complex
void launch_pion_corr(int T, int n, const double* O, int mode, double* partial, double* corr, hipStream_t s) {
  MomPairs mp{};
  mp.nm = 1;
  launch_pair_corr(T, n, 1, 1, mode == 0, mp, (double)T * n * (mode == 0 ? n - 1 : n), O, partial, corr, s);
}

// ------------------------------------------------------------------------------------
// pi-pi zero-momentum pieces from four disjoint noise groups of m = N/4 sources
// (Sec. 7: independent noise for each propagator of a diagram).  B^{gh}(t) is the m x m
// block of O(t) with rows in group g and columns in group h.
//   L^{gh}(t1,t2) = tr[B^{gh}(t1) B^{hg}(t2)] / m^2
//   D0(dt) = 1/T sum_t0 L^{12}(t1,t0) L^{34}(t1,t0)          t1 = t0 + dt
//   D1(dt) = 1/T sum_t0 L^{12}(t1,t1) L^{34}(t0,t0)          (no vacuum subtraction)
//   D2(dt) = 1/T sum_t0 tr[B^{12}(t0) B^{23}(t1) B^{34}(t1) B^{41}(t0)] / m^4
//   D3(dt) = 1/T sum_t0 tr[B^{12}(t1) B^{23}(t1) B^{34}(t0) B^{41}(t0)] / m^4
//   vac(t) = L^{12}(t,t)
// By cyclicity the 4-fold traces are tr[P(t0) Q(t1)] and tr[R(t1) S(t0)] with P = B^{41} B^{12},
// Q = B^{23} B^{34}, R = B^{12} B^{23}, S = B^{34} B^{41}, so the matrix products are made once per
// timeslice (4 T of them, not 4 T^2) and every (t0, t1) needs four sums over m^2 entries.  One block per
// dt that formed the products for each t0 in turn took 620 us for T = 64 and 48 sources, these two 35.
// ------------------------------------------------------------------------------------
constexpr int PIPI_MMAX = 32;

// w [6][T][m][m]: P, R and, transposed, Q, S, B^{21}, B^{43}; loops [2][T]: tr[B^{12} B^{21}], tr[B^{34} B^{43}]
__global__ __launch_bounds__(256) void k_pipi_products(int T, int N, const double* O, double* w, double* loops) {
  __shared__ double2 A[PIPI_MMAX * PIPI_MMAX], B[PIPI_MMAX * (PIPI_MMAX + 1)];
  const int t = blockIdx.x, k = blockIdx.y, m = N / 4;
  const double2* Ot = (const double2*)O + (size_t)t * N * N;
  // groups of the factors (rows, columns): P, R, Q, S, then the two loops
  const int gr[6] = {3, 0, 1, 2, 0, 2}, gm[6] = {0, 1, 2, 3, 1, 3}, gc[6] = {1, 2, 3, 0, 0, 2};
  for (int e = threadIdx.x; e < m * m; e += 256) {
    const int i = e / m, j = e % m;
    A[e] = Ot[(size_t)(gr[k] * m + i) * N + gm[k] * m + j];
    B[i * (m + 1) + j] = Ot[(size_t)(gm[k] * m + i) * N + gc[k] * m + j];
  }
  __syncthreads();
  double2* out = (double2*)w + ((size_t)k * T + t) * m * m;
  double v[2] = {0.0, 0.0};
  for (int e = threadIdx.x; e < m * m; e += 256) {
    const int i = e / m, j = e % m;
    if (k >= 4) {  // the loop's second factor, transposed, and its trace with the first
      const double2 x = A[e], y = B[j * (m + 1) + i];
      out[e] = y;
      v[0] += x.x * y.x - x.y * y.y;
      v[1] += x.x * y.y + x.y * y.x;
      continue;
    }
    // outputs of a row (P, R) or of a column (Q, S: stored transposed) are consecutive threads
    const int r = k < 2 ? i : j, c = k < 2 ? j : i;
    double2 s = make_double2(0.0, 0.0);
    for (int l = 0; l < m; ++l) {
      const double2 x = A[r * m + l], y = B[l * (m + 1) + c];
      s.x += x.x * y.x - x.y * y.y;
      s.y += x.x * y.y + x.y * y.x;
    }
    out[e] = s;
  }
  if (k >= 4) {
    block_sum_n<2, 256>(v);
    if (threadIdx.x < 2) loops[2 * ((size_t)(k - 4) * T + t) + threadIdx.x] = threadIdx.x == 0 ? v[0] : v[1];
  }
}

// one block per dt, waves over t0
constexpr int PIPI_WAVES = 16;
__global__ __launch_bounds__(64 * PIPI_WAVES) void k_pipi(int T, int N, const double* O, const double* w,
                                                         const double* loops, double* diag, double* vac) {
  __shared__ double red[PIPI_WAVES][8];
  const int dt = blockIdx.x, m = N / 4, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const size_t mm = (size_t)m * m;
  const double2 *W = (const double2*)w, *Oc = (const double2*)O;
  const double2 *v12 = (const double2*)loops, *v34 = v12 + T;
  double d[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int t0 = wv; t0 < T; t0 += PIPI_WAVES) {
    const int t1 = (t0 + dt) % T;
    double v[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // L12, L34, the two 4-fold traces
    auto add = [&](int k, const double2& x, const double2& y) {
      v[2 * k] += x.x * y.x - x.y * y.y;
      v[2 * k + 1] += x.x * y.y + x.y * y.x;
    };
    for (int e = lane; e < (int)mm; e += 64) {
      const int i = e / m, j = e % m;
      add(0, Oc[((size_t)t1 * N + i) * N + m + j], W[(4 * (size_t)T + t0) * mm + e]);
      add(1, Oc[((size_t)t1 * N + 2 * m + i) * N + 3 * m + j], W[(5 * (size_t)T + t0) * mm + e]);
      add(2, W[(size_t)t0 * mm + e], W[(2 * (size_t)T + t1) * mm + e]);
      add(3, W[((size_t)T + t1) * mm + e], W[(3 * (size_t)T + t0) * mm + e]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = wave_sum(v[k]);
    const double2 x = v12[t1], y = v34[t0];
    d[0] += v[0] * v[2] - v[1] * v[3];
    d[1] += v[0] * v[3] + v[1] * v[2];
    d[2] += x.x * y.x - x.y * y.y;
    d[3] += x.x * y.y + x.y * y.x;
#pragma unroll
    for (int k = 4; k < 8; ++k) d[k] += v[k];
  }
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 8; ++k) red[wv][k] = d[k];
  __syncthreads();
  if (threadIdx.x < 8) {
    double s = 0.0;
    for (int k = 0; k < PIPI_WAVES; ++k) s += red[k][threadIdx.x];
    const double m4 = (double)mm * (double)mm;
    diag[2 * ((size_t)(threadIdx.x / 2) * T + dt) + threadIdx.x % 2] = s / m4 / T;
  }
  if (vac && threadIdx.x == 0) {
    vac[2 * dt] = v12[dt].x / (double)mm;
    vac[2 * dt + 1] = v12[dt].y / (double)mm;
  }
}

size_t pipi_work(int T, int n) { return (size_t)T * (6 * (size_t)(n / 4) * (n / 4) + 2); }

void launch_pipi(int T, int n, const double* O, double* work, double* diag, double* vac, hipStream_t s) {
  double* loops = work + 2 * (size_t)T * 6 * (n / 4) * (n / 4);
  hipLaunchKernelGGL(k_pipi_products, dim3((unsigned)T, 6), dim3(256), 0, s, T, n, O, work, loops);
  hipLaunchKernelGGL(k_pipi, dim3((unsigned)T), dim3(64 * PIPI_WAVES), 0, s, T, n, O, work, loops, diag, vac);
}

}  // namespace a2a
