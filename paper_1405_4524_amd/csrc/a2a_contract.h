// a2a_contract.h -- host-side declarations of the contraction, fill, dilution and point-source
// launchers (internal to liba2a).
#pragma once

#include <hip/hip_runtime.h>

#include "a2a_device.h"

namespace a2a {

// stochastic operators O[t][a][b] (Sec. 7, eq. stoop) and the correlators built from them
// (g5 = 0: without gamma_5, the Gram matrices <eta_a, X_b>_t; timeslices t_first .. + nt)
// phase (complex [na / ns][V3], or null): momentum projection O = sum_y phase(y) eta^dag g5 X, row r of
// O(t) being source r % ns with phase r / ns (ns <= 0: one phase, ns = na)
// rows (or null), [T][ns]: row r of O(t) is source rows[t ns + r % ns] (time-diluted sources);
// without rows, na > 0 takes rows 0 .. na - 1 of eta (O is na x n), na <= 0 means na = n
// partial: nchunk x nt x na x n complex (not used when nchunk is 1)
void launch_stoch_ops(const Geo& g, int n, const double* eta, const double* X, double* partial, int nchunk,
                      double* O, hipStream_t s, int g5 = 1, int t_first = 0, int nt = -1,
                      const double* phase = nullptr, const int* rows = nullptr, int na = 0, int ns = 0);
int stoch_chunks(const Geo& g, int na, int n, int nt);
// A batch of momenta: the distinct phases exp(-i p.y) they need (p reduced to [0, L)), and for each
// momentum the phases of O(t, p) and O(t, -p)
constexpr int MOM_BATCH = 16;
struct MomBatch {
  int nph;
  long long p[2 * MOM_BATCH][3];
};
struct MomPairs {
  int nm;
  int ip[MOM_BATCH], im[MOM_BATCH];
};
// Support of spin-colour diluted sources: off [SC_CHECK_BLOCKS] is not zero where one has entries other than
// zero outside its own component (off null: not asked for)
constexpr int SC_CHECK_BLOCKS = 1024;
struct ScCheck {
  const double* eta;
  int nv, group, time;
  int* off;
};
// f: complex [nph][V3]
void launch_phases(const Geo& g, const MomBatch& m, double* f, const ScCheck& check, hipStream_t s);
// operators O [T][nph][12 nv][n] of spin-colour diluted sources (row 12 i + c: noise vector i, component
// c; source i group + c, plus 12 t if time is set); partial: nchunk times that (not used for one chunk)
int stoch_sc_chunks(const Geo& g, int nv, int nph, int n);
void launch_stoch_sc(const Geo& g, int n, int nv, int nph, int group, int time, const double* eta, const double* X,
                     const double* phase, double* partial, int nchunk, double* O, hipStream_t s);
// corr [nm][T] from O [T][nph][N][N], partial: pair_corr_partials complex; rows: from O [T][nph][na][N],
// partial: nm T^2 complex
size_t pair_corr_partials(int T, int n, int nm);
void launch_pion_mom(int T, int N, int nph, int group, int mode, const MomPairs& mp, const double* O, double* partial,
                     double* corr, hipStream_t s);
void launch_pion_mom_rows(int T, int N, int na, int nph, const int* rows, int group, int mode, const MomPairs& mp,
                          const double* O, double* partial, double* corr, hipStream_t s);
// the 12 unit sources at one site (canonical complex128 [12][V][12])
void launch_point_sources(const Geo& g, long site, double* out, hipStream_t s);
// pi-pi diagrams from point and stochastic propagators, from the timeslice Gram matrices
// Pn [T][12][12], G and Fp [T][n1][n2], A [12][n1] (at t0), B [T][n2][12]; partial holds
// pipi_mixed_chunks(n1) x T x 6 doubles; diag [4][T] and pieces [3][T] complex (device)
int pipi_mixed_chunks(int n1);
void launch_pipi_mixed(int T, int t0, int n1, int n2, const double* Pn, const double* G, const double* Fp,
                       const double* A, const double* B, double* partial, double* diag, double* pieces,
                       hipStream_t s);
void launch_dilute(const Geo& g, int nnoise, int scheme, int D, const double* noise, double* out, hipStream_t s);
void launch_gram_corr(int T, int n, const double* E, const double* F, double* corr, hipStream_t s);

// outer-product fill (Sec. 7, eq. Sfill) on the FP64 matrix cores:
// C(m, n) = scale sum_k P(m, k) conj(Q(n, k)), complex operands with element strides
struct FillArgs {
  const double* P[2];  // operand pairs: [0] the product to store or S1, [1] S2 (contract mode)
  const double* Q[2];
  long long pk, qk;          // P(m, k) = P[m + k pk], Q(n, k) = Q[n + k qk] (complex elements)
  long long pz;              // contract mode: P's offset per grid.y index (sink timeslice)
  int M, N, K;  // M and N multiples of 96
  double scale;
  double* out;               // fill mode: C(m, n) at out[m om + n]
  long long om;
  int dagger;                // store the spin-colour dagger of every 12 x 12 block
  double* partial;           // contract mode: [z][block] complex partials of sum C1 conj(C2)
};
// most rows M of a fill, whose (M / 32)^2 one-wave blocks must be fewer than 2^32 threads, and of the
// contractions (fill or Gram matrices), which launch the same for every larger M
constexpr long long FILL_MAX_ROWS = (1LL << 18) - 1, FILL_CONTRACT_MAX_ROWS = 1LL << 21;
int fill_blocks(int M, int N);  // blocks and partials of a contraction, per z
void launch_fill(const FillArgs& a, hipStream_t s);
void launch_fill_contract(const FillArgs& a, int nz, double* corr, hipStream_t s);
void launch_pion_corr(int T, int n, const double* O, int mode, double* partial, double* corr, hipStream_t s);
// work: pipi_work(T, n) complex
size_t pipi_work(int T, int n);
void launch_pipi(int T, int n, const double* O, double* work, double* diag, double* vac, hipStream_t s);

}  // namespace a2a
