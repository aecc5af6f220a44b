// hop_mfma.hip -- the Wilson-clover hopping stencil on the matrix cores for lane-interleaved
// groups of right-hand sides (FP16 or BF16 storage, FP32 accumulation).
//
// At one output site x the hopping term H (the sum over the eight neighbours in the
// hopping-parameter form of the Wilson-clover operator, Sec. 7) is a real 24 x 192 matrix
// acting on the eight neighbour spinors stacked as 8 x 24 reals: block d = 2 mu + f of the
// matrix is the real form of (1 -+ gamma_mu) (x) V_d with V_d the site's hop link of
// direction d (the link, or the daggered backward link, with the fermion boundary sign).
// Every RHS of a group sees the same matrix, so one wavefront takes one site at a time and
// multiplies the matrix with the 192 x 16 block of neighbour data of each 16-lane tile on the
// matrix cores: v_mfma_f32_16x16x32 over 2 row tiles (24 rows + 8 unused) x 7 K steps.  The
// clover term A_x psi(x) is one more K step (24 columns + 8 zero columns).  The inverse-clover
// epilogue is a second product after a register -> LDS -> register transpose of the hop result
// (which rounds that intermediate to the storage format).  Calls with an axpy term (aux1) use
// the per-thread stencil.
//
// The matrix is rebuilt per site in LDS by the 64 lanes of the wave: lane (d, s, c') writes
// the three row blocks (colour a = 0..2) of its direction d for output spin s and real /
// imaginary part c'.  Each entry is the real or imaginary part of a link element, possibly
// swapped and negated; which one is fixed per lane and selected once before the site loop.
// Half of the entries are zero (the spin projector has two non-zero entries per row) and are
// written once; the per-site build writes only the other half (7% faster Schur operator).
//
// Layout of one wavefront's LDS matrix: 24 rows of 464 bytes = 232 halves: columns 0..191
// the hopping blocks (d, spin s', colour b, re/im), 192..215 the clover block, 216..231 zero.
// Rows are 464 B apart so that the 16-byte fragment reads of 16 consecutive rows fall on
// distinct banks.
#include <type_traits>

#include "a2a_kernels.h"

namespace a2a {

namespace {

typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <typename S>
struct MM;

template <>
struct MM<_Float16> {
  static __device__ __forceinline__ f4v mma(const uint4& a, const uint4& b, const f4v& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8v, a), __builtin_bit_cast(h8v, b), c, 0, 0,
                                                  0);
  }
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const _Float16 a = (_Float16)lo, b = (_Float16)hi;
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
  }
  static __device__ __forceinline__ float lo(uint32_t u) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xffffu));
  }
  static __device__ __forceinline__ float hi(uint32_t u) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16)); }
};

template <>
struct MM<bf16_t> {
  static __device__ __forceinline__ f4v mma(const uint4& a, const uint4& b, const f4v& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8v, a), __builtin_bit_cast(b8v, b), c, 0, 0,
                                                   0);
  }
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    return (uint32_t)float_to_bf16(lo).v | ((uint32_t)float_to_bf16(hi).v << 16);
  }
  static __device__ __forceinline__ float lo(uint32_t u) { return bf16_to_float(bf16_t{(uint16_t)(u & 0xffffu)}); }
  static __device__ __forceinline__ float hi(uint32_t u) { return bf16_to_float(bf16_t{(uint16_t)(u >> 16)}); }
};

constexpr int WAVES = BS / 64;
constexpr int SITES_PER_WAVE = BS / WAVES;  // a block covers BS sites, like every reducing kernel
constexpr int TROW = 29;                    // uint4 per matrix row (464 B)
constexpr int TCLO = 24;                    // uint4 column of the clover K step (half 192)
constexpr int TRW = 5;                      // uint4 per transpose row (80 B)

__device__ __forceinline__ uint32_t rot16(uint32_t v) { return (v >> 16) | (v << 16); }

// Pointers read from the group and operator tables are generic; accesses through them would be
// FLAT instructions, which count against the LDS counter too and so make every LDS wait also
// wait for outstanding HBM traffic.  All of these fields point to device global memory.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) uint32_t* gptr1;
typedef const __attribute__((address_space(1))) v4u* gptr4;
__device__ __forceinline__ uint32_t gld1(const void* p) { return *(gptr1)p; }
__device__ __forceinline__ uint4 gld4(const void* p) {
  const v4u v = *(gptr4)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}
// single-use operands (the site's own aux / shadow chunks, the output): streaming access
__device__ __forceinline__ uint4 gld4nt(const void* p) {
  const v4u v = __builtin_nontemporal_load((gptr4)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void gst4nt(void* p, const uint4& v) {
  v4u w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  __builtin_nontemporal_store(w, (__attribute__((address_space(1))) v4u*)p);
}

// (1 + sg gamma_mu)[s][t] in the chiral basis as a unit complex (re, im), entries in {-1, 0, 1}.
// gamma_mu = [[0, a_mu], [a_mu^dag, 0]] with a_k = -i sigma_k (mu = 0, 1, 2) and a_4 = 1.
__device__ __forceinline__ void proj_entry(int mu, int sg, int s, int t, int& re, int& im) {
  re = 0;
  im = 0;
  if (s == t) {
    re = 1;
    return;
  }
  if ((s < 2) == (t < 2)) return;
  const int u = s < 2 ? s : t, v = s < 2 ? t - 2 : s - 2;  // entry a[u][v] (conjugated below the diagonal)
  int ar = 0, ai = 0;
  if (mu == 0) {
    if (u != v) ai = -1;  // -i sigma_1
  } else if (mu == 1) {
    if (u == 0 && v == 1) ar = -1;  // -i sigma_2
    if (u == 1 && v == 0) ar = 1;
  } else if (mu == 2) {
    if (u == v) ai = u == 0 ? -1 : 1;  // -i sigma_3
  } else {
    if (u == v) ar = 1;
  }
  if (s >= 2) ai = -ai;
  re = sg * ar;
  im = sg * ai;
}

// Real-form row c' of (P v) for a unit complex P and a link element v = (vr, vi) packed as two
// 16-bit halves: c' = 0 gives (Re Pv, -Im Pv), c' = 1 gives (Im Pv, Re Pv).  All eight cases
// are one of (vr,-vi), (vi,vr), (-vr,vi), (-vi,-vr): a byte permutation (identity, half swap,
// or all-zero for a vanishing projector entry) and a sign mask.
struct Variant {
  uint32_t sel, xm;
};
__device__ __forceinline__ Variant variant(int re, int im, int cp) {
  int T = -1;
  if (re == 1) T = cp ? 1 : 0;
  if (re == -1) T = cp ? 3 : 2;
  if (im == 1) T = cp ? 0 : 3;
  if (im == -1) T = cp ? 2 : 1;
  Variant r;
  r.sel = T < 0 ? 0x0c0c0c0cu : (T == 1 || T == 3) ? 0x01000302u : 0x03020100u;
  r.xm = T == 0 ? 0x80000000u : T == 2 ? 0x00008000u : T == 3 ? 0x80008000u : 0u;
  return r;
}
__device__ __forceinline__ uint32_t apply(const Variant& V, uint32_t v) {
  return __builtin_amdgcn_perm(v, v, V.sel) ^ V.xm;
}

// LDS traffic of one wavefront is executed in issue order, so lanes of the same wave see each
// other's LDS writes without waiting on any counter; only the compiler must keep the order.
__device__ __forceinline__ void wave_lds_sync() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_wave_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

}  // namespace

// Data one site needs beside its x neighbours and the y neighbour it shares with its pair, for each 16-lane
// tile the lane's 16 bytes in the B-fragment layout (chunk gq of its RHS; lanes gq = 3 repeat chunk 0): the
// other y neighbour, the three K steps of z and t neighbours, the clover input (EPI_CLOV) and the other
// operand of the ALPHA reduction (OMEGA's is the clover input).  One 16-byte load per lane and operand keeps
// the count of memory instructions, which is what the address units spend their cycles on, low.
template <int NT>
struct SiteIn {
  uint4 SD;  // this lane's 16 bytes of the site's links (lanes 0..17) and clover (18..35)
  uint4 O[NT];
  uint4 Z[NT][3];
  uint4 Bc[NT];
  uint4 Bx[NT];
  int site, up;  // up: O is the forward y neighbour
};

// A block takes all NT lane tiles of a group over a 1 / nsub part of BS sites of 4D bricks of the lattice
// (the whole x row, then y, z, t extents), so that most neighbours of a block's sites are sites of the same
// block.  A wave builds a site's matrix and applies it to every tile of the group.
//
// What bounds it: gathered lines that miss the CU's vector L1.  At 48 RHS a CU has about 85 128-byte requests
// to its L2 in flight, 570 cycles each, its address units are busy or waiting 93% of the time and the matrix
// cores 24% (32^3x64, inverse epilogue; 68 requests of 490 cycles with eight gathers a site), so the count
// of gathered lines sets the time (with every gather in one L2-resident line set the pair below took 2.9 ms).
// A wave therefore sweeps pairs of output sites in adjacent y rows along x: each new pair needs one new
// input per row, the inputs behind them and each other's row stay in registers, and a site gathers six
// spinors instead of eight.  To share registers across K steps, each x and y direction is a K step of its own
// (three chunks and a zero chunk; seven K steps instead of six).  The fragments of the matrix are read from
// LDS once per K step for all tiles, and each operand's registers are refilled with the next site's data as
// soon as its products are issued, so a site's requests are in flight for a whole site.  Schur pair, 32^3x64,
// 48 RHS: one tile at a time with eight gathers 4080 us, tiles sharing fragments 3945, pairs 3641, pairs in
// compact cells of bricks 3557 (its reads and writes alone take 2.6 ms at the rate of a
// copy); 24^3x48, 32 RHS: 954, 933, 910, 895; 16^3x32, 16 RHS: 114, 114, 113, 111.
//
// Registers: one tile (DEPTH 2: requests two sites ahead) takes 124-152 of the 168 that three waves per SIMD
// leave a wave, two tiles 148-162, three 184-232 of the 256 of two waves.  With a reduction two tiles do not
// quite fit: the compiler spills 2 (RED_OMEGA), 7 (RED_ALPHA, EPI 3) or 36 (RED_ALPHA, EPI 1) of them.  Two
// tiles two sites ahead at two waves take 86 us for 73 at 12^3x24 and the same on larger lattices.
template <class P, int EPI, int RED, int NT>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(NT == 3 ? 2 : 3))) void k_hop_mfma(HopMArgs a) {
  using S = typename P::S;
  using M = MM<S>;
  constexpr int DEPTH = NT == 1 ? 2 : 1;  // sites requested ahead
  __shared__ uint4 tbl[WAVES][24][TROW];  // the site's matrix
  // register-layout transposes, one row per RHS lane; before them the site's links (chunks 0..17) and
  // clover (18..35)
  __shared__ uint4 trb[WAVES][16][TRW];

  const int2 tile = a.tiles[blockIdx.x];  // {group, site block}
  const ILGroupDev& grp = a.groups[tile.x];
  const OpDev& op = a.ops[grp.op];
  const Geo g = op.g;
  const int hv = g.hv;
  const int po = a.out_par;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, gq = lane >> 4;
  uint4(*T)[TROW] = tbl[w];
  uint2* tr2 = (uint2*)&trb[w][n][0];  // this lane's transpose row as 8-byte pieces
  uint4* stg = &trb[w][0][0];

  // ---- lane constants: matrix-building role (d, s, c') and the four spin-column variants
  const int bd = lane & 7, bs = (lane >> 3) & 3, bc = lane >> 5;
  Variant var[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    int re, im;
    proj_entry(bd >> 1, (bd & 1) ? 1 : -1, bs, t, re, im);
    var[t] = variant(re, im, bc);
  }
  // Each row of (1 -+ gamma_mu) has two non-zero entries: the diagonal (spin s' = s) and one
  // partner spin p2 in the other chiral block.  Only those two column triplets of a row block
  // are ever written; the other entries keep the zeros written once below.
  int p2 = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    int re, im;
    proj_entry(bd >> 1, (bd & 1) ? 1 : -1, bs, t, re, im);
    if (t != bs && (re != 0 || im != 0)) p2 = t;
  }
  Variant var_d = var[0], var_p = var[0];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (t == bs) var_d = var[t];
    if (t == p2) var_p = var[t];
  }
  // clover-building role: row o, column half h (lanes 48..63 repeat lanes 0..15: same values)
  const int co = (lane >> 1) % 24, ch = lane & 1;
  const int cs = co / 6, ca_ = (co % 6) >> 1, ccp = co & 1;
  const int cblk = cs >> 1, ci = 3 * cs + ca_ - 6 * cblk;
  const int cdw = 72 + (cblk * 6 + ci) * 6;  // staged dword of the row's six block entries
  // fragment rows (rows 24..31 of the second row tile read valid rows; their outputs are unused)
  const int frow0 = n, frow1 = n + 16 < 24 ? n + 16 : n + 8;
  const int ochunk = gq < 3 ? gq : 0;  // the chunk this lane loads / stores (gq = 3 repeats 0)

  double kp = 1.0;
  for (int i = 0; i < a.gpow; ++i) kp *= op.kappa;
  const float gam = (float)(a.gsign * kp);
  const float cbv = (float)a.cb;

  const char* hl = (const char*)op.HL[po];
  const char* cf = (const char*)(EPI >= 2 ? op.AIF[po] : op.AF[po]);
  const long long vs = grp.vs;
  const char* vin = grp.base + (long long)a.vin * vs;
  char* vout = grp.base + (long long)a.vout * vs;
  const char* vaux2 = a.vaux2 >= 0 ? grp.base + (long long)a.vaux2 * vs : nullptr;
  const char* vrh = a.vrhat >= 0 ? grp.base + (long long)a.vrhat * vs : nullptr;

  unsigned used = 0;  // bit t: lane n of tile t holds a source
#pragma unroll
  for (int t = 0; t < NT; ++t) used |= ((int)gld1(&grp.slot[t * 16 + n]) >= 0 ? 1u : 0u) << t;
  float red[NT][3];
#pragma unroll
  for (int t = 0; t < NT; ++t) red[t][0] = red[t][1] = red[t][2] = 0.f;

  // zero the matrix once: the padding columns stay zero
  for (int e = lane; e < 24 * TROW; e += 64) (&T[0][0])[e] = make_uint4(0, 0, 0, 0);
  wave_lds_sync();

  // the wave's share of the BS sites of the block's brick position: part tile.y % nsub of its
  // SITES_PER_WAVE sites, so that the waves of a block keep the same (x, y) positions
  const int nsub = __builtin_amdgcn_readfirstlane(op.nsub);
  const int spw = SITES_PER_WAVE / nsub;
  const int s0 = __builtin_amdgcn_readfirstlane(tile.y / nsub * BS + w * SITES_PER_WAVE + tile.y % nsub * spw);
  const int cnt = s0 < hv ? (hv - s0 < spw ? hv - s0 : spw) : 0;

  // a site's links and clover: 36 chunks of 16 bytes, one per lane (lanes 36.. repeat)
  const int sdl = lane < 36 ? lane : lane - 36;
  const bool sd_clover = EPI != 0 && sdl >= 18;
  const char* sd_base = sd_clover ? cf + (sdl - 18) * 16 : hl + (sdl % 18) * 16;
  auto build = [&](const uint4& SD) {
    stg[lane] = SD;
    wave_lds_sync();
    const uint32_t* st32 = (const uint32_t*)stg;
    uint32_t L[9];
#pragma unroll
    for (int j = 0; j < 9; ++j) L[j] = st32[bd * 9 + j];
#pragma unroll
    for (int ca = 0; ca < 3; ++ca) {  // the non-zero triplets (s' = s and s' = p2) of the row block
      uint32_t* row = (uint32_t*)&T[6 * bs + 2 * ca + bc][bd * 3];
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        row[3 * bs + b] = apply(var_d, L[ca * 3 + b]);
        row[3 * p2 + b] = apply(var_p, L[ca * 3 + b]);
      }
    }
    if (EPI != 0) {
      uint32_t o[6];
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        const uint32_t c = st32[cdw + j];
        o[j] = ccp ? rot16(c) : (c ^ 0x80000000u);
      }
      uint2* dst = (uint2*)((char*)&T[co][TCLO] + 24 * ch);
      if (ch == cblk) {  // the other chiral block's half stays zero
        dst[0] = make_uint2(o[0], o[1]);
        dst[1] = make_uint2(o[2], o[3]);
        dst[2] = make_uint2(o[4], o[5]);
      }
    }
  };

  constexpr long long SITE = NT * 768;  // bytes of a site in a group's vector
  unsigned hoff[3];                     // chunk (4 kt + gq) % 3 of this lane's RHS, kt = 0..2
#pragma unroll
  for (int t = 0; t < 3; ++t) hoff[t] = ((4 * t + gq) % 3) * 256 + n * 16;
  const int own = ochunk * 256 + n * 16;
  // fragment columns of the x and y K steps: the direction's three chunks and a zero chunk
  const int xcol = gq < 3 ? gq : TCLO + 3, xstep = gq < 3 ? 3 : 0;

  // Loads are unconditional (past the range the last pair is loaded again), so that the number of memory
  // operations in flight is the same on every path and the waits on them stay exact; only the two extra
  // inputs of a pair that starts a row are requested under a branch.
  auto in4 = [&](int site, int t) { return gld4(vin + (site * SITE + t * 768) + own); };
  auto own4 = [&](const char* v, int site, int t) { return gld4nt(v + (site * SITE + t * 768) + own); };
  PairCursor cu;  // the pair requested last
  struct Row {
    int site, nb[5], up, row;
  };
  auto locate = [&](int r) {
    Row w;
    w.site = pair_site(g, cu, po, r, w.nb, &w.up, &w.row);
    return w;
  };
  auto wrap = [&](int j) { return j < 0 ? j + g.Xh : j >= g.Xh ? j - g.Xh : j; };
  // One output site.  S: its data, refilled for the site `to`; xp, xm, tw: its forward and backward x
  // neighbours and the y neighbour in the pair's other row; xm is refilled with input x_to.  At the end of
  // a row xp and tw are refilled too (xp_to, tw_to).
  auto step = [&](SiteIn<NT>& r, uint4* xp, uint4* xm, uint4* tw, const Row& to, int x_to, bool fresh, int xp_to,
                  int tw_to) {
    const int site = r.site, up = r.up;
    const int nbs[3] = {gq >= 3 ? to.nb[2] : to.nb[1], gq >= 2 ? to.nb[3] : to.nb[2], gq >= 1 ? to.nb[4] : to.nb[3]};
    const char* zad[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      unsigned h = hoff[k];
      asm volatile("" : "+v"(h));  // keeps the 64-bit sums vin + hoff out of registers of their own (they spilled)
      zad[k] = vin + ((unsigned long long)(unsigned)nbs[k] * (unsigned)SITE + h);
    }
    r.site = to.site;
    r.up = to.up;
    build(r.SD);
    r.SD = gld4(sd_base + (size_t)to.site * 288);
    wave_lds_sync();
    f4v acc0[NT], acc1[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc0[t] = acc1[t] = f4v{0.f, 0.f, 0.f, 0.f};
    uint4 A0 = T[frow0][xcol], A1 = T[frow1][xcol];
    // K step k's products with B, the fragments of column c after it requested first
    auto products = [&](auto B, int c) {
      const uint4 a0 = A0, a1 = A1;
      if (c >= 0) {
        A0 = T[frow0][c];
        A1 = T[frow1][c];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc0[t] = M::mma(a0, B(t), acc0[t]);
        acc1[t] = M::mma(a1, B(t), acc1[t]);
      }
    };
    products([&](int t) { return xp[t]; }, xcol + xstep);
    products([&](int t) { return xm[t]; }, xcol + (up ? 3 : 2) * xstep);
#pragma unroll
    for (int t = 0; t < NT; ++t) xm[t] = in4(x_to, t);
    __builtin_amdgcn_sched_barrier(0);  // keeps the requests here
    products([&](int t) { return tw[t]; }, xcol + (up ? 2 : 3) * xstep);
    if (fresh) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        tw[t] = in4(tw_to, t);
        xp[t] = in4(xp_to, t);
      }
    }
    products([&](int t) { return r.O[t]; }, 12 + gq);
#pragma unroll
    for (int t = 0; t < NT; ++t) r.O[t] = in4(to.nb[0], t);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {  // the clover block follows the last K step
      products([&](int t) { return r.Z[t][k]; }, k < 2 || EPI != 0 ? 12 + 4 * (k + 1) + gq : -1);
#pragma unroll
      for (int t = 0; t < NT; ++t) r.Z[t][k] = gld4(zad[k] + t * 768);
      __builtin_amdgcn_sched_barrier(0);
    }
    float v0[NT][4], v1[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v0[t][q] = gam * acc0[t][q];
        v1[t][q] = gam * acc1[t][q];
      }
    const f4v zero = {0.f, 0.f, 0.f, 0.f};
    if (EPI == 1) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f4v c0 = M::mma(A0, r.Bc[t], zero), c1 = M::mma(A1, r.Bc[t], zero);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v0[t][q] += cbv * c0[q];
          v1[t][q] += cbv * c1[q];
        }
      }
    }
    if (EPI == 2 || EPI == 3) {  // o = A^{-1} (.): transpose the rounded result through LDS, second product
      uint4 B2[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        tr2[gq] = make_uint2(M::pack2(v0[t][0], v0[t][1]), M::pack2(v0[t][2], v0[t][3]));
        tr2[4 + gq] = gq < 2 ? make_uint2(M::pack2(v1[t][0], v1[t][1]), M::pack2(v1[t][2], v1[t][3])) : make_uint2(0, 0);
        wave_lds_sync();
        B2[t] = trb[w][n][gq];
        wave_lds_sync();
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f4v c0 = M::mma(A0, B2[t], zero), c1 = M::mma(A1, B2[t], zero);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v0[t][q] = c0[q];
          v1[t][q] = c1[q];
        }
      }
    }
    if (EPI == 3) {  // o = aux2 + A^{-1} (.): the site's aux2 chunk to output rows through LDS
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        trb[w][n][gq] = r.Bc[t];
        wave_lds_sync();
        const uint2 x0 = tr2[gq], x1 = tr2[4 + gq];
        wave_lds_sync();
        v0[t][0] += M::lo(x0.x);
        v0[t][1] += M::hi(x0.x);
        v0[t][2] += M::lo(x0.y);
        v0[t][3] += M::hi(x0.y);
        v1[t][0] += M::lo(x1.x);
        v1[t][1] += M::hi(x1.x);
        v1[t][2] += M::lo(x1.y);
        v1[t][3] += M::hi(x1.y);
      }
    }
    // rows 16 m + 4 gq .. +3 of row tile m, rounded to the storage format
    uint2 q0[NT], q1[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      q0[t] = make_uint2(M::pack2(v0[t][0], v0[t][1]), M::pack2(v0[t][2], v0[t][3]));
      q1[t] = make_uint2(M::pack2(v1[t][0], v1[t][1]), M::pack2(v1[t][2], v1[t][3]));
    }
    if (RED == RED_ALPHA || RED == RED_OMEGA) {  // over the values as stored
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        trb[w][n][gq] = RED == RED_ALPHA ? r.Bx[t] : r.Bc[t];  // the partner, to output rows
        wave_lds_sync();
        const uint2 xr0 = tr2[gq], xr1 = tr2[4 + gq];
        wave_lds_sync();
        float r0 = 0.f, r1 = 0.f, r2 = 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          if (m == 1 && gq >= 2) continue;
          const uint2 q = m ? q1[t] : q0[t];
          const uint2 x = m ? xr1 : xr0;
          const float o0 = M::lo(q.x), o1 = M::hi(q.x), o2 = M::lo(q.y), o3 = M::hi(q.y);
          const float x0 = M::lo(x.x), x1 = M::hi(x.x), x2 = M::lo(x.y), x3 = M::hi(x.y);
          if (RED == RED_ALPHA) {  // (rhat, o)
            r0 += x0 * o0 + x1 * o1 + x2 * o2 + x3 * o3;
            r1 += x0 * o1 - x1 * o0 + x2 * o3 - x3 * o2;
          } else {  // (o, aux2), |o|^2
            r0 += o0 * x0 + o1 * x1 + o2 * x2 + o3 * x3;
            r1 += o0 * x1 - o1 * x0 + o2 * x3 - o3 * x2;
            r2 += o0 * o0 + o1 * o1 + o2 * o2 + o3 * o3;
          }
        }
        // a select, not a product with 0 or 1: an idle lane's column holds whatever its memory
        // held, and 0 * NaN would reach the partial sums of the same lane in the other tiles
        const bool keep = (used >> t) & 1;
        red[t][0] += keep ? r0 : 0.f;
        red[t][1] += keep ? r1 : 0.f;
        red[t][2] += keep ? r2 : 0.f;
      }
    }
    if (EPI == 1 || EPI == 3)
#pragma unroll
      for (int t = 0; t < NT; ++t) r.Bc[t] = own4(vaux2, to.site, t);
    if (RED == RED_ALPHA)
#pragma unroll
      for (int t = 0; t < NT; ++t) r.Bx[t] = own4(vrh, to.site, t);
    // to the storage layout through LDS: one 16-byte store per lane (idle lanes write their own
    // unread lane slots; lanes gq = 3 repeat the chunk-0 store of lane gq = 0)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      tr2[gq] = q0[t];
      tr2[4 + gq] = q1[t];
      wave_lds_sync();
      gst4nt(vout + (site * SITE + t * 768) + own, trb[w][n][ochunk]);
      wave_lds_sync();
    }
  };

  if (cnt > 0) {
    SiteIn<NT> sites[DEPTH];
    uint4 ip[2][NT], iq[2][NT];  // inputs in the rows of site 0 and site 1
    cu.init(g, s0 >> 1);
    int left = cnt >> 1, ahead = left;  // pairs to compute, pairs to request (this one included)
    auto fill = [&](SiteIn<NT>& r, const Row& to) {
      r.site = to.site;
      r.up = to.up;
      r.SD = gld4(sd_base + (size_t)to.site * 288);
      const int nbs[3] = {gq >= 3 ? to.nb[2] : to.nb[1], gq >= 2 ? to.nb[3] : to.nb[2], gq >= 1 ? to.nb[4] : to.nb[3]};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        r.O[t] = in4(to.nb[0], t);
#pragma unroll
        for (int k = 0; k < 3; ++k) r.Z[t][k] = gld4(vin + (nbs[k] * SITE + t * 768) + hoff[k]);
        if (EPI == 1 || EPI == 3) r.Bc[t] = own4(vaux2, to.site, t);
        if (RED == RED_ALPHA) r.Bx[t] = own4(vrh, to.site, t);
      }
    };
    {
      const Row l = locate(0), m = locate(1);
      const int i = cu.X0 + cu.rx;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        ip[0][t] = in4(l.row + i, t);
        ip[1][t] = in4(l.row + wrap(i - 1), t);
        iq[0][t] = in4(m.row + i, t);
        iq[1][t] = in4(m.row + wrap(i + 1), t);
      }
      fill(sites[0], l);
      if (DEPTH == 2) fill(sites[DEPTH - 1], m);
    }
    // the two sites of a pair; ph: ip[ph], iq[ph] hold the inputs at the pair's own x_h, ip[ph ^ 1] the one
    // behind, iq[ph ^ 1] the one ahead
    auto pair = [&](auto ph_c) {
      constexpr int ph = decltype(ph_c)::value;
      const Row m0 = locate(1);
      bool fresh = false;
      if (ahead > 1) {
        --ahead;
        fresh = cu.next(g);
      }
      const Row l = locate(0), m = locate(1);
      const int i = cu.X0 + cu.rx;
      step(sites[0], ip[ph], ip[ph ^ 1], iq[ph], DEPTH == 2 ? l : m0, l.row + i, false, 0, 0);
      step(sites[DEPTH - 1], iq[ph ^ 1], iq[ph], ip[ph], DEPTH == 2 ? m : l, m.row + wrap(i + 1), fresh, m.row + i,
           l.row + wrap(i - 1));
    };
    for (;;) {
      pair(std::integral_constant<int, 0>{});
      if (--left == 0) break;
      pair(std::integral_constant<int, 1>{});
      if (--left == 0) break;
    }
  }

  if (RED == RED_ALPHA || RED == RED_OMEGA) {
    __syncthreads();  // every wave is done with its matrix: reuse the LDS as scratch
    double* scr = (double*)&tbl[0][0][0];  // [tile][wave][lane][3]
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        double x = (double)red[t][q];
        x += __shfl_xor(x, 16, 64);
        x += __shfl_xor(x, 32, 64);
        if (lane < 16) scr[((t * WAVES + w) * 16 + lane) * 3 + q] = x;
      }
    __syncthreads();
    if (threadIdx.x < 48 * NT) {
      const int t = threadIdx.x / 48, m = (threadIdx.x / 3) % 16, q = threadIdx.x % 3;
      const int sl = grp.slot[t * 16 + m];
      if (sl >= 0) {
        double sum = 0.0;
#pragma unroll
        for (int j = 0; j < WAVES; ++j) sum += scr[((t * WAVES + j) * 16 + m) * 3 + q];
        store_partial(a.rb, a.slots[sl].sid, tile.y, q, sum);
      }
    }
  }
}

template <class P, int NT>
static void launch_mfma_nt(const HopMArgs& a, int ntiles, int epi, hipStream_t s) {
  const dim3 g(ntiles), b(BS);
  if (epi == 3) {
    if (a.red == RED_ALPHA)
      hipLaunchKernelGGL((k_hop_mfma<P, 3, RED_ALPHA, NT>), g, b, 0, s, a);
    else if (a.red == RED_OMEGA)
      hipLaunchKernelGGL((k_hop_mfma<P, 3, RED_OMEGA, NT>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_hop_mfma<P, 3, RED_NONE, NT>), g, b, 0, s, a);
  } else if (epi == 2) {
    hipLaunchKernelGGL((k_hop_mfma<P, 2, RED_NONE, NT>), g, b, 0, s, a);
  } else if (epi == 1) {
    if (a.red == RED_ALPHA)
      hipLaunchKernelGGL((k_hop_mfma<P, 1, RED_ALPHA, NT>), g, b, 0, s, a);
    else if (a.red == RED_OMEGA)
      hipLaunchKernelGGL((k_hop_mfma<P, 1, RED_OMEGA, NT>), g, b, 0, s, a);
    else
      hipLaunchKernelGGL((k_hop_mfma<P, 1, RED_NONE, NT>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_hop_mfma<P, 0, RED_NONE, NT>), g, b, 0, s, a);
  }
}

template <class P>
static void launch_mfma_p(const HopMArgs& a, int ntiles, int epi, hipStream_t s) {
  switch (a.nt) {
    case 1: launch_mfma_nt<P, 1>(a, ntiles, epi, s); break;
    case 2: launch_mfma_nt<P, 2>(a, ntiles, epi, s); break;
    case 3: launch_mfma_nt<P, 3>(a, ntiles, epi, s); break;
    default: break;
  }
}

// A block's four waves sweep BS / nsub sites one after another, about half a microsecond each, so nsub
// sets how many of the chip's ~512 resident blocks there are and how long the last of them run (Schur
// pair, 16 sources: 8^3x16, 16 bricks, 199 us whole and 20 us in 16 parts; 16^3x32, 256 blocks, 199 us
// whole, 107 in two and 113 in four; 48 sources: 248 in two, 229 in four; 24^3x48, 1296 blocks, 32 sources
// 982 in two, 896 in four; 32^3x64, 4096 blocks, 48 sources 3537 in two, 3613 in four).
int il_subblocks(int hv) {
  const int nblk = (hv + BS - 1) / BS;
  return nblk >= 2048 ? 2 : nblk >= 128 ? 4 : 16;
}

bool hop_mfma_supports(int prec, int inv, bool clov, int red, bool aux1) {
  if ((prec != 2 && prec != 3) || aux1) return false;
  if (inv == 2) return red == RED_NONE || red == RED_ALPHA || red == RED_OMEGA;
  if (inv) return red == RED_NONE;
  if (clov) return red == RED_NONE || red == RED_ALPHA || red == RED_OMEGA;
  return red == RED_NONE;
}

void launch_hop_mfma(int prec, const HopMArgs& a, int ntiles, int inv, bool clov, hipStream_t s) {
  if (ntiles <= 0) return;
  const int epi = inv == 2 ? 3 : inv ? 2 : clov ? 1 : 0;
  if (prec == 2) launch_mfma_p<PrecF16>(a, ntiles, epi, s);
  if (prec == 3) launch_mfma_p<PrecB16>(a, ntiles, epi, s);
}

}  // namespace a2a
