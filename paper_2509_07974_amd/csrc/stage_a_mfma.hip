// Stage (a) of the mixed paths on the matrix cores: per-centre multipoles in
// radial bins from binary16 hi/lo operands with binary32 accumulation.
//
// The sums S_f,k = sum_j v_f(j) z_ij^k over the neighbours j of centre i in a
// bin are a contraction over j.  With every order written as k = p + r or
// p - r, p a multiple of 17 and 0 <= r <= 8,
//
//     cos((p +- r) phi) = cos(p phi) cos(r phi) -+ sin(p phi) sin(r phi)
//     sin((p +- r) phi) = sin(p phi) cos(r phi) +- cos(p phi) sin(r phi),
//
// all of them follow from one small matrix product per bin,
//
//     D[row][col] = sum_j A[row][j] B[j][col],
//     rows    v_f,  v_f cos(p phi),  v_f sin(p phi)   (p = 17, 34),
//     columns cos(r phi), sin(r phi), r = 1..8, and 1,
//
// in which every product that the matrix cores form is a wanted one, and a
// neighbour needs some 30 operand values (orders up to 25) where a vector kernel
// issues 426 multiply-adds.  Every operand x is split x = hi + lo into two
// binary16 values (22 significant bits), and hi hi + lo hi + hi lo is
// accumulated in binary32 by v_mfma_f32_16x16x32_f16: products are exact,
// sums are rounded to nearest.  The dominant accumulators are added to
// binary64 every 2 or 4 chunks.  The weights carry a power-of-two scale per
// family (MatScale) that puts their largest value below 2^15.
//
// Mapping on CDNA4 (wave64):
//  * one wave owns one (centre, group of bins) at a time (per-XCD queues over
//    the Morton-ordered centre list, with stealing); no barriers between
//    waves.  The centres of a block take the groups in turn, the widest bins
//    first.  Where the octets around a centre do not fit the L2 of an XCD, the
//    block is the whole queue, so that its waves read the same galaxies at the
//    same time: the octets are 96 bytes a galaxy, and in a dense field one row
//    of cells of one group is as large as a share of L2.  Elsewhere it is 64
//    centres, so that units of several lengths overlap (launch_pairs_mm);
//  * the annulus is a list of octets (8 consecutive sorted galaxies, aligned)
//    with an 8-bit mask of those inside the row segment.  A chunk is 8
//    octets: lane l forms neighbour l&7 of octet l>>3.  r^2 is formed in
//    binary64 without contraction and tested against the squared edges, the
//    oracle's arithmetic, so binning is bit-exact; neighbours outside the bin
//    get z = 0 and with it zero columns and zero p > 0 rows;
//  * the rows p = 0 (weights alone) do not depend on the centre: they are
//    kept split and transposed per octet in memory (octet_kernel below) and
//    loaded straight into matrix operand layout;
//  * the columns and the rows p > 0 are formed one neighbour per lane and
//    transposed through LDS: 16-byte stores of 8 values of a neighbour, read
//    back with ds_read_b64_tr_b16, 4 neighbours of one value per lane.
//
// The unit vector z and its powers 2 and 4 are formed in binary64 from the
// reciprocal root of one Newton step, and every higher power takes at most
// three products from those: an error of z^4 in binary32 alone grows eightfold
// on the way to z^34.  Errors against binary64, worst order of a family relative
// to its rms, at nmax 5 to 16 in uniform and clustered catalogues, this kernel
// / vector kernel: G and Q 2.4e-7 to 3.5e-7 / 5.5e-7 to 1.6e-6, W, A and V
// 1.6e-7 to 4.3e-7 / 2.4e-7 to 1.4e-6, T_-8 1.5e-7 / 4e-7, T_-4 and M_-4
// 1.4e-7 / 2.4e-7, U 2.6e-8 / 4.5e-8.  Where no power of z adds to it the
// operands' 22 bits show: M_0 7.6e-8 to 2.0e-7 / 8.2e-8 to 2.5e-7 (larger in 10
// of 60 catalogues and orders), and A_2 of the 3PCF plan 1.8e-7 / 1.2e-7; both
// are same-galaxy terms beside products of G, and every shear correlator of
// an estimate is closer to binary64 than with the vector kernel.
//
// What bounds it: the vector ALUs, 79 % of the cycles issuing (220 lane
// instructions per in-bin pair, 84 % of the candidates of a chunk in the bin),
// at a clock that the card's power limit holds between 2.0 and 2.1 GHz; LDS is
// 41 % busy and the matrix cores 24 %.  258 GB miss L2, 0.4 TB/s.  (nmax 15, 8192
// of 1e7 galaxies: 66, 37 and 24 %.)  Three waves per SIMD (168 registers) is
// what the accumulators leave without spills.  Measured against the vector
// kernel, 12 bins to 100', nmax 10: 1e6 galaxies 613 ms at 2.11 GHz, 647 at 2.00,
// against 914 at 2.37.
#include <algorithm>
#include <type_traits>

#include "stage_a_plan.hpp"

namespace fpcf4 {
namespace sa {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef __fp16 tr4v __attribute__((__vector_size__(4 * sizeof(__fp16))));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int RC = 8;              // largest column order
constexpr int PSTEP = 2 * RC + 1;  // row orders p = 0, 17, 34
constexpr int DPP_ROW_ROR8 = 0x128;  // lane i <- i xor 8 within 16
// Chunks of 64 candidates per binary32 block.  Neighbours of a chunk lie close
// together, so a block's partial sums are far larger than the bin's sum after
// cancellation, and every matrix product rounds at their size: with blocks of
// 16 chunks the multipoles W of a dense field had errors of 6.5e-7 of their rms
// (at every order up to nmax 10), with 4 up to 3.4e-7 and with 2 1.8e-7; the vector
// kernel has 2e-7 to 8e-7, growing with the order.  The lower orders get the
// shorter blocks.  The low-part accumulators stay in binary32 over the whole
// bin: their sums, and with them their roundings, are 2^-11 of the others'.
constexpr int fold_chunks(int n) { return nord(n) <= 6 ? 2 : 4; }

// row orders p > 0 of a plan
__host__ __device__ constexpr int nrow_orders(int n) {
  return ktop(n) <= RC ? 0 : (ktop(n) - RC + PSTEP - 1) / PSTEP;
}

// Operand planes in LDS: 8 binary16 values of each of 64 neighbours, 64 bytes
// of padding per 16 neighbours, so that the lane groups of a transposing read
// use different banks.  The planes' offsets (modulo 256 bytes: 0, 128, 128, 0
// for the columns, 0, 128 for z^p) do the same for the planes read together.
constexpr int PLANE_BYTES = 64 * 16 + 4 * 64;
__host__ __device__ constexpr int plane_at(int n) { return 16 * n + 64 * (n >> 4); }
constexpr int COL_PLANE[4] = {0, 1408, 2944, 4352};   // hi 0..7, hi 8..15, lo 0..7, lo 8..15
constexpr int ZP_PLANE = 5632, ZP_LO = 1408, ZP_STEP = 2816;
static_assert(COL_PLANE[1] >= PLANE_BYTES && COL_PLANE[2] - COL_PLANE[1] >= PLANE_BYTES &&
              COL_PLANE[3] - COL_PLANE[2] >= PLANE_BYTES && ZP_PLANE - COL_PLANE[3] >= PLANE_BYTES &&
              ZP_LO >= PLANE_BYTES && ZP_STEP - ZP_LO >= PLANE_BYTES, "planes overlap");
// Column pairs (cos, sin)(r phi) in plane order; z^4 and z^8 share a group of
// four values, which the triple blocks read alone.
constexpr int COL_R[RC] = {1, 2, 3, 5, 6, 7, 4, 8};
__host__ __device__ constexpr int col_of(int r) {   // column of cos(r phi)
  return r <= 3 ? 2 * r - 2 : r == 4 ? 12 : r == 8 ? 14 : 2 * r - 4;
}
// Columns of the second right operand: z^17 hi, the in-bin flag, z^17 lo,
// (z^4, z^8) hi, lo.
constexpr int X_P = 0, X_FLAG = 2, X_PLO = 4, X_4 = 8, X_8 = 10, X_LO = 4;

template <int N> struct MConf {
  static constexpr int NP = nrow_orders(N);
  static constexpr int NS = is3(N) ? 0 : 1;               // triple blocks
  static constexpr bool TOP = ktop(N) >= 2 * PSTEP;       // order 34 itself is needed
  // accumulator tiles: p = 0 by the columns; p = 0 by the second operand
  // (orders 0 and 17); triple blocks by the second operand; p = 17, 34 by the
  // columns; p = 0 by z^34
  static constexpr int TT = 0, TX = 1, TS = 2, TP = 2 + NS, T34 = TP + NP, NT = T34 + (TOP ? 1 : 0);
  // the sums that the epilogue reads (row, column), in doubles: high and low
  // rows of a weight are added, so that p = 0 and triple blocks have 8 rows
  static constexpr int OT = 0, OX = 128, OS = 256, OP = 256 + 128 * NS, O34 = OP + 256 * NP,
                       OZERO = O34 + (TOP ? 128 : 0), NSUM = OZERO + 1;
  static_assert(NP >= 1 && NP <= 2 && ktop(N) <= PSTEP * 2 + RC, "row orders");
};

// A record entry is a sum of at most four of those sums per component; bit 15
// of an index negates the term.
struct Terms {
  uint16_t v[8];   // re, re, re, re, im, im, im, im
};
struct TermList {
  Terms t;
  int n[2];
};
constexpr uint16_t TERM_NEG = 0x8000;
constexpr void add_term(TermList& l, int comp, int idx, bool neg) {
  l.t.v[4 * comp + l.n[comp]++] = (uint16_t)(idx | (neg ? TERM_NEG : 0));
}
// adds component `part` of sum_j v_f z^k (k >= 0) to component `comp` of the entry
template <int N>
constexpr void add_sum(TermList& l, int comp, int f, int k, int part, bool neg) {
  using C = MConf<N>;
  if (k == 0) {
    if (part == 0) add_term(l, comp, C::OX + 16 * f + X_FLAG, neg);
  } else if (k <= RC) {
    add_term(l, comp, C::OT + 16 * f + col_of(k) + part, neg);
  } else if (k == PSTEP || k == 2 * PSTEP) {
    const int o = (k == PSTEP ? C::OX : C::O34) + 16 * f + X_P + part;
    add_term(l, comp, o, neg);
    add_term(l, comp, o + X_PLO - X_P, neg);
  } else {
    // rows c, s (p phi) by columns c, s (r phi):
    // cos((p + d) phi) = c c - sg s s, sin = s c + sg c s, r = |d|, sg = sign d
    const int t = k > PSTEP + RC ? 2 : 1, d = k - PSTEP * t, r = d < 0 ? -d : d;
    const int row = C::OP + 256 * (t - 1) + 32 * f + col_of(r);
    add_term(l, comp, part == 0 ? row : row + 16, neg);
    add_term(l, comp, part == 0 ? row + 17 : row + 1, neg != ((part == 0) == (d > 0)));
  }
}
// a complex weight (families f, f + 1) at order k of either sign
template <int N>
constexpr void add_pair(TermList& l, int f, int k) {
  const int ko = k < 0 ? -k : k;
  if (ko > kmax_f(N, f)) return;   // orders the plan does not form (3PCF plan) are zero
  add_sum<N>(l, 0, f, ko, 0, false);
  add_sum<N>(l, 0, f + 1, ko, 1, k >= 0);
  add_sum<N>(l, 1, f + 1, ko, 0, false);
  add_sum<N>(l, 1, f, ko, 1, k < 0);
}
template <int N>
constexpr void add_real(TermList& l, int f, int k) {
  const int ko = k < 0 ? -k : k;
  if (ko > kmax_f(N, f)) return;
  add_sum<N>(l, 0, f, ko, 0, false);
  add_sum<N>(l, 1, f, ko, 1, k < 0);
}
// triple-block weight q at z^4 or z^8 (column of its cos)
template <int N>
constexpr void add_triple(TermList& l, int comp, int q, int col, bool neg) {
  add_term(l, comp, MConf<N>::OS + 16 * q + col, neg);
  add_term(l, comp, MConf<N>::OS + 16 * q + col + X_LO, neg);
}
template <int N>
constexpr Terms entry_terms(int e) {
  using C = MConf<N>;
  constexpr Layout L = make_layout(nord(N));
  TermList l{};
  for (int i = 0; i < 8; ++i) l.t.v[i] = (uint16_t)C::OZERO;
  if (e < L.offW) add_pair<N>(l, FA, e - (2 * nord(N) + 3));               // G_k
  else if (e < L.offQ) add_real<N>(l, FW, e - L.offW - 2 * nord(N));       // W_k
  else if (e < L.offA) add_pair<N>(l, FC, e - L.offQ + L.qlo);             // Q_k
  else if (e < L.offV) add_real<N>(l, FE, e - L.offA);                     // A_k, k >= 0
  else if (e < L.offS) add_real<N>(l, FV, e - L.offV);                     // V_k, k >= 0
  else if (C::NS) {                                                        // T_-8, T_-4, M_-4, M_0, U
    const int sp = e - L.offS;
    if (sp == S_T8 || sp == S_T4 || sp == S_M4) {
      const int col = sp == S_T8 ? X_8 : X_4, q = sp == S_M4 ? 2 : 0;
      add_triple<N>(l, 0, q, col, false);
      add_triple<N>(l, 0, q + 1, col + 1, false);
      add_triple<N>(l, 1, q + 1, col, false);
      add_triple<N>(l, 1, q, col + 1, true);
    } else if (sp == S_M0) {
      add_term(l, 0, C::OS + 16 * 2 + X_FLAG, false);
      add_term(l, 1, C::OS + 16 * 3 + X_FLAG, false);
    } else {
      add_term(l, 0, C::OS + 16 * 4 + X_FLAG, false);
    }
  }
  return l.t;
}
template <int N> struct alignas(16) EntryTable {
  Terms t[make_layout(nord(N)).mpc];
};
template <int N>
constexpr EntryTable<N> make_entry_table() {
  EntryTable<N> t{};
  for (int e = 0; e < make_layout(nord(N)).mpc; ++e) t.t[e] = entry_terms<N>(e);
  return t;
}
template <int N> __device__ const EntryTable<N> entry_table = make_entry_table<N>();

// Per wave: planes of the columns and, per p > 0, of z^p: hi (c, s, flag, 0,
// c, s, c, s) and lo (c, s, 0, 0, c, s, c, s).  The window of octets being
// listed and the epilogue's sums take their place.
template <int N> union alignas(256) WaveBuf {
  unsigned char planes[ZP_PLANE + MConf<N>::NP * ZP_STEP];
  int first[64];
  double sums[MConf<N>::NSUM];
};

// x, y -> binary16 pairs hi, lo with hi + lo = x, y to 22 bits.  The
// remainder has to be taken from the very hi that is stored, so the
// conversion is opaque to the compiler, which would otherwise form a second
// hi from the unrounded value for it.  v_fma_mix_f32 reads a binary16 half in
// place; its binary16-result forms run at half its rate.
__device__ __forceinline__ unsigned pack2(float x, float y) {
  unsigned r;
  asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}
__device__ __forceinline__ void split2(float x, float y, unsigned& hi, unsigned& lo) {
  hi = pack2(x, y);
  float rx, ry;
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(rx) : "v"(hi), "v"(x));
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(ry) : "v"(hi), "v"(y));
  lo = pack2(rx, ry);
}
// (vh + vl) (xh + xl) -> hi, lo: hi = vh xh rounded, lo its exact remainder
// plus vh xl + vl xh.  Four packed instructions per pair of products.
__device__ __forceinline__ void product2(half8v vh, half8v vl, half8v xh, half8v xl, half8v& hi, half8v& lo) {
  hi = vh * xh;
  lo = __builtin_elementwise_fma(vh, xh, -hi);
  lo = __builtin_elementwise_fma(vh, xl, lo);
  lo = __builtin_elementwise_fma(vl, xh, lo);
}

// every lane's dwords replaced by those of another lane of its quad
constexpr int DPP_QUAD_EVEN = 0xA0, DPP_QUAD_ODD = 0xF5;   // [0,0,2,2], [1,1,3,3]
template <int CTRL>
__device__ __forceinline__ half8v quad(half8v v) {
  u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
  for (int k = 0; k < 4; ++k) u[k] = (unsigned)__builtin_amdgcn_mov_dpp((int)u[k], CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(half8v, u);
}

__device__ __forceinline__ f32x4 mma(half8v a, half8v b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// One operand, 16 values x 32 neighbours: lane (i = l & 15, g = l >> 4) gets
// value i of neighbours 16 g + 8 s + 0..7.  The 16 lanes of a transposing read
// address 4 neighbours x 4 groups of 4 values (lane i: neighbour i >> 2, group
// i & 3); p is the lane's address for neighbour 16 g + 8 s + (i >> 2).
__device__ __forceinline__ half8v read_operand(const unsigned char* p) {
  typedef __attribute__((address_space(3))) tr4v* lds_tr4;
  const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_tr4)(p)));
  const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_tr4)(p + 4 * 16)));
  return __builtin_bit_cast(half8v, u32x4{a.x, a.y, b.x, b.y});
}

// inclusive prefix sum / maximum over the wave: within rows of 16 lanes, then
// across them (row_shr 1, 2, 4, 8, row_bcast 15 and 31)
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_scan_add(int v) {
  v += dpp_or<0x111, 0xf>(0, v);
  v += dpp_or<0x112, 0xf>(0, v);
  v += dpp_or<0x114, 0xf>(0, v);
  v += dpp_or<0x118, 0xf>(0, v);
  v += dpp_or<0x142, 0xa>(0, v);
  v += dpp_or<0x143, 0xc>(0, v);
  return v;
}
__device__ __forceinline__ int wave_scan_max(int v) {   // v >= 0
  v = imax(v, dpp_or<0x111, 0xf>(0, v));
  v = imax(v, dpp_or<0x112, 0xf>(0, v));
  v = imax(v, dpp_or<0x114, 0xf>(0, v));
  v = imax(v, dpp_or<0x118, 0xf>(0, v));
  v = imax(v, dpp_or<0x142, 0xa>(0, v));
  v = imax(v, dpp_or<0x143, 0xc>(0, v));
  return v;
}

__device__ __forceinline__ int lane_get(int v, int src) { return __builtin_amdgcn_ds_bpermute(src << 2, v); }

template <int N, bool RED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void stage_mm_kernel(StageAArgs a) {
  using C = MConf<N>;
  constexpr int NP = C::NP, NS = C::NS, NT = C::NT;
  __shared__ WaveBuf<N> bufs[4];
  __shared__ unsigned bmax[2][FPCF4_NBINS_SUPPORTED];
  __shared__ double unscale[TREE_LEVELS_MAX + 1][NWEIGHTS + 4];
  if (ruled_out(a)) return;

  const unsigned lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  WaveBuf<N>& wb = bufs[wv];
  const int c = (int)lane & 15, g = (int)lane >> 4;

  for (int q = (int)threadIdx.x; q < 2 * FPCF4_NBINS_SUPPORTED; q += (int)blockDim.x)
    bmax[q / FPCF4_NBINS_SUPPORTED][q % FPCF4_NBINS_SUPPORTED] = 0u;
  if (threadIdx.x < (TREE_LEVELS_MAX + 1) * NWEIGHTS)
    unscale[threadIdx.x / NWEIGHTS][threadIdx.x % NWEIGHTS] =
        a.ms[threadIdx.x / NWEIGHTS].inv[threadIdx.x % NWEIGHTS];
  __syncthreads();

  const Gal<float>* __restrict__ cgal = reinterpret_cast<const Gal<float>*>(a.cgal);
  const Grid gr = a.cat.g;
  constexpr Layout L = make_layout(nord(N));
  constexpr int MPC = L.mpc;
  const int nb = a.nb;
  const int ng = a.ngroups;

  // LDS addresses of this lane's part of the transposing reads
  const int nb0 = plane_at(16 * g) + 16 * (c >> 2), grp4 = c & 3;
  const unsigned char* cread = wb.planes + (grp4 >> 1) * COL_PLANE[1] + nb0 + (grp4 & 1) * 8;
  const unsigned char* lread = wb.planes + COL_PLANE[2 + (grp4 >> 1)] + nb0 + (grp4 & 1) * 8;
  const unsigned char* zread = wb.planes + ZP_PLANE + nb0 + (grp4 == 3 ? 0 : 8);
  const unsigned char* xread =
      wb.planes + (grp4 < 2 ? ZP_PLANE + grp4 * ZP_LO : (grp4 == 2 ? COL_PLANE[1] : COL_PLANE[3]) + 8) + nb0;
  // octet blocks: rows c of p = 0 and of the triple blocks
  const unsigned toff = 128u + 16u * (unsigned)c, soff = 384u + 16u * (unsigned)imin(c, 9);

  unsigned long long wave_pairs = 0;
  float xmax = 0.f, wxmax = 0.f;
  const int xcd0 = blockIdx.x & 7;
  int xs = 0;
  // asked for one unit ahead, so that the round trip hides behind the current one
  auto request = [&]() -> int {
    return lane == 0 ? atomicAdd(a.work_counter + SCHED_STRIDE * ((xcd0 + xs) & 7), 1) : 0;
  };
  int next = request();

  for (;;) {
    // ---- next unit: (centre, bin group) of this XCD's part of the centre
    // list, then of the others'
    int idx = -1, grp = 0;
    while (xs < 8) {
      const int xcd = (xcd0 + xs) & 7;
      const int lo = (int)(((int64_t)a.ncent * xcd) >> 3);
      const int hi = (int)(((int64_t)a.ncent * (xcd + 1)) >> 3);
      const unsigned u = (unsigned)__builtin_amdgcn_readfirstlane(next);
      if (u < (unsigned)(hi - lo) * (unsigned)ng) {
        const unsigned per = (unsigned)a.block * (unsigned)ng, blk = u / per, rem = u - blk * per;
        const int b0 = lo + (int)(blk * (unsigned)a.block);
        const unsigned nc = (unsigned)imin(a.block, hi - b0);
        grp = (int)(rem / nc);
        idx = b0 + (int)(rem - (unsigned)grp * nc);
        next = request();
        break;
      }
      // exhausted: the next XCD's queue, where a look at its counter (a load,
      // which does not queue up as the grabs do) finds units left
      for (++xs; xs < 8; ++xs) {
        const int x = (xcd0 + xs) & 7;
        const int l = (int)(((int64_t)a.ncent * x) >> 3), h = (int)(((int64_t)a.ncent * (x + 1)) >> 3);
        const int seen = __hip_atomic_load(a.work_counter + SCHED_STRIDE * x, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        if ((unsigned)__builtin_amdgcn_readfirstlane(seen) < (unsigned)(h - l) * (unsigned)ng) {
          next = request();
          break;
        }
      }
    }
    if (idx < 0) break;
    idx = __builtin_amdgcn_readfirstlane(a.order ? a.order[idx] : idx);
    grp = __builtin_amdgcn_readfirstlane(grp);
    const Gal<float> gi = cgal[a.centres[idx]];
    const double xi = gi.x, yi = gi.y;
    if (!RED && grp == 0 && lane == 0) {
      float* xg = reinterpret_cast<float*>(a.xg);
      xg[2 * idx] = gi.a;
      xg[2 * idx + 1] = gi.b;
      reinterpret_cast<float*>(a.xw)[idx] = gi.w;
      xmax = fmaxf(xmax, fmaxf(fabsf(gi.a), fabsf(gi.b)));
      wxmax = fmaxf(wxmax, fabsf(gi.w));
    }

    for (int b = (int)a.gend[grp] - 1; b >= (int)a.gfirst[grp]; --b) {
      const int lev = RED ? a.level[b] : 0;
      const int32_t* __restrict__ cstart = RED ? a.rcell[lev - 1] : a.cat.cell_start;
      const unsigned char* __restrict__ octets = reinterpret_cast<const unsigned char*>(a.octets[lev]);
      const double e2lo = a.e2[b], e2hi = a.e2[b + 1];
      // conservative culling radii and cell margin (binning itself is exact)
      const double rin = a.edges[b] * (1.0 - 1e-9);
      const double rout = a.edges[b + 1] * (1.0 + 1e-9);
      const double dlt = 1e-9 * gr.h;
      int cy0 = (int)floor((yi - rout - gr.y0) * gr.inv_h) - 1;
      int cy1 = (int)floor((yi + rout - gr.y0) * gr.inv_h) + 1;
      cy0 = imax(cy0, 0);
      cy1 = imin(cy1, gr.ncy - 1);
      const int nrows = cy1 - cy0 + 1;

      f32x4 acc[NT], low[1 + NP];   // low: the products by the columns' low parts
      double m[NT][4];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) m[t][i] = 0.0;
      }
#pragma unroll
      for (int t = 0; t < 1 + NP; ++t) low[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      auto fold = [&]() {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
          for (int i = 0; i < 4; ++i) m[t][i] += (double)acc[t][i];
          acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      };
      int cnt = 0, nfold = 0;

      for (int rg = 0; rg < nrows; rg += 64) {
        // ---- row table, one row per lane: segments [s1, s1 + l1) and
        // [s2, s2 + l2) of the sorted catalogue (cells entirely inside the
        // inner circle are skipped), as octets
        int s1 = 0, l1 = 0, s2 = 0, l2 = 0;
        const int cy = cy0 + rg + (int)lane;
        if (rg + (int)lane < nrows) {
          const double ylo = gr.y0 + cy * gr.h - dlt;
          const double yhi = gr.y0 + (cy + 1) * gr.h + dlt;
          const double dymin = fmax(0.0, fmax(ylo - yi, yi - yhi));
          if (dymin < rout) {
            const double hw = sqrt(rout * rout - dymin * dymin) + dlt;
            int cx0 = (int)floor((xi - hw - gr.x0) * gr.inv_h);
            int cx1 = (int)floor((xi + hw - gr.x0) * gr.inv_h);
            cx0 = imax(cx0, 0);
            cx1 = imin(cx1, gr.ncx - 1);
            if (cx0 <= cx1) {
              const double dymax = fmax(fabs(ylo - yi), fabs(yhi - yi));
              int hx0 = cx1 + 1, hx1 = cx1;
              if (dymax < rin) {
                const double hwi = sqrt(rin * rin - dymax * dymax) - 2.0 * dlt;
                hx0 = (int)ceil((xi - hwi - gr.x0) * gr.inv_h + 1e-7);
                hx1 = (int)floor((xi + hwi - gr.x0) * gr.inv_h - 1e-7) - 1;
                hx0 = imax(hx0, cx0);
                hx1 = imin(hx1, cx1);
                if (hx0 > hx1) { hx0 = cx1 + 1; hx1 = cx1; }
              }
              const int32_t* cs = cstart + (int64_t)cy * gr.ncx;
              s1 = cs[cx0];
              l1 = cs[hx0] - s1;
              s2 = cs[hx1 + 1];
              l2 = cs[cx1 + 1] - s2;
            }
          }
        }
        const int n1 = l1 > 0 ? ((s1 + l1 - 1) >> 3) - (s1 >> 3) + 1 : 0;
        const int n2 = l2 > 0 ? ((s2 + l2 - 1) >> 3) - (s2 >> 3) + 1 : 0;
        const int pe = wave_scan_add(n1 + n2);   // inclusive prefix over rows
        const int ex = pe - n1 - n2;
        const int tot = __builtin_amdgcn_readlane(pe, 63);

        for (int w0 = 0; w0 < tot; w0 += 64) {
          // ---- a window of 64 octets, one per lane: every row marks its first
          // octet of the window, a running maximum spreads the row index, then
          // the octet and its in-segment mask
          wb.first[lane] = 0;
          wave_sync();
          if (ex < w0 + 64 && pe > w0 && pe > ex) wb.first[imax(ex - w0, 0)] = (int)lane;
          wave_sync();
          const int r = wave_scan_max(wb.first[lane]);
          wave_sync();
          unsigned wo = 0;   // byte offset of the octet's block | mask
          {
            const int o = w0 + (int)lane;
            const int off = o - lane_get(ex, r);
            const int k1 = lane_get(n1, r);
            const int a1 = lane_get(s1, r), b1 = lane_get(l1, r);
            const int a2 = lane_get(s2, r), b2 = lane_get(l2, r);
            const bool first = off < k1;
            const int st = first ? a1 : a2, ln = first ? b1 : b2;
            if (o < tot) {
              const int oc = (st >> 3) + (first ? off : off - k1);
              const int lo8 = imax(st - 8 * oc, 0), hi8 = imin(st + ln - 8 * oc, 8);
              wo = (unsigned)oc * (unsigned)OCTET_BYTES | (((1u << hi8) - 1u) & ~((1u << lo8) - 1u));
            }
          }
          const int nch = imin(8, (tot - w0 + 7) >> 3);

          // position of this lane's neighbour of a chunk, and its octet's
          // entry (a chunk past the window reads some octet of it again)
          auto load = [&](int ch, double2& xy, unsigned& o) {
            o = (unsigned)lane_get((int)wo, 8 * ch + ((int)lane >> 3));
            xy = *reinterpret_cast<const double2*>(octets + ((o & ~255u) | (lane & 7u) << 4));
          };
          auto process = [&](double2 xy, unsigned o) {
            // ---- bin (binary64 r^2, no contraction)
            const double dx = xy.x - xi, dy = xy.y - yi;
            const double rr = r2_exact(dx, dy);
            const bool inb = ((o & (1u << (lane & 7u))) != 0u) & (rr >= e2lo) & (rr < e2hi);
            const unsigned long long mm = __builtin_amdgcn_ballot_w64(inb);
            if (mm == 0ull) return;
            cnt += (int)__popcll(mm);
            // ---- rows p = 0 and triple blocks, in operand layout (in flight
            // while the columns are formed).  K step s of lane group g is the
            // octet of lanes 16 g + 8 s + 0..7.
            const unsigned own = o & ~255u;
            const unsigned oth = (unsigned)__builtin_amdgcn_mov_dpp((int)own, DPP_ROW_ROR8, 0xf, 0xf, false);
            const unsigned oc[2] = {c < 8 ? own : oth, c < 8 ? oth : own};
            half8v v0[2], vs[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              v0[s] = *reinterpret_cast<const half8v*>(octets + (oc[s] + toff));
              if constexpr (NS) vs[s] = *reinterpret_cast<const half8v*>(octets + (oc[s] + soff));
            }
            // ---- z and its powers; z = 0 outside the bin
            const double i0 = (double)__frsqrt_rn(fmaxf((float)rr, 1.17549435e-38f));
            const double er = 1.0 - (rr * i0) * i0;
            double i1 = i0 + (0.5 * i0) * er;
            i1 = inb ? i1 : 0.0;
            const double zr6 = dx * i1, zi6 = dy * i1;
            const float zr = (float)zr6, zi = (float)zi6, c2 = 2.f * zr;
            float pr[RC + 1], pi[RC + 1];
            pr[1] = zr;
            pi[1] = zi;
            const double ar = zr6 * zr6 - zi6 * zi6, ai = zr6 * zi6;   // z^2 = ar + 2 i ai
            pr[2] = (float)ar;
            pi[2] = 2.f * (float)ai;
            pr[4] = (float)(ar * ar - 4.0 * (ai * ai));
            pi[4] = 4.f * (float)(ar * ai);
            pr[8] = pr[4] * pr[4] - pi[4] * pi[4];
            pi[8] = 2.f * pr[4] * pi[4];
            const int at = plane_at((int)lane);
            const unsigned flag = inb ? 0x3c00u : 0u;   // 1 in binary16
            // z^17 = (z^8)^2 z, z^34 = (z^17)^2
            const float sr = pr[8] * pr[8] - pi[8] * pi[8], si = 2.f * pr[8] * pi[8];
            float qr = sr * zr - si * zi, qi = sr * zi + si * zr;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
              unsigned h, l;
              split2(qr, qi, h, l);
              unsigned char* zp = wb.planes + ZP_PLANE + ZP_STEP * p + at;
              *reinterpret_cast<u32x4*>(zp) = u32x4{h, flag, h, h};
              *reinterpret_cast<u32x4*>(zp + ZP_LO) = u32x4{l, 0u, l, l};
              const float tr = qr * qr - qi * qi;
              qi = 2.f * qr * qi;
              qr = tr;
            }
            pr[3] = c2 * pr[2] - zr;
            pi[3] = c2 * pi[2] - zi;
            pr[5] = c2 * pr[4] - pr[3];
            pi[5] = c2 * pi[4] - pi[3];
            pr[6] = pr[3] * pr[3] - pi[3] * pi[3];
            pi[6] = 2.f * pr[3] * pi[3];
            pr[7] = c2 * pr[6] - pr[5];
            pi[7] = c2 * pi[6] - pi[5];
            u32x4 chi[2], clo[2];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
              unsigned h, l;
              split2(pr[COL_R[r]], pi[COL_R[r]], h, l);
              chi[r >> 2][r & 3] = h;
              clo[r >> 2][r & 3] = l;
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              *reinterpret_cast<u32x4*>(wb.planes + COL_PLANE[k] + at) = chi[k];
              *reinterpret_cast<u32x4*>(wb.planes + COL_PLANE[2 + k] + at) = clo[k];
            }
            wave_sync();
            // ---- operands and products, two K steps of 32 neighbours
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              const half8v bh = read_operand(cread + 128 * s);
              const half8v bl = read_operand(lread + 128 * s);
              const half8v bx = read_operand(xread + 128 * s);
              acc[C::TT] = mma(v0[s], bh, acc[C::TT]);
              low[0] = mma(v0[s], bl, low[0]);
              acc[C::TX] = mma(v0[s], bx, acc[C::TX]);
              if constexpr (NS) acc[C::TS] = mma(vs[s], bx, acc[C::TS]);
              // rows 2 f, 2 f + 1 of p > 0 take both parts of weight f, which sit
              // in those two rows of p = 0
              const half8v vh = quad<DPP_QUAD_EVEN>(v0[s]), vl = quad<DPP_QUAD_ODD>(v0[s]);
#pragma unroll
              for (int p = 0; p < NP; ++p) {
                const half8v xh = read_operand(zread + ZP_STEP * p + 128 * s);
                const half8v xl = read_operand(zread + ZP_STEP * p + ZP_LO + 128 * s);
                half8v ah, al;
                product2(vh, vl, xh, xl, ah, al);
                acc[C::TP + p] = mma(ah, bh, acc[C::TP + p]);
                low[1 + p] = mma(ah, bl, low[1 + p]);
                low[1 + p] = mma(al, bh, low[1 + p]);
              }
              if constexpr (C::TOP) {
                // z^34: the second operand's addresses, one p on; its flag and
                // (z^4, z^8) columns are not used
                const half8v b34 = read_operand((grp4 < 2 ? xread + ZP_STEP : xread) + 128 * s);
                acc[C::T34] = mma(v0[s], b34, acc[C::T34]);
              }
            }
            if (++nfold >= fold_chunks(N)) {
              fold();
              nfold = 0;
            }
            wave_sync();
          };
          double2 xy0, xy1;
          unsigned o0, o1;
          load(0, xy0, o0);
          for (int ch = 0; ch < nch; ch += 2) {
            load(ch + 1, xy1, o1);
            process(xy0, o0);
            if (ch + 1 == nch) break;
            load(ch + 2, xy0, o0);
            process(xy1, o1);
          }
        }
      }
      fold();
      wave_sync();

      // ---- epilogue: unscaled sums -> LDS -> record entries.  Rows 2 f and
      // 2 f + 1 are the high and low part of weight f in p = 0 (of triple-block
      // weight f), and cos and sin in p > 0; this lane holds rows 4 g + 0..3.
      const double u0 = unscale[lev][2 * g], u1 = unscale[lev][2 * g + 1];
      double* S = wb.sums;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int row = 16 * (2 * g + j) + c;
        const double u = j ? u1 : u0;
        auto both = [&](int t) { return m[t][2 * j] + m[t][2 * j + 1]; };
        S[C::OT + row] = (both(C::TT) + ((double)low[0][2 * j] + (double)low[0][2 * j + 1])) * u;
        S[C::OX + row] = both(C::TX) * u;
        if constexpr (NS) S[C::OS + row] = both(C::TS) * unscale[lev][NF + 2 * g + j];
        if constexpr (C::TOP) S[C::O34 + row] = both(C::T34) * u;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            S[C::OP + 256 * p + 16 * (4 * g + 2 * j + i) + c] =
                (m[C::TP + p][2 * j + i] + (double)low[1 + p][2 * j + i]) * u;
      }
      if (lane == 0) S[C::OZERO] = 0.0;
      wave_sync();
      float2* rec = reinterpret_cast<float2*>(a.rec_aos) + ((int64_t)idx * nb + b) * MPC;
      float gmax = 0.f, wmax = 0.f;   // block maxima for the fp16 operand scaling
#pragma unroll
      for (int e0 = 0; e0 < MPC; e0 += 64) {
        const int e = e0 + (int)lane;
        if (e < MPC) {
          const u32x4 q = *reinterpret_cast<const u32x4*>(&entry_table<N>.t[e]);
          double v[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const unsigned t = i & 1 ? q[i >> 1] >> 16 : q[i >> 1] & 0xffffu;
            const double x = S[t & 0x7fffu];
            v[i] = t & TERM_NEG ? -x : x;
          }
          const double re = (v[0] + v[1]) + (v[2] + v[3]), im = (v[4] + v[5]) + (v[6] + v[7]);
          rec[e] = make_float2((float)re, (float)im);
          const float mx = (float)fmax(fabs(re), fabs(im));
          if (e < L.offW) gmax = fmaxf(gmax, mx);
          else if (e < L.offQ) wmax = fmaxf(wmax, mx);
        }
      }
      if (a.maxima != nullptr) {
        // bits of non-negative floats order as integers; lane 63 ends with all
        const int gm = wave_scan_max((int)__float_as_uint(gmax)), wm = wave_scan_max((int)__float_as_uint(wmax));
        if (lane == 63) {
          atomicMax(&bmax[0][b], (unsigned)gm);
          atomicMax(&bmax[1][b], (unsigned)wm);
        }
      }
      if (a.counts != nullptr && lane == 0) a.counts[(int64_t)idx * nb + b] = cnt;
      wave_pairs += (unsigned long long)cnt;
      wave_sync();
    }
  }
  if (a.pairs != nullptr && lane == 0 && wave_pairs) atomicAdd(a.pairs, wave_pairs);
  if (a.maxima != nullptr) {
    __syncthreads();
    for (int q = (int)threadIdx.x; q < nb; q += (int)blockDim.x) {
      if (bmax[0][q]) atomicMax(a.maxima + MAXIMA_G + q, bmax[0][q]);
      if (bmax[1][q]) atomicMax(a.maxima + MAXIMA_W + q, bmax[1][q]);
    }
    if (!RED && lane == 0) {
      atomicMax(a.maxima + MAXIMA_X, __float_as_uint(xmax));
      atomicMax(a.maxima + MAXIMA_X + 1, __float_as_uint(wxmax));
    }
  }
}

template <int N, bool RED>
static int resident_blocks_mm() {
  static int resident = -1;
  if (resident < 0) {
    int per_cu = 0, dev = 0, ncu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, stage_mm_kernel<N, RED>, 256, 0) != hipSuccess ||
        per_cu < 1)
      per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
      ncu = 256;
    resident = per_cu * ncu;
  }
  return resident;
}

template <int N, bool RED>
hipError_t launch_pairs_mm(StageAArgs a, hipStream_t s) {
  // bin groups, widest bins first: a group closes once it holds an eighth of
  // the annulus area, so that a centre's bins spread over several waves and
  // the narrow inner bins share one
  const double* e = a.host_edges;
  const double total = a.b_hi > a.b_lo ? e[a.b_hi] * e[a.b_hi] - e[a.b_lo] * e[a.b_lo] : 0.0;
  int cut[FPCF4_NBINS_SUPPORTED + 1], nc = 0;
  cut[nc++] = a.b_hi;
  double acc = 0.0;
  for (int b = a.b_hi - 1; b >= a.b_lo; --b) {
    acc += e[b + 1] * e[b + 1] - e[b] * e[b];
    if (b == a.b_lo || acc >= 0.125 * total) {
      cut[nc++] = b;
      acc = 0.0;
    }
  }
  if (nc == 1) cut[nc++] = a.b_hi;   // no bins: the centre factors are still written
  a.ngroups = nc - 1;
  for (int q = 0; q < nc - 1; ++q) {
    a.gfirst[q] = (uint8_t)cut[q + 1];
    a.gend[q] = (uint8_t)cut[q];
  }
  // Octets within the outermost radius of a centre, against 4 MB of L2.  1e6
  // galaxies, 12 bins to 100', nmax 8, at 3, 10, 60 and 120 per square arcmin
  // (9 MB and more): 52, 189, 134 and 197 ms with blocks of 64, where six groups are
  // in flight at once, 48, 172, 111 and 162 with the whole queue; at 1 (3 MB) 22.1
  // and 21.5, at 0.5 15.7 and 16.1, and 30011 galaxies at 1, 13 bins to 57' (1 MB)
  // 3.06 and 3.12.
  const double near = a.density * M_PI * e[a.nb] * e[a.nb] * (OCTET_BYTES / 8.0);
  a.block = near > 2.5e6 ? imax(a.ncent, 1) : 64;
  const int resident = resident_blocks_mm<N, RED>();
  const int64_t units = (int64_t)a.ncent * a.ngroups;
  int nblocks = (int)std::min<int64_t>((units + 3) / 4, resident);
  nblocks = ((nblocks + 7) / 8) * 8;   // blocks are dealt round-robin to the 8 XCDs
  if (nblocks < 8) nblocks = 8;
  hipLaunchKernelGGL((stage_mm_kernel<N, RED>), dim3(nblocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

#if defined(FPCF4_STAGE_A_N)
// One translation unit per nmax, as for the vector kernel.
// matrix_order, for the preprocessor
#define FPCF4_MM4 (FPCF4_STAGE_A_N >= 5)
#define FPCF4_MM3 (FPCF4_STAGE_A_N >= 8 && FPCF4_STAGE_A_N != 12)
static_assert(FPCF4_MM4 == matrix_order(4, FPCF4_STAGE_A_N) && FPCF4_MM3 == matrix_order(3, FPCF4_STAGE_A_N),
              "instantiated where they are used");
#if FPCF4_MM4
template hipError_t launch_pairs_mm<FPCF4_STAGE_A_N, false>(StageAArgs, hipStream_t);
template hipError_t launch_pairs_mm<FPCF4_STAGE_A_N, true>(StageAArgs, hipStream_t);
#endif
#if FPCF4_MM3
template hipError_t launch_pairs_mm<PLAN3 + FPCF4_STAGE_A_N, false>(StageAArgs, hipStream_t);
template hipError_t launch_pairs_mm<PLAN3 + FPCF4_STAGE_A_N, true>(StageAArgs, hipStream_t);
#endif
#else
// ---------------------------------------------------------------------------
// Octet blocks: OCTET_BYTES per 8 consecutive neighbours, four parts that each
// load of the pair kernel reads whole lines of:
//   byte   0: 8 positions (x, y)
//   byte 128: 16 rows of 8 binary16 values, the high and low parts of each of
//             the seven weights, and two rows of zeros
//   byte 384: 10 rows, the high and low parts of each of the triple-block
//             weights (w g)^3, |w g|^2 w g, w^3
// Neighbours past the last one are zero.  One thread forms one row or two
// positions; the octet's records come from L1.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double weight_of(const Gal<float>& q, int f) {
  const double x = q.a, y = q.b, w = q.w;
  switch (f) {
    case FA: return x;
    case FB: return y;
    case FC: return x * x - y * y;
    case FD: return 2.0 * x * y;
    case FW: return w;
    case FE: return x * x + y * y;
    case FV: return w * w;
    case NF + 0: return (x * x - y * y) * x - 2.0 * x * y * y;
    case NF + 1: return (x * x - y * y) * y + 2.0 * x * y * x;
    case NF + 2: return (x * x + y * y) * x;
    case NF + 3: return (x * x + y * y) * y;
    default: return w * w * w;
  }
}
__device__ __forceinline__ double weight_of(const GalR<float>& q, int f) {
  const float v[NWEIGHTS] = {q.a, q.b, q.c, q.d, q.w, q.e, q.v, q.p3, q.q3, q.ea, q.eb, q.u};
  float r = v[0];
#pragma unroll
  for (int k = 1; k < NWEIGHTS; ++k) r = f == k ? v[k] : r;
  return r;
}

constexpr int kOctetParts = 30;   // 4 pairs of positions, 26 rows
// weights whose second component is the next one: real and imaginary part
__device__ __forceinline__ bool complex_weight(int f) { return f == FA || f == FC || f == NF || f == NF + 2; }
__device__ __forceinline__ bool second_part(int f) { return f > 0 && complex_weight(f - 1); }
template <typename Rec>
__global__ __launch_bounds__(256) void octet_kernel(const Rec* gal, int64_t n, MatScale ms, unsigned char* out,
                                                    unsigned* faint) {
  const int64_t parts = ((n + 7) / 8) * kOctetParts;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < parts; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t oc = i / kOctetParts;
    const int part = (int)(i - oc * kOctetParts);
    unsigned char* o = out + oc * OCTET_BYTES;
    if (part < 4) {
#pragma unroll
      for (int j = 2 * part; j < 2 * part + 2; ++j) {
        const int64_t q = 8 * oc + j;
        reinterpret_cast<double2*>(o)[j] = q < n ? double2{gal[q].x, gal[q].y} : double2{0.0, 0.0};
      }
      continue;
    }
    const int row = part - 4;
    const bool low = (row & 1) != 0;
    const int f = row < 16 ? imin(row >> 1, NF - 1) : NF + ((row - 16) >> 1);
    const bool none = row == 14 || row == 15;
    const double scale = 1.0 / ms.inv[f];   // exact: a power of two
    const bool judge = !low && !none && !second_part(f), pair = judge && complex_weight(f);
    const double scale2 = pair ? 1.0 / ms.inv[f + 1] : 0.0;
    double most = 0.0;   // of a real or complex weight
    half8v v;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t q = 8 * oc + j;
      float x = 0.f;
      if (q < n && !none) {
        const double s = weight_of(gal[q], f) * scale;
        x = (float)s;
        most = fmax(most, fabs(s));
        if (pair) most = fmax(most, fabs(weight_of(gal[q], f + 1) * scale2));
      }
      const _Float16 h = (_Float16)x;
      v[j] = low ? (_Float16)(x - (float)h) : h;
    }
    *reinterpret_cast<half8v*>(o + 128 + 16 * row) = v;
    if (judge && most < OCTET_MIN) {
      // a last octet of fewer than eight counts with the one before it, since a
      // galaxy or two alone may well have a small shear
      if (8 * oc + 8 > n && oc > 0)
        for (int64_t q = 8 * oc - 8; q < 8 * oc; ++q) {
          most = fmax(most, fabs(weight_of(gal[q], f) * scale));
          if (pair) most = fmax(most, fabs(weight_of(gal[q], f + 1) * scale2));
        }
      if (most > 0.0 && most < OCTET_MIN) *faint = 1u;   // every writer stores the same
    }
  }
}
#endif

}  // namespace sa

#if !defined(FPCF4_STAGE_A_N)
size_t octet_bytes(int64_t n) { return (size_t)((n + 7) / 8) * OCTET_BYTES; }

template <typename Rec>
hipError_t build_octets(const Rec* gal, int64_t n, const MatScale& ms, void* out, unsigned* faint, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (((n + 7) / 8) * sa::kOctetParts + 255) / 256;
  hipLaunchKernelGGL(sa::octet_kernel<Rec>, dim3((unsigned)(blocks < 16384 ? blocks : 16384)), dim3(256), 0, s, gal,
                     n, ms, static_cast<unsigned char*>(out), faint);
  return hipGetLastError();
}
template hipError_t build_octets<Gal<float>>(const Gal<float>*, int64_t, const MatScale&, void*, unsigned*, hipStream_t);
template hipError_t build_octets<GalR<float>>(const GalR<float>*, int64_t, const MatScale&, void*, unsigned*,
                                              hipStream_t);
#endif

}  // namespace fpcf4
