// Shear 3PCF multipoles from the per-centre records of stage (a): the
// order-N construction of the appendix on N-th order shear statistics,
// taken at N = 3 (beta rows (+,+,+), (-,+,+), (+,-,+), (+,+,-) for
// Gamma_0..Gamma_3, generalised x-projection zeta_0 = (phi_1 + phi_2)/2):
//
//   Upsilon_{mu,n}(b1, b2) = sum_i x_i F1_mu(i, b1; n) F2_mu(i, b2; n)
//
//   mu  x_i        F1 at Theta_1      F2 at Theta_2      same-neighbour block
//   0   w g        G_{n-3}            G_{-n-3}           Q_{-6}
//   1   conj(w g)  G_{n-1}            G_{-n-1}           Q_{-2}
//   2   w g        conj G_{-n-1}      G_{-n-3}           A_{-2} = conj A_2
//   3   w g        G_{n-3}            conj G_{n-1}       A_{-2}
//   N   w          W_n                W_{-n}             V_0
//
// (a slot with exponent coefficient c is G_c, or conj G_{-c} where its shear
// is conjugated).  The natural components are products of three projected
// shears -gamma_c e^{-2 i zeta} (Sect. 2.1), so the shear components carry a
// factor (-1)^3 that the block products above do not: the output is
// -Upsilon_mu for mu = 0..3 (the normalisation has no shear and no sign).  For distinct neighbour pairs the j = k terms, which exist
// only for Theta_1 = Theta_2, are removed:
//   Upsilon'(b, b) = Upsilon(b, b) - sum_i x_i D_mu(i, b),
// D_mu = sum_j (slot-1 weight)(slot-2 weight) e^{i (c1 + c2) phi_ij}, the
// block in the last column (c1 + c2 does not depend on n).
//
// A stage (a) record of order n4 holds G_k for k = -2 n4 - 3 .. 2 n4 - 1,
// W_k for |k| <= 2 n4, Q_-6, Q_-2, A_2 and V_0, so 3PCF multipoles up to
// |n| <= 2 n4 are read from it directly.
//
// The contraction (5 (2m+1) nb^2 complex products per centre) is binary64
// throughout (the records are converted on load).  A wave takes a tile of T1 x
// T2 outputs (b1, b2) of one (n, mu, centre slice), a lane every 64th centre
// of the slice: T1 + T2 loads feed T1 T2 products, all in registers, and the
// lanes' sums are added at the end.  Each slice writes its own partial buffer;
// the slices are added in slice order (deterministic).
#include "fpcf4_internal.hpp"

namespace fpcf4 {
namespace {

struct Slot3 {
  bool w;      // W block (else G)
  bool conj;
  int s, o;    // order = s * n + o
};
struct Row3 {
  int x;       // centre factor: 0 = w g, 1 = conj(w g), 2 = w
  Slot3 f1, f2;
  int dfam;    // same-neighbour block: 0 = Q, 1 = A, 2 = V
  int dord;
  bool dconj;
};
__host__ __device__ constexpr Row3 row3(int mu) {
  return mu == 0 ? Row3{0, {false, false, 1, -3}, {false, false, -1, -3}, 0, -6, false}
       : mu == 1 ? Row3{1, {false, false, 1, -1}, {false, false, -1, -1}, 0, -2, false}
       : mu == 2 ? Row3{0, {false, true, -1, -1}, {false, false, -1, -3}, 1, 2, true}
       : mu == 3 ? Row3{0, {false, false, 1, -3}, {false, true, 1, -1}, 1, 2, true}
                 : Row3{2, {true, false, 1, 0}, {true, false, -1, 0}, 2, 0, false};
}

constexpr int CH3 = 64;   // centres of a slice, a multiple of the wave

__device__ inline int slot_entry(const Layout& L, const Slot3& f, int n) {
  const int k = f.s * n + f.o;
  return f.w ? eW(L, k) : eG(L, k);
}

template <typename T>
__device__ inline void centre_factor(const ThreeArgs& a, int x, int ci, double& xr, double& xi) {
  if (x == 2) {
    xr = (double)static_cast<const T*>(a.xw)[ci];
    xi = 0.0;
  } else {
    const T* g = static_cast<const T*>(a.xg);
    xr = (double)g[2 * ci];
    xi = (double)g[2 * ci + 1];
    if (x == 1) xi = -xi;
  }
}

// slice s of `parts` covers centres [s * per, min((s + 1) * per, ncent))
__host__ __device__ inline int slice_len(int ncent, int parts) {
  const int per = (ncent + parts - 1) / parts;
  return (per + CH3 - 1) / CH3 * CH3;
}

// Bin tiles of a dimension: as many of t bins as cover nb.
__host__ __device__ inline int tiles3(int nb, int t) { return (nb + t - 1) / t; }

// Lane l ends with the sum over the lanes of value l of v[0, 64): lanes that
// differ in bit W exchange halves of the values (indexes known at compile time,
// so that they stay in registers).
template <int W>
__device__ __forceinline__ void transpose_sum(double (&v)[64], int lane) {
  const bool up = (lane & W) != 0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const double keep = up ? v[k + W] : v[k], send = up ? v[k] : v[k + W];
    v[k] = keep + __shfl_xor(send, W, 64);
  }
  if constexpr (W > 1) transpose_sum<W / 2>(v, lane);
}

// One wave per (n, mu, slice, tile); blockIdx.x = n times the workgroups of
// four consecutive tiles, which share slot-1 records through L1.  Bound by the
// binary64 multiply-adds, four per product (and per 64 centres of a tile 6 T1 +
// 3 T2 + 12 more for conversions and the centre factor), and in binary64 by
// the records' way from L2 (T1 + T2 of 16 bytes per centre and tile).  27000
// galaxies, 65 bins, |n| <= 15, binary64: 6.6 ms; the three tree levels' sums of
// 1e6 galaxies, 12 bins, |n| <= 10: 13 ms.  One output per thread with the
// records staged in LDS read 32 bytes of LDS for every four multiply-adds and
// took 9.0 and 42 ms.
static_assert(THREE_SLICES % 8 == 0, "equal shares for the XCDs");
template <typename T, int T1, int T2>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void contract3_kernel(ThreeArgs a) {
  static_assert(2 * T1 * T2 <= 64, "one lane per component of the tile's sums");
  const int nt2 = tiles3(a.nb2, T2), ntt = tiles3(a.nb1, T1) * nt2, groups = (ntt + 3) / 4;
  // workgroups are dealt to the 8 XCDs round-robin: give each XCD a contiguous
  // range of (slice, mu, n, tile), so that the tiles of one (n, mu, slice) read
  // its records through one L2
  const unsigned all = gridDim.x * 5u * THREE_SLICES;
  const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + 5u * blockIdx.z);
  const unsigned id = (lin & 7u) * (all / 8u) + (lin >> 3);
  const int bx = (int)(id % gridDim.x), mu = (int)(id / gridDim.x % 5u), sl = (int)(id / gridDim.x / 5u);
  const int ni = bx / groups;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tile = (bx - ni * groups) * 4 + wv;
  if (tile >= ntt) return;
  const int lane = (int)(threadIdx.x & 63);
  const int u1 = tile / nt2 * T1, u2 = (tile - tile / nt2 * nt2) * T2;   // first bins of the tile in the slot ranges
  const int n = ni - a.m, nb = a.nb;
  const Layout L = make_layout(a.n4);
  const Row3 r = row3(mu);
  const int per = slice_len(a.ncent, THREE_SLICES);
  const int c0 = sl * per, c1 = min(a.ncent, c0 + per);
  // records of the tile's bins (past the range: the last bin again, not stored)
  const T* r1 = static_cast<const T*>(a.rec) + 2 * ((size_t)slot_entry(L, r.f1, n) * nb + a.lo1) * a.ldc;
  const T* r2 = static_cast<const T*>(a.rec2) + 2 * ((size_t)slot_entry(L, r.f2, n) * nb + a.lo2) * a.ldc2;
  const T* p1[T1];
  const T* p2[T2];
#pragma unroll
  for (int b = 0; b < T1; ++b) p1[b] = r1 + 2 * (size_t)min(u1 + b, a.nb1 - 1) * a.ldc;
#pragma unroll
  for (int b = 0; b < T2; ++b) p2[b] = r2 + 2 * (size_t)min(u2 + b, a.nb2 - 1) * a.ldc2;
  const double s1 = r.f1.conj ? -1.0 : 1.0;
  const T s2 = r.f2.conj ? T(-1) : T(1);
  double v[64];
#pragma unroll
  for (int k = 0; k < 64; ++k) v[k] = 0.0;
  for (int cb = c0; cb < c1; cb += 64) {
    const int ci = min(cb + lane, c1 - 1);
    const int col1 = a.par1 ? a.par1[ci] : ci, col2 = a.par2 ? a.par2[ci] : ci;
    T f1[T1][2], f2[T2][2];
#pragma unroll
    for (int b = 0; b < T1; ++b) {
      f1[b][0] = p1[b][2 * (size_t)col1];
      f1[b][1] = p1[b][2 * (size_t)col1 + 1];
    }
#pragma unroll
    for (int b = 0; b < T2; ++b) {
      f2[b][0] = p2[b][2 * (size_t)col2];
      f2[b][1] = p2[b][2 * (size_t)col2 + 1];
    }
    double xr, xi;
    centre_factor<T>(a, r.x, ci, xr, xi);
    if (cb + lane >= c1) xr = xi = 0.0;
    const double yr = s1 * xr, yi = s1 * xi;
    double gr[T2], gi[T2];
#pragma unroll
    for (int b = 0; b < T2; ++b) {
      gr[b] = (double)f2[b][0];
      gi[b] = (double)(s2 * f2[b][1]);
    }
#pragma unroll
    for (int b = 0; b < T1; ++b) {
      const double fr = (double)f1[b][0], fi = (double)f1[b][1];
      const double lr = fma(xr, fr, -(yi * fi)), li = fma(xi, fr, yr * fi);
#pragma unroll
      for (int q = 0; q < T2; ++q) {
        double& ar = v[2 * (b * T2 + q)];
        double& ai = v[2 * (b * T2 + q) + 1];
        ar = fma(lr, gr[q], ar);
        ai = fma(lr, gi[q], ai);
        ar = fma(-li, gi[q], ar);
        ai = fma(li, gr[q], ai);
      }
    }
  }
  transpose_sum<32>(v, lane);
  const int k = lane >> 1, b1 = u1 + k / T2, b2 = u2 + k % T2;
  if (k < T1 * T2 && b1 < a.nb1 && b2 < a.nb2)
    a.part[2 * ((size_t)sl * three_elems(nb, a.m) + ((size_t)mu * a.nn + ni) * nb * nb + (size_t)(a.lo1 + b1) * nb +
                a.lo2 + b2) + (lane & 1)] = v[0];
}

// same-neighbour sums sum_i x_i D_mu(i, b) for every bin: one workgroup per
// (mu, centre slice, bin tile), centres strided over the threads, then a
// fixed-order tree reduction over the workgroup.
template <typename T>
__global__ __launch_bounds__(256) void diag3_kernel(ThreeArgs a) {
  const int mu = blockIdx.x;
  const int sl = blockIdx.y;
  const int nb = a.nb;
  const BinTiles bt = bin_tiles(a.nb1);   // bins [lo1, lo1 + nb1) of the slot-1 records
  const int ob = a.lo1 + (int)blockIdx.z * bt.tb, nbt = min(bt.tb, a.lo1 + a.nb1 - ob);
  const Layout L = make_layout(a.n4);
  const Row3 r = row3(mu);
  const int ed = r.dfam == 0 ? eQ(L, r.dord) : r.dfam == 1 ? eA(L, r.dord) : eV(L, r.dord);
  const int per = slice_len(a.ncent, THREE_SLICES);
  const int c0 = sl * per;
  const int c1 = min(a.ncent, c0 + per);
  const T* rec = static_cast<const T*>(a.rec);
  double accr[BIN_TILE_MAX], acci[BIN_TILE_MAX];
#pragma unroll
  for (int b = 0; b < BIN_TILE_MAX; ++b) accr[b] = acci[b] = 0.0;
  for (int ci = c0 + (int)threadIdx.x; ci < c1; ci += blockDim.x) {
    double xr, xi;
    centre_factor<T>(a, r.x, ci, xr, xi);
#pragma unroll
    for (int b = 0; b < BIN_TILE_MAX; ++b) {
      if (b < nbt) {
        const size_t o = (((size_t)ed * nb + ob + b) * a.ldc + ci) * 2;
        const double vr = (double)rec[o];
        const double vi = r.dconj ? -(double)rec[o + 1] : (double)rec[o + 1];
        accr[b] = fma(xr, vr, fma(-xi, vi, accr[b]));
        acci[b] = fma(xr, vi, fma(xi, vr, acci[b]));
      }
    }
  }
  __shared__ double2 red[256];
  const int t = threadIdx.x;
  double* out = a.part + 2 * ((size_t)sl * three_elems(nb, a.m) + (size_t)5 * a.nn * nb * nb +
                              (size_t)mu * nb);
#pragma unroll
  for (int b = 0; b < BIN_TILE_MAX; ++b) {
    if (b < nbt) {
      red[t] = make_double2(accr[b], acci[b]);
      __syncthreads();
      for (int s = 128; s > 0; s >>= 1) {
        if (t < s) {
          red[t].x += red[t + s].x;
          red[t].y += red[t + s].y;
        }
        __syncthreads();
      }
      if (t == 0) {
        out[2 * (ob + b)] = red[0].x;
        out[2 * (ob + b) + 1] = red[0].y;
      }
      __syncthreads();
    }
  }
}

// acc[i] += sum over slices of part[s][i], slices in order
__global__ void reduce3_kernel(const double* part, size_t elems2, double* acc) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= elems2) return;
  double v = 0.0;
  for (int s = 0; s < THREE_SLICES; ++s) v += part[(size_t)s * elems2 + i];
  acc[i] += v;
}

// out[mu][b1][b2][n] = acc[mu][n][b1][b2] - [b1 == b2] diag[mu][b1]
__global__ void finalize3_kernel(const double* acc, int nb, int m, int subtract, double* out) {
  const int nn = 2 * m + 1;
  const size_t total = (size_t)5 * nb * nb * nn;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int ni = (int)(i % nn);
  const int b2 = (int)((i / nn) % nb);
  const int b1 = (int)((i / ((size_t)nn * nb)) % nb);
  const int mu = (int)(i / ((size_t)nn * nb * nb));
  const size_t src = ((size_t)mu * nn + ni) * nb * nb + (size_t)b1 * nb + b2;
  double vr = acc[2 * src], vi = acc[2 * src + 1];
  if (subtract && b1 == b2) {
    const size_t d = (size_t)5 * nn * nb * nb + (size_t)mu * nb + b1;
    vr -= acc[2 * d];
    vi -= acc[2 * d + 1];
  }
  // (-1)^3 of the three projected shears (exact)
  const double sg = mu < 4 ? -1.0 : 1.0;
  out[2 * i] = sg * vr;
  out[2 * i + 1] = sg * vi;
}

template <typename T, int T1, int T2>
void launch_tile3(const ThreeArgs& a, hipStream_t s) {
  const int groups = (tiles3(a.nb1, T1) * tiles3(a.nb2, T2) + 3) / 4;
  hipLaunchKernelGGL((contract3_kernel<T, T1, T2>), dim3(a.nn * groups, 5, THREE_SLICES), dim3(256), 0, s, a);
}
template <typename T, int T1>
void launch_row3(const ThreeArgs& a, int t2, hipStream_t s) {
  switch (t2) {
    case 2: return launch_tile3<T, T1, 2>(a, s);
    case 3: return launch_tile3<T, T1, 3>(a, s);
    case 4: return launch_tile3<T, T1, 4>(a, s);
    case 5: return launch_tile3<T, T1, 5>(a, s);
    default: return launch_tile3<T, T1, 6>(a, s);
  }
}
// The tile shape of the least work: binary64 operations of a tile (four per
// product, two conversions per record, four more for the centre factor at
// slot 1, the sign at slot 2, about twelve per centre) times the tiles,
// surplus bins of the last ones included.
template <typename T>
void launch_contract3(const ThreeArgs& a, hipStream_t s) {
  int best1 = 0, best2 = 0;
  int64_t least = INT64_MAX;
  for (int t1 = 2; t1 <= 5; ++t1)
    for (int t2 = 2; t2 <= 6; ++t2) {
      const int64_t work = (int64_t)tiles3(a.nb1, t1) * tiles3(a.nb2, t2) * (4 * t1 * t2 + 6 * t1 + 3 * t2 + 12);
      if (work < least) {
        least = work;
        best1 = t1;
        best2 = t2;
      }
    }
  switch (best1) {
    case 2: return launch_row3<T, 2>(a, best2, s);
    case 3: return launch_row3<T, 3>(a, best2, s);
    case 4: return launch_row3<T, 4>(a, best2, s);
    default: return launch_row3<T, 5>(a, best2, s);
  }
}

}  // namespace

template <typename T>
hipError_t launch_three(const ThreeArgs& a, hipStream_t s) {
  if (a.ncent <= 0) return hipSuccess;
  if (a.nb < 1 || a.nb > FPCF4_NBINS_SUPPORTED || a.m < 0 || a.m > 2 * a.n4) return hipErrorInvalidValue;
  if (a.lo1 < 0 || a.nb1 < 1 || a.lo1 + a.nb1 > a.nb || a.lo2 < 0 || a.nb2 < 1 || a.lo2 + a.nb2 > a.nb)
    return hipErrorInvalidValue;
  launch_contract3<T>(a, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the same-neighbour sums exist where both slots share bins and records
  if (a.lo1 == a.lo2 && a.nb1 == a.nb2 && a.rec2 == a.rec && a.par1 == nullptr && a.par2 == nullptr)
    hipLaunchKernelGGL(diag3_kernel<T>, dim3(5, THREE_SLICES, bin_tiles(a.nb1).nt), dim3(256), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t elems2 = 2 * three_elems(a.nb, a.m);
  hipLaunchKernelGGL(reduce3_kernel, dim3((unsigned)((elems2 + 255) / 256)), dim3(256), 0, s,
                     (const double*)a.part, elems2, a.acc);
  return hipGetLastError();
}
template hipError_t launch_three<float>(const ThreeArgs&, hipStream_t);
template hipError_t launch_three<double>(const ThreeArgs&, hipStream_t);

hipError_t launch_finalize3(const double* acc, int nb, int m, int subtract, double* out, hipStream_t s) {
  const size_t total = (size_t)5 * nb * nb * (2 * m + 1);
  hipLaunchKernelGGL(finalize3_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, acc, nb,
                     m, subtract, out);
  return hipGetLastError();
}

}  // namespace fpcf4
