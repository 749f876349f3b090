// Multipoles -> bin-averaged natural components, binary64 (Sect. 2.3 and the
// multipole expansion of Sect. 3.1):
//   Ubar(T, Phi_a, Phi_b) = (2 pi)^-2 sum_{n2,n3} Upsilon_n I_n2(Phi_a) I_n3(Phi_b),
//   I_0(Phi) = |Delta Phi|, I_m(Phi) = (e^{i m Phi_up} - e^{i m Phi_low}) / (i m),
// on nphi linear angular bins of [0, 2 pi), done as two small complex
// contractions (over n2, then over n3).  Gamma_mu = Ubar_mu / Nbar.
//
// I_-m is the conjugate of I_m, and so is I_m of the mirrored bin
// nphi - 1 - a.  With the sums s_m = u_m + u_-m and differences
// d_m = u_m - u_-m (m >= 1; s_0 = u_0, d_0 = 0),
//   sum_m u_m I_m(a) = P + i Q,  P = sum_{m >= 0} s_m Re I_m(a), Q = sum d_m Im I_m(a),
// and the mirrored bin has P - i Q: a quarter of the multiply-adds of the
// plain sum.
#include "fpcf4_internal.hpp"

namespace fpcf4 {

__device__ inline void ang_int(int m, int a, int nphi, double& re, double& im) {
  const double lo = 2.0 * M_PI * a / nphi, hi = 2.0 * M_PI * (a + 1) / nphi;
  if (m == 0) {
    re = hi - lo;
    im = 0.0;
    return;
  }
  double sh, ch, sl, cl;
  sincos(m * hi, &sh, &ch);
  sincos(m * lo, &sl, &cl);
  // (e^{i m hi} - e^{i m lo}) / (i m)
  re = (sh - sl) / m;
  im = -(ch - cl) / m;
}

// table[m][a] = I_m(Phi_a), complex, 0 <= m <= nmax, of the lower half of the bins
__global__ void nat_table(int nmax, int nphi, double* table) {
  const int nh = (nphi + 1) / 2;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < (nmax + 1) * nh; t += gridDim.x * blockDim.x) {
    double re, im;
    ang_int(t / nh, t % nh, nphi, re, im);
    table[2 * t] = re;
    table[2 * t + 1] = im;
  }
}

// Sums over n2 of one (triplet, correlator) per block, as sums and differences
// in n3: tmp[t][a][mu][m] = (s_m, d_m)(a), complex.  The multipoles are folded
// over both orders in LDS; a thread then takes one (a, m) for both a and its
// mirror.  trip lists the triplets of bins, or is null for all in order.
__global__ __launch_bounds__(256) void nat_sum_n2(const double* ups, int nb, int nmax, int nphi, const int32_t* trip,
                                                  int64_t ntrip, const double* table, double* tmp) {
  const int nn = 2 * nmax + 1, n1 = nmax + 1, nh = (nphi + 1) / 2;
  __shared__ double fold[(FPCF4_NMAX_SUPPORTED + 1) * (FPCF4_NMAX_SUPPORTED + 1) * 8];   // [j][m]: ss, sd, ds, dd
  for (int64_t q = blockIdx.x; q < 9 * ntrip; q += gridDim.x) {
    const int64_t t = q / 9;
    const int mu = (int)(q - 9 * t);
    int64_t src = t;
    if (trip) src = ((int64_t)trip[3 * t] * nb + trip[3 * t + 1]) * nb + trip[3 * t + 2];
    const double* u = ups + 2 * ((int64_t)mu * nb * nb * nb + src) * nn * nn;
    for (int e = (int)threadIdx.x; e < n1 * n1; e += (int)blockDim.x) {
      const int j = e / n1, m = e - j * n1;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double pp = u[2 * ((nmax + j) * nn + nmax + m) + c];
        const double pm = m ? u[2 * ((nmax + j) * nn + nmax - m) + c] : 0.0;
        const double mp = j ? u[2 * ((nmax - j) * nn + nmax + m) + c] : 0.0;
        const double mm = j && m ? u[2 * ((nmax - j) * nn + nmax - m) + c] : 0.0;
        const double sp = pp + pm, sm = mp + mm;                      // sums over +-m at +j, -j
        const double dp = m ? pp - pm : 0.0, dm = m ? mp - mm : 0.0;  // differences
        fold[8 * e + c] = sp + sm;
        fold[8 * e + 2 + c] = dp + dm;
        fold[8 * e + 4 + c] = j ? sp - sm : 0.0;
        fold[8 * e + 6 + c] = j ? dp - dm : 0.0;
      }
    }
    __syncthreads();
    for (int e = (int)threadIdx.x; e < nh * n1; e += (int)blockDim.x) {
      const int a = e / n1, m = e - a * n1;
      double P[4] = {0.0, 0.0, 0.0, 0.0}, Q[4] = {0.0, 0.0, 0.0, 0.0};   // of s, d: re, im
      for (int j = 0; j < n1; ++j) {
        const double ir = table[2 * (j * nh + a)], ii = table[2 * (j * nh + a) + 1];
        const double* f = fold + 8 * (j * n1 + m);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          P[c] += f[c] * ir;
          Q[c] += f[4 + c] * ii;
        }
      }
      const int b = nphi - 1 - a;
      double* o = tmp + (((t * nphi + a) * 9 + mu) * n1 + m) * 4;
      double* r = tmp + (((t * nphi + b) * 9 + mu) * n1 + m) * 4;
#pragma unroll
      for (int c = 0; c < 4; c += 2) {   // P + i Q, P - i Q
        o[c] = P[c] - Q[c + 1];
        o[c + 1] = P[c + 1] + Q[c];
        if (b != a) {
          r[c] = P[c] + Q[c + 1];
          r[c + 1] = P[c + 1] - Q[c];
        }
      }
    }
    __syncthreads();
  }
}

// Sums over n3 of all nine correlators and the division by the norm, a wave
// per (triplet, a, 64 bins b and their mirrors): gamma[mu][t][a][b] =
// Ubar_mu / Re Nbar, norm[t][a][b] = Re Nbar.  The operands (s, d) are the
// same for the whole wave and come through scalar loads; the nine
// correlators' 36 sums share each load of the table.
// 256 triplets, nmax 10, 129 x 129 angular bins: 280 us, of which writing the
// 579 MB of results takes 122 at the rate of a copy.  The rest are the sums: an
// odd number of bins leaves every second wave with one lane's work (nh = 65).
// The whole conversion takes 393 us; with a plain sum per output (one thread
// each, its operands read again for every output) and a division pass over the
// stored sums it took 1232 us.
__global__ __launch_bounds__(256) void nat_sum_n3(const double* __restrict__ tmp, int64_t ntrip, int nmax, int nphi,
                                                  const double* __restrict__ table, double* __restrict__ gamma,
                                                  double* __restrict__ norm) {
  const int n1 = nmax + 1, nh = (nphi + 1) / 2, nchunk = (nh + 63) / 64;
  const double scale = 1.0 / (4.0 * M_PI * M_PI);
  const int64_t per_mu = ntrip * nphi * nphi, waves = ntrip * nphi * nchunk;
  const int lane = (int)(threadIdx.x & 63);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int64_t w = blockIdx.x * (int64_t)4 + wv; w < waves; w += (int64_t)gridDim.x * 4) {
    const int64_t ta = w / nchunk;                 // t * nphi + a
    const int b = (int)(w - ta * nchunk) * 64 + lane;
    const int bl = b < nh ? b : nh - 1;
    const double* __restrict__ u = tmp + ta * 9 * n1 * 4;
    double P[9][2], Q[9][2];
#pragma unroll
    for (int mu = 0; mu < 9; ++mu) P[mu][0] = P[mu][1] = Q[mu][0] = Q[mu][1] = 0.0;
    for (int m = 0; m < n1; ++m) {
      const double ir = table[2 * (m * nh + bl)], ii = table[2 * (m * nh + bl) + 1];
#pragma unroll
      for (int mu = 0; mu < 9; ++mu) {
        const double* f = u + (mu * n1 + m) * 4;
        P[mu][0] += f[0] * ir;
        P[mu][1] += f[1] * ir;
        Q[mu][0] += f[2] * ii;
        Q[mu][1] += f[3] * ii;
      }
    }
    if (b < nh) {
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const int bo = side ? nphi - 1 - b : b;
        if (side && bo == b) break;
        const double sg = side ? -1.0 : 1.0;
        const int64_t o = ta * nphi + bo;
        const double nv = (P[8][0] - sg * Q[8][1]) * scale;
        norm[o] = nv;
#pragma unroll
        for (int mu = 0; mu < 8; ++mu) {
          const double re = (P[mu][0] - sg * Q[mu][1]) * scale, im = (P[mu][1] + sg * Q[mu][0]) * scale;
          gamma[2 * (mu * per_mu + o)] = nv != 0.0 ? re / nv : 0.0;
          gamma[2 * (mu * per_mu + o) + 1] = nv != 0.0 ? im / nv : 0.0;
        }
      }
    }
  }
}

size_t natural_tmp_bytes(int64_t ntrip, int nmax, int nphi) {
  return (size_t)(ntrip * nphi * 9 * (nmax + 1)) * 32;
}

hipError_t natural_triplets(const double* ups, int nb, int nmax, int nphi, const int32_t* trip,
                            int64_t ntrip, double* tmp, double* gamma, double* norm, hipStream_t s) {
  const int64_t nh = (nphi + 1) / 2;
  double* table = nullptr;
  hipError_t e = hipMallocAsync(reinterpret_cast<void**>(&table), (size_t)((nmax + 1) * nh) * 16, s);
  if (e != hipSuccess) return e;
  const int64_t b2 = 9 * ntrip, b3 = (ntrip * nphi * ((nh + 63) / 64) + 3) / 4;
  hipLaunchKernelGGL(nat_table, dim3(64), dim3(256), 0, s, nmax, nphi, table);
  hipLaunchKernelGGL(nat_sum_n2, dim3((unsigned)(b2 < 65536 ? b2 : 65536)), dim3(256), 0, s, ups, nb, nmax, nphi, trip,
                     ntrip, table, tmp);
  hipLaunchKernelGGL(nat_sum_n3, dim3((unsigned)(b3 < 65536 ? b3 : 65536)), dim3(256), 0, s, tmp, ntrip, nmax, nphi,
                     table, gamma, norm);
  e = hipGetLastError();
  (void)hipFreeAsync(table, s);
  return e;
}

}  // namespace fpcf4
