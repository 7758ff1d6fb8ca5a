// Gram-based QR of the range finder's large sketches (QR classes 2 and 3)
// where its products run in FP32: two passes of G = Y^H Y, G = L L^H,
// Y <- Y L^-H (into Qc, then Qc and Y trade places).
//
// Its sums keep one fixed order.  An FP32 product rounds Q first, so a last
// bit of Q that differs flips a rounding of 6e-8 here and there, and one flip
// moves the truncated matrix by 1e-9 to 7e-8 (measured, 900 x 700 to 1024^2,
// l = 74 to 110): another order of the FP64 sums gives results that agree to
// the FP32 products' precision only.  Elsewhere rounding differences stay
// 1e-14 and the faster gramqr.hip takes over (here too for the QR of B^H,
// after the last FP32 product).
//
// A Cholesky pivot at or below kCholTol times the Gram's largest diagonal
// (kappa(Y) beyond about 1e7, where two passes lose orthogonality) refuses the
// problem: TEBD_DEV_QR_FALLBACK, and the Householder kernels (gate 2) take it
// over from what the passes left in Y, which spans the same space.
#include <cfloat>

#include "householder.hpp"
#include "kinds.hpp"
#include "loaders.hpp"

namespace tebd {

constexpr double kCholTol = 1e-14;
constexpr int kCholLdsL = 96;  // Gram in LDS up to this width (147 KiB), else in global memory

using CfgGram = ZCfg<kSketchTileM, kSketchTileN, 16, 2, 2>;

// G = Y^H Y into C (l x l column-major): the tiles that meet the lower
// triangle, all that the factorisation reads.  In the second pass only the
// problems whose first pass succeeded take part.
template <int WHICH>
__global__ __launch_bounds__(256) void k_gram_f32(Prob* probs, const int32_t* offs, int nprob,
                                                  int tebd, int pass) {
  __shared__ zt smem[CfgGram::lds_elems];
  for_each_tile<TK_GRAM>(probs, offs, nprob, tebd, [&](Prob& P, int, int, int m0, int n0, int) {
    if (!(P.chol & (WHICH ? kGramF32N : kGramF32M)) || (pass && !P.chol_ok)) return;
    if (n0 > m0) return;
    const int rows = WHICH ? P.n : P.m;
    const zt* Yc = WHICH ? P.Yt : P.Y;
    LdAdjColA la{Yc, rows};
    LdColB lb{Yc, rows};
    StCol st{P.C, P.l};
    zgemm_tile<CfgGram>(P.l, P.l, rows, m0, n0, la, lb, st, smem);
  });
}

// Q = Y R^-1 into Qc (R^-1 from k_chol_f32 in J).
template <int WHICH>
__global__ __launch_bounds__(256) void k_qapply_f32(Prob* probs, const int32_t* offs, int nprob,
                                                    int tebd) {
  __shared__ zt smem[CfgGram::lds_elems];
  for_each_tile<WHICH ? TK_QAPN : TK_QAPM>(probs, offs, nprob, tebd,
                                           [&](Prob& P, int, int, int m0, int n0, int) {
    if (!P.chol_ok || !(P.chol & (WHICH ? kGramF32N : kGramF32M))) return;
    const int rows = WHICH ? P.n : P.m;
    LdColA la{WHICH ? P.Yt : P.Y, rows};
    LdColB lb{P.J, P.l};
    StCol st{P.Qc, rows};
    zgemm_tile<CfgGram>(rows, P.l, P.l, m0 / 2, n0 / 2, la, lb, st, smem);
  });
}

// Cholesky G = L L^H of the Gram in C (column-major l x l, lower triangle
// used), then X = R^-1 = (L^-1)^H, upper triangular, into J: column c of
// L^-1 by forward substitution, one wavefront per column, the column held
// across the lanes (lane t keeps rows t, t + 64, ...).
template <int WHICH>
__global__ __launch_bounds__(1024) void k_chol_f32(Prob* probs, int pass) {
  Prob& P = probs[blockIdx.x];
  const int l = P.l, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool elig = l > 0 && (P.chol & (WHICH ? kGramF32N : kGramF32M)) && (pass == 0 || P.chol_ok);
  if (!elig) {
    if (tid == 0 && pass == 0) P.chol_ok = 0;
    return;
  }
  __shared__ zt g_lds[kCholLdsL * kCholLdsL];
  __shared__ double dmax_s;
  __shared__ int fail_s;
  const bool in_lds = l <= kCholLdsL;
  zt* G = in_lds ? g_lds : P.C;
  if (in_lds)
    for (int e = tid; e < l * l; e += 1024) g_lds[e] = P.C[e];
  __syncthreads();
  if (tid == 0) {
    double dm = 0.0;
    for (int j = 0; j < l; ++j) dm = fmax(dm, G[j + size_t(j) * l].x);
    dmax_s = dm;
    fail_s = !(dm > 0.0) || !isfinite(dm);
  }
  __syncthreads();
  for (int j = 0; j < l && !fail_s; ++j) {
    if (tid == 0) {
      const double d = G[j + size_t(j) * l].x;
      if (!(d > kCholTol * dmax_s) || !isfinite(d))
        fail_s = 1;
      else
        G[j + size_t(j) * l] = make_double2(sqrt(d), 0.0);
    }
    __syncthreads();
    if (fail_s) break;
    const double inv = 1.0 / G[j + size_t(j) * l].x;
    for (int i = j + 1 + tid; i < l; i += 1024) G[i + size_t(j) * l] = zscale(G[i + size_t(j) * l], inv);
    __syncthreads();
    const int nt = l - j - 1;
    for (int e = tid; e < nt * nt; e += 1024) {
      const int kk = e / nt, ii = e - kk * nt;
      if (ii < kk) continue;
      const int k = j + 1 + kk, i = j + 1 + ii;
      const zt lij = G[i + size_t(j) * l], lkj = G[k + size_t(j) * l];
      G[i + size_t(k) * l] = zsub(G[i + size_t(k) * l], zmul(lij, zconj(lkj)));
    }
    __syncthreads();
  }
  if (fail_s) {
    if (tid == 0) {
      P.chol_ok = 0;
      P.flags |= TEBD_DEV_QR_FALLBACK;
    }
    return;
  }
  // X = (L^-1)^H: row c of X holds conj of column c of L^-1
  zt* X = P.J;
  for (int c = wave; c < l; c += 16) {
    zt xr[kMaxL / 64];  // rows lane, lane + 64, ... of column c of L^-1
#pragma unroll
    for (int q = 0; q < kMaxL / 64; ++q) xr[q] = make_double2(0.0, 0.0);
    for (int i = c; i < l; ++i) {
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int q = 0; q < kMaxL / 64; ++q) {
        const int k = lane + 64 * q;
        if (k >= c && k < i) {
          const zt lik = G[i + size_t(k) * l];
          sr += lik.x * xr[q].x - lik.y * xr[q].y;
          si += lik.x * xr[q].y + lik.y * xr[q].x;
        }
      }
      sr = wave_sum(sr);
      si = wave_sum(si);
      const double lii = G[i + size_t(i) * l].x;
      const zt x = i == c ? make_double2(1.0 / lii, 0.0) : make_double2(-sr / lii, -si / lii);
#pragma unroll
      for (int q = 0; q < kMaxL / 64; ++q)
        if (lane + 64 * q == i) xr[q] = x;
    }
#pragma unroll
    for (int q = 0; q < kMaxL / 64; ++q) {
      const int i = lane + 64 * q;
      if (i < l) X[c + size_t(i) * l] = i >= c ? zconj(xr[q]) : make_double2(0.0, 0.0);
    }
  }
  if (tid == 0) P.chol_ok = 1;
}

template <int WHICH>
__global__ void k_qswap_f32(Prob* probs, int nprob) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nprob) return;
  Prob& P = probs[p];
  if (!P.chol_ok) return;
  zt* t = WHICH ? P.Yt : P.Y;
  if (WHICH)
    P.Yt = P.Qc;
  else
    P.Y = P.Qc;
  P.Qc = t;
}

bool gram_f32_any(const Common& c, int which) {
  return c.mixed && c.chol && qr_class(which ? c.nmax : c.mmax, c.lmax) >= 2;
}

hipError_t launch_gram_f32(Prob* probs, const Common& c, int which, hipStream_t s) {
  const dim3 gg(grid_for(c, TK_GRAM)), gq(grid_for(c, which ? TK_QAPN : TK_QAPM));
  const dim3 gs((c.nprob + 63) / 64);
  hipError_t e = hipSuccess;
  for (int pass = 0; pass < 2 && e == hipSuccess; ++pass) {
    if (which) {
      TEBD_LAUNCH("k_gram_f32<1>", k_gram_f32<1>, gg, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd, pass);
      TEBD_LAUNCH("k_chol_f32<1>", k_chol_f32<1>, dim3(c.nprob), dim3(1024), 0, s, probs, pass);
      TEBD_LAUNCH("k_qapply_f32<1>", k_qapply_f32<1>, gq, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd);
      TEBD_LAUNCH("k_qswap_f32<1>", k_qswap_f32<1>, gs, dim3(64), 0, s, probs, c.nprob);
    } else {
      TEBD_LAUNCH("k_gram_f32<0>", k_gram_f32<0>, gg, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd, pass);
      TEBD_LAUNCH("k_chol_f32<0>", k_chol_f32<0>, dim3(c.nprob), dim3(1024), 0, s, probs, pass);
      TEBD_LAUNCH("k_qapply_f32<0>", k_qapply_f32<0>, gq, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd);
      TEBD_LAUNCH("k_qswap_f32<0>", k_qswap_f32<0>, gs, dim3(64), 0, s, probs, c.nprob);
    }
    e = hipGetLastError();
  }
  return e;
}

}  // namespace tebd
