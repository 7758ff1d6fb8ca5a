// Gram-based QR of the range finder's large sketches (QR classes 2 and 3)
// where its products run in FP32: two passes of G = Y^H Y, G = L L^H,
// Y <- Y L^-H (into Qc, then Qc and Y trade places).
//
// Its sums keep one fixed order, and of each complex product the same real
// products are fused (zmul_fixed: left to the compiler, copies of one unrolled
// loop choose differently).  An FP32 product rounds Q first, so a last bit of Q
// that differs flips a rounding of 6e-8 here and there, and one flip moves the
// truncated matrix by 1e-9 to 7e-8 (measured, 900 x 700 to 1024^2, l = 74 to
// 110; 2 matrices in 100): another order or rounding of the FP64 sums gives
// results that agree to the FP32 products' precision only.  Elsewhere rounding differences stay
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

// a b and a conj(b), the second real product of each sum rounded on its own.
__device__ __forceinline__ zt zmul_fixed(zt a, zt b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ zt zmul_conj_fixed(zt a, zt b) {
  return make_double2(fma(a.x, b.x, a.y * b.y), fma(a.y, b.x, -(a.x * b.y)));
}

using CfgGram = ZCfg<kSketchTileM, kSketchTileN, 16, 2, 2>;

// G = Y^H Y into C (l x l column-major), the 16 x 16 tiles of the lower
// triangle, all that the factorisation reads: a wavefront each, operands
// straight from memory kAhead slabs of 16 rows ahead (a 32 x 32 tile takes
// four of the queue's wavefronts).  The sums run over the rows in order, four to a
// matrix-core step, as in zgemm_tile.  Eight 1024 x 74 sketches: 108 us
// through LDS with a barrier per slab, 96 us so (columns 16 KB apart share a
// cache channel; 26 us of it is matrix-core time).  In the second pass only the
// problems whose first pass succeeded take part.
constexpr int kAhead = 4;

template <int WHICH>
__global__ __launch_bounds__(256) void k_gram_f32(Prob* probs, const int32_t* offs, int nprob,
                                                  int tebd, int pass) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4, w = wave_id();
  for_each_tile<TK_GRAM>(probs, offs, nprob, tebd, [&](Prob& P, int, int, int m0, int n0, int) {
    if (!(P.chol & (WHICH ? kGramF32N : kGramF32M)) || (pass && !P.chol_ok)) return;
    const int rows = WHICH ? P.n : P.m, l = P.l;
    const int r0 = m0 + (w >> 1) * 16, c0 = n0 + (w & 1) * 16;
    if (c0 > r0 || r0 >= l) return;
    const zt* Y = WHICH ? P.Yt : P.Y;
    const zt* pa = Y + size_t(r0 + ti < l ? r0 + ti : l - 1) * rows;
    const zt* pb = Y + size_t(c0 + ti < l ? c0 + ti : l - 1) * rows;
    auto load = [&](int k0, zt (&a)[4], zt (&b)[4]) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = k0 + 4 * s + tk, kc = k < rows ? k : rows - 1;
        a[s] = pa[kc];
        b[s] = pb[kc];
        if (k >= rows) a[s] = b[s] = make_double2(0.0, 0.0);
      }
    };
    v4d re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    zt a[kAhead][4], b[kAhead][4];
#pragma unroll
    for (int p = 0; p < kAhead; ++p) load(16 * p, a[p], b[p]);
    for (int k0 = 0; k0 < rows; k0 += 16 * kAhead) {
#pragma unroll
      for (int p = 0; p < kAhead; ++p) {  // (slabs beyond the rows are zeros)
#pragma unroll
        for (int s = 0; s < 4; ++s) {  // conj(a) b
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p][s].x, b[p][s].x, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p][s].x, b[p][s].y, im, 0, 0, 0);
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p][s].y, b[p][s].y, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[p][s].y, b[p][s].x, im, 0, 0, 0);
        }
        load(k0 + 16 * (p + kAhead), a[p], b[p]);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = r0 + tk + 4 * r, col = c0 + ti;
      if (row < l && col < l) P.C[row + size_t(col) * l] = make_double2(re[r], im[r]);
    }
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
// used), then X = R^-1 = (L^-1)^H, upper triangular, into J.
//
// Up to kCholLdsL columns: the Gram in registers, element (i, k) with thread
// (i mod 32, k mod 32), the scaled column of a step broadcast through LDS (one
// barrier a step); L goes to LDS by rows for the inverse.  There column c of
// L^-1 by forward substitution, four columns per wavefront, 16 lanes each: the
// sum of row i adds 64 products in a binary tree over the columns k mod 64
// (lane u holds k = 4u ... 4u + 3), so LDS holds a row with those four 16
// apart, and no read conflicts.  l = 74, eight problems: 250 us column by
// column in LDS and with a wavefront per column, 84 us so.
__device__ __forceinline__ int chol_slot(int k) {  // place of column k in a row
  const int u = (k >> 2) & 15, m = k & 3;
  return k < 64 ? 16 * m + u : 64 + 8 * m + u;
}
__device__ __forceinline__ int chol_ld(int l) { return l > 64 ? 97 : 65; }
static_assert(kCholLdsL <= 96, "chol_slot: two blocks of 64 and 32 columns");

struct CholShared {
  zt L[kCholLdsL * (kCholLdsL + 1)];
  zt col[2][kCholLdsL];
  double diag[kCholLdsL];
  int refused[2];  // verdict on the pivots of the even and the odd steps
};

// False when a pivot is refused (uniform).  sh.refused is zero on entry.  Step j
// writes its verdict before its barrier and everyone reads it after; the slot
// is next written in step j + 2, past the barrier of step j + 1.
__device__ __forceinline__ bool chol_factor(const zt* G, int l, double dmax, CholShared& sh) {
  constexpr int NB = kCholLdsL / 32;
  const int tid = threadIdx.x, ti = tid & 31, tk = tid >> 5, ld = chol_ld(l);
  zt g[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int i = ti + 32 * a, k = tk + 32 * b;
      g[a][b] = zload_if(i < l && k <= i, G + i + size_t(k) * l);
    }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    for (int jt = 0; jt < 32; ++jt) {
      const int j = 32 * b + jt;
      if (j >= l) break;
      zt* col = sh.col[j & 1];
      if (tk == jt) {  // the half wavefront that holds column j
        const double d = __shfl(g[b][b].x, (tid & 32) | jt, 64);
        if (!(d > kCholTol * dmax) || !isfinite(d)) {
          sh.refused[j & 1] = 1;
        } else {
          const double root = sqrt(d), inv = 1.0 / root;
          if (ti == jt) sh.diag[j] = root;
#pragma unroll
          for (int a = b; a < NB; ++a) {
            const int i = ti + 32 * a;
            if (i > j && i < l) {
              const zt v = zscale(g[a][b], inv);
              col[i] = v;
              sh.L[i * ld + chol_slot(j)] = v;
            }
          }
        }
      }
      __syncthreads();
      if (sh.refused[j & 1]) return false;
#pragma unroll
      for (int c = b; c < NB; ++c) {  // rows and columns beyond j (the others are done with)
        const zt lkj = col[tk + 32 * c];
#pragma unroll
        for (int a = c; a < NB; ++a) {
          const zt lij = col[ti + 32 * a];
          g[a][c] = zsub(g[a][c], zmul_conj_fixed(lij, lkj));
        }
      }
    }
  }
  __syncthreads();
  return true;
}

__device__ __forceinline__ void chol_inverse(zt* X, int l, const CholShared& sh) {
  const int lane = threadIdx.x & 63, u = lane & 15, ld = chol_ld(l);
  for (int c0 = 4 * wave_id(); c0 < l; c0 += 64) {
    const int c = c0 + (lane >> 4);
    zt x[2][4];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int m = 0; m < 4; ++m) x[q][m] = make_double2(0.0, 0.0);
#pragma unroll
    for (int qi = 0; qi < 2; ++qi) {
      const int from = c0 > 64 * qi ? (c0 - 64 * qi) >> 2 : 0;
      for (int v = from; v < 16 && 64 * qi + 4 * v < l; ++v) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
          const int i = 64 * qi + 4 * v + mi;
          if (i >= l) break;
          const zt* row = sh.L + i * ld + u;
          double sr[4], si[4];
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            sr[m] = 0.0;
            si[m] = 0.0;
#pragma unroll
            for (int q = 0; q <= qi; ++q) {
              const int k = 64 * q + 4 * u + m;
              zt lik = row[q == 0 ? 16 * m : 64 + 8 * m];
              if (k >= i) lik = make_double2(0.0, 0.0);
              const zt t = zmul_fixed(lik, x[q][m]);
              sr[m] += t.x;
              si[m] += t.y;
            }
          }
          const double tr = group_sum((sr[0] + sr[1]) + (sr[2] + sr[3]), 16);
          const double ts = group_sum((si[0] + si[1]) + (si[2] + si[3]), 16);
          const double lii = sh.diag[i];
          const zt xi = i == c ? make_double2(1.0 / lii, 0.0) : make_double2(-tr / lii, -ts / lii);
          if (u == v && i >= c) x[qi][mi] = xi;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int i = 64 * q + 4 * u + m;
        if (i < l && c < l)
          X[c + size_t(i) * l] = i >= c ? zconj(x[q][m]) : make_double2(0.0, 0.0);
      }
  }
}

// Wider ones work on the Gram in global memory, a wavefront per column of the
// inverse (lane t keeps rows t, t + 64, ...).
template <int WHICH>
__global__ __launch_bounds__(1024) void k_chol_f32(Prob* probs, int pass) {
  Prob& P = probs[blockIdx.x];
  const int l = P.l, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool elig = l > 0 && (P.chol & (WHICH ? kGramF32N : kGramF32M)) && (pass == 0 || P.chol_ok);
  if (!elig) {
    if (tid == 0 && pass == 0) P.chol_ok = 0;
    return;
  }
  __shared__ CholShared sh;
  __shared__ double dmax_s;
  __shared__ int fail_s;
  const bool in_lds = l <= kCholLdsL;
  zt* G = P.C;
  if (wave == 0) {
    double dm = 0.0;
    for (int j = lane; j < l; j += 64) {
      const double d = G[j + size_t(j) * l].x;
      dm = fmax(dm, d);
    }
    dm = wave_max(dm);
    if (lane == 0) {
      dmax_s = dm;
      fail_s = !(dm > 0.0) || !isfinite(dm);
      sh.refused[0] = sh.refused[1] = 0;
    }
  }
  __syncthreads();
  bool refused = fail_s != 0;
  __syncthreads();  // fail_s is read before a step writes it
  if (in_lds && !refused) refused = !chol_factor(G, l, dmax_s, sh);
  for (int j = 0; j < l && !in_lds && !refused; ++j) {
    if (tid == 0) {
      const double d = G[j + size_t(j) * l].x;
      if (!(d > kCholTol * dmax_s) || !isfinite(d))
        fail_s = 1;
      else
        G[j + size_t(j) * l] = make_double2(sqrt(d), 0.0);
    }
    __syncthreads();
    refused = fail_s != 0;  // (two barriers before the next step's write)
    if (refused) break;
    const double inv = 1.0 / G[j + size_t(j) * l].x;
    for (int i = j + 1 + tid; i < l; i += 1024) G[i + size_t(j) * l] = zscale(G[i + size_t(j) * l], inv);
    __syncthreads();
    const int nt = l - j - 1;
    for (int e = tid; e < nt * nt; e += 1024) {
      const int kk = e / nt, ii = e - kk * nt;
      if (ii < kk) continue;
      const int k = j + 1 + kk, i = j + 1 + ii;
      const zt lij = G[i + size_t(j) * l], lkj = G[k + size_t(j) * l];
      G[i + size_t(k) * l] = zsub(G[i + size_t(k) * l], zmul_conj_fixed(lij, lkj));
    }
    __syncthreads();
  }
  if (refused) {
    if (tid == 0) {
      P.chol_ok = 0;
      P.flags |= TEBD_DEV_QR_FALLBACK;
    }
    return;
  }
  if (in_lds) {
    chol_inverse(P.J, l, sh);
    if (tid == 0) P.chol_ok = 1;
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
          const zt t = zmul_fixed(lik, xr[q]);
          sr += t.x;
          si += t.y;
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
