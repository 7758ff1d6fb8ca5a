// Householder QR by one workgroup (qr_core) and the pivot order shared by
// every pivoted QR.
#pragma once

#include "zdev.hpp"

namespace tebd {

// Householder QR of a rows x l column-major matrix (ld = rows), in place,
// followed by the explicit thin Q (backward accumulation).  Reflector j is
// H_j = I - 2 u u^H with ||u|| = 1, u supported on rows >= j, chosen so that
// H_j x = beta e_j with beta = -phase(x_j) ||x||; a zero column gives H_j = I.
// With want_r the l x l upper factor (column-major) is written to P.Rb first.
//
// qr_core serves the two larger size classes: problems with
// (l + 2) rows <= kLdsElems keep the whole matrix in LDS; larger ones work
// on the matrix in global memory (L2-resident) with one wavefront per
// trailing column, the column held in registers between its dot product and
// its update when it has at most 64 * kRegRows rows left.  The small
// problems that dominate a TEBD sweep run register-resident (k_qr_reg).
constexpr int kLdsElems = 9600;  // complex elements of LDS a workgroup may claim (150 KiB)
constexpr int kRegRows = 16;

// Size classes of the batched QR, by (rows, l): 0 and 1 are register-
// resident (512 threads with 8 rows per lane, 1024 threads with 12), 2 keeps
// the matrix in LDS (1024 threads), 3 works on global memory.  The class
// index never decreases when rows or l grow, so a box of sizes
// [rmin, rmax] x [lmin, lmax] reaches exactly the classes between
// qr_class(rmin, lmin) and qr_class(rmax, lmax).
constexpr int kRegGroupMax = 32;  // lanes per column of the register classes

__host__ __device__ __forceinline__ int reg_group(int nt, int l) {
  int lp2 = 1;
  while (lp2 < l) lp2 <<= 1;
  const int g = nt / lp2;
  return g > kRegGroupMax ? kRegGroupMax : g;
}

__host__ __device__ __forceinline__ bool qr_reg_fits(int nt, int rpl, int rows, int l) {
  if (l < 1 || l > kMaxL) return false;
  const int g = reg_group(nt, l);
  return g >= 1 && rows <= g * rpl;
}

__host__ __device__ __forceinline__ int qr_class(int rows, int l) {
  if (qr_reg_fits(512, 8, rows, l)) return 0;
  if (qr_reg_fits(1024, 12, rows, l)) return 1;
  if (int64_t(l + 2) * rows <= kLdsElems) return 2;
  return 3;
}

// Route bits (kGram*) of a problem with sketches m x l and n x l.  queue: the
// tile queue is open to it (in a sweep from size class 2 on); first: the first QR tries the Gram.  With FP32
// products (mixed) the range finder's QRs of classes 2 and 3 take
// launch_gram_f32 and the others the Householder kernels; the other bits
// then only serve the QR of B^H.
__host__ __device__ __forceinline__ int gram_bits(int m, int n, int l, bool queue, bool first,
                                                  bool mixed, bool sweep) {
  int b = first && (l > kGramFirstMinL || qr_class(m, l) >= 2) ? kGramFirst : 0;
  if (queue && gram_queue_size(m, l) && (!sweep || qr_class(m, l) >= 2)) b |= kGramTileM;
  if (queue && gram_queue_size(n, l) && (!sweep || qr_class(n, l) >= 2)) b |= kGramTileN;
  if (mixed && qr_class(m, l) >= 2) b |= kGramF32M;
  if (mixed && qr_class(n, l) >= 2) b |= kGramF32N;
  return b;
}

// y_c[j0..rows) -= 2 u (u^H y_c) for one column, by one wavefront.  Rows
// below `skip` are treated as zero on input (they held R entries).
template <int REG>
__device__ __forceinline__ void reflect_column(const zt* __restrict__ u, zt* yc, int j0, int skip,
                                               int rows, int lane, double* nrm_out = nullptr) {
  double nn = 0.0;  // sum |y_c[r]|^2 over r > j0 after the update
  const int nr = rows - j0;
  double dr = 0.0, di = 0.0;
  if (REG > 0 && nr <= 64 * REG) {
    zt cache[REG > 0 ? REG : 1];
#pragma unroll
    for (int i = 0; i < REG; ++i) {
      const int r = j0 + lane + 64 * i;
      cache[i] = (r < rows && r >= skip) ? yc[r] : make_double2(0.0, 0.0);
      if (r < rows) {
        const zt t = zcmul(u[r], cache[i]);
        dr += t.x;
        di += t.y;
      }
    }
    dr = wave_sum(dr);
    di = wave_sum(di);
    const zt d2 = make_double2(2.0 * dr, 2.0 * di);
#pragma unroll
    for (int i = 0; i < REG; ++i) {
      const int r = j0 + lane + 64 * i;
      if (r < rows) {
        const zt v = zsub(cache[i], zmul(u[r], d2));
        yc[r] = v;
        if (r > j0) nn += zabs2(v);
      }
    }
  } else {
    for (int r = j0 + lane; r < rows; r += 64) {
      if (r < skip) continue;
      const zt t = zcmul(u[r], yc[r]);
      dr += t.x;
      di += t.y;
    }
    dr = wave_sum(dr);
    di = wave_sum(di);
    const zt d2 = make_double2(2.0 * dr, 2.0 * di);
    for (int r = j0 + lane; r < rows; r += 64) {
      const zt old = r < skip ? make_double2(0.0, 0.0) : yc[r];
      const zt v = zsub(old, zmul(u[r], d2));
      yc[r] = v;
      if (r > j0) nn += zabs2(v);
    }
  }
  if (nrm_out) {
    nn = wave_sum(nn);
    if (lane == 0) *nrm_out = nn;
  }
}

// Pivot order key of a remaining column: larger for a larger trailing norm
// v; norms that agree to 2^-36 relative count as equal, and then the lower
// position wins.  0 (no candidate) for a NaN norm.  The low byte carries a
// payload (the group of the register QR).  One 64-bit maximum picks the
// pivot, and the norm it returns is v to 2^-36 relative.
__device__ __forceinline__ unsigned long long pivot_key(double v, int pos, int payload) {
  if (!(v >= 0.0)) return 0ull;
  const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(v));
  return (1ull << 63) | (b & 0x7FFFFFFFFFFF0000ull) |
         (static_cast<unsigned long long>(255 - pos) << 8) | static_cast<unsigned>(payload);
}
__device__ __forceinline__ double pivot_key_norm(unsigned long long k) {
  return __longlong_as_double(static_cast<long long>(k & 0x7FFFFFFFFFFF0000ull));
}
__device__ __forceinline__ int pivot_key_pos(unsigned long long k) {
  return 255 - static_cast<int>((k >> 8) & 0xff);
}
__device__ __forceinline__ unsigned long long key_max(unsigned long long a, unsigned long long b) {
  return a > b ? a : b;
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ unsigned long long key_dpp(unsigned long long k) {
  return static_cast<unsigned long long>(
      __double_as_longlong(dpp_move<CTRL, ROW_MASK>(__longlong_as_double(static_cast<long long>(k)))));
}
// Wavefront maximum of keys (uniform result): the row steps of
// wave_max_nonneg, masked-off rows reading 0 (no candidate).
__device__ __forceinline__ unsigned long long key_wave_max(unsigned long long k) {
  k = key_max(k, key_dpp<0xb1>(k));
  k = key_max(k, key_dpp<0x4e>(k));
  k = key_max(k, key_dpp<0x141>(k));
  k = key_max(k, key_dpp<0x140>(k));
  k = key_max(k, key_dpp<0x142, 0xa>(k));
  k = key_max(k, key_dpp<0x143, 0xc>(k));
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(k & 0xffffffffu), 63));
  const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(k >> 32), 63));
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}
__device__ __forceinline__ unsigned long long key_max_xor(unsigned long long k, int off) {
  const double o = __shfl_xor(__longlong_as_double(static_cast<long long>(k)), off, 64);
  const unsigned long long ok = static_cast<unsigned long long>(__double_as_longlong(o));
  return ok > k ? ok : k;
}

// Column pivoting for the range-finder QRs of Alg. 1: before step j the
// remaining column with the largest trailing norm (pivot_key order) is
// swapped into place, and the factorisation stops at the first j >= 1 whose
// pivot norm |R_jj| is <= kRankTol |R_00|.  The kept rank r replaces the
// sketch width l of the problem, so later products and the small SVD work on
// the numerical range only.
//
// Work split: column c belongs to wavefront c mod NW.  Step j is prepared by
// the owner of column j alone (pivot search, swap, reflector), published in
// a double-buffered LDS vector, and applied by every wavefront to its own
// trailing columns, which also yields their new trailing norms (double-
// buffered, so the next pivot search reads a stable copy).  One barrier per
// step, two with pivoting; the thin Q is accumulated the same way backwards.
constexpr double kRankTol = 1e-13;

template <int NT, int REG>
__device__ __forceinline__ int qr_core(zt* Y, int rows, int l, zt* u_s /* 2 * rows */,
                                       zt* rdiag, zt* Rb, bool piv, bool allow_stop,
                                       int32_t* perm /* l, or nullptr */,
                                       double* nrm /* 2 * kMaxL */, int* sh_i) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int NW = NT / 64;
  int rank = l;
  double best00 = 0.0;  // squared pivot norm of step 0
  if (piv) {
    for (int c = wave; c < l; c += NW) {
      double s = 0.0;
      for (int r = lane; r < rows; r += 64) s += zabs2(Y[size_t(c) * rows + r]);
      s = wave_sum(s);
      if (lane == 0) nrm[c] = s;
    }
  }
  for (int j = 0; j < l; ++j) {
    double* ncur = nrm + (j & 1) * kMaxL;
    double* nnext = nrm + ((j + 1) & 1) * kMaxL;
    zt* u = u_s + (j & 1) * rows;
    if (piv) __syncthreads();  // trailing norms of step j-1 are complete
    if (wave == (j % NW)) {
      int stop = 0;
      if (piv) {
        unsigned long long bk = 0ull;
        for (int c = j + lane; c < l; c += 64) {
          const unsigned long long k = pivot_key(ncur[c], c, 0);
          bk = k > bk ? k : bk;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) bk = key_max_xor(bk, off);
        const int bi = bk ? pivot_key_pos(bk) : j;
        const double best = pivot_key_norm(bk);  // |R_jj|^2 to 2^-36
        if (j == 0) best00 = best;
        if (allow_stop && j > 0 && !(best > kRankTol * kRankTol * best00)) stop = 1;
        if (!stop && bi != j) {
          zt* ya = Y + size_t(j) * rows;
          zt* yb = Y + size_t(bi) * rows;
          for (int r = lane; r < rows; r += 64) {
            const zt t = ya[r];
            ya[r] = yb[r];
            yb[r] = t;
          }
          if (perm && lane == 0) {
            const int32_t t = perm[j];
            perm[j] = perm[bi];
            perm[bi] = t;
          }
        }
      }
      if (!stop) {
        zt* yj = Y + size_t(j) * rows;
        double s = 0.0;
        for (int r = j + 1 + lane; r < rows; r += 64) s += zabs2(yj[r]);
        s = wave_sum(s);
        const zt alpha = yj[j];
        const double aa = sqrt(zabs2(alpha));
        const double xnorm = sqrt(aa * aa + s);
        zt beta = make_double2(0.0, 0.0), v0 = make_double2(0.0, 0.0);
        double vinv = 0.0;  // 1 / ||x - beta e_j||
        if (xnorm > 0.0) {
          const zt ph = aa > 0.0 ? zscale(alpha, 1.0 / aa) : make_double2(1.0, 0.0);
          beta = zscale(ph, -xnorm);
          v0 = zsub(alpha, beta);
          vinv = 1.0 / sqrt(2.0 * xnorm * (xnorm + aa));
        }
        for (int r = j + lane; r < rows; r += 64) {
          const zt uu = zscale(r == j ? v0 : yj[r], vinv);
          u[r] = uu;
          yj[r] = uu;
        }
        if (lane == 0) rdiag[j] = beta;
      }
      if (lane == 0) sh_i[j & 1] = stop;
    }
    __syncthreads();  // reflector j (or the stop decision) is published
    if (sh_i[j & 1]) {
      rank = j;
      break;
    }
    for (int c = j + 1 + ((wave - (j + 1) % NW + NW) % NW); c < l; c += NW)
      reflect_column<REG>(u, Y + size_t(c) * rows, j, j, rows, lane, piv ? nnext + c : nullptr);
  }
  __syncthreads();
  if (Rb) {
    for (int e = tid; e < rank * rank; e += NT) {
      const int c = e / rank, i = e - c * rank;
      zt v;
      if (i < c)
        v = Y[size_t(c) * rows + i];
      else if (i == c)
        v = rdiag[c];
      else
        v = make_double2(0.0, 0.0);
      Rb[e] = v;
    }
    __syncthreads();
  }
  // Q = H_0 H_1 ... H_{r-1} [I; 0], accumulated from the last reflector: the
  // owner of column j publishes u_j and turns its column into H_j e_j, then
  // every wavefront applies H_j to its columns c > j (row j treated as 0).
  for (int j = rank - 1; j >= 0; --j) {
    zt* u = u_s + (j & 1) * rows;
    if (wave == (j % NW)) {
      zt* yj = Y + size_t(j) * rows;
      for (int r = j + lane; r < rows; r += 64) u[r] = yj[r];
      const zt uj = yj[j];
      for (int r = lane; r < rows; r += 64) {
        zt v = make_double2(0.0, 0.0);
        if (r >= j) {
          v = zscale(zmul(r == j ? uj : yj[r], zconj(uj)), -2.0);
          if (r == j) v.x += 1.0;
        }
        yj[r] = v;
      }
    }
    __syncthreads();
    for (int c = j + 1 + ((wave - (j + 1) % NW + NW) % NW); c < rank; c += NW)
      reflect_column<REG>(u, Y + size_t(c) * rows, j, j + 1, rows, lane);
  }
  __syncthreads();
  return rank;
}

}  // namespace tebd
