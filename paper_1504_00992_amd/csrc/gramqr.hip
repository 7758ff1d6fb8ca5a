// Gram-based QR of the sketches (the QR steps of Alg. 1 and of Sec. IV step
// i-ii; Tamascelli, Rosenbach, Plenio, arXiv:1504.00992, leave the method
// open): G = Y^H Y, G = L L^H, Q = Y L^-H, R = L^H.
//
// Why it may be used.  The columns of a power iteration's sketch A^H Q (or
// A Q~, or B^H) are graded like the singular values, kappa(Y) is up to 1e13,
// and a Gram matrix squares it; but Cholesky does not see a scaling of the
// columns (its rounding errors are relative to sqrt(G_ii G_jj)), and scaled
// to unit length those columns are nearly orthogonal, because Q already
// is a basis ordered by singular value.  Measured over spin-boson, Ising and
// XX evolutions and matrices of exponential spectra, the smallest scaled
// pivot d_j / G_jj (the squared sine between a column and those before it) is
// 3e-3 in the first power iteration and 0.27 or more later.  One pass then
// leaves Q orthonormal to about eps / (smallest pivot).  So the passes check
// that ratio: below kRelRefuse the Householder QR takes the problem, and where
// the columns must be orthonormal to rounding (the last basis, B^H) a second
// pass follows below kRelStrict.
// The QR of Y0 = A Omega has no such grading: it accepts kappa(Y0) up to
// about 1e7 (kAbsRefuse, against the largest diagonal entry).
//
// Cost.  A Householder QR of 100 x 32 is a chain of 32 dependent steps of a
// whole workgroup (2400 cycles each, 45 us with the accumulation of Q); here
// the chain is the factorisation of the 16 x 16 diagonal blocks, one
// wavefront each, 4 columns at a time, and everything else is matrix-core
// products.
#include <cfloat>

#include "householder.hpp"
#include "kinds.hpp"
#include "loaders.hpp"

namespace tebd {

constexpr double kRelRefuse = 1e-10;
constexpr double kRelStrict = 0.25;
constexpr double kAbsRefuse = 1e-14;

// A 16 x 16 complex tile in the result layout of v_mfma_f64_16x16x4: element
// r of lane t is entry (t / 16 + 4 r, t % 16).
struct ZTile {
  v4d re, im;
};
__device__ __forceinline__ ZTile tile_zero() {
  return {v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}};
}
// c += a b for one k-step of 4 (lane t: a = A[t % 16][t / 16], b = B[t / 16][t % 16])
__device__ __forceinline__ void tile_mma(ZTile& c, zt a, zt b) {
  c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, c.re, 0, 0, 0);
  c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, c.im, 0, 0, 0);
  c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, c.re, 0, 0, 0);
  c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, c.im, 0, 0, 0);
}
// Row-major storage with leading dimension ld.
__device__ __forceinline__ ZTile tile_load(const zt* p, int ld) {
  const int lane = threadIdx.x & 63;
  ZTile t;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const zt v = p[((lane >> 4) + 4 * r) * ld + (lane & 15)];
    t.re[r] = v.x;
    t.im[r] = v.y;
  }
  return t;
}
__device__ __forceinline__ void tile_store(zt* p, int ld, const ZTile& t) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    p[((lane >> 4) + 4 * r) * ld + (lane & 15)] = make_double2(t.re[r], t.im[r]);
}
// Operands of k-step s from row-major tiles: A[r][k] and B[k][c].
__device__ __forceinline__ zt op_a(const zt* p, int ld, int s) {
  const int lane = threadIdx.x & 63;
  return p[(lane & 15) * ld + 4 * s + (lane >> 4)];
}
__device__ __forceinline__ zt op_b(const zt* p, int ld, int s) {
  const int lane = threadIdx.x & 63;
  return p[(4 * s + (lane >> 4)) * ld + (lane & 15)];
}
__device__ __forceinline__ zt zneg(zt a) { return make_double2(-a.x, -a.y); }

// Verdict on the pivot d of a column whose Gram diagonal is g (the largest
// one is gmax): bit 0 refused, bit 1 below kRelStrict.  first: refused by size
// against the largest diagonal entry instead of its own.
__device__ __forceinline__ int pivot_verdict(double d, double g, bool first, double gmax) {
  const bool ok = d > (first ? kAbsRefuse * gmax : kRelRefuse * g) && d > DBL_MIN && d <= DBL_MAX;
  return (ok ? 0 : 1) | (d >= kRelStrict * g ? 0 : 2);
}

// Whether a refused sketch sets TEBD_DEV_QR_FALLBACK: in any QR, on the tile
// queue or by a workgroup, in the size classes 2 and 3.
__device__ __forceinline__ bool refusal_reported(const Prob& P, int rows, int mode) {
  return !(mode & QRM_QUIET) && qr_class(rows, P.l1) >= 2;
}

// One wavefront: G = L L^H of a 16 x 16 Hermitian tile (both triangles valid)
// by Gaussian elimination on [G | I], both in one array: step j subtracts m_i
// times row j from the rows i > j, m_i = conj(G_ji) / d_j, d_j = G_jj; columns
// k > j of a row belong to G, columns k < j to the growing inverse, each scaled
// by d_k, and column j becomes -conj(G_ji) = -m_i d_j (its old entries are
// dropped, the pivot row holds 1 there).  On return column k < i of row i holds
// d_k times the unit-lower inverse, the diagonal the pivots and columns k > i
// the pivot rows.
// The inverse takes nothing from the lower triangle of G, which differs from
// the upper one by its rounding, u |G|: with it, X R = I held to u / (smallest
// scaled pivot) only, and so did the QR of B^H (measured with pivots of 5e-6:
// singular values off by 4e-12 s_1, 1e-15 so, for 40 cycles a step).
// A step is bound by its instructions (five cycles each for one wavefront, a
// branch about twenty) and the LDS round trip, about 480 cycles, so it has no
// branch but the loop's own and leaves tests and scalings to the end.  One
// wavefront does a whole tile: with the rows spread over eight, a barrier per
// step and the multipliers by readlane, a step took 900.  Row j goes through
// 16 entries of LDS, in order within a wavefront; it holds the multipliers
// too, conj(G_ij).
// n: columns from n on are the identity's.
__device__ __forceinline__ void chol_tile(ZTile& w, zt* buf, int n) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4;
#pragma unroll
  for (int rj = 0; rj < 4; ++rj) {
    if (4 * rj >= n) break;
#pragma unroll 1
    for (int tj = 0; tj < 4; ++tj) {
      const int j = 4 * rj + tj;
      if (tk == tj) buf[ti] = make_double2(w.re[rj], w.im[rj]);
      asm volatile("" ::: "memory");
      zt rv = buf[ti];
      const double d = buf[j].x;
      zt m[4];
#pragma unroll
      for (int r = rj; r < 4; ++r) m[r] = buf[tk + 4 * r];
      asm volatile("" ::: "memory");
      const double inv = rcp_pos(d);
      const bool below = tk > tj;  // rows of register rj up to j stay
      const double keep = ti == j ? 0.0 : 1.0;
      const double rj_keep = ti == j && below ? 0.0 : 1.0;
      rv.x = ti == j ? 1.0 : rv.x * inv;
      rv.y = ti == j ? 0.0 : rv.y * inv;
      const zt rj_v = make_double2(below ? rv.x : 0.0, below ? rv.y : 0.0);
#pragma unroll
      for (int r = rj; r < 4; ++r) {  // w -= conj(m) rv, in column j w = -conj(m)
        const zt v = r == rj ? rj_v : rv;
        const double k = r == rj ? rj_keep : keep;
        w.re[r] = fma(-m[r].x, v.x, fma(-m[r].y, v.y, w.re[r] * k));
        w.im[r] = fma(-m[r].x, v.y, fma(m[r].y, v.x, w.im[r] * k));
      }
    }
  }
}

// The end of chol_tile: L^-1 into w, and R = L^H into rb (or null;
// column-major, ld rld, rows and columns below n only).  gd: the Gram
// diagonal of the tile's columns (LDS).  Returns the verdict on the pivots.
__device__ __forceinline__ int chol_tile_end(ZTile& w, int j0, int n, const double* gd, bool first,
                                             double gmax, zt* rb, int rld) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4;
  int bad = 0;
  double dk = 0.0;  // the pivot of this lane's column
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (tk + 4 * r == ti) dk = w.re[r];
  dk += __shfl_xor(dk, 16, 64);
  dk += __shfl_xor(dk, 32, 64);
  const double ik = rcp_pos(dk);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = tk + 4 * r;
    // d_i sits in the lane of column i of this 16-lane row
    const double d = __shfl(w.re[r], (lane & 48) | i, 64);
    const double rs = rsqrt_pos(d);
    if (j0 + i < n) bad |= pivot_verdict(d, gd[i], first, gmax);
    if (rb && j0 + i < n && j0 + ti < n)
      rb[size_t(j0 + ti) * rld + j0 + i] =
          ti > i ? make_double2(w.re[r] * rs, w.im[r] * rs) : make_double2(ti == i ? d * rs : 0.0, 0.0);
    const double f = rs * ik;
    w.re[r] = ti < i ? w.re[r] * f : ti == i ? rs : 0.0;
    w.im[r] = ti < i ? w.im[r] * f : 0.0;
  }
  const uint64_t refused = __ballot(bad & 1), loose = __ballot(bad & 2);
  return (refused ? 1 : 0) | (loose ? 2 : 0);
}

// Whole workgroup of NW wavefronts: G (nb x nb 16 x 16 blocks, block-lower
// part, row-major, leading dimension ld; rows beyond n hold the identity) =
// L L^H, replaced by X = L^-1 (block-lower; the diagonal blocks' upper parts
// are zero); gd: its diagonal.  Right-looking: block column kb is factored and
// inverted by wavefront 0, its panel L_ik = G_ik X_kk^H goes to
// pn (nb blocks of 16 x 17), row kb of the inverse is finished, and the rows
// below take the update of both the trailing matrix and the inverse.
// Wavefront 0 updates only the next diagonal block and factors it while the
// others finish the update: the chain is the diagonal blocks and their panels.
template <int NW>
__device__ __forceinline__ int chol_invert(zt* G, int ld, int nb, zt* pn, int n, const double* gd,
                                           bool first, double gmax, zt* rb, int rld,
                                           int* sh_flags, zt* buf) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  constexpr int PL = 17, PB = 16 * PL;
  int verdict = 0;
  // step kb - 1 on block (i, j), i >= kb: D_ij -= L_ik L_jk^H (j >= kb),
  // E_ij -= L_ik X_kj (j < kb; E_ik is new)
  auto update = [&](int kb, int i, int j) {
    const int k = kb - 1;
    ZTile c = j == k ? tile_zero() : tile_load(G + size_t(i) * 16 * ld + j * 16, ld);
    const zt* li = pn + i * PB;
    const zt* q = j > k ? pn + j * PB : G + size_t(k) * 16 * ld + j * 16;
    zt a[4], b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a[s] = zneg(op_a(li, PL, s));
      b[s] = j > k ? zconj(op_a(q, PL, s)) : op_b(q, ld, s);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) tile_mma(c, a[s], b[s]);
    return c;
  };
  for (int kb = 0; kb < nb; ++kb) {
    zt* gkk = G + size_t(kb) * 16 * ld + kb * 16;
    if (wave == 0) {
      ZTile d = kb > 0 ? update(kb, kb, kb) : tile_load(gkk, ld);
      chol_tile(d, buf, n - kb * 16);
      verdict |= chol_tile_end(d, kb * 16, n, gd + kb * 16, first, gmax, rb, rld);
      tile_store(gkk, ld, d);
      if (lane == 0) *sh_flags = verdict;
    } else if (kb > 0) {
      int t = 0;
      for (int i = kb; i < nb; ++i)
        for (int j = 0; j <= i; ++j) {
          if (i == kb && j == i) continue;
          if (t++ % (NW - 1) == wave - 1)
            tile_store(G + size_t(i) * 16 * ld + j * 16, ld, update(kb, i, j));
        }
    }
    __syncthreads();
    const int flags = *sh_flags;
    if (flags & 1) return flags;
    // the panel below, and row kb of the inverse
    for (int t = wave; t < nb - 1; t += NW) {
      const int i = t < kb ? t : t + 1;
      zt* p = i > kb ? G + size_t(i) * 16 * ld + kb * 16 : G + size_t(kb) * 16 * ld + i * 16;
      zt a[4], b[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {  // L_ik = G_ik X_kk^H, X_ki = X_kk E_ki
        a[s] = op_a(i > kb ? p : gkk, ld, s);
        b[s] = i > kb ? zconj(op_a(gkk, ld, s)) : op_b(p, ld, s);
      }
      ZTile c = tile_zero();
#pragma unroll
      for (int s = 0; s < 4; ++s) tile_mma(c, a[s], b[s]);
      if (i > kb) {
        tile_store(pn + i * PB, PL, c);
        if (rb) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = i * 16 + (lane >> 4) + 4 * r, col = kb * 16 + (lane & 15);
            if (row < n) rb[size_t(row) * rld + col] = make_double2(c.re[r], -c.im[r]);
          }
        }
      } else {
        tile_store(p, ld, c);
      }
    }
    if (rb) {  // R is upper triangular
      for (int e = threadIdx.x; e < 16 * (n - kb * 16 - 16); e += NW * 64) {
        const int r = e & 15, cidx = kb * 16 + 16 + (e >> 4);
        rb[size_t(kb * 16 + r) * rld + cidx] = make_double2(0.0, 0.0);
      }
    }
    __syncthreads();
  }
  return *sh_flags;
}

// R_B = L_2^H R_1 after a second pass: conj(L_2) is in rb (row-major, so
// column-major it is R_2), R_1 in r1; the product through t.
template <int NT>
__device__ __forceinline__ void compose_r(zt* rb, const zt* r1, zt* t, int l) {
  for (int e = threadIdx.x; e < l * l; e += NT) {
    const int c = e / l, r = e - c * l;
    double sr = 0.0, si = 0.0;
    for (int k = r; k <= c; ++k) {
      const zt a = rb[size_t(k) * l + r], b = r1[size_t(c) * l + k];
      sr = fma(a.x, b.x, fma(-a.y, b.y, sr));
      si = fma(a.x, b.y, fma(a.y, b.x, si));
    }
    t[e] = make_double2(sr, si);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < l * l; e += NT) rb[e] = t[e];
  __syncthreads();
}

// --------------------------------------------------------------------------
// One wavefront: 16 rows from r0 of column block bc of Q = Y X^H.  X
// row-major (ld), block-lower, zero in the columns beyond l.  get reads Y, put
// writes Q, both in range only.
template <class Get, class Put>
__device__ __forceinline__ void apply_block(int rows, int l, int bc, int r0, const zt* X, int ld,
                                            Get&& get, Put&& put) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4;
  const int r = r0 + ti, rc = r < rows ? r : rows - 1;
  ZTile c = tile_zero();
  const zt* xr = X + size_t(bc) * 16 * ld;
#pragma unroll 2
  for (int kk = 0; kk <= bc; ++kk) {
    zt a[4], b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = kk * 16 + 4 * s + tk;
      a[s] = op_a(xr + kk * 16, ld, s);
      b[s] = get(rc, k < l ? k : l - 1);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) tile_mma(c, zconj(a[s]), b[s]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int col = bc * 16 + tk + 4 * q;
    if (col < l && r < rows) put(r, col, make_double2(c.re[q], c.im[q]));
  }
}
// All of them, in place: block bc of Q needs the blocks <= bc of Y, so the
// blocks go from the last to the first and the strip needs no second buffer.
template <class Get, class Put>
__device__ __forceinline__ void apply_strip(int rows, int l, int nb, int r0, const zt* X, int ld,
                                            Get&& get, Put&& put) {
  for (int bc = nb - 1; bc >= 0; --bc) apply_block(rows, l, bc, r0, X, ld, get, put);
}

// One wavefront: tile (bi, bj) of G = Y^H Y over the rows [ra, re), Y
// column-major with leading dimension ldy.  Lane t takes rows t / 16, 4 + t / 16,
// ... of columns 16 bi + t % 16 and 16 bj + t % 16 per 16 rows: the order of
// zgemm_tile, so that a sketch has the same Gram matrix on the tile queue.
// Columns beyond l repeat the last one (the caller masks their products).
// From LDS: the rows up to the next multiple of 16 hold zeros, no tests.
__device__ __forceinline__ ZTile gram_tile_lds(const zt* ys, int ldy, int l, int bi, int bj, int ra,
                                               int re) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4;
  const int ca = bi * 16 + ti, cb = bj * 16 + ti;
  const zt* pa = ys + (ca < l ? ca : l - 1) * ldy + tk;
  const zt* pb = ys + (cb < l ? cb : l - 1) * ldy + tk;
  ZTile c = tile_zero();
#pragma unroll 2
  for (int r = ra; r < re; r += 16) {
    zt a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = pa[r + 4 * u];
      b[u] = pb[r + 4 * u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) tile_mma(c, zconj(a[u]), b[u]);
  }
  return c;
}
// From global memory: the next 16 rows are loaded while the current ones are
// multiplied.
__device__ __forceinline__ ZTile gram_tile_glb(const zt* Y, int rows, int l, int bi, int bj, int ra,
                                               int re) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4;
  const int ca = bi * 16 + ti, cb = bj * 16 + ti;
  const zt* pa = Y + size_t(ca < l ? ca : l - 1) * rows;
  const zt* pb = Y + size_t(cb < l ? cb : l - 1) * rows;
  auto load = [&](int r, zt (&a)[4], zt (&b)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = r + 4 * u + tk;
      a[u] = zload_if(k < re, pa + k);
      b[u] = pb[k < re ? k : re - 1];
    }
  };
  ZTile c = tile_zero();
  zt a[4], b[4];
  load(ra, a, b);
  for (int r = ra; r < re; r += 16) {
    zt an[4], bn[4];
    load(r + 16, an, bn);
#pragma unroll
    for (int u = 0; u < 4; ++u) tile_mma(c, zconj(a[u]), b[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = an[u];
      b[u] = bn[u];
    }
  }
  return c;
}

// The identity in the rows and columns beyond n of block (bi, bj).
__device__ __forceinline__ void pad_identity(ZTile& c, int bi, int bj, int n) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = bi * 16 + (lane >> 4) + 4 * r, j = bj * 16 + (lane & 15);
    if (i >= n || j >= n) {
      c.re[r] = i == j ? 1.0 : 0.0;
      c.im[r] = 0.0;
    }
  }
}

// Largest of n non-negative values in LDS, in every lane.
__device__ __forceinline__ double largest_of(const double* v, int n) {
  double m = 0.0;
  for (int j = threadIdx.x & 63; j < n; j += 64) m = fmax(m, v[j]);
  return wave_max_nonneg(m);
}

// Block pair t of the block-lower triangle (row by row).
__device__ __forceinline__ void lower_pair(int t, int& bi, int& bj) {
  bi = 0;
  while (t > bi) {
    t -= bi + 1;
    ++bi;
  }
  bj = t;
}

constexpr int kGqThreads = 512, kGqWaves = kGqThreads / 64;
// Largest width whose Gram matrix a workgroup keeps in LDS (80: 104 KiB and
// the panel); wider ones live in the problem's X and W (free until the SVD).
// Where some width may be beyond that (often only a capacity), the narrow
// ones get LDS for 48 columns.
constexpr int kGqLdsBlocks = 5, kGqWideBlocks = 3;
constexpr int kGqLdsMax = 9940;  // complex elements of dynamic LDS (155 KiB)

__host__ __device__ constexpr int gq_ld(int blocks) { return 16 * blocks + 1; }
// After the Gram matrix: the panel, or the partial tiles of the depth slices
// (narrow sketches only: at most 6 tiles).
__host__ __device__ constexpr int gq_tail(int max_blocks) {
  return max_blocks * 16 * 17 > 1536 ? max_blocks * 16 * 17 : 1536;
}
// Then the sketch itself when it fits: columns of rows rounded up to 16, plus one.
__host__ __device__ inline int gq_ldy(int rows) { return ((rows + 15) & ~15) + 1; }

struct GqShared {
  double gd[kMaxL];  // Gram diagonal
  zt row[16];        // pivot row of the diagonal block
  int flags;
  int todo[kGqWaves];  // small problems their wavefront leaves to the workgroup
  int sh_i[2];
};

// The whole QR of one problem's sketch by one workgroup: Gram tiles (over
// depth slices when there are fewer tiles than wavefronts), Cholesky and
// inverse, Q.  The sketch is read once into LDS where it fits (a read of what
// another XCD wrote takes about a microsecond, so all of them are in flight
// together), else streamed twice.  A refusal (kRelRefuse) runs the
// Householder QR here, on global memory: it takes a column that vanishes or
// repeats others, which a graded sketch of revealed rank does not have, so
// this path need not be fast.
__device__ __forceinline__ void gram_qr_problem(Prob& P, int which, int mode, int lds_blocks,
                                                int lds_elems, zt* smem, GqShared& sh) {
  const int l = P.l, tid = threadIdx.x, wave = wave_id(), lane = tid & 63;
  const int rows = which ? P.n : P.m;
  zt* Y = which ? P.Yt : P.Y;
  const int nb = (l + 15) / 16;
  const bool in_lds = nb <= lds_blocks;
  const int ld = in_lds ? gq_ld(lds_blocks) : 16 * nb;
  zt* G = in_lds ? smem : P.X;
  zt* pn = smem + 16 * lds_blocks * gq_ld(lds_blocks);
  const int ys_at = 16 * lds_blocks * gq_ld(lds_blocks) + gq_tail(nb);
  const int ldy = gq_ldy(rows);
  const bool y_lds = ys_at + ldy * l <= lds_elems;
  zt* ys = smem + ys_at;
  const bool first = mode & QRM_FIRST, want_r = mode & QRM_WANT_R;
  const int ntile = nb * (nb + 1) / 2;
  // depth slices: 4 for one tile, 2 for three, else 1; of a sketch that is the
  // tile queue's elsewhere, its chunks (one or two, see kGramQueueRegRows)
  int lsl = rows < 64 || nb > 2 ? 0 : nb == 1 ? 2 : 1;
  if (P.chol & (which ? kGramTileN : kGramTileM))
    lsl = nb <= 2 && gram_chunks(rows, P.l1, gram_room(P)) > 1 ? 1 : 0;
  const int slices = 1 << lsl;
  const int chunk = (((rows + slices - 1) >> lsl) + 15) & ~15;
  bool failed = false;
  for (int pass = 0; pass < 2; ++pass) {
    if (y_lds) {
      // a wavefront takes columns wave, wave + 8, ... in pieces of 64 rows, eight
      // pieces in flight; rows up to the next multiple of 16 become zero
      const int last = rows * l - 1, rows16 = ldy - 1;
      for (int c0 = wave, r0 = 0; c0 < l;) {
        zt v[8];
        int cu = c0, ru = r0;
  #pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int e = cu * rows + ru + lane;
          v[u] = Y[e < last ? e : last];
          ru += 64;
          if (ru >= rows16) {
            ru = 0;
            cu += kGqWaves;
          }
        }
  #pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int r = r0 + lane;
          if (c0 < l && r < rows16) ys[c0 * ldy + r] = r < rows ? v[u] : make_double2(0.0, 0.0);
          r0 += 64;
          if (r0 >= rows16) {
            r0 = 0;
            c0 += kGqWaves;
          }
        }
      }
      __syncthreads();
    }
    for (int u = wave; u < ntile * slices; u += kGqWaves) {
      const int t = u >> lsl, s = u - (t << lsl);
      int bi, bj;
      lower_pair(t, bi, bj);
      const int ra = s * chunk, re = ra + chunk < rows ? ra + chunk : rows;
      ZTile c = y_lds ? gram_tile_lds(ys, ldy, l, bi, bj, ra, re)
                      : gram_tile_glb(Y, rows, l, bi, bj, ra, re);
      if (slices > 1) {
        tile_store(pn + u * 256, 16, c);
      } else {
        pad_identity(c, bi, bj, l);
        tile_store(G + size_t(bi) * 16 * ld + bj * 16, ld, c);
      }
    }
    __syncthreads();
    if (slices > 1) {
      for (int e = tid; e < ntile * 256; e += kGqThreads) {
        const int t = e >> 8, w = e & 255, i = w >> 4, j = w & 15;
        int bi, bj;
        lower_pair(t, bi, bj);
        zt v = pn[(t * slices) * 256 + w];
        for (int s = 1; s < slices; ++s) v = zadd(v, pn[(t * slices + s) * 256 + w]);
        if (bi * 16 + i >= l || bj * 16 + j >= l)
          v = make_double2(bi == bj && i == j ? 1.0 : 0.0, 0.0);
        G[size_t(bi * 16 + i) * ld + bj * 16 + j] = v;
      }
      __syncthreads();
    }
    for (int j = tid; j < 16 * nb; j += kGqThreads) sh.gd[j] = G[size_t(j) * ld + j].x;
    if (want_r && pass)  // keep R_1 while R_2 is written
      for (int e = tid; e < l * l; e += kGqThreads) P.C[e] = P.Rb[e];
    __syncthreads();
    const double gmax = first ? largest_of(sh.gd, l) : 0.0;
    zt* rb = want_r ? P.Rb : nullptr;
    const int flags = chol_invert<kGqWaves>(G, ld, nb, pn, l, sh.gd, first, gmax, rb, l, &sh.flags,
                                            sh.row);
    if (flags & 1) {
      failed = pass == 0;
      if (pass && want_r) {  // Q_1 and R_1 stand
        __syncthreads();
        for (int e = tid; e < l * l; e += kGqThreads) P.Rb[e] = P.C[e];
      }
      break;
    }
    const bool again = pass == 0 && (mode & QRM_STRICT) && (flags & 2);
    auto put = [&](int r, int k, zt v) { Y[size_t(k) * rows + r] = v; };
    const int strips = (rows + 15) >> 4;
    if (y_lds) {  // every block of a strip on its own, the deepest first
      int bc = nb - 1, st = wave;
      for (;;) {
        while (st >= strips && bc >= 0) {
          st -= strips;
          --bc;
        }
        if (bc < 0) break;
        apply_block(rows, l, bc, st * 16, G, ld, [&](int r, int k) { return ys[k * ldy + r]; }, put);
        st += kGqWaves;
      }
    } else {
      for (int st = wave; st < strips; st += kGqWaves)
        apply_strip(rows, l, nb, st * 16, G, ld,
                    [&](int r, int k) { return Y[size_t(k) * rows + r]; }, put);
    }
    if (want_r && pass) compose_r<kGqThreads>(P.Rb, P.C, P.J, l);
    if (!again) break;
    __syncthreads();
  }
  if (tid == 0 && failed && refusal_reported(P, rows, mode)) P.flags |= TEBD_DEV_QR_FALLBACK;
  if (first) {
    if (tid == 0) P.chol_ok = failed ? 0 : 1;
    return;
  }
  if (failed && (mode & QRM_LEAVE) && qr_class(rows, P.l1) < 2) {
    if (tid == 0) P.chol_ok = 0;
    return;
  }
  if (failed) {
    __syncthreads();
    zt* rdiag = smem;
    double* nrm = reinterpret_cast<double*>(smem + kMaxL);
    qr_core<kGqThreads, 0>(Y, rows, l, P.qru, rdiag, want_r ? P.Rb : nullptr, false, false,
                           nullptr, nrm, sh.sh_i);
  }
  if (want_r)
    for (int c = tid; c < l; c += kGqThreads) P.piv[c] = c;
  if (tid == 0) P.chol_ok = 1;
}

// Whether a sketch goes to the Householder kernels without an attempt.
__device__ __forceinline__ bool not_tried(const Prob& P, int rows, int mode) {
  return ((mode & QRM_FIRST) && !(P.chol & kGramFirst)) ||
         ((mode & QRM_LARGE) && qr_class(rows, P.l1) < 2);
}

// The same by one wavefront, for l <= 16 columns of at most 64 rows (most
// bonds of a sweep): one Gram tile, one factorisation, no barrier.  False
// when the workgroup has to do it (a later QR that is refused, or a second pass
// is wanted); nothing is written then that it does not write again.
__device__ __forceinline__ bool gram_qr_small(Prob& P, int which, int mode, zt* xs) {
  constexpr int NS = kGqSmallRows / 16;
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4;
  const int l = P.l, rows = which ? P.n : P.m;
  if (l == 0) return true;
  if (l > 16 || rows > kGqSmallRows) return false;
  const bool first = mode & QRM_FIRST, want_r = mode & QRM_WANT_R;
  if (not_tried(P, rows, mode)) {
    if (lane == 0) P.chol_ok = 0;
    return true;
  }
  zt* Y = which ? P.Yt : P.Y;
  ZTile g = tile_zero();
  {
    // addresses clamped instead of loads skipped: a branch each costs more
    zt f[NS][4];
    const zt* yc = Y + size_t(ti < l ? ti : l - 1) * rows;
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      if (16 * st >= rows) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 16 * st + 4 * tk + u;
        f[st][u] = yc[k < rows ? k : rows - 1];
      }
    }
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      if (16 * st >= rows) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = 16 * st + 4 * tk + u < rows;
        const zt v = make_double2(in ? f[st][u].x : 0.0, in ? f[st][u].y : 0.0);
        tile_mma(g, zconj(v), v);
      }
    }
  }
  pad_identity(g, 0, 0, l);
  // the Gram diagonal, in LDS beside the pivot row
  double* gd = reinterpret_cast<double*>(xs + 16);
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (tk + 4 * r == ti) gd[ti] = g.re[r];
  // the strips again as operands of Q = Y X^H: in flight during the factorisation
  zt yb[NS][4];
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    if (16 * st >= rows) break;
    const int r = 16 * st + ti, rc = r < rows ? r : rows - 1;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 4 * s + tk;
      yb[st][s] = Y[size_t(k < l ? k : l - 1) * rows + rc];
    }
  }
  asm volatile("" ::: "memory");
  chol_tile(g, xs, l);
  const double gmax = first ? largest_of(gd, l) : 0.0;
  const int flags = chol_tile_end(g, 0, l, gd, first, gmax, want_r ? P.Rb : nullptr, l);
  if (first && (flags & 1)) {  // the pivoted Householder QR is next (class 0: no report)
    if (lane == 0) P.chol_ok = 0;
    return true;
  }
  if ((flags & 1) || ((mode & QRM_STRICT) && (flags & 2))) return false;
  asm volatile("" ::: "memory");  // the diagonal is read
  tile_store(xs, 17, g);
  zt a[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = zconj(op_a(xs, 17, s));
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    if (16 * st >= rows) break;
    ZTile c = tile_zero();
#pragma unroll
    for (int s = 0; s < 4; ++s) tile_mma(c, a[s], yb[st][s]);
    const int r = 16 * st + ti;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = tk + 4 * q;
      if (col < l && r < rows) Y[size_t(col) * rows + r] = make_double2(c.re[q], c.im[q]);
    }
  }
  if (want_r && lane < l) P.piv[lane] = lane;
  if (lane == 0) P.chol_ok = 1;
  return true;
}

// Items of the launch: packs of kGqWaves small problems, a wavefront each,
// then the problems of a workgroup each, both from their queues (TK_GQ_S,
// TK_GQ_L).  direct, a batch of up to one problem per CU: item i is problem i,
// a small one taken by the first wavefront.  The queues cost two dependent
// reads before a problem is known, and wavefronts of a pack wait for each
// other's instructions on a CU while others idle: 90 launches over 14 bonds
// of a few states each take 0.68 ms in packs, 0.53 so.
constexpr int kGqDirect = 256;

__global__ __launch_bounds__(kGqThreads) void k_gram_qr(Prob* probs, const int32_t* offs, int nprob,
                                                        int which, int mode, int lds_blocks,
                                                        int lds_elems) {
  extern __shared__ zt smem[];
  __shared__ GqShared sh;
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const bool direct = nprob <= kGqDirect;
  const int32_t* ol = offs + size_t(TK_GQ_L) * (nprob + 1);
  const int32_t* os = offs + size_t(TK_GQ_S) * (nprob + 1);
  const int nl = direct ? nprob : ol[nprob], ns = direct ? 0 : os[nprob];
  const int packs = (ns + kGqWaves - 1) / kGqWaves, items = nl + packs;
  for (int it = blockIdx.x; it < items; it += gridDim.x) {
    int mine = -1;  // a problem for the workgroup
    if (it >= packs) {
      if (wave == 0) {
        mine = direct ? it : find_problem(ol, nprob, it - packs);
        if (direct) {
          Prob& P = probs[mine];
          if (gram_small(P.m, P.n, P.l1) && gram_qr_small(P, which, mode, smem)) mine = -1;
        }
      }
    } else {
      const int t = it * kGqWaves + wave;
      if (t < ns) {
        const int p = find_problem(os, nprob, t);
        if (!gram_qr_small(probs[p], which, mode, smem + wave * 272)) mine = p;
      }
    }
    if (lane == 0) sh.todo[wave] = mine;
    if (!__syncthreads_or(mine >= 0)) continue;  // (todo is not read)
    for (int w = 0; w < kGqWaves; ++w) {
      const int p = sh.todo[w];
      if (p < 0) continue;
      Prob& P = probs[p];
      if (P.l == 0 || (!(mode & QRM_ALL) && (P.chol & (which ? kGramTileN : kGramTileM)))) continue;
      if (not_tried(P, which ? P.n : P.m, mode)) {
        if (threadIdx.x == 0) P.chol_ok = 0;
        continue;
      }
      gram_qr_problem(P, which, mode, lds_blocks, lds_elems, smem, sh);
      __syncthreads();
    }
    __syncthreads();
  }
}

// --------------------------------------------------------------------------
// The large sketches (kGramQueueWork): Gram partials on the tile queue, the
// Cholesky factorisation by one workgroup, Q in strips of 64 rows.  The l x l
// Gram matrix alone has too few tiles for the chip, so the rows are split
// into chunks whose partial sums the Cholesky kernel adds in order; only the
// block-lower half is computed.  Measured on two 4900 x 200 sketches, before
// (one chunk, both halves; column-by-column Cholesky in global memory) and
// after: Gram 530 -> 97 us, Cholesky 2500 -> 307 us per launch.
template <int WHICH>
__global__ __launch_bounds__(256) void k_gram(Prob* probs, const int32_t* offs, int nprob, int tebd,
                                              int pass) {
  using Cfg = ZCfg<kGramTile, kGramTile, 16, 2, 2>;
  __shared__ zt smem[Cfg::lds_elems];
  for_each_tile<TK_GRAM>(probs, offs, nprob, tebd, [&](Prob& P, int M, int N, int m0, int n0, int) {
    if (!(P.chol & (WHICH ? kGramTileN : kGramTileM)) || (pass && !P.chol_again)) return;
    const int rows = WHICH ? P.n : P.m, l = P.l;
    const int wide = gram_blocks(l) * kGramTile;
    const int ch = n0 / wide, c0 = n0 - ch * wide;
    const int nch = gram_chunks(rows, P.l1, gram_room(P));
    if (ch >= nch || c0 > m0) return;
    const int len = ((rows + nch - 1) / nch + 15) & ~15;
    const int ra = ch * len, rl = rows - ra < len ? rows - ra : len;
    const zt* Yc = (WHICH ? P.Yt : P.Y) + ra;
    LdAdjColA la{Yc, rows};
    LdColB lb{Yc, rows};
    StRow st{(gram_room(P) ? P.Qc : P.C) + size_t(ch) * l * l, l};
    zgemm_tile<Cfg>(M, l, rl > 0 ? rl : 0, m0, c0, la, lb, st, smem);
  });
}

// The sum of the partial Gram matrices, Cholesky and inverse; X = L^-1 goes
// to C and what follows it (row-major, ld padded to whole blocks).  It fits the
// four buffers from C on, which have room for the l1 x l1 the pass began with: a
// sketch of the queue has l1 >= 8 (kGramQueueMinL), where one block of 16 x 16 is
// 4 x 8 x 8, and (16 ceil(l1 / 16))^2 <= 4 l1^2 beyond.
constexpr int kCholThreads = 512, kCholWaves = kCholThreads / 64;

template <int WHICH>
__global__ __launch_bounds__(kCholThreads) void k_chol(Prob* probs, int pass, int mode,
                                                       int lds_blocks) {
  extern __shared__ zt smem[];
  __shared__ double gd[kMaxL];
  __shared__ zt buf[16];
  __shared__ int sh_flags;
  Prob& P = probs[blockIdx.x];
  const int l = P.l, tid = threadIdx.x;
  const bool mine = l > 0 && (P.chol & (WHICH ? kGramTileN : kGramTileM));
  const bool first = mode & QRM_FIRST, want_r = mode & QRM_WANT_R;
  if (!mine || (first && !(P.chol & kGramFirst))) {
    if (tid == 0 && pass == 0) {
      P.chol_ok = 0;
      P.chol_again = 0;
    }
    return;
  }
  if (pass && !P.chol_again) return;
  const int rows = WHICH ? P.n : P.m;
  const int nb = (l + 15) / 16, lj = 16 * nb;
  const bool in_lds = nb <= lds_blocks;
  const int ld = in_lds ? gq_ld(lds_blocks) : lj;
  zt* G = in_lds ? smem : P.X;
  zt* pn = smem + 16 * lds_blocks * gq_ld(lds_blocks);
  const int nch = gram_chunks(rows, P.l1, gram_room(P));
  const zt* part = gram_room(P) ? P.Qc : P.C;
  for (int e = tid; e < lj * lj; e += kCholThreads) {
    const int i = e / lj, j = e - i * lj;
    if (j / 16 > i / 16) continue;
    zt v = make_double2(i == j ? 1.0 : 0.0, 0.0);
    if (i < l && j < l) {
      // above the diagonal of a diagonal block: its mirror image (a tile of
      // the block-lower half holds both)
      v = part[size_t(i) * l + j];
      for (int c = 1; c < nch; ++c) v = zadd(v, part[size_t(c) * l * l + size_t(i) * l + j]);
    }
    G[size_t(i) * ld + j] = v;
  }
  __syncthreads();
  for (int j = tid; j < lj; j += kCholThreads) gd[j] = G[size_t(j) * ld + j].x;
  if (want_r && pass)
    for (int e = tid; e < l * l; e += kCholThreads) P.C[e] = P.Rb[e];
  __syncthreads();
  const double gmax = first ? largest_of(gd, l) : 0.0;
  const int flags = chol_invert<kCholWaves>(G, ld, nb, pn, l, gd, first, gmax,
                                            want_r ? P.Rb : nullptr, l, &sh_flags, buf);
  if (flags & 1) {
    __syncthreads();
    if (pass && want_r)  // Q_1 and R_1 stand
      for (int e = tid; e < l * l; e += kCholThreads) P.Rb[e] = P.C[e];
    if (tid == 0) {
      if (pass == 0) {
        P.chol_ok = 0;
        if (refusal_reported(P, rows, mode)) P.flags |= TEBD_DEV_QR_FALLBACK;
      }
      P.chol_again = 0;
    }
    return;
  }
  if (want_r) {
    if (pass) compose_r<kCholThreads>(P.Rb, P.C, P.J, l);
    for (int c = tid; c < l; c += kCholThreads) P.piv[c] = c;
  }
  for (int e = tid; e < lj * lj; e += kCholThreads) {
    const int i = e / lj, j = e - i * lj;
    if (j / 16 <= i / 16) P.C[e] = G[size_t(i) * ld + j];
  }
  if (tid == 0) {
    P.chol_ok = 1;
    // (the second pass leaves it set: Q takes its factor too)
    if (pass == 0) P.chol_again = (mode & QRM_STRICT) && (flags & 2);
  }
}

template <int WHICH>
__global__ __launch_bounds__(256) void k_qapply(Prob* probs, const int32_t* offs, int nprob,
                                                int tebd, int pass) {
  for_each_tile<WHICH ? TK_QAPN : TK_QAPM>(probs, offs, nprob, tebd,
                                           [&](Prob& P, int, int, int m0, int n0, int) {
    if (n0 || !P.chol_ok || (pass && !P.chol_again)) return;
    const int rows = WHICH ? P.n : P.m, nb = (P.l + 15) / 16;
    const int r0 = m0 + 16 * wave_id();
    zt* Y = WHICH ? P.Yt : P.Y;
    if (r0 < rows)
      apply_strip(rows, P.l, nb, r0, P.C, 16 * nb,
                  [&](int r, int k) { return Y[size_t(k) * rows + r]; },
                  [&](int r, int k, zt v) { Y[size_t(k) * rows + r] = v; });
  });
}

__global__ void k_chol_mark(Prob* probs, int nprob) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nprob) return;
  Prob& P = probs[p];
  P.chol = P.l > 0 ? gram_bits(P.m, P.n, P.l1, true, true, P.mixed != 0, true) : 0;
  P.chol_ok = 0;
  P.chol_again = 0;
}

hipError_t launch_chol_mark(Prob* probs, const Common& c, hipStream_t s) {
  TEBD_LAUNCH("k_chol_mark", k_chol_mark, dim3((c.nprob + 63) / 64), dim3(64), 0, s, probs,
              c.nprob);
  return hipGetLastError();
}

bool gram_on_queue(const Common& c, int which) {
  const int rows = which ? c.nmax : c.mmax;
  return c.chol && gram_queue_size(rows, c.lmax) &&
         (qr_class(rows, c.lmax) >= 2 || (!c.tebd && rows > kGramQueueRegRows));
}

hipError_t launch_gram_qr(Prob* probs, const Common& c, int which, int mode, hipStream_t s) {
  static const hipError_t attr = []() {
    const void* fns[3] = {reinterpret_cast<const void*>(&k_gram_qr),
                          reinterpret_cast<const void*>(&k_chol<0>),
                          reinterpret_cast<const void*>(&k_chol<1>)};
    for (const void* f : fns) {
      hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         kGqLdsMax * int(sizeof(zt)));
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }();
  if (attr != hipSuccess) return attr;
  const int blocks = (c.lmax + 15) / 16;
  const int lds_blocks = blocks <= kGqLdsBlocks ? blocks : kGqWideBlocks;
  const int base = 16 * lds_blocks * gq_ld(lds_blocks) + gq_tail(blocks);
  const size_t lds = size_t(base) * sizeof(zt);
  hipError_t e = hipSuccess;
  const bool queue = gram_on_queue(c, which);
  if (!queue) mode |= QRM_ALL;
  if (queue) {
    const int passes = mode & QRM_STRICT ? 2 : 1;
    for (int pass = 0; pass < passes && e == hipSuccess; ++pass) {
      const dim3 gg(grid_for(c, TK_GRAM)), gq(grid_for(c, which ? TK_QAPN : TK_QAPM));
      if (which) {
        TEBD_LAUNCH("k_gram<1>", k_gram<1>, gg, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd, pass);
        TEBD_LAUNCH("k_chol<1>", k_chol<1>, dim3(c.nprob), dim3(kCholThreads), lds, s, probs, pass, mode, lds_blocks);
        TEBD_LAUNCH("k_qapply<1>", k_qapply<1>, gq, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd, pass);
      } else {
        TEBD_LAUNCH("k_gram<0>", k_gram<0>, gg, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd, pass);
        TEBD_LAUNCH("k_chol<0>", k_chol<0>, dim3(c.nprob), dim3(kCholThreads), lds, s, probs, pass, mode, lds_blocks);
        TEBD_LAUNCH("k_qapply<0>", k_qapply<0>, gq, dim3(256), 0, s, probs, c.offs, c.nprob, c.tebd, pass);
      }
      e = hipGetLastError();
    }
  }
  // the sketches of a workgroup or a wavefront each, unless every one of the batch is large
  if (e == hipSuccess && !(queue && gram_queue_size(which ? c.nmin : c.mmin, c.lmin))) {
    // LDS for the sketch too, up to the CU's whole: a workgroup per CU suffices
    // (in a batch of more than kGqDirect the small problems go eight to a workgroup)
    const int64_t want = int64_t(base) + int64_t(gq_ldy(which ? c.nmax : c.mmax)) * c.lmax;
    int elems = int(want < kGqLdsMax ? want : kGqLdsMax);
    if (elems < kGqWaves * 272) elems = kGqWaves * 272;
    const int nl = c.ktiles[TK_GQ_L], ns = c.ktiles[TK_GQ_S];
    int g = nl + (ns + kGqWaves - 1) / kGqWaves;
    if (c.nprob <= kGqDirect)
      g = c.nprob;
    else if (nl < 0 || ns < 0)
      g = c.nprob;
    TEBD_LAUNCH("k_gram_qr", k_gram_qr, dim3(g < 1 ? 1 : g), dim3(kGqThreads),
                size_t(elems) * sizeof(zt), s, probs, c.offs, c.nprob, which, mode, lds_blocks,
                elems);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace tebd
