// Small SVD of the projected matrix by one-sided Jacobi, and the truncation
// rule with lambda renormalisation (one workgroup per problem).
//
// Paper: Tamascelli, Rosenbach, Plenio, arXiv:1504.00992.  The SVD of B = Q^H A
// of Sec. IV step ii (computed as B^H = Q_B R_B, then a one-sided Jacobi SVD of
// R_B^H, which keeps small singular values to high relative accuracy), and the
// discarded weight of Sec. II.C, Eq. (defdiscweigt), evaluated with the
// Frobenius identity of Sec. IV.
#include <cfloat>
#include <type_traits>

#include "householder.hpp"
#include "kinds.hpp"
#include "sidestreams.hpp"
#include "zgemm.hpp"

namespace tebd {

// --------------------------------------------------------------------------
// Small SVD of B (l x n) from B^H = Q_B R_B: one-sided Jacobi on C = R_B^H
// (l x l).  Column pairs are rotated in the round-robin order of the circle
// method, l/2 disjoint pairs per round, one pair per wavefront at a time.
// A pair (p, q) with Gram entries a = |c_p|^2, b = |c_q|^2, g = c_p^H c_q is
// rotated when |g| > tol sqrt(a b):  phi = arg g, zeta = (b - a) / (2|g|),
// t = sign(zeta) / (|zeta| + sqrt(1 + zeta^2)), cs = 1/sqrt(1+t^2), sn = t cs,
//   c_p <- cs c_p - sn e^{-i phi} c_q,  c_q <- sn c_p + cs e^{-i phi} c_q,
// which zeroes the (p, q) Gram entry.  The same rotation accumulates into J.
// At convergence C J = X Sigma with orthogonal columns, so
// B = X Sigma (Q_B J)^H: left vectors X (normalised columns), values Sigma,
// right vectors Q_B J (formed later).  Outputs are sorted descending.
// C and J live in LDS when 2 l^2 fits, else in global memory; a pair's
// columns are held in registers (l <= 64 * REGS) for the whole rotation.

// Rotation of a column pair with Gram entries a = |c_p|^2, b = |c_q|^2 and
// g = c_p^H c_q (given as gr + i gi): false when |g| <= tol sqrt(a b).
// Otherwise zeta = (b - a) / (2|g|), t = sign(zeta) / (|zeta| + sqrt(1 +
// zeta^2)), cs = 1 / sqrt(1 + t^2), sn = t cs, em = e^{-i arg g}, and
// ag = |g| (the carried norms move by t |g|).  Every lane of the group computes
// it on the critical path of a round: square root and division go through the
// hardware estimates (rsqrt_pos, rcp_pos), 8 instructions instead of 15.
__device__ __forceinline__ bool jacobi_rotation(double gr, double gi, double a, double b,
                                                double tol, double& ag, double& t, double& cs,
                                                double& sn, zt& em) {
  const double g2 = gr * gr + gi * gi;
  if (!(g2 > tol * tol * (a * b)) || g2 == 0.0) return false;
  const double ig = rsqrt_pos(g2);  // 1 / |g|
  ag = g2 * ig;
  const double zeta = 0.5 * (b - a) * ig, az = fabs(zeta);
  const bool far = az > 1e100;  // zeta^2 would overflow; there sqrt(1 + zeta^2) = |zeta|
  const double z2 = far ? 1.0 : fma(zeta, zeta, 1.0);
  const double root = far ? az : z2 * rsqrt_pos(z2);
  t = copysign(rcp_pos(az + root), zeta);
  cs = rsqrt_pos(fma(t, t, 1.0));
  sn = t * cs;
  em = make_double2(gr * ig, -gi * ig);
  return true;
}

// Round-robin (circle method) pairing of lp players: position 0 stays, the
// others rotate by one place per round.  pos < lp and round < lp - 1, so
// one conditional subtraction reduces modulo lp - 1 (no integer division).
__device__ __forceinline__ int circle_player(int pos, int round, int lp) {
  if (pos == 0) return 0;
  const int x = pos - 1 + round;
  return 1 + (x >= lp - 1 ? x - (lp - 1) : x);
}


// Column norms are recomputed exactly at the start of every sweep and then
// carried through the rotations analytically (a' = a - t|g|, b' = b + t|g|),
// so each pair needs a single complex reduction, g = c_p^H c_q.
// A sweep whose rotations all turned by less than about 1e-7 rad (|g|^2 <=
// kSmallTurn a b) leaves the columns so close to orthogonal that the next
// sweep would likely rotate nothing; instead of running that sweep,
// pairs_below_tol tests every pair of the current C at once.
constexpr double kSmallTurn = 1e-14;
constexpr int kMaxSweeps = 40;

// True when no pair of columns of C (column c at C + c S) would be rotated:
// every |c_p^H c_q| <= tol |c_p| |c_q| with nrm[c] = |c_c|^2 recomputed and
// visible to the workgroup (the test of jacobi_rotation).  The verdict of a
// sweep that rotates nothing, from l (l - 1) / 2 independent dot products
// instead of l - 1 dependent rounds.  Whole workgroup (one barrier).
template <int NT>
__device__ __forceinline__ bool pairs_below_tol(const zt* C, int S, int l, double tol,
                                                const double* nrm) {
  // thread t: columns {2a, 2a + 1} x {2b, 2b + 1}, a <= b, four dot products
  // per pass over the rows (a missing last column repeats the one before)
  const int nh = (l + 1) / 2;
  int bad = 0;
  for (int t = threadIdx.x; t < nh * nh; t += NT) {
    const int a = t / nh, b = t - a * nh;
    if (a > b) continue;
    const int p0 = 2 * a, q0 = 2 * b;
    const int p1 = p0 + 1 < l ? p0 + 1 : p0, q1 = q0 + 1 < l ? q0 + 1 : q0;
    const zt* x0 = C + size_t(p0) * S;
    const zt* x1 = C + size_t(p1) * S;
    const zt* y0 = C + size_t(q0) * S;
    const zt* y1 = C + size_t(q1) * S;
    double g[4][2] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    for (int r = 0; r < l; ++r) {
      const zt u0 = x0[r], u1 = x1[r], v0 = y0[r], v1 = y1[r];
      zdot_acc(u0, v0, g[0][0], g[0][1]);
      zdot_acc(u0, v1, g[1][0], g[1][1]);
      zdot_acc(u1, v0, g[2][0], g[2][1]);
      zdot_acc(u1, v1, g[3][0], g[3][1]);
    }
    const int ps[4] = {p0, p0, p1, p1}, qs[4] = {q0, q1, q0, q1};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double g2 = g[i][0] * g[i][0] + g[i][1] * g[i][1];
      if (ps[i] < qs[i] && g2 > tol * tol * (nrm[ps[i]] * nrm[qs[i]]) && g2 != 0.0) bad = 1;
    }
  }
  return __syncthreads_or(bad) == 0;
}

// Whether singular value a of column i comes before b of column j: descending,
// equal ones by column, NaN last (every column has a place of its own: places
// without a column would be read from uninitialised LDS).
__device__ __forceinline__ bool sorts_before(double a, int i, double b, int j) {
  const bool na = a != a, nb = b != b;
  return a > b || (nb && !na) || ((a == b || (na && nb)) && i < j);
}

// Column norms, descending order, and the sorted outputs X, W, sig.
template <int NT>
__device__ __forceinline__ void jacobi_finish(Prob& P, const zt* C, const zt* J, int l,
                                              double* sig_s, int* perm_s) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int c = wave; c < l; c += NW) {
    double s = 0.0;
    for (int r = lane; r < l; r += 64) s += zabs2(C[size_t(c) * l + r]);
    s = wave_sum(s);
    if (lane == 0) sig_s[c] = sqrt(s);
  }
  __syncthreads();
  for (int j = tid; j < l; j += NT) {
    const double sj = sig_s[j];
    int rank = 0;
    for (int i = 0; i < l; ++i) rank += sorts_before(sig_s[i], i, sj, j);
    perm_s[rank] = j;
  }
  __syncthreads();
  for (int c = wave; c < l; c += NW) {
    const int src = perm_s[c];
    const double sv = sig_s[src], inv = sv > 0.0 ? 1.0 / sv : 0.0;
    const zt* cc = C + size_t(src) * l;
    const zt* jc = J + size_t(src) * l;
    for (int r = lane; r < l; r += 64) {
      const zt x = cc[r], w = jc[r];
      P.X[size_t(c) * l + r] = sv > 0.0 ? zscale(x, inv) : make_double2(0.0, 0.0);
      P.W[size_t(c) * l + r] = w;
    }
  }
  for (int c = tid; c < l; c += NT) P.sig[c] = sig_s[perm_s[c]];
}

// --------------------------------------------------------------------------
// Truncation: chi' = min(chi_max, smallest c with w(c) <= eps), where
// w(c) = (||A||_F^2 - sum_{j<=c} s_j^2) / ||A||_F^2; eps <= 0 keeps
// min(chi_max, l).  TEBD: lambda' = s / ||s_{1..chi'}|| and chi' are written
// into the MPS.  Run by the whole workgroup of the problem's small SVD after
// it (sorted(c): the c-th largest singular value, from LDS); the scans run
// on thread 0 so the summation order is fixed.  The global reads (partial
// sums, outer lambdas) are spread over the workgroup first: one thread
// reading them one after another waited for each.
constexpr int kTailChunk = 64;

template <int NT, class Sorted>
__device__ __forceinline__ void truncate_tail(Prob& P, int l, double eps, int tebd,
                                              int32_t* retry_count, Sorted sorted, double* scan) {
  __shared__ int chi_s, first_s;
  __shared__ double norm_s, frob_s;
  __shared__ double part_s[kTailChunk];
  const int tid = threadIdx.x;
  // ||A||_F^2 from the partial sums, the gate product's (TEBD) or k_frob's:
  // loaded kTailChunk at a time, added by thread 0 in index order
  const int npart =
      tebd ? gate_partials(P.dl * P.dr, P.gcol0, P.chi_l * P.chi_r) : kFrobSlices;
  __syncthreads();  // the singular values are in place
  // one round of global reads: the first chunk of partial sums, and whether
  // an outer lambda is at or below the floor (its inverse was taken as 0)
  if (tid < kTailChunk && tid < npart) part_s[tid] = P.part[tid];
  bool floor_hit = false;
  if (tebd) {
    if (P.lam_l)
      for (int a = tid; a < P.chi_l; a += NT) floor_hit |= !(P.lam_l[a] > P.lambda_floor);
    if (P.lam_r)
      for (int b = tid; b < P.chi_r; b += NT) floor_hit |= !(P.lam_r[b] > P.lambda_floor);
  }
  floor_hit = __syncthreads_or(floor_hit) != 0;
  double frob2 = 0.0;
  for (int i0 = 0; i0 < npart; i0 += kTailChunk) {
    if (i0 > 0) {
      __syncthreads();  // the previous chunk is summed
      if (tid < kTailChunk && i0 + tid < npart) part_s[tid] = P.part[i0 + tid];
      __syncthreads();
    }
    if (tid == 0) {
      const int n = npart - i0 < kTailChunk ? npart - i0 : kTailChunk;
      for (int i = 0; i < n; ++i) frob2 += part_s[i];
    }
  }
  // kept(c) = s_1^2 + ... + s_c^2 in index order (thread 0, into scan[c - 1]);
  // then every c at once: w(c) = (||A||_F^2 - kept(c)) / ||A||_F^2, and chi'
  // the smallest c <= cap with w(c) <= eps.  The same operations as one
  // thread scanning c = 1, 2, ..., without its chain of divisions.
  // A first stage that may still be retried only accepts a rank <= k1.
  const bool can_retry = P.l2 > P.l1;
  int cap = P.kcap < l ? P.kcap : l;
  if (can_retry && P.k1 < cap) cap = P.k1;
  if (tid == 0) {
    double kept = 0.0;
    for (int c = 0; c < l; ++c) {
      const double sv = sorted(c);
      kept += sv * sv;
      scan[c] = kept;
    }
    frob_s = frob2;
    first_s = INT32_MAX;
  }
  __syncthreads();
  const double fr = frob_s;
  int first = INT32_MAX;
  bool nonfinite = false;
  for (int c = tid + 1; c <= l; c += NT) {
    nonfinite |= !isfinite(sorted(c - 1));
    const double wc = fr > 0.0 ? (fr - scan[c - 1]) / fr : 0.0;
    if (eps > 0.0 && c <= cap && wc <= eps && c < first) first = c;
  }
  if (first != INT32_MAX) atomicMin(&first_s, first);
  nonfinite = __syncthreads_or(nonfinite) != 0;
  if (tid == 0) {
    int flags = P.flags;
    P.frob2 = frob2;
    const bool found = first_s != INT32_MAX;
    const int chi = found ? first_s : cap;
    // the discarded weight at chi' (or at cap when no c qualifies)
    double w = fr > 0.0 ? (fr - scan[chi - 1]) / fr : 0.0;
    const double nk = scan[chi - 1];  // the kept squares summed up to chi'
    const bool finite = isfinite(frob2) && !nonfinite;
    int out = chi;
    if (can_retry && !(eps > 0.0 && found)) {
      // stage 1 rejected: leave every output untouched, run stage 2
      P.retry = 1;
      if (retry_count) atomicAdd(retry_count, 1);
      out = -1;
    }
    if (eps > 0.0 && !found) flags |= TEBD_DEV_CHI_BOUND;
    if (!finite) flags |= TEBD_DEV_NONFINITE;
    if (w < 0.0) w = 0.0;
    if (floor_hit) flags |= TEBD_DEV_LAMBDA_FLOOR;
    if (out >= 0) {
      P.chi_new = chi;
      P.flags = flags;
      *P.disc = w;
      *P.status = flags;
      if (P.chi_out) *P.chi_out = chi;
    }
    chi_s = out;
    norm_s = sqrt(nk);
  }
  __syncthreads();
  const int chi = chi_s;
  if (chi < 0) return;
  if (tebd) {
    const double inv = norm_s > 0.0 ? 1.0 / norm_s : 0.0;
    for (int j = threadIdx.x; j < P.chi_cap; j += NT) P.lam_mid[j] = j < chi ? sorted(j) * inv : 0.0;
    if (threadIdx.x == 0) *P.chi_slot = chi;
  } else {
    for (int j = threadIdx.x; j < P.kcap; j += NT) P.S[j] = j < chi ? sorted(j) : 0.0;
  }
}

// Size classes of the small SVD, by l: 0 (l <= 32, 256 threads) and 1
// (l <= 64, 512 threads) rotate every pair of a round at once (k_svd_pairs);
// 2 and 3 rotate the pairs of two blocks of columns (jac_pair), 2 up to where
// C and J would fit in LDS.
__host__ __device__ __forceinline__ int svd_class(int l) {
  if (l <= 32) return 0;
  if (l <= 64) return 1;
  if (2 * l * l <= kLdsElems) return 2;
  return 3;
}

// One column's rows of C and J: lane h of n holds rows h + n i.
template <int REGS>
struct JacColumn {
  zt c[REGS], j[REGS];
};

// All l/2 pairs of a round are rotated at once by 16 lanes each (a group), in
// the odd-even order: the columns stand in a row of lp = l (+ 1) positions,
// rounds rotate the pairs of positions (0 1)(2 3)... and (1 2)(3 4)... in
// turn, and every pair changes places as it is rotated, so that after lp rounds
// each two columns have met once and the row is reversed.
// Group k keeps the columns at positions 2k and 2k + 1 in registers (lane h
// rows h, h + 16, ... of C and J, zeros beyond l); only the column at 2k goes
// to group k - 1 and back, through LDS, one transfer and one barrier a round.
// A round is bound by the instructions of a wavefront (about five cycles
// each, a branch twenty) and the LDS traffic: the rows per lane are a template
// argument, and a pair that need not rotate has the rotation by zero.
// Measured, one problem, l = 34 / l = 42: 240 / 229 us with every column of C
// and J read from LDS and written back in each round (104 KB at l = 34), 141 /
// 156 us so; rotation parameters without the branch around them 154 / 176 us;
// J one round behind C, in the gaps of C's chain, 177 / 174 us.
// Same rotation, tolerance, carried norms (recomputed in every sweep) and
// sweep limit as jac_pair.
constexpr int kPairGroup = 16;

// Rotation of columns (x, y) that change places: x becomes sn x + cs em y, y
// becomes cs x - sn em y.  Bit 0 of the result: rotated, bit 1: by more than a
// small turn.
template <int RPR>
__device__ __forceinline__ int pair_rotate(JacColumn<RPR>& x, JacColumn<RPR>& y, double tol,
                                           double& na, double& nb) {
  double g0 = 0.0, g1 = 0.0;
#pragma unroll
  for (int i = 0; i < RPR; ++i) zdot_acc(x.c[i], y.c[i], g0, g1);
  g0 = group_sum(g0, kPairGroup);
  g1 = group_sum(g1, kPairGroup);
  double ag, t, cs, sn;
  zt em;
  const bool on = jacobi_rotation(g0, g1, na, nb, tol, ag, t, cs, sn, em);
  const double turn = on ? t * ag : 0.0;
  cs = on ? cs : 1.0;
  sn = on ? sn : 0.0;
  em.x = on ? em.x : 1.0;
  em.y = on ? em.y : 0.0;
#pragma unroll
  for (int i = 0; i < RPR; ++i) {
    const zt u = x.c[i], v = zmul(em, y.c[i]), uj = x.j[i], vj = zmul(em, y.j[i]);
    x.c[i] = zrot_hi(u, v, cs, sn);
    y.c[i] = zrot_lo(u, v, cs, sn);
    x.j[i] = zrot_hi(uj, vj, cs, sn);
    y.j[i] = zrot_lo(uj, vj, cs, sn);
  }
  const int r = !on ? 0 : ag * ag > kSmallTurn * (na * nb) ? 3 : 1;
  const double a = na;
  na = nb + turn;
  nb = fmax(a - turn, 0.0);
  return r;
}

// LDS elements: the columns in transfer, or C for pairs_below_tol.
constexpr int pair_lds(int groups, int rpr) {
  return 2 * groups * (kPairGroup * rpr + 1);
}

template <int NT, int RPR>
__device__ __forceinline__ void svd_pairs(Prob& P, int l, double eps, int tebd,
                                          int32_t* retry_count, zt* lds, double* nrm,
                                          double* sig_s, double* srt_s) {
  constexpr int G = kPairGroup, RP = G * RPR, S = RP + 1;
  const int tid = threadIdx.x, k = tid / G, h = tid & (G - 1);
  const int np = (l + 1) / 2, lp = 2 * np;  // groups with columns, positions
  const double tol = DBL_EPSILON * sqrt(double(l));
  JacColumn<RPR> x, y;
  auto load = [&](int c, JacColumn<RPR>& v) {
    const int cc = c < l ? c : l - 1;
#pragma unroll
    for (int i = 0; i < RPR; ++i) {
      const int r = h + G * i;
      const zt a = P.Rb[size_t(r < l ? r : l - 1) * l + cc];
      const bool in = r < l && c < l;
      v.c[i] = make_double2(in ? a.x : 0.0, in ? -a.y : 0.0);
      v.j[i] = make_double2(in && r == c ? 1.0 : 0.0, 0.0);
    }
  };
  load(2 * k, x);
  load(2 * k + 1, y);
  // slot k: C and J of the column at position 2k, and its norm
  auto put = [&](int slot, const JacColumn<RPR>& v, double n) {
    zt* at = lds + slot * 2 * RP + h;
#pragma unroll
    for (int i = 0; i < RPR; ++i) {
      at[G * i] = v.c[i];
      at[RP + G * i] = v.j[i];
    }
    if (h == 0) nrm[slot] = n;
  };
  auto get = [&](int slot, JacColumn<RPR>& v) {
    const zt* at = lds + slot * 2 * RP + h;
#pragma unroll
    for (int i = 0; i < RPR; ++i) {
      v.c[i] = at[G * i];
      v.j[i] = at[RP + G * i];
    }
    return nrm[slot];
  };
  auto norm2 = [&](const JacColumn<RPR>& v) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < RPR; ++i) s += zabs2(v.c[i]);
    return group_sum(s, G);
  };
  const bool have = k < np, right = k + 1 < np, left = k > 0 && have;
  bool converged = l == 1;
  int sweep = 0;
  for (; sweep < kMaxSweeps && !converged; ++sweep) {
    double na = norm2(x), nb = norm2(y);
    int bits = 0;
    for (int round = 0; round < np; ++round) {
      if (have) {
        bits |= pair_rotate(x, y, tol, na, nb);
        put(k, x, na);
      }
      __syncthreads();
      if (right) {
        JacColumn<RPR> z;
        double nz = get(k + 1, z);
        bits |= pair_rotate(y, z, tol, nb, nz);
        put(k + 1, z, nz);
      }
      __syncthreads();
      if (left) na = get(k, x);
    }
    const bool rotated = __syncthreads_or(bits & 1) != 0;
    const bool turned_far = __syncthreads_or(bits & 2) != 0;
    converged = !rotated;
    if (rotated && !turned_far) {
      // every pair at once, C by position (the empty one, if any, is first or
      // last: it has no column in C below and above)
      const int skip = lp > l && !(sweep & 1) ? 1 : 0;
      na = norm2(x);
      nb = norm2(y);
      auto column = [&](int pos, const JacColumn<RPR>& v, double n) {
        const int c = pos - skip;
        if (c < 0 || c >= l) return;
#pragma unroll
        for (int i = 0; i < RPR; ++i) lds[c * S + h + G * i] = v.c[i];
        if (h == 0) sig_s[c] = n;
      };
      if (have) {
        column(2 * k, x, na);
        column(2 * k + 1, y, nb);
      }
      __syncthreads();
      converged = pairs_below_tol<NT>(lds, S, l, tol, sig_s);
    }
  }
  if (!converged && tid == 0) P.flags |= TEBD_DEV_JACOBI_NOCONV;
  // singular values, descending order, sorted outputs; the empty position is
  // the last one after an even number of sweeps, the first one else
  const int skip = lp > l && (sweep & 1) ? 1 : 0;
  const int cx = have ? 2 * k - skip : -1, cy = have ? 2 * k + 1 - skip : -1;
  const double sx = sqrt(norm2(x)), sy = sqrt(norm2(y));
  __syncthreads();
  if (h == 0 && cx >= 0 && cx < l) sig_s[cx] = sx;
  if (h == 0 && cy >= 0 && cy < l) sig_s[cy] = sy;
  __syncthreads();
  auto out = [&](int c, double sv, const JacColumn<RPR>& v) {
    if (c < 0 || c >= l) return;
    int rank = 0;
    for (int i = h; i < l; i += G) rank += sorts_before(sig_s[i], i, sv, c);
    rank = static_cast<int>(group_sum(double(rank), G));
    const double inv = sv > 0.0 ? 1.0 / sv : 0.0;
#pragma unroll
    for (int i = 0; i < RPR; ++i) {
      const int r = h + G * i;
      if (r < l) {
        P.X[size_t(rank) * l + r] = zscale(v.c[i], inv);
        P.W[size_t(rank) * l + r] = v.j[i];
      }
    }
    if (h == 0) {
      srt_s[rank] = sv;
      P.sig[rank] = sv;
    }
  };
  out(cx, sx, x);
  out(cy, sy, y);
  truncate_tail<NT>(P, l, eps, tebd, retry_count, [&](int c) { return srt_s[c]; }, nrm);
}

template <int NT, int CLS>
__global__ __launch_bounds__(NT) void k_svd_pairs(Prob* probs, double eps, int tebd,
                                                  int32_t* retry_count) {
  extern __shared__ zt lds[];
  __shared__ double nrm[64], sig_s[64];
  __shared__ double srt_s[64];  // singular values in descending order
  Prob& P = probs[blockIdx.x];
  const int l = P.l;
  if (l == 0 || svd_class(l) != CLS) return;
  static_assert(NT / kPairGroup == (CLS == 0 ? 16 : 32), "a group for every two columns");
  if (l <= (CLS == 0 ? 16 : 48))
    svd_pairs<NT, (CLS == 0 ? 1 : 3)>(P, l, eps, tebd, retry_count, lds, nrm, sig_s, srt_s);
  else
    svd_pairs<NT, (CLS == 0 ? 2 : 4)>(P, l, eps, tebd, retry_count, lds, nrm, sig_s, srt_s);
}

// --------------------------------------------------------------------------
// Classes 2 and 3.  The columns are split into blocks of kJacBlock; a
// workgroup rotates every pair of columns across two blocks at a time
// (jac_pair), the block pairs follow the circle method, and the first round
// of a sweep also rotates the pairs inside the blocks.  A wavefront keeps one
// column of the first block (its rows of C and J) in registers and meets the
// second block's columns, in LDS, one after another.  Rotation, tolerance,
// carried norms (recomputed for every block pair) and sweep limit as in
// k_svd_pairs; 5 to 7 sweeps.
//
// The rounds are launches of a workgroup per block pair (k_jac_round) where the
// host knows that there are such problems: one CU's arithmetic and memory
// are the bound of a single workgroup (l = 200: 1.4 GFLOP of rotations).
// k_small_svd then goes on where kJacSweeps sweeps were not enough; without
// the launches it runs all of them, the same operations in the same order, so
// that every rank mode of a sweep gives the same bits.
// Measured, the whole small SVD of one workgroup that rotated single pairs /
// these launches: l = 200, two problems 33.8 / 3.1 ms; l = 74, 20 problems
// 2.86 / 0.90 ms; by one workgroup in blocks, l = 74 2.28 ms.  A launch takes
// 4.5 us with nothing to do, 13 us (l = 74) to 17 us (l = 200) with.
constexpr int kJacBlock = 8, kJacThreads = 64 * kJacBlock, kJacSweeps = 7, kJacCheckFrom = 2;

// Per launched sweep s, in Prob::jac: bit s a rotation happened, bit 8 + s one
// of them by more than a small turn, bit 16 + s the test of all pairs after it
// failed.
__device__ __forceinline__ bool sweep_ended(bool rotated, bool more, int sweep) {
  return !rotated || (!more && sweep >= kJacCheckFrom);
}
__device__ __forceinline__ bool jac_done(int bits, int sweep) {
  for (int s = 0; s < sweep; ++s)
    if (sweep_ended(bits >> s & 1, (bits >> 8 | bits >> 16) >> s & 1, s)) return true;
  return false;
}
static_assert(kJacSweeps <= 8, "bits per sweep in Prob::jac");

// The problems of these classes (indices, in order, then their number in the
// low 22 bits of list[nprob] and the largest l above), one workgroup.
__global__ __launch_bounds__(1024) void k_jac_list(Prob* probs, int nprob, int32_t* list) {
  __shared__ int wsum[16], wmax[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  int base = 0, lmax = 0;
  for (int p0 = 0; p0 < nprob; p0 += 1024) {
    const int p = p0 + tid;
    const int l = p < nprob ? probs[p].l : 0;
    const bool in = l > 0 && svd_class(l) >= 2;
    const unsigned long long m = __ballot(in);
    if (lane == 0) wsum[wave] = __popcll(m);
    __syncthreads();
    int at = base + __popcll(m & ((1ull << lane) - 1));
    for (int w = 0; w < 16; ++w) {
      at += w < wave ? wsum[w] : 0;
      base += wsum[w];
    }
    if (in) {
      list[at] = p;
      probs[p].jac = 0;
      lmax = l > lmax ? l : lmax;
    }
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) {
    const int o = __shfl_xor(lmax, off, 64);
    lmax = o > lmax ? o : lmax;
  }
  if (lane == 0) wmax[wave] = lmax;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; ++w) lmax = wmax[w] > lmax ? wmax[w] : lmax;
    list[nprob] = base | lmax << 22;
  }
}
constexpr int kJacCountMask = (1 << 22) - 1;

template <int REGS>
__device__ __forceinline__ double jac_norm2(const JacColumn<REGS>& x) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < REGS; ++i) s += zabs2(x.c[i]);
  return wave_sum(s);
}

// One wavefront: rotates columns x and y (squared norms na, nb, carried);
// bit 0 of the result: rotated, bit 1: by more than a small turn.
template <int REGS>
__device__ __forceinline__ int jac_rotate(JacColumn<REGS>& x, JacColumn<REGS>& y, double tol,
                                          double& na, double& nb) {
  double g0 = 0.0, g1 = 0.0;
#pragma unroll
  for (int i = 0; i < REGS; ++i) zdot_acc(x.c[i], y.c[i], g0, g1);
  g0 = wave_sum(g0);
  g1 = wave_sum(g1);
  double ag, t, cs, sn;
  zt em;
  if (!jacobi_rotation(g0, g1, na, nb, tol, ag, t, cs, sn, em)) return 0;
#pragma unroll
  for (int i = 0; i < REGS; ++i) {
    const zt u = x.c[i], v = zmul(em, y.c[i]), uj = x.j[i], vj = zmul(em, y.j[i]);
    x.c[i] = zrot_lo(u, v, cs, sn);
    y.c[i] = zrot_hi(u, v, cs, sn);
    x.j[i] = zrot_lo(uj, vj, cs, sn);
    y.j[i] = zrot_hi(uj, vj, cs, sn);
  }
  const int r = ag * ag > kSmallTurn * (na * nb) ? 3 : 1;
  na = fmax(na - t * ag, 0.0);
  nb += t * ag;
  return r;
}

// kJacBlock wavefronts (this one is w): blocks a and b of round `round`; start:
// C and J are still R_B^H and the identity.  Returns bit 0: something rotated,
// bit 8: by more than a small turn (in any such group of the workgroup: they
// run in step, each with lds and sh of its own).  lds: columns of C, then of
// J, per slot: kJacBlock slots of the second block, and in round 0 as many of
// the first.  Columns beyond l count as zero.
struct JacShared {
  double nrm[2 * kJacBlock];
  int changed[kJacBlock];
};

template <int REGS>
__device__ __forceinline__ int jac_pair(Prob& P, int a, int b, int round, bool start, int w,
                                        zt* lds, JacShared& sh) {
  constexpr int S = 64 * REGS;
  const int lane = threadIdx.x & 63, l = P.l;
  auto put = [&](int slot, const JacColumn<REGS>& x) {
    zt* at = lds + slot * 2 * S + lane;
#pragma unroll
    for (int i = 0; i < REGS; ++i) {
      at[64 * i] = x.c[i];
      at[S + 64 * i] = x.j[i];
    }
  };
  auto get = [&](int slot, JacColumn<REGS>& x) {
    const zt* at = lds + slot * 2 * S + lane;
#pragma unroll
    for (int i = 0; i < REGS; ++i) {
      x.c[i] = at[64 * i];
      x.j[i] = at[S + 64 * i];
    }
  };
  auto load = [&](int col, JacColumn<REGS>& x) {
    const int cc = col < l ? col : l - 1;
#pragma unroll
    for (int u = 0; u < REGS; ++u) {
      const int r = lane + 64 * u, rc = r < l ? r : l - 1;
      const bool in = r < l && col < l;
      const zt v = start ? zconj(P.Rb[size_t(rc) * l + cc]) : P.C[size_t(cc) * l + rc];
      const zt vj = start ? make_double2(r == col ? 1.0 : 0.0, 0.0) : P.J[size_t(cc) * l + rc];
      x.c[u] = make_double2(in ? v.x : 0.0, in ? v.y : 0.0);
      x.j[u] = make_double2(in ? vj.x : 0.0, in ? vj.y : 0.0);
    }
  };
  auto store = [&](int col, const JacColumn<REGS>& x) {
    if (col >= l) return;
#pragma unroll
    for (int u = 0; u < REGS; ++u) {
      const int r = lane + 64 * u;
      if (r < l) {
        P.C[size_t(col) * l + r] = x.c[u];
        P.J[size_t(col) * l + r] = x.j[u];
      }
    }
  };
  const int p = (a < b ? a : b) * kJacBlock + w, q = (a < b ? b : a) * kJacBlock + w;
  const double tol = DBL_EPSILON * sqrt(double(l));
  JacColumn<REGS> x, y;
  load(p, x);
  load(q, y);
  int bits = 0;
  double na = jac_norm2(x);
  {
    const double n = jac_norm2(y);
    if (lane == 0) {
      sh.nrm[w] = n;
      sh.nrm[kJacBlock + w] = na;
      sh.changed[w] = start;
    }
  }
  put(w, y);
  bool moved = start;  // the first block's column
  if (round == 0) {    // the pairs inside either block
    put(kJacBlock + w, x);
    for (int r = 0; r < kJacBlock - 1; ++r) {
      const int h = w & (kJacBlock / 2 - 1), side = w < kJacBlock / 2 ? 0 : kJacBlock;
      const int s0 = circle_player(h, r, kJacBlock),
                s1 = circle_player(kJacBlock - 1 - h, r, kJacBlock);
      const int lo = side + (s0 < s1 ? s0 : s1), hi = side + (s0 < s1 ? s1 : s0);
      __syncthreads();
      get(lo, x);
      get(hi, y);
      double nl = sh.nrm[lo], nh = sh.nrm[hi];
      const int c = jac_rotate(x, y, tol, nl, nh);
      if (c) {
        put(lo, x);
        put(hi, y);
        if (lane == 0) {
          sh.nrm[lo] = nl;
          sh.nrm[hi] = nh;
        }
      }
      bits |= c;
    }
    const bool inner = __syncthreads_or(bits) != 0;
    moved |= inner;
    if (lane == 0 && inner) sh.changed[w] = 1;
    get(kJacBlock + w, x);
    na = sh.nrm[kJacBlock + w];
  }
  for (int s = 0; s < kJacBlock; ++s) {
    const int slot = (w + s) & (kJacBlock - 1);
    __syncthreads();
    get(slot, y);
    double n = sh.nrm[slot];
    const int c = jac_rotate(x, y, tol, na, n);
    if (c) {
      put(slot, y);
      if (lane == 0) {
        sh.nrm[slot] = n;
        sh.changed[slot] = 1;
      }
      moved = true;
    }
    bits |= c;
  }
  if (moved) store(p, x);
  const int all = (__syncthreads_or(bits & 1) ? 1 : 0) | (__syncthreads_or(bits & 2) ? 1 << 8 : 0);
  if (sh.changed[w]) {
    get(w, y);
    store(q, y);
  }
  __syncthreads();  // the slots are free, and C and J in place for the workgroup
  return all;
}

// Blocks of a problem, an even number of them (with one that is none).
__host__ __device__ __forceinline__ int jac_blocks(int l) {
  return ((l + kJacBlock - 1) / kJacBlock + 1) & ~1;
}

template <int REGS>
__global__ __launch_bounds__(kJacThreads) void k_jac_round(Prob* probs, const int32_t* list,
                                                           int nprob, int pairs, int sweep,
                                                           int round) {
  extern __shared__ zt lds[];
  __shared__ JacShared sh;
  const int items = (list[nprob] & kJacCountMask) * pairs;
  for (int it = blockIdx.x; it < items; it += gridDim.x) {
    const int i = it / pairs, k = it - i * pairs;
    Prob& P = probs[list[i]];
    const int nb = jac_blocks(P.l);
    if (k >= nb / 2 || round >= nb - 1 || jac_done(P.jac, sweep)) continue;
    const int a = circle_player(k, round, nb), b = circle_player(nb - 1 - k, round, nb);
    // an odd number of blocks: the last player is none (its partner's inner
    // pairs still rotate)
    if (round > 0 && (a > b ? a : b) * kJacBlock >= P.l) continue;
    const int bits = jac_pair<REGS>(P, a, b, round, sweep == 0 && round == 0, wave_id(), lds, sh);
    if (threadIdx.x == 0 && bits) atomicOr(&P.jac, bits << sweep);
  }
}

// The test of all pairs after a sweep of small turns only (jacobi_rotation's,
// norms recomputed).  One wavefront: tile (bi, bj) of the Gram matrix; true
// when a pair of it would still be rotated.
__device__ __forceinline__ bool jac_tile_bad(const Prob& P, int bi, int bj) {
  const int lane = threadIdx.x & 63, ti = lane & 15, tk = lane >> 4, l = P.l;
  const int p = bi * 16 + ti, q = bj * 16 + ti;
  const zt* cp = P.C + size_t(p < l ? p : l - 1) * l;
  const zt* cq = P.C + size_t(q < l ? q : l - 1) * l;
  v4d re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
  double np = 0.0, nq = 0.0;
  for (int k0 = 0; k0 < l; k0 += 16) {
    zt u[4], v[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * s + tk, kc = k < l ? k : l - 1;
      u[s] = cp[kc];
      v[s] = cq[kc];
      if (k >= l) u[s] = v[s] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {  // g = conj(u) v
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(u[s].x, v[s].x, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(u[s].x, v[s].y, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(u[s].y, v[s].y, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(-u[s].y, v[s].x, im, 0, 0, 0);
      np += zabs2(u[s]);
      nq += zabs2(v[s]);
    }
  }
  np += __shfl_xor(np, 16, 64);
  np += __shfl_xor(np, 32, 64);
  nq += __shfl_xor(nq, 16, 64);
  nq += __shfl_xor(nq, 32, 64);
  const double tol = DBL_EPSILON * sqrt(double(l));
  bool bad = false;
#pragma unroll
  for (int r = 0; r < 4; ++r) {  // entry (tk + 4 r, ti) of the tile
    const int row = tk + 4 * r;
    const double nr = __shfl(np, row, 64), g2 = re[r] * re[r] + im[r] * im[r];
    const bool pair = bi * 16 + row < q && q < l;
    bad |= pair && g2 > tol * tol * (nr * nq) && g2 != 0.0;
  }
  return __any(bad);
}

__global__ __launch_bounds__(256) void k_jac_check(Prob* probs, const int32_t* list, int nprob,
                                                   int blocks, int sweep) {
  const int tiles = blocks * blocks;
  const int items = (list[nprob] & kJacCountMask) * tiles;
  for (int it = blockIdx.x * 4 + wave_id(); it < items; it += gridDim.x * 4) {
    const int i = it / tiles, t = it - i * tiles, bi = t / blocks, bj = t - bi * blocks;
    Prob& P = probs[list[i]];
    const int bits = P.jac >> sweep;
    if (bi > bj || bj * 16 >= P.l || !(bits & 1) || (bits & (1 << 8)) || jac_done(P.jac, sweep))
      continue;
    if (jac_tile_bad(P, bi, bj) && (threadIdx.x & 63) == 0) atomicOr(&P.jac, 1 << (16 + sweep));
  }
}

// The rest of the iteration (all of it without the launches above: first = 0),
// one workgroup per problem, then the sorted outputs and the truncation.
// PAR block pairs of a round at a time (two as long as their LDS fits).
template <int REGS, int PAR>
__global__ __launch_bounds__(kJacThreads* PAR) void k_small_svd(Prob* probs, double eps, int tebd,
                                                                int32_t* retry_count, int first) {
  extern __shared__ zt lds[];
  constexpr int NT = kJacThreads * PAR;
  __shared__ JacShared sh[PAR];
  __shared__ double sig_s[kMaxL];
  __shared__ double scan[kMaxL];
  __shared__ int perm_s[kMaxL];
  Prob& P = probs[blockIdx.x];
  const int l = P.l;
  if (l == 0 || svd_class(l) < 2) return;
  const int nb = jac_blocks(l), blocks = (l + 15) / 16;
  bool converged = first > 0 && jac_done(P.jac, first);
  for (int sweep = first; sweep < kMaxSweeps && !converged; ++sweep) {
    int bits = 0;
    for (int round = 0; round < nb - 1; ++round)
      for (int k0 = 0; k0 < nb / 2; k0 += PAR) {
        const int g = wave_id() / kJacBlock, k = k0 + g;
        const bool any = k < nb / 2;  // else a pair of blocks beyond l
        bits |= jac_pair<REGS>(P, any ? circle_player(k, round, nb) : nb,
                               any ? circle_player(nb - 1 - k, round, nb) : nb + 1, round,
                               sweep == 0 && round == 0, wave_id() % kJacBlock,
                               lds + size_t(g) * 4 * kJacBlock * 64 * REGS, sh[g]);
      }
    bool bad = false;
    if (sweep >= kJacCheckFrom && bits == 1) {
      for (int t = wave_id(); t < blocks * blocks; t += NT / 64)
        if (t / blocks <= t % blocks) bad |= jac_tile_bad(P, t / blocks, t % blocks);
      bad = __syncthreads_or(bad) != 0;
    }
    converged = sweep_ended(bits & 1, bits >> 8 & 1 || bad, sweep);
  }
  if (!converged && threadIdx.x == 0) P.flags |= TEBD_DEV_JACOBI_NOCONV;
  jacobi_finish<NT>(P, P.C, P.J, l, sig_s, perm_s);
  truncate_tail<NT>(P, l, eps, tebd, retry_count, [&](int c) { return sig_s[perm_s[c]]; }, scan);
}

// LDS of one column of C and J.
size_t jac_column_bytes(int lmax) { return (lmax <= 128 ? 2 * 128 : 2 * 256) * sizeof(zt); }

// The launches of the wide small SVD (classes 2 and 3) for at most `count`
// problems of at most lmax columns.
void launch_jacobi_rounds(Prob* probs, const int32_t* list, int nprob, int count, int lmax,
                          hipStream_t s) {
  const int nb = jac_blocks(lmax), pairs = nb / 2;
  const int blocks = (lmax + 15) / 16;
  const int64_t items = int64_t(count) * pairs, tiles = int64_t(count) * blocks * blocks;
  const dim3 g(unsigned(items < 1024 ? items : 1024)), gt(unsigned(tiles < 4096 ? (tiles + 3) / 4 : 1024));
  const size_t column = jac_column_bytes(lmax);
  for (int sweep = 0; sweep < kJacSweeps; ++sweep) {
    for (int r = 0; r < nb - 1; ++r) {
      const size_t lds = (r == 0 ? 2 : 1) * kJacBlock * column;
      if (lmax <= 128)
        TEBD_LAUNCH("k_jac_round<2>", k_jac_round<2>, g, dim3(kJacThreads), lds, s, probs, list, nprob, pairs, sweep, r);
      else
        TEBD_LAUNCH("k_jac_round<4>", k_jac_round<4>, g, dim3(kJacThreads), lds, s, probs, list, nprob, pairs, sweep, r);
    }
    if (sweep >= kJacCheckFrom)
      TEBD_LAUNCH("k_jac_check", k_jac_check, gt, dim3(256), 0, s, probs, list, nprob, blocks, sweep);
  }
}

// The list lies where the queue of the Theta products was.
int32_t* jac_list(const Common& c) { return c.offs + size_t(TK_THETA) * (c.nprob + 1); }

// Classes 2 and 3 take launch_jacobi_rounds where the host can know that there
// are such problems: in a truncation of matrices by the widths it asked for,
// in a sweep that synchronises with the host by reading what the range finder
// revealed (15 us, against 0.3 ms of empty launches).  Sweeps that only
// enqueue know the capacity alone and keep to one launch.  A truncation, which
// does not wait for the device either, pays for the empty launches where its
// matrices turn out to be of rank 64 or less: 96 x 80 of rank 10 at l = 74 takes
// 411 us, 241 with one launch and Householder QRs; of full rank 72 x 72, l = 72
// 1.4 ms and 3.7; 256 x 256 of rank 10 0.85 and 2.05.
bool wide_svd(const Common& c) {
  return svd_class(c.lmax) >= 2 && (!c.tebd || c.adaptive >= 2);
}

hipError_t launch_wide_list(Prob* probs, const Common& c, const int32_t** found, hipStream_t s) {
  TEBD_LAUNCH("k_jac_list", k_jac_list, dim3(1), dim3(1024), 0, s, probs, c.nprob, jac_list(c));
  *found = jac_list(c) + c.nprob;
  return hipGetLastError();
}

void wide_found(Common& c, int32_t found) {
  c.wide_n = found & kJacCountMask;
  c.wide_l = found >> 22;
}

hipError_t launch_small_svd(Prob* probs, const Common& c, hipStream_t s) {
  static const hipError_t attr = []() {
    const struct {
      const void* fn;
      size_t elems;
    } lds[] = {{reinterpret_cast<const void*>(&k_small_svd<2, 2>), size_t(8 * kJacBlock * 128)},
               {reinterpret_cast<const void*>(&k_small_svd<4, 1>), size_t(4 * kJacBlock * 256)},
               {reinterpret_cast<const void*>(&k_svd_pairs<512, 1>), size_t(pair_lds(32, 4))},
               {reinterpret_cast<const void*>(&k_jac_round<2>), size_t(4 * kJacBlock * 128)},
               {reinterpret_cast<const void*>(&k_jac_round<4>), size_t(4 * kJacBlock * 256)}};
    for (const auto& f : lds) {
      const hipError_t e = hipFuncSetAttribute(f.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               int(f.elems * sizeof(zt)));
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }();
  if (attr != hipSuccess) return attr;
  // the problem's l here is the rank the range finder revealed
  const int lo = svd_class(c.lmin < 1 ? 1 : c.lmin);
  int hi = svd_class(c.lmax);
  int32_t* retry = c.pass2 ? nullptr : c.retry_count;
  const bool wide = c.wide_n > 0;
  if (c.wide_n == 0 && hi > 1) hi = 1;
  auto pairs0 = [&](hipStream_t t) {
    TEBD_LAUNCH("k_svd_pairs<256, 0>", (k_svd_pairs<256, 0>), dim3(c.nprob), dim3(256),
                pair_lds(16, 2) * sizeof(zt), t, probs, c.eps, c.tebd, retry);
  };
  auto pairs1 = [&](hipStream_t t) {
    TEBD_LAUNCH("k_svd_pairs<512, 1>", (k_svd_pairs<512, 1>), dim3(c.nprob), dim3(512),
                pair_lds(32, 4) * sizeof(zt), t, probs, c.eps, c.tebd, retry);
  };
  auto wider = [&](hipStream_t t) {
    if (wide) launch_jacobi_rounds(probs, jac_list(c), c.nprob, c.wide_n, c.wide_l, t);
    const int first = wide ? kJacSweeps : 0;
    const int l = wide ? c.wide_l : c.lmax;
    const size_t lds = 2 * kJacBlock * jac_column_bytes(l);
    if (l <= 128)
      TEBD_LAUNCH("k_small_svd<2, 2>", (k_small_svd<2, 2>), dim3(c.nprob), dim3(2 * kJacThreads), 2 * lds, t, probs, c.eps, c.tebd, retry, first);
    else
      TEBD_LAUNCH("k_small_svd<4, 1>", (k_small_svd<4, 1>), dim3(c.nprob), dim3(kJacThreads), lds, t, probs, c.eps, c.tebd, retry, first);
  };
  auto run = [&](int k, hipStream_t t) {
    if (k == 0)
      pairs0(t);
    else if (k == 1)
      pairs1(t);
    else
      wider(t);
  };
  struct Item {
    const decltype(run)* fn;
    int k;
    void operator()(hipStream_t t) const { (*fn)(k, t); }
  };
  Item items[3];
  int n = 0;
  for (int k = lo < 2 ? lo : 2; k <= (hi < 2 ? hi : 2); ++k) items[n++] = {&run, k};
  return fork_join(s, items, n, c);
}

}  // namespace tebd

extern "C" int32_t tebd_size_class(int32_t factorization, int32_t rows, int32_t l) {
  using namespace tebd;
  if (l < 1 || l > kMaxL) return -1;
  if (factorization == 0) return rows < 1 || rows > kMaxRows ? -1 : qr_class(rows, l);
  if (factorization == 1) return svd_class(l);
  return -1;
}
