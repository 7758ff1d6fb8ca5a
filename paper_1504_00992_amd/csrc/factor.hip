// Wavefront-level kernels of the RRSVD pipeline (one workgroup per problem):
// planning of a TEBD sweep, ||A||_F^2, Householder QR with explicit Q, and the
// Accuracy Check.
//
// Paper: Tamascelli, Rosenbach, Plenio, arXiv:1504.00992.  QR steps of Alg. 1
// (the paper leaves the QR method open; Householder reflections are used
// because the sketch of a TEBD Theta is often rank deficient; the QRs after
// the first are Gram-based, gramqr.hip), and the Accuracy Check of Sec. IV.
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "householder.hpp"
#include "sidestreams.hpp"
#include "kinds.hpp"
#include "zgemm.hpp"

namespace tebd {

// --------------------------------------------------------------------------
// TEBD sweep planning: one thread per (chain, bond of the parity), problems
// numbered chain-major.  Chains that share a bond's gate form gate groups
// (up to kGateGroup consecutive chains; their problems nb apart): the
// group's Theta matrices sit side by side in one row-major block, and one
// gate product covers all their columns, reading the gate once per output
// tile instead of once per chain.  The Theta blocks are laid out bond-major.
//
// Columns chi_l chi_r of chain ch in its gate group (0 when its bond or
// local dimensions are out of range: such a problem is skipped, and has no
// columns in the group).
__device__ __forceinline__ int group_cols(const tebd_mps& mps, int ch, int bond) {
  const int32_t* chi = mps.chi + size_t(ch) * (mps.n_sites + 1);
  const int cl = chi[bond], cm = chi[bond + 1], cr = chi[bond + 2], cap = mps.chi_max;
  const int dl = mps.d[bond], dr = mps.d[bond + 1];
  const bool ok = cl >= 1 && cl <= cap && cm >= 1 && cm <= cap && cr >= 1 && cr <= cap &&
                  dl >= 1 && dl <= mps.d_max && dr >= 1 && dr <= mps.d_max;
  return ok ? cl * cr : 0;
}

// Plan item t (the thread layout below) of a sweep: writes one descriptor.
// Called by whole wavefronts (the group sums are lane shuffles).
__device__ __forceinline__ void plan_item(int t, Prob* probs, int nprob, const tebd_mps& mps,
                                          const zt* gates, int64_t gate_chain_stride, int parity,
                                          int single_chain, int single_bond, int kcap, int p_over,
                                          char* slab_base, size_t slab_sz, int64_t mcap,
                                          int64_t ncap, int64_t lcap, int64_t lslab,
                                          int64_t npart_cap, double* disc, int32_t* status,
                                          double lambda_floor, int mixed, int adaptive, char* tape,
                                          size_t tape_stride, char* theta_base,
                                          size_t theta_stride, int chol) {
  // Items run group by group: a group's chains are the lanes of one aligned
  // kGateGroup-lane segment of a wavefront, so its column offsets are a
  // segmented prefix sum over the lanes.
  const int N = mps.n_sites, cap = mps.chi_max, dmax = mps.d_max;
  const int nb = (N - 1 - parity + 1) / 2;
  int chain, bond, bi = 0, p = 0;
  bool live;
  if (single_chain >= 0) {
    chain = single_chain;
    bond = single_bond;
    live = t == 0;
  } else {
    const int ncb = (mps.n_chains + kGateGroup - 1) / kGateGroup;
    const int g = t / kGateGroup;
    bi = g / ncb;
    chain = (g - bi * ncb) * kGateGroup + (t - g * kGateGroup);
    bond = parity + 2 * bi;
    live = bi < nb && chain < mps.n_chains;
    p = chain * nb + bi;
  }
  const int w = live ? group_cols(mps, chain, bond) : 0;
  int incl = w;
#pragma unroll
  for (int off = 1; off < kGateGroup; off <<= 1) {
    const int v = __shfl_up(incl, off, kGateGroup);
    if ((threadIdx.x & (kGateGroup - 1)) >= off) incl += v;
  }
  int gtot = __shfl(incl, kGateGroup - 1, kGateGroup), gcol0 = incl - w;
  // gate group: chains c0 .. c0 + gsz - 1 of this bond when they share the
  // gate, else this problem alone
  int c0 = chain, gsz = 1;
  if (single_chain < 0 && gate_chain_stride == 0) {
    c0 = chain / kGateGroup * kGateGroup;
    gsz = mps.n_chains - c0 < kGateGroup ? mps.n_chains - c0 : kGateGroup;
  } else {
    gcol0 = 0;
    gtot = w;
  }
  if (!live || p >= nprob) return;
  Prob P;
  const int32_t* chi = mps.chi + size_t(chain) * (N + 1);
  const int cl = chi[bond], cm = chi[bond + 1], cr = chi[bond + 2];
  const int dl = mps.d[bond], dr = mps.d[bond + 1];
  const bool bad = cl < 1 || cl > cap || cm < 1 || cm > cap || cr < 1 || cr > cap || dl < 1 ||
                   dl > dmax || dr < 1 || dr > dmax;
  P.chi_l = cl;
  P.chi_m = cm;
  P.chi_r = cr;
  P.dl = dl;
  P.dr = dr;
  P.m = dl * cl;
  P.n = dr * cr;
  int l2 = kcap + p_over;
  if (l2 > P.m) l2 = P.m;
  if (l2 > P.n) l2 = P.n;
  int k1 = kcap, l = l2;
  if (adaptive == 1 || adaptive == 2) {  // first stage: the current bond dimension plus a margin
    const int margin = (cm + 3) / 4 > 4 ? (cm + 3) / 4 : 4;
    k1 = cm + margin < kcap ? cm + margin : kcap;
    l = k1 + p_over;
    if (l > P.m) l = P.m;
    if (l > P.n) l = P.n;
  }
  P.ac_r = 0;
  P.ac_col = 0;
  P.ac_cap = l2;
  P.ac_grow = 0;
  P.chol_ok = 0;
  if (adaptive == 3) {  // Accuracy Check: from the current bond dimension, probes of p columns
    l = cm + p_over;
    if (l > P.m) l = P.m;
    if (l > P.n) l = P.n;
    P.ac_r = p_over < 1 ? 1 : (p_over > kAccMaxR ? kAccMaxR : p_over);
    P.ac_col = l;
    l2 = l;  // no second stage
  }
  P.l = bad ? 0 : l;
  P.k1 = k1;
  P.l1 = l;
  P.chol = bad ? 0 : gram_bits(P.m, P.n, l, chol != 0, chol != 0 || cm >= kcap || qr_class(P.m, l) >= 3, mixed != 0, true);
  P.l2 = l2;
  P.retry = 0;
  P.kcap = kcap;
  P.pid = chain * (N - 1) + bond;
  P.chi_new = 0;
  P.flags = bad ? TEBD_DEV_BAD_STATE : 0;
  P.npart = 0;
  P.mixed = mixed;
  P.om_ext = 0;
  P.frob2 = 0.0;
  carve_slab(P, slab_base + size_t(p) * slab_sz, mcap, ncap, lslab, 1, mixed, npart_cap);
  P.gcol0 = gcol0;
  P.gtot = gtot;
  P.gn = chain == c0 ? gsz : 0;
  P.gstride = nb;
  P.T = reinterpret_cast<zt*>(theta_base + (size_t(bi) * mps.n_chains + c0) * theta_stride);
  P.lda = P.n;
  P.ldom = P.l;
  P.U = nullptr;
  P.ldu = 0;
  P.S = nullptr;
  P.VH = nullptr;
  P.ldvh = 0;
  P.chi_out = nullptr;
  const size_t site_stride = size_t(dmax) * cap * cap;
  P.gk = mps.gamma ? reinterpret_cast<zt*>(mps.gamma) + (size_t(chain) * N + bond) * site_stride
                   : nullptr;
  P.gk1 = P.gk + site_stride;
  double* lam_chain = mps.lambda + size_t(chain) * (N - 1) * cap;
  P.lam_l = bond >= 1 ? lam_chain + size_t(bond - 1) * cap : nullptr;
  P.lam_mid = lam_chain + size_t(bond) * cap;
  P.lam_r = bond + 1 <= N - 2 ? lam_chain + size_t(bond + 1) * cap : nullptr;
  P.chi_slot = mps.chi + size_t(chain) * (N + 1) + bond + 1;
  // single-bond mode: `gates` is that bond's gate
  P.gate = single_chain >= 0 ? gates
                             : gates + size_t(chain) * gate_chain_stride +
                                   size_t(bond) * dmax * dmax * dmax * dmax;
  P.gate_ld = dmax * dmax;
  P.chi_cap = cap;
  P.lambda_floor = lambda_floor;
  if (tape) {
    tape_slot(tape + size_t(p) * tape_stride, mcap, lcap, P.tape_hdr, P.tape_sig, P.tape_u,
              P.tape_vh);
    P.tape_ldu = int32_t(lcap);
    P.tape_ldvh = int32_t(ncap);
  } else {
    P.tape_u = P.tape_vh = nullptr;
    P.tape_sig = nullptr;
    P.tape_hdr = nullptr;
    P.tape_ldu = P.tape_ldvh = 0;
  }
  if (single_chain >= 0) {
    P.disc = disc;
    P.status = status;
  } else {
    P.disc = disc + size_t(chain) * (N - 1) + bond;
    P.status = status + size_t(chain) * (N - 1) + bond;
  }
  probs[p] = P;
  if (bad) {
    *P.status = TEBD_DEV_BAD_STATE;
    *P.disc = 0.0;
  }
}

__global__ __launch_bounds__(64) void k_plan_sweep(
    Prob* probs, int nprob, tebd_mps mps, const zt* gates, int64_t gate_chain_stride, int parity,
    int single_chain, int single_bond, int kcap, int p_over, char* slab_base, size_t slab_sz,
    int64_t mcap, int64_t ncap, int64_t lcap, int64_t lslab, int64_t npart_cap, double* disc,
    int32_t* status, double lambda_floor, int mixed, int adaptive, char* tape, size_t tape_stride,
    int32_t* retry_count, char* theta_base, size_t theta_stride, int chol) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t == 0 && retry_count) {
    *retry_count = 0;
    retry_count[kAccCountSlot] = 0;  // the Accuracy Check's two round counters
    retry_count[kAccCountSlot + 1] = 0;
    retry_count[kAccCountSlot + 2] = 0;  // and its widest pass
  }
  plan_item(t, probs, nprob, mps, gates, gate_chain_stride, parity, single_chain, single_bond,
            kcap, p_over, slab_base, slab_sz, mcap, ncap, lcap, lslab, npart_cap, disc, status,
            lambda_floor, mixed, adaptive, tape, tape_stride, theta_base, theta_stride, chol);
}

hipError_t launch_plan_sweep(Prob* probs, const Common& c, const tebd_mps& mps, const zt* gates,
                             int64_t gate_chain_stride, int32_t parity, int32_t single_chain,
                             int32_t single_bond, int32_t p_over, char* slab_base,
                             size_t slab_sz, double* disc, int32_t* status, double lambda_floor,
                             int32_t mixed, int32_t adaptive, char* tape, size_t tape_stride,
                             int32_t* retry_count, int64_t lslab, char* theta_base,
                             size_t theta_stride, hipStream_t s) {
  const int64_t mcap = int64_t(c.dmax) * c.chimax;
  const int64_t lcap = c.lmax;
  const int64_t npart_cap = gate_partials_cap(c.dmax * c.dmax, c.chimax * c.chimax);
  // one kGateGroup-lane segment per (bond, block of kGateGroup chains)
  int64_t items = 1;
  if (single_chain < 0) {
    const int64_t nb = c.nprob / mps.n_chains, ncb = (mps.n_chains + kGateGroup - 1) / kGateGroup;
    items = nb * ncb * kGateGroup;
  }
  static_assert(64 % kGateGroup == 0, "segments do not straddle wavefronts");
  TEBD_LAUNCH("k_plan_sweep", k_plan_sweep, dim3((items + 63) / 64), dim3(64), 0, s, probs,
              c.nprob, mps, gates, gate_chain_stride, parity, single_chain, single_bond, c.kcap,
              p_over, slab_base, slab_sz, mcap, mcap, lcap, lslab, npart_cap, disc, status,
              lambda_floor, mixed, adaptive, tape, tape_stride, retry_count, theta_base,
              theta_stride, c.chol);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// ||A||_F^2 for caller-supplied matrices (fixed summation order): workgroup
// (problem, slice) sums |A|^2 over its slice of rows (threads along the
// columns) into part[slice].  With the FP32 products it also writes the
// complex64 copy of A they read.
// A wavefront takes a row at a time, eight pieces of 64 elements in flight:
// there are 32 workgroups to a matrix only, so each has to keep its CU's
// share of the memory busy (two 4900 x 4900: 1470 us with one load in flight
// per thread, 263 us so).
constexpr int kFrobThreads = 1024;

__global__ __launch_bounds__(kFrobThreads) void k_frob(Prob* probs) {
  __shared__ double red[kFrobThreads / 64];
  const int pi = blockIdx.x / kFrobSlices, sl = blockIdx.x - pi * kFrobSlices;
  Prob& P = probs[pi];
  if (P.l == 0) return;
  const int rs = (P.m + kFrobSlices - 1) / kFrobSlices;
  const int r0 = sl * rs, r1 = r0 + rs < P.m ? r0 + rs : P.m;
  const int lane = threadIdx.x & 63;
  constexpr int U = 8;
  double s = 0.0;
  for (int r = r0 + wave_id(); r < r1; r += kFrobThreads / 64) {
    const zt* row = P.A + size_t(r) * P.lda;
    float2* rowf = P.Af ? P.Af + size_t(r) * P.n : nullptr;
    for (int c0 = lane; c0 < P.n; c0 += 64 * U) {
      zt v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + 64 * u;
        v[u] = row[c < P.n ? c : P.n - 1];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + 64 * u;
        if (c >= P.n) break;
        s += zabs2(v[u]);
        if (rowf) rowf[c] = make_float2(float(v[u].x), float(v[u].y));
      }
    }
  }
  s = block_sum<kFrobThreads>(s, red);
  if (threadIdx.x == 0) P.part[sl] = s;
}

hipError_t launch_frob(Prob* probs, const Common& c, hipStream_t s) {
  TEBD_LAUNCH("k_frob", k_frob, dim3(c.nprob * kFrobSlices), dim3(kFrobThreads), 0, s,
              probs);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// A problem a gated QR launch leaves alone: gate 1 runs only the bases the
// Accuracy Check grew; gate 2 only what the Gram-based QR did not finish.
__device__ __forceinline__ bool qr_gated(const Prob& P, int gate) {
  return (gate == 1 && !P.ac_grow) || (gate == 2 && P.chol_ok);
}

// Register-resident QR.  Column c of the rows x l matrix belongs to a group
// of G lanes (G = NT / l rounded up to a power of two, at most 32, so a
// group never straddles wavefronts); lane h of the group keeps rows h,
// h + G, ... of the column in registers.  Dot products, updates and
// trailing norms of a column are register arithmetic plus a DPP sum over
// the group; only the reflector is broadcast through LDS, where all groups
// read the same G addresses at a time.  The reflector buffer holds zeros
// outside the reflector's rows, so the row loops run without branches (their
// LDS loads overlap) and rows outside [j, rows) are left exactly unchanged.
//
// Columns never move.  Pivoting picks the unfactored group first in
// pivot_key order, over the positions the swaps of qr_core would have
// produced (each group tracks its own): every trailing group posts its key
// in LDS, and after the barrier each wavefront takes their maximum.  The
// pivot group is recorded as logical column j; R, the pivot order and the
// thin Q are written out in logical order.  Same reflectors (stored
// unnormalised), pivoting rule and rank tolerance as qr_core.
// With pivoting, two barriers per factorisation step (trailing norms,
// reflector); without, one.  Every reflector keeps an LDS slot of its own
// when they all fit (always for 512 threads x 8 rows), and then each group
// accumulates its column of Q with no barrier at all; otherwise two
// alternating buffers serve, and the backward accumulation takes one
// barrier per step.
template <int RPL>
struct RegQrShared {
  // rows x l elements always fit for 512 x 8; 144 KiB for 1024 x 12
  static constexpr int kBuf = RPL <= 8 ? 4096 : 9216;
  zt buf[kBuf];  // reflector slots (zero outside the reflector's rows)
  zt rdiag[kMaxL];
  double tau_s[kMaxL];              // tau of each reflector (H = I - tau v v^H)
  unsigned long long key_s[kMaxL];  // pivot key of each group; 0 once pivoted
  int32_t piv_grp[kMaxL];
};

// The body for one group width G and RPL rows per lane (compile-time
// constants, so the row offsets of the register loops are immediates; RPL
// may be below the class's RS when the rows fit, which shortens every
// register loop); SLOTS: every reflector keeps its own slot
// (G * RPL * l <= RegQrShared<RS>::kBuf); PIV: column pivoting.
template <int NT, int RPL, int G, bool SLOTS, bool PIV, int RS>
__device__ __forceinline__ void qr_reg_body(Prob& P, int rows, int l, zt* Yg, int want_r,
                                            RegQrShared<RS>& sh) {
  constexpr bool piv = PIV;
  constexpr int UST = G * RPL;               // rows a group can hold
  constexpr int KEEP = RPL <= 8 ? RPL : 1;  // reflector rows kept in registers
  auto& rdiag = sh.rdiag;
  auto& key_s = sh.key_s;
  auto& piv_grp = sh.piv_grp;
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = tid / G, h = tid - g * G;
  const bool have = g < l;
  // the QR of B^H keeps every column; without pivoting no rank is revealed
  const bool allow_stop = piv && !want_r;
  const zt zero = make_double2(0.0, 0.0);
  // reflector j: slot j, or the alternating buffers
  constexpr bool slots = SLOTS;
  auto slot = [&](int j) { return sh.buf + (slots ? j : (j & 1)) * UST; };
  zt y[RPL];
  double nn = 0.0;
#pragma unroll
  for (int i = 0; i < RPL; ++i) {
    const int r = h + G * i;
    y[i] = zload_if(have && r < rows, Yg + size_t(g) * rows + r);
    nn += zabs2(y[i]);
  }
  nn = group_sum(nn, G);
  for (int c = tid; c < l; c += NT) piv_grp[c] = c;
  if (piv && have && h == 0) key_s[g] = pivot_key(nn, g, g);
  __syncthreads();
  // trailing norm (rows >= the next step) and position of this group
  double my_tn = nn;
  int my_pos = g;
  int mine = kMaxL;  // logical column of this group once it has been the pivot
  // Reflectors are kept unnormalised, H_j = I - tau_j v v^H with
  // v = x - beta e_j (x: the column at step j, zero above row j) and
  // tau_j = 2 / ||v||^2 = 1 / (||x|| (||x|| + |x_j|)): rows > j of v are the
  // column itself, so they are written before beta and tau are known.  The
  // group of logical column j keeps x unscaled in its registers and v_j, tau_j
  // in my_v0, my_tau.
  double my_tau = 0.0;
  zt my_v0 = zero;
  // rows > j of v into buffer ub, zeros elsewhere in the group's range (so no
  // earlier reflector survives in the buffer)
  auto write_v = [&](zt* ub, int j) {
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const bool on = h + G * i > j && h + G * i < rows;
      zt w;
      w.x = on ? y[i].x : 0.0;
      w.y = on ? y[i].y : 0.0;
      ub[h + G * i] = w;
    }
  };
  // The rest of reflector j from the column of group p (pn = ||column p,
  // rows >= j||), called by the whole group p after write_v: row j of v,
  // tau_j and R_jj = beta.
  auto finish_reflector = [&](int j, int p, double pn, zt* ub) {
    // row j sits in register j / G of the group's lane j % G (uniform)
    const int i0 = j / G, hj = j - i0 * G, lj = (p * G + hj) & 63;
    double ax = 0.0, ay = 0.0;
#pragma unroll
    for (int i = 0; i < RPL; ++i)
      if (i == i0) {
        ax = read_lane(y[i].x, lj);
        ay = read_lane(y[i].y, lj);
      }
    const zt alpha = make_double2(ax, ay);
    const double a2 = zabs2(alpha);
    const double ia = a2 > 0.0 ? rsqrt(a2) : 0.0;  // 1 / |alpha|
    const double aa = a2 * ia;
    const double xnorm = pn;
    zt beta = zero, v0 = zero;
    double tau = 0.0;
    if (xnorm > 0.0) {
      const zt ph = aa > 0.0 ? zscale(alpha, ia) : make_double2(1.0, 0.0);
      beta = zscale(ph, -xnorm);
      v0 = zsub(alpha, beta);
      tau = 1.0 / (xnorm * (xnorm + aa));
    }
    if (h == hj) ub[j] = v0;
    if (h == 0) {
      rdiag[j] = beta;
      sh.tau_s[j] = tau;
    }
    my_tau = tau;
    my_v0 = v0;
    mine = j;
  };
  auto reflector = [&](int j, int p, double pn, zt* ub) {
    write_v(ub, j);
    finish_reflector(j, p, pn, ub);
  };
  // trailing column: y -= tau_j v (v^H y) with v in ub, zero outside its
  // rows; with want_norm (uniform over the wavefront) the norm of rows > j is
  // returned (else 0); with vout (the next reflector's group) rows > j + 1 of
  // the updated column are written there as the next v, before the norm is
  // reduced
  auto apply = [&](const zt* ub, int j, bool want_norm, zt* vout) {
    const double tau = sh.tau_s[j];
    zt uu[KEEP];  // v kept in registers between the two loops when they fit
    double dr0 = 0.0, di0 = 0.0, dr1 = 0.0, di1 = 0.0;
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const zt u = ub[h + G * i];
      if (i < KEEP) uu[i < KEEP ? i : 0] = u;
      if (i & 1)
        zdot_acc(u, y[i], dr1, di1);
      else
        zdot_acc(u, y[i], dr0, di0);
    }
    const double dr = group_sum(dr0 + dr1, G), di = group_sum(di0 + di1, G);
    const zt d2 = make_double2(tau * dr, tau * di);
    // without the kept copy, the second read of u must not be hoisted
    // above this point (it would hold every row twice in registers)
    if (KEEP < RPL) __builtin_amdgcn_sched_barrier(0);
    double tn = 0.0;
    if (want_norm) {
      double tn0 = 0.0, tn1 = 0.0;
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int r = h + G * i;
        const zt u = i < KEEP ? uu[i < KEEP ? i : 0] : ub[r];
        y[i] = zsub_mul(y[i], u, d2);
        const double yx = r > j ? y[i].x : 0.0, yy = r > j ? y[i].y : 0.0;
        if (i & 1)
          tn1 = fma(yx, yx, fma(yy, yy, tn1));
        else
          tn0 = fma(yx, yx, fma(yy, yy, tn0));
      }
      if (vout) write_v(vout, j + 1);
      tn = group_sum(tn0 + tn1, G);
    } else {
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const zt u = i < KEEP ? uu[i < KEEP ? i : 0] : ub[h + G * i];
        y[i] = zsub_mul(y[i], u, d2);
      }
    }
    return tn;
  };
  int rank = l;
  if constexpr (!piv) {
    // Logical column j is group j, which builds reflector j as soon as its
    // own update by reflector j - 1 is done (with its trailing norm summed
    // in the same pass), while the other groups are still applying j - 1;
    // reflector j + 1 goes to another slot or buffer than reflector j, so
    // one barrier per step suffices.
    if (g == 0) reflector(0, 0, sqrt(nn), slot(0));
    __syncthreads();
    for (int j = 0; j + 1 < l; ++j) {
      if (have && g > j) {
        // the wavefront that holds group j + 1 sums trailing norms
        const bool lead = (tid >> 6) == (((j + 1) * G) >> 6);
        const double tn = apply(slot(j), j, lead, g == j + 1 ? slot(j + 1) : nullptr);
        if (g == j + 1) finish_reflector(j + 1, g, sqrt(tn), slot(j + 1));
      }
      __syncthreads();  // reflector j + 1 is published; reflector j is read
    }
  }
  double best00 = 0.0;  // squared pivot norm of step 0
  for (int j = 0; piv && j < l; ++j) {
    unsigned long long key = 0ull;
    for (int c = lane; c < l; c += 64) key = key_max(key, key_s[c]);
    key = key_wave_max(key);
    if (key == 0ull) {  // only NaN norms left: stop here
      rank = j;
      break;
    }
    const int p = static_cast<int>(key & 0xff), pp = pivot_key_pos(key);
    const double best = pivot_key_norm(key);  // |R_jj|^2 to 2^-36
    if (j == 0) best00 = best;
    if (allow_stop && j > 0 && !(best > kRankTol * kRankTol * best00)) {
      rank = j;
      break;
    }
    if (g == p) reflector(j, p, sqrt(my_tn), slot(j));
    __syncthreads();  // reflector j is published; every key read is done
    if (tid == 0) piv_grp[j] = p;
    if (have && mine == kMaxL) {
      if (my_pos == j) my_pos = pp;  // the swap of qr_core moves it to the pivot's place
      my_tn = apply(slot(j), j, true, nullptr);
      if (h == 0) key_s[g] = pivot_key(my_tn, my_pos, g);
    }
    if (g == p && h == 0) key_s[g] = 0ull;
    __syncthreads();  // the keys of step j + 1 are in
  }
  if (want_r) {
    if (have && mine < rank) {
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int r = h + G * i;
        if (r < rank) {  // value selects only (no select between addresses)
          const zt d = rdiag[r];
          const bool up = r < mine, dg = r == mine;
          zt v;
          v.x = up ? y[i].x : (dg ? d.x : 0.0);
          v.y = up ? y[i].y : (dg ? d.y : 0.0);
          P.Rb[size_t(mine) * rank + r] = v;
        }
      }
    }
    for (int c = tid; c < rank; c += NT) P.piv[c] = piv_grp[c];
  }
  // Q = H_0 ... H_{r-1} [I; 0]: the group of logical column c < rank starts
  // from H_c e_c = e_c - tau_c v_c conj(v_c[c]) and applies H_{c-1}, ..., H_0.
  // With a slot per reflector the groups need no barrier.  With the
  // alternating buffers, the group of column j publishes v_j one step
  // ahead, while H_{j+1} is being applied (column j is not touched by H_j or
  // later reflectors): one barrier per step.
  auto start_q = [&](zt* ub) {  // by the group with mine < rank; ub: publish v_c there
    const int c = mine, i0 = c / G, hc = c - i0 * G;
    // -tau_c conj(v_c[c])
    const zt m = make_double2(-my_tau * my_v0.x, my_tau * my_v0.y);
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const bool on = h + G * i > c && h + G * i < rows;
      zt w;
      w.x = on ? y[i].x : 0.0;
      w.y = on ? y[i].y : 0.0;
      if (ub) ub[h + G * i] = w;  // zeros outside [c, rows)
      y[i] = zmul(w, m);
    }
    if (ub && h == hc) ub[c] = my_v0;
#pragma unroll
    for (int i = 0; i < RPL; ++i)
      if (i == i0 && h == hc) {
        y[i] = zmul(my_v0, m);
        y[i].x += 1.0;
      }
  };
  if constexpr (slots) {
    // Every reflector keeps its slot, so any group can accumulate any column,
    // and column c costs c applications.  The columns go out in blocks of the
    // 64 / G groups of a wavefront, costliest block first, dealt to the four
    // SIMDs back and forth (SIMD 0 1 2 3 3 2 1 0 0 1 ..., wavefront w on SIMD
    // w mod 4, the k-th block of a SIMD to its k-th wavefront), so that the
    // SIMDs carry similar sums.  The start H_c e_c comes from slot c: its
    // rows > c are the column as it was when reflector c was built, row c
    // holds v_c[c].  The same operations, in the same order, as when the
    // group of column c accumulates it.
    constexpr int GPW = 64 / G;
    const int nblk = (rank + GPW - 1) / GPW;
    const int wv = tid >> 6, kq = wv >> 2, sq = wv & 3;
    const int dq = 4 * kq + ((kq & 1) ? 3 - sq : sq);  // deal position of this wavefront
    const int qc = dq < nblk ? (nblk - 1 - dq) * GPW + g % GPW : rank;
    if (qc < rank) {
      const zt* vs = slot(qc);
      const zt v0 = vs[qc];
      const double tau = sh.tau_s[qc];
      const zt m = make_double2(-tau * v0.x, tau * v0.y);  // -tau_c conj(v_c[c])
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int r = h + G * i;
        y[i] = zmul(zload_if(r > qc && r < rows, vs + r), m);
        if (r == qc) {
          y[i] = zmul(v0, m);
          y[i].x += 1.0;
        }
      }
      for (int j = qc - 1; j >= 0; --j) apply(slot(j), j, false, nullptr);
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int r = h + G * i;
        if (r < rows) Yg[size_t(qc) * rows + r] = y[i];
      }
    }
  } else {
    if (rank > 0 && mine == rank - 1) start_q(slot(rank - 1));
    for (int j = rank - 1; j >= 0; --j) {
      __syncthreads();  // v_j is published; the reads of the other buffer are done
      if (j > 0 && mine == j - 1) start_q(slot(j - 1));
      if (have && mine > j && mine < rank) apply(slot(j), j, false, nullptr);
    }
    if (have && mine < rank) {
#pragma unroll
      for (int i = 0; i < RPL; ++i) {
        const int r = h + G * i;
        if (r < rows) Yg[size_t(mine) * rows + r] = y[i];
      }
    }
  }
  if (tid == 0) P.l = rank;
}

template <int NT, int RPL, bool PIV>
__global__ __launch_bounds__(NT) void k_qr_reg(Prob* probs, int which, int want_r, int cls,
                                                 int gate) {
  __shared__ RegQrShared<RPL> sh;
  Prob& P = probs[blockIdx.x];
  const int l = P.l;
  const int rows = which ? P.n : P.m;
  // class from the width the pass started with: P.l shrinks as QRs run
  if (l == 0 || qr_class(rows, P.l1) != cls || qr_gated(P, gate)) return;
  zt* Yg = which ? P.Yt : P.Y;
  // l <= kMaxL, so G >= NT / kMaxL
  static_assert(NT / kMaxL >= 2, "group widths below 2 are not instantiated");
  const int G = reg_group(NT, l);
  auto run = [&](auto gc) {
    constexpr int GC = decltype(gc)::value, HALF = RPL / 2;
    // the revealed rank of the later QRs of a pass is often below the width
    // that set the class: G doubles, and half the rows per lane may do
    if (rows <= GC * HALF) {
      // G * HALF * l <= NT * HALF <= kBuf: every reflector has its slot
      static_assert(NT * HALF <= RegQrShared<RPL>::kBuf, "slots for the half-height body");
      qr_reg_body<NT, HALF, GC, true, PIV>(P, rows, l, Yg, want_r, sh);
    } else if (RPL <= 8 || GC * RPL * l <= RegQrShared<RPL>::kBuf) {
      // 512 x 8: G * 8 * l <= 4096 for every l (G * l <= 512, or G = 32 and l <= 16)
      qr_reg_body<NT, RPL, GC, true, PIV>(P, rows, l, Yg, want_r, sh);
    } else {
      qr_reg_body<NT, RPL, GC, (RPL <= 8), PIV>(P, rows, l, Yg, want_r, sh);
    }
  };
  if (G == 32)
    run(std::integral_constant<int, 32>());
  else if (G == 16)
    run(std::integral_constant<int, 16>());
  else if (G == 8)
    run(std::integral_constant<int, 8>());
  else if (NT / kMaxL <= 4 && G == 4)
    run(std::integral_constant<int, (NT / kMaxL <= 4 ? 4 : 8)>());
  else if (NT / kMaxL <= 2)
    run(std::integral_constant<int, (NT / kMaxL <= 2 ? 2 : 8)>());
}

// Class 2, (l + 2) * rows <= kLdsElems beyond the register classes:
// qr_core's column ownership with 1024 threads (one wavefront per column at
// a time), the matrix in up to 150 KiB of LDS.
template <int NT>
__global__ __launch_bounds__(NT) void k_qr_lds(Prob* probs, int which, int want_r, int pivot,
                                                 int gate) {
  extern __shared__ zt lds[];  // rows * l matrix, then 2 * rows for u
  __shared__ zt rdiag[kMaxL];
  Prob& P = probs[blockIdx.x];
  const int l = P.l;
  const int rows = which ? P.n : P.m;
  if (l == 0 || qr_class(rows, P.l1) != 2 || qr_gated(P, gate)) return;
  __shared__ double nrm[2 * kMaxL];
  __shared__ int sh_i[2];
  zt* Yg = which ? P.Yt : P.Y;
  const int tot = rows * l;
  for (int e = threadIdx.x; e < tot; e += NT) lds[e] = Yg[e];
  __syncthreads();
  __shared__ int32_t perm_s[kMaxL];
  for (int c = threadIdx.x; c < l; c += NT) perm_s[c] = c;
  __syncthreads();
  const int rank = qr_core<NT, 0>(lds, rows, l, lds + tot, rdiag, want_r ? P.Rb : nullptr,
                                  pivot != 0, pivot != 0 && !want_r, want_r ? perm_s : nullptr, nrm,
                                  sh_i);
  if (want_r)
    for (int c = threadIdx.x; c < l; c += NT) P.piv[c] = perm_s[c];
  const int keep = rows * rank;
  for (int e = threadIdx.x; e < keep; e += NT) Yg[e] = lds[e];
  if (threadIdx.x == 0) P.l = rank;
}

// Class 3, everything larger, runs on global memory (L2-resident) with
// 1024 threads, qr_core's column ownership, and each column held in
// registers between its dot product and its update.
// The two reflector buffers live in LDS up to kGlbLdsRows rows (147 KiB)
// and in the problem's slab beyond.
constexpr int kGlbLdsRows = 4608;

template <int NT>
__global__ __launch_bounds__(NT) void k_qr_glb(Prob* probs, int which, int want_r, int pivot,
                                                 int gate) {
  extern __shared__ zt u_lds[];  // 2 * min(rows, kGlbLdsRows)
  __shared__ zt rdiag[kMaxL];
  Prob& P = probs[blockIdx.x];
  const int l = P.l;
  const int rows = which ? P.n : P.m;
  if (l == 0 || qr_class(rows, P.l1) != 3 || qr_gated(P, gate)) return;
  zt* u_s = rows <= kGlbLdsRows ? u_lds : P.qru;
  __shared__ double nrm[2 * kMaxL];
  __shared__ int sh_i[2];
  __shared__ int32_t perm_s[kMaxL];
  for (int c = threadIdx.x; c < l; c += NT) perm_s[c] = c;
  __syncthreads();
  const int rank = qr_core<NT, kRegRows>(which ? P.Yt : P.Y, rows, l, u_s, rdiag,
                                         want_r ? P.Rb : nullptr, pivot != 0,
                                         pivot != 0 && !want_r, want_r ? perm_s : nullptr, nrm,
                                         sh_i);
  if (want_r)
    for (int c = threadIdx.x; c < l; c += NT) P.piv[c] = perm_s[c];
  if (threadIdx.x == 0) P.l = rank;
}

hipError_t launch_qr(Prob* probs, const Common& c, int which, int want_r, int pivot,
                     hipStream_t s, int gate) {
  const int rows_max = which ? c.nmax : c.mmax;
  const int rows_min = which ? c.nmin : c.mmin;
  static const hipError_t attr = []() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_qr_glb<1024>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       int(2 * size_t(kGlbLdsRows) * sizeof(zt)));
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_qr_lds<1024>),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               int(size_t(kLdsElems) * sizeof(zt)));
  }();
  if (attr != hipSuccess) return attr;
  typedef void (*Launch)(hipStream_t, Prob*, int, int, int, int, int, int);
  struct Item {
    Launch fn;
    Prob* probs;
    int which, want_r, pivot, nprob, rows, grow;
    void operator()(hipStream_t t) const { fn(t, probs, which, want_r, pivot, nprob, rows, grow); }
  };
  const Launch fns[4] = {
      [](hipStream_t t, Prob* p, int w, int r, int v, int np, int, int g) {
        if (v)
          TEBD_LAUNCH("k_qr_reg<512, 8, true>", (k_qr_reg<512, 8, true>), dim3(np), dim3(512), 0, t, p, w, r, 0, g);
        else
          TEBD_LAUNCH("k_qr_reg<512, 8, false>", (k_qr_reg<512, 8, false>), dim3(np), dim3(512), 0, t, p, w, r, 0, g);
      },
      [](hipStream_t t, Prob* p, int w, int r, int v, int np, int, int g) {
        if (v)
          TEBD_LAUNCH("k_qr_reg<1024, 12, true>", (k_qr_reg<1024, 12, true>), dim3(np), dim3(1024), 0, t, p, w, r, 1, g);
        else
          TEBD_LAUNCH("k_qr_reg<1024, 12, false>", (k_qr_reg<1024, 12, false>), dim3(np), dim3(1024), 0, t, p, w, r, 1, g);
      },
      [](hipStream_t t, Prob* p, int w, int r, int v, int np, int, int g) {
        TEBD_LAUNCH("k_qr_lds<1024>", k_qr_lds<1024>, dim3(np), dim3(1024), size_t(kLdsElems) * sizeof(zt),
                           t, p, w, r, v, g);
      },
      [](hipStream_t t, Prob* p, int w, int r, int v, int np, int rw, int g) {
        TEBD_LAUNCH("k_qr_glb<1024>", k_qr_glb<1024>, dim3(np), dim3(1024),
                    2 * size_t(rw < kGlbLdsRows ? rw : kGlbLdsRows) * sizeof(zt), t,
                           p, w, r, v, g);
      }};
  // the classes between those of the smallest and the largest possible size
  int lo = qr_class(rows_min, c.lmin);
  const int hi = qr_class(rows_max, c.lmax);
  // gate 2 of a QR that every sketch took the Gram in: only sketches of the
  // tile queue's size may be left, in their classes
  if (gate == 2 && !pivot && !c.mixed) {
    int least = 3;
    for (int l = c.lmin; l <= c.lmax && least > lo; ++l) {
      const int rows = std::max(rows_min, gram_queue_rows(l));
      if (rows <= rows_max) least = std::min(least, qr_class(rows, l));
    }
    lo = std::min(std::max(lo, least), hi);
  }
  Item items[4];
  int n = 0;
  for (int k = lo; k <= hi; ++k)
    items[n++] = {fns[k], probs, which, want_r, pivot, c.nprob, rows_max, gate};
  return fork_join(s, items, n, c);
}

// --------------------------------------------------------------------------
// Accuracy Check (Sec. IV, Alg. 2), one workgroup per problem still probing:
// with Q the current basis (columns 0..l-1 of Y) and B = A Omega_r in the
// next r columns, D = B - Q (Q^H B) and MAX = max_i ||d_i||.  Theorem 2 with
// Fact 1 bounds the Frobenius residual ||(I - QQ^H) A||_F by (10/3) pi MAX
// (with probability 1 - 10^-r), so MAX is compared with
// tol = sqrt(eps) ||A||_F / ((10/3) pi), eps the relative discarded weight.
// MAX > tol: the basis takes B's first min(r, cap - l) columns (its QR runs
// next, grow_only), or, with no room left, the check stops with
// TEBD_DEV_ACC_CAPPED.  The check goes on while MAX > tol and l <= n - r;
// problems still probing are counted in count[round & 1] for the host, and
// count[(round + 1) & 1] is cleared for the next round.
// Both products are a tile wide (r <= 16) and run on the matrix cores, a tile
// per wavefront straight from memory: 22.7 us a round with a wavefront per
// column and a thread per row (a sweep of 4 x 40 spin-boson sites), 6.9 us so.
__global__ __launch_bounds__(256) void k_acc_resid(Prob* probs, double eps, int32_t* count,
                                                   int round) {
  Prob& P = probs[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0 && tid == 0) count[(round + 1) & 1] = 0;
  const int l = P.l, r = P.ac_r;
  if (l == 0 || r == 0) {
    if (tid == 0) P.ac_grow = 0;
    return;
  }
  const int m = P.m, ti = lane & 15, tk = lane >> 4;
  const zt* Q = P.Y;
  const zt* B = P.Y + size_t(l) * m;
  __shared__ zt cs[kMaxL * kAccMaxR];  // C = Q^H B, l x r, column j of Q in row j
  __shared__ double part[4][kAccMaxR], frob_s[64];
  static_assert(kAccMaxR <= 16, "the probes are one tile wide");
  const int npart = gate_partials(P.dl * P.dr, P.gcol0, P.chi_l * P.chi_r);
  if (wave == 3 && lane < npart) frob_s[lane] = P.part[lane];
  const zt zero = make_double2(0.0, 0.0);
  const zt* bi = B + size_t(ti < r ? ti : r - 1) * m;
  // one wavefront per 16 columns of Q
  for (int j0 = 16 * wave; j0 < l; j0 += 64) {
    const zt* qj = Q + size_t(j0 + ti < l ? j0 + ti : l - 1) * m;
    v4d re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < m; k0 += 16) {
      zt u[4], v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = k0 + 4 * t + tk, kc = k < m ? k : m - 1;
        u[t] = qj[kc];
        v[t] = bi[kc];
        if (k >= m) u[t] = v[t] = zero;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {  // conj(u) v
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t].x, v[t].x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t].x, v[t].y, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t].y, v[t].y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(-u[t].y, v[t].x, im, 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + tk + 4 * q;
      if (j < l && ti < r) cs[j * kAccMaxR + ti] = make_double2(re[q], im[q]);
    }
  }
  __syncthreads();
  // 16 rows of D = B - Q C per wavefront
  double nrm = 0.0;  // of column ti, this lane's rows
  for (int r0 = 16 * wave; r0 < m; r0 += 64) {
    const zt* qr = Q + (r0 + ti < m ? r0 + ti : m - 1);
    v4d re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    zt d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = r0 + tk + 4 * q;
      d[q] = bi[row < m ? row : m - 1];
    }
    for (int k0 = 0; k0 < l; k0 += 16) {
      zt u[4], v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = k0 + 4 * t + tk, kc = k < l ? k : l - 1;
        u[t] = qr[size_t(kc) * m];
        v[t] = cs[kc * kAccMaxR + (ti < r ? ti : r - 1)];
        if (k >= l) u[t] = v[t] = zero;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t].x, v[t].x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t].x, v[t].y, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-u[t].y, v[t].y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t].y, v[t].x, im, 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const zt v = make_double2(d[q].x - re[q], d[q].y - im[q]);
      if (r0 + tk + 4 * q < m) nrm += zabs2(v);
    }
  }
  nrm += __shfl_xor(nrm, 16, 64);
  nrm += __shfl_xor(nrm, 32, 64);
  if (lane < r) part[wave][lane] = nrm;
  __syncthreads();
  if (tid != 0) return;
  double mx = 0.0;
  bool finite = true;
  for (int i = 0; i < r; ++i) {
    const double v = (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
    finite = finite && isfinite(v);
    mx = fmax(mx, sqrt(v));
  }
  double frob2 = 0.0;
  for (int i = 0; i < npart; ++i) frob2 += i < 64 ? frob_s[i] : P.part[i];
  const double tol = sqrt(eps) * sqrt(frob2) / kAccConst;
  const bool grow = finite && mx > tol;
  int lnew = l;
  P.ac_grow = 0;
  if (!finite) P.flags |= TEBD_DEV_NONFINITE;
  if (grow) {
    const int w = P.ac_cap - l < r ? P.ac_cap - l : r;
    if (w <= 0) {
      P.flags |= TEBD_DEV_ACC_CAPPED;
      P.ac_r = 0;
      atomicMax(count + 2, P.l1);
      return;
    }
    lnew = l + w;
    P.l = lnew;
    if (P.l1 < lnew) P.l1 = lnew;
    P.ac_grow = 1;
  }
  P.ac_col += r;
  atomicMax(count + 2, P.l1);  // the widest pass so far (it sets the QR classes of later launches)
  if (grow && lnew <= P.n - r)
    atomicAdd(count + (round & 1), 1);
  else
    P.ac_r = 0;
}

hipError_t launch_acc_resid(Prob* probs, const Common& c, int round, hipStream_t s) {
  TEBD_LAUNCH("k_acc_resid", k_acc_resid, dim3(c.nprob), dim3(256), 0, s, probs, c.eps,
              c.acc_count, round);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Adaptive rank, between the passes: problems whose first stage was rejected
// get the fixed-rank width (and are marked), every other problem is skipped.
__global__ void k_stage2(Prob* probs, int nprob) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nprob) return;
  Prob& P = probs[p];
  if (P.retry) {
    P.l = P.l2;
    P.l1 = P.l2;
    P.k1 = P.kcap;
    P.ldom = P.l2;
    P.retry = 0;
    P.flags |= TEBD_DEV_RANK_RETRY;
  } else {
    P.l = 0;
  }
}

hipError_t launch_stage2(Prob* probs, const Common& c, hipStream_t s) {
  TEBD_LAUNCH("k_stage2", k_stage2, dim3((c.nprob + 63) / 64), dim3(64), 0, s, probs, c.nprob);
  return hipGetLastError();
}

}  // namespace tebd
