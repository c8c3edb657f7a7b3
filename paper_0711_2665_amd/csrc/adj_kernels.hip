// adj_kernels.hip -- reverse (adjoint) pass of the coupled step.
//
// The coupled step maps (A, r, v) -> (B, r', v') through four stages (gather,
// MD sub-cycle, spreading, LB sweep; Sec. 2).  Its transpose, applied to the
// adjoint (lam_B, lam_r', lam_v') of the step's output, gives the adjoint of
// its input and the contributions to dL/dgamma and dL/dF_drive:
//   LB^T      lam_f(x) = (dcoll/df)^T lam_B(x) [+ (du/df)^T lam_u(x) where a
//             bead stencil touches x], then lam_A = pull^T lam_f (each element
//             of A is pulled by exactly one (node, direction), so the
//             transpose is a scatter with one writer per element);
//   spread^T  lam_J_p = sum_k W_k lam_Fn(x_k), lam_Fn(x) = sum_i 3 w_i c_i
//             lam_B_i(x); d/dr of W_k gives a position term;
//   MD^T      the sub-steps in reverse; the force Jacobian enters as
//             (dF/dr)^T lam_F, which for conservative forces equals the
//             directional derivative of F along lam_F (evaluated with dual
//             numbers);
//   gather^T  lam_u(x_k) += W_k lam_up_p (summed per node like the forward
//             spreading), and d/dr of W_k gives a position term.
// The fields the reverse step needs (populations, r, v, u_p, J of the step)
// come from a tape written while the segment is recomputed from a checkpoint.
#include <type_traits>

#include "lbmd_kernels.h"
#include "lbmd_lattice.h"

namespace lbmd {

// ---------------------------------------------------------------------------
// Dual numbers: value and derivative along one direction.
// ---------------------------------------------------------------------------
struct Dd {
  double v, d;
};
__device__ inline Dd mkd(double v, double d = 0.0) { return Dd{v, d}; }
__device__ inline Dd operator+(Dd a, Dd b) { return Dd{a.v + b.v, a.d + b.d}; }
__device__ inline Dd operator-(Dd a, Dd b) { return Dd{a.v - b.v, a.d - b.d}; }
__device__ inline Dd operator-(Dd a) { return Dd{-a.v, -a.d}; }
__device__ inline Dd operator*(Dd a, Dd b) { return Dd{a.v * b.v, a.d * b.v + a.v * b.d}; }
__device__ inline Dd operator*(double s, Dd a) { return Dd{s * a.v, s * a.d}; }
__device__ inline Dd operator/(Dd a, Dd b) {
  double q = a.v / b.v;
  return Dd{q, (a.d - q * b.d) / b.v};
}
__device__ inline Dd dsqrt(Dd x) {
  double s = sqrt(x.v);
  return Dd{s, s > 0.0 ? x.d / (2.0 * s) : 0.0};
}
__device__ inline Dd datan2(Dd y, Dd x) {
  double den = x.v * x.v + y.v * y.v;
  return Dd{atan2(y.v, x.v), (x.v * y.d - y.v * x.d) / den};
}

// ---- force laws in dual arithmetic (the same expressions as the forward
// force laws; positions carry the direction in their derivative part) -----
__device__ inline void bond_dd(const MdParams& P, const Dd* rp, const Dd* rq, Dd F[3]) {
  Dd d0 = rp[0] - rq[0], d1 = rp[1] - rq[1], d2 = rp[2] - rq[2];
  Dd dist = dsqrt(d0 * d0 + d1 * d1 + d2 * d2);
  Dd coef = -(P.k_bond * (dist - mkd(P.r0))) / dist;
  F[0] = F[0] + coef * d0; F[1] = F[1] + coef * d1; F[2] = F[2] + coef * d2;
}

// Component a of the three vertex forces of the bending term (out[0] on
// the bead before the centre, out[1] on the centre, out[2] on the bead after
// it), each 0 + its term; 0 for a straight or folded angle.
__device__ inline void angle_dd_comp(const MdParams& P, const Dd* ra, const Dd* rb, const Dd* rc, int a,
                                     Dd out[3]) {
  out[0] = mkd(0.0); out[1] = mkd(0.0); out[2] = mkd(0.0);
  Dd b1[3] = {rb[0] - ra[0], rb[1] - ra[1], rb[2] - ra[2]};
  Dd b2[3] = {rc[0] - rb[0], rc[1] - rb[1], rc[2] - rb[2]};
  Dd n[3] = {b1[1] * b2[2] - b1[2] * b2[1], b1[2] * b2[0] - b1[0] * b2[2], b1[0] * b2[1] - b1[1] * b2[0]};
  Dd s = dsqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  Dd c = b1[0] * b2[0] + b1[1] * b2[1] + b1[2] * b2[2];
  if (s.v == 0.0) return;
  Dd phi = datan2(s, c);
  Dd den = s * s + c * c;
  Dd kp = P.kappa * phi;
  // component a of b2 x n and of n x b1 (constant indices in each branch)
  Dd g1, g2, b1a, b2a;
  if (a == 0) {
    g1 = b2[1] * n[2] - b2[2] * n[1]; g2 = n[1] * b1[2] - n[2] * b1[1]; b1a = b1[0]; b2a = b2[0];
  } else if (a == 1) {
    g1 = b2[2] * n[0] - b2[0] * n[2]; g2 = n[2] * b1[0] - n[0] * b1[2]; b1a = b1[1]; b2a = b2[1];
  } else {
    g1 = b2[0] * n[1] - b2[1] * n[0]; g2 = n[0] * b1[1] - n[1] * b1[0]; b1a = b1[2]; b2a = b2[2];
  }
  Dd d1 = (c * g1 / s - s * b2a) / den;
  Dd d2 = (c * g2 / s - s * b1a) / den;
  out[0] = out[0] + kp * d1;
  out[1] = out[1] + -(kp * (d1 - d2));
  out[2] = out[2] + -(kp * d2);
}

// The dual LJ force of one pair (separation d0, d1, d2), if within r_c.
__device__ inline bool lj_term(const MdParams& P, Dd d0, Dd d1, Dd d2, Dd t[3]) {
  Dd r2 = d0 * d0 + d1 * d1 + d2 * d2;
  if (!(r2.v < P.rc2)) return false;
  Dd sr2 = mkd(P.sig2) / r2;
  Dd sr6 = sr2 * sr2 * sr2;
  Dd sr12 = sr6 * sr6;
  Dd coef = P.eps24 * (2.0 * sr12 - sr6) / r2;
  t[0] = coef * d0; t[1] = coef * d1; t[2] = coef * d2;
  return true;
}
__device__ inline void lj_dd(const MdParams& P, Dd d0, Dd d1, Dd d2, Dd F[3]) {
  Dd t[3];
  if (!lj_term(P, d0, d1, d2, t)) return;
  F[0] = F[0] + t[0]; F[1] = F[1] + t[1]; F[2] = F[2] + t[2];
}

// Wall sites within r_c of the bead (r_c <= 3): the sites of the wall plane
// at offsets P.wlo..P.whi (1 - ceil(r_c)..ceil(r_c), within -2..3) around the
// base node, minus the pore block -- the rows outside hold no site within
// r_c, so the hit sites and their order are those of the full 6 x 6 window;
// the derivative of the wrapped position is that of r.  Sites are numbered
// row by row over the window; the caller's lane `part` of `nparts` stores
// the dual force of each of its sites (number part modulo nparts) within
// r_c in wv/wd and marks it in whit (0 for the others).
constexpr int ADJ_WIN = 36;   // sites in the largest window (a multiple of 4)
__device__ inline void wall_terms(const MdParams& P, const Geom& g, const Dd* rp, int part, int nparts,
                                  double (*wv)[3], double (*wd)[3], int8_t* whit) {
  const int nw = P.whi - P.wlo + 1;
  for (int num = part; num < nw * nw; num += nparts) whit[num] = 0;
  if (g.wall_axis < 0) return;
  const double w[3] = {wrapc(rp[0].v, g.nx), wrapc(rp[1].v, g.ny), wrapc(rp[2].v, g.nz)};
  const int b[3] = {(int)floor(w[0]), (int)floor(w[1]), (int)floor(w[2])};
  const int n[3] = {g.nx, g.ny, g.nz};
  const int a = g.wall_axis, t0 = g.t0, t1 = g.t1;
  int off = g.wall_pos - b[a];               // offset along the normal reaching the plane
  if (off < -2) off += n[a];
  if (off > 3) off -= n[a];
  if (off < P.wlo || off > P.whi) return;
  int site[3];
  site[a] = b[a] + off;
  for (int num = part; num < nw * nw; num += nparts) {
    const int o1 = P.wlo + num / nw, o0 = P.wlo + num % nw;
    const int u1 = b[t1] + o1;
    const int v1 = u1 < 0 ? u1 + n[t1] : (u1 >= n[t1] ? u1 - n[t1] : u1);
    const bool in1 = v1 >= g.lo1 && v1 <= g.hi1;
    const int u0 = b[t0] + o0;
    const int v0 = u0 < 0 ? u0 + n[t0] : (u0 >= n[t0] ? u0 - n[t0] : u0);
    const bool in0 = v0 >= g.lo0 && v0 <= g.hi0;
    if (in0 && in1) continue;              // pore node: fluid
    site[t0] = u0;
    site[t1] = u1;
    const double e0 = w[0] - (double)site[0], e1 = w[1] - (double)site[1], e2 = w[2] - (double)site[2];
    if (!(e0 * e0 + e1 * e1 + e2 * e2 < P.rc2)) continue;
    Dd t3[3];
    if (!lj_term(P, Dd{e0, rp[0].d}, Dd{e1, rp[1].d}, Dd{e2, rp[2].d}, t3)) continue;
    for (int c = 0; c < 3; ++c) { wv[num][c] = t3[c].v; wd[num][c] = t3[c].d; }
    whit[num] = 1;
  }
}

// ---------------------------------------------------------------------------
// Initial adjoint: lam_r = dL/dr(final), lam_v = dL/dv(final) or 0, lam_A = 0,
// parameter accumulators 0.
// ---------------------------------------------------------------------------
__global__ void k_adj_init(const double* __restrict__ dLdr, const double* __restrict__ dLdv, AdjBufs a, int n3) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n3) {
    a.lr[k] = dLdr[k];
    a.lv[k] = dLdv ? dLdv[k] : 0.0;
  }
  if (k < 4) a.par[k] = 0.0;
}

// d W_k / d r_a of the trilinear weight of corner k.
__device__ inline double dweight(const Stencil& s, int k, int a) {
  double w[3], dw[3];
  for (int b = 0; b < 3; ++b) {
    bool hi = (k >> b) & 1;
    w[b] = hi ? s.d[b] : 1.0 - s.d[b];
    dw[b] = hi ? 1.0 : -1.0;
  }
  return a == 0 ? dw[0] * w[1] * w[2] : (a == 1 ? w[0] * dw[1] * w[2] : w[0] * w[1] * dw[2]);
}

// 0 + the values of the group's eight lanes where on, in order, on every lane.
__device__ inline double corner_sum(double x, bool on) {
  const int base = threadIdx.x & 63 & ~7;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double y = __shfl(x, base + k, 64);
    if (__shfl(on ? 1 : 0, base + k, 64)) s += y;
  }
  return s;
}

// ---------------------------------------------------------------------------
// Spreading transpose, eight lanes per bead (one per corner; the terms are
// then added in corner order): lam_J and the position term of the spreading
// (J_p of the step from the tape).  With one thread per bead, the corners'
// loads one after the other, 22 us (the gather transpose 37) at 100 beads.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_adj_spread_t(const T* __restrict__ lamB, Dev d, AdjBufs a, const double* __restrict__ Jt, int nb) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, p = e >> 3, k = e & 7;
  if (e == 0) *a.lok = 0;                      // the list check of this step follows
  if (p >= nb) return;                         // whole groups of eight lanes
  const Rep& R = d.reps[0];
  const size_t N = (size_t)R.lp.N;
  double rp[3] = {d.rs[3 * p], d.rs[3 * p + 1], d.rs[3 * p + 2]};
  Stencil st = make_stencil(R.g, rp);
  double lJ[3] = {0.0, 0.0, 0.0}, lr[3] = {0.0, 0.0, 0.0};
  const double J[3] = {Jt[3 * p], Jt[3 * p + 1], Jt[3 * p + 2]};
  const int n = (int)corner_node(R.g, st, k);
  const bool fluid = !(d.flags[n] & F_SOLID);
  if (fluid) {
    double lf[Q];
    for (int i = 0; i < Q; ++i) lf[i] = (double)lamB[(size_t)i * N + n];
    double lF[3];
    lF[0] = 3.0 * (wgt(1) * (lf[1] - lf[2]) + wgt(7) * (lf[7] - lf[8] + lf[9] - lf[10] + lf[11] - lf[12] + lf[13] - lf[14]));
    lF[1] = 3.0 * (wgt(3) * (lf[3] - lf[4]) + wgt(7) * (lf[7] - lf[8] - lf[9] + lf[10] + lf[15] - lf[16] + lf[17] - lf[18]));
    lF[2] = 3.0 * (wgt(5) * (lf[5] - lf[6]) + wgt(11) * (lf[11] - lf[12] - lf[13] + lf[14] + lf[15] - lf[16] - lf[17] + lf[18]));
    double W = corner_weight(st, k);
    double JdotL = J[0] * lF[0] + J[1] * lF[1] + J[2] * lF[2];
    for (int b = 0; b < 3; ++b) {
      lJ[b] = W * lF[b];
      lr[b] = dweight(st, k, b) * JdotL;
    }
  }
  for (int b = 0; b < 3; ++b) {
    const double sJ = corner_sum(lJ[b], fluid), sr = corner_sum(lr[b], fluid);
    if (k == b) {
      a.lJ[3 * p + b] = sJ;
      a.lrs[3 * p + b] = sr;
    }
  }
}

// ---------------------------------------------------------------------------
// MD sub-cycle transpose.  Up to ADJ_CHAIN beads k_adj_terms and k_adj_chain,
// below; longer chains one launch per sub-step (in reverse order), four
// beads per three-wave workgroup.  The force positions r_mid and the
// velocities at the start of every sub-step come from the tape the forward
// sub-cycle wrote (while the segment was recomputed, or in the forward pass
// of a one-segment horizon).  On
// entry lr, lv hold the adjoint of r, v after the step and lJ that of the
// impulse J; the launches alternate between (lr, lv) and (lr2, lv2), so that
// a launch reads every bead's adjoint before the sub-step and writes the
// other pair; k_adj_md_fin leaves the adjoint of r_n, v_n through the
// sub-cycle in lr, lv.  lup collects the adjoint of u_p, gacc per bead the
// terms of dL/dgamma and dL/dF_drive, which k_adj_md_fin adds over the
// beads in a fixed order to par[0] and par[1].
//
// Per sub-step and bead, with lvt = lv + hh lr (the second half drift):
// the direction of the force derivative is dir = cf lvt (the kick), the
// derivative dF of the conservative force along the field of directions
// (for conservative forces (dF/dr)^T lvt = dF/dr lvt) enters lr, and lv
// goes back through the kick and the first half drift.
// ---------------------------------------------------------------------------
constexpr int ADJ_LANES = 16;                // lanes per bead in the pair wave (a power of two)
constexpr int AS_BPB = 64 / ADJ_LANES;       // beads per workgroup
constexpr int AS_WG = 192;                   // wave 0: pair terms; wave 1: bonds and angles; wave 2: wall sites
constexpr int ADJ_PER_LANE = MAXNBR / ADJ_LANES;   // list entries per lane
constexpr int AS_FIN = 1024;                 // threads of k_adj_md_fin
static_assert((ADJ_LANES & (ADJ_LANES - 1)) == 0 && 64 % ADJ_LANES == 0, "lanes per bead: a power of two");
static_assert(MAXNBR % ADJ_LANES == 0 && MAXNBR % 4 == 0 && MAXNBR <= 64, "whole list entries per lane, one mask");
static_assert(ADJ_WIN % 4 == 0 && ADJ_WIN <= 64, "wall sites: whole words, one mask");
static_assert(3 * (AS_BPB + 2) <= 32 && 32 + 2 * AS_BPB <= 64, "one thread of wave 1 per angle component and per bond");

// Bead q's force position (from the tape rows rms) and direction as duals.
__device__ inline void bead_dual(const double* __restrict__ rms, const double* __restrict__ dirin, int q, Dd r[3]) {
  for (int c = 0; c < 3; ++c) r[c] = Dd{rms[6 * (size_t)q + c], dirin[3 * q + c]};
}

// Dual LJ term of the pair (bead at xp with direction dp, partner at rj
// with direction dj), if within r_c.
__device__ inline void lj_pair(const MdParams& P, const Geom& g, const double* xp, const double* dp,
                               const double* rj, const double* dj, Dd S[3]) {
  const double e0 = min_image(xp[0] - rj[0], g.nx);
  const double e1 = min_image(xp[1] - rj[1], g.ny);
  const double e2 = min_image(xp[2] - rj[2], g.nz);
  lj_dd(P, Dd{e0, dp[0] - dj[0]}, Dd{e1, dp[1] - dj[1]}, Dd{e2, dp[2] - dj[2]}, S);
}

// One bead's reverse sub-step given its force (value f, derivative df along
// the directions): with lvt = lv + hh lr, adds the sub-step's terms of
// dL/dgamma and dL/dF_drive to accg, accf and that of u_p to lu, and gives
// the adjoint before the sub-step (lrm, lvn) and the bead's next direction
// dn = cf (lvn + hh lrm).  xp, dp: the bead's force position and direction.
__device__ inline void bead_reverse(const MdParams& P, const Geom& g, double kT, const double* xp, const double* dp,
                                    const Dd* S, const double* lr, const double* lv, const double* lJ,
                                    const double* u, const double* vo, const double* xi, double* lu, double& accg,
                                    double& accf, double* lrm, double* lvn, double* dn) {
  double f[3] = {S[0].v, S[1].v, S[2].v}, df[3] = {S[0].d, S[1].d, S[2].d};
  const double h = 2.0 * P.hh;
  const double gam = P.gamma;
  const double de = -h * P.e, domE = h * P.e;
  const double dcf = (h * P.e) / (P.m * gam) - P.omE / (P.m * gam * gam);
  const double dsig = P.sig > 0.0 ? ((kT / P.m) * (h * P.e * P.e)) / P.sig : 0.0;
  const bool field = P.field_on && in_field(g, xp);
  if (field) f[g.wall_axis] += P.f_drive;
  for (int c = 0; c < 3; ++c) {
    const double lvt = lv[c] + P.hh * lr[c];
    accg += lvt * (vo[c] * de + (f[c] + gam * u[c]) * dcf + P.cf * u[c] + xi[c] * dsig);
    accg += lJ[c] * (-P.m) * ((u[c] - vo[c]) * domE + xi[c] * dsig);
    lu[c] = lu[c] + (P.cf * gam * lvt - P.m * P.omE * lJ[c]);
    lrm[c] = lr[c] + df[c];
    lvn[c] = P.e * lvt + P.m * P.omE * lJ[c] + P.hh * lrm[c];
    dn[c] = P.cf * (lvn[c] + P.hh * lrm[c]);
  }
  if (field) accf += dp[g.wall_axis];
}

// The bead noise of every sub-step of the step being reversed, drawn in
// parallel before the reverse sub-cycle (the forward's draws: key (seed,
// replica), counter (step, s, p, 0)); one thread per (s, p).
__global__ void k_adj_noise(Dev d, double* __restrict__ xi, uint32_t step, int nb, int n_sub) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nb * n_sub) return;
  const MdParams& P = d.reps[0].mp;
  const int s = t / nb, p = t - s * nb;
  double x[3];
  gauss3(P.seed, P.replica, step, (uint32_t)s, (uint32_t)p, x);
  for (int c = 0; c < 3; ++c) xi[(size_t)t * 3 + c] = x[c];
}

// The neighbour lists built at the reversed step's start positions hold
// every pair within r_c at the sub-steps' force positions while no bead is
// farther than half the skin from where they were built (and no bucket of
// the cell table overflowed); else the reverse sub-steps scan all pairs.
// Also writes the directions the first reversed sub-step reads.
__global__ void k_adj_lcheck(Dev d, AdjBufs a, const double* __restrict__ mdt, int nb, int n_sub) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t == 0 && d.rb[3] != 0u) atomicOr(a.lok, 1);
  if (t < nb) {
    // the first reversed sub-step's directions cf (lv + hh lr)
    const MdParams& P = d.reps[0].mp;
    for (int c = 0; c < 3; ++c) a.dirA[3 * t + c] = P.cf * (a.lv[3 * t + c] + P.hh * a.lr[3 * t + c]);
  }
  if (t >= nb * n_sub) return;
  const int p = t % nb;
  double d2 = 0.0;
  for (int c = 0; c < 3; ++c) {
    const double x = mdt[(size_t)t * 6 + c] - d.ref[3 * p + c];
    d2 += x * x;
  }
  if (!(d2 <= d.reps[0].mp.halfskin2)) atomicOr(a.lok, 1);
}

// S += the terms (v, d)[k] for the set bits k of mask, in ascending k; the
// loads of four terms are issued before their additions.
__device__ inline void add_masked(Dd S[3], uint64_t mask, const double (*v)[3], const double (*d)[3]) {
  while (mask) {
    int k[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      k[i] = mask ? __builtin_ctzll(mask) : -1;
      mask &= mask - 1;
    }
    double tv[4][3], td[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kk = k[i] >= 0 ? k[i] : k[0];
      for (int c = 0; c < 3; ++c) { tv[i][c] = v[kk][c]; td[i][c] = d[kk][c]; }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k[i] >= 0)
        for (int c = 0; c < 3; ++c) S[c] = S[c] + Dd{tv[i][c], td[i][c]};
  }
}

// Reverse sub-step s, the k-th launch of the reversed cycle (k = n_sub - 1 - s),
// for beads p0 .. p0 + AS_BPB - 1.  The conservative force on bead p (value
// and derivative along the directions dir) is evaluated by three waves side
// by side:
//   wave 0, ADJ_LANES lanes per bead: lane l takes the dual LJ term of list
//   entries l, l + ADJ_LANES, ... (those within r_c), stored by list
//   position;
//   wave 1: each component of the angles centred at p0 - 1 .. p0 + AS_BPB
//   (one lane each) and the two bonds of each bead, into LDS;
//   wave 2, ADJ_LANES lanes per bead: the wall sites numbered lane modulo
//   ADJ_LANES, stored by site.
// The terms are then added in one fixed order: lane l < 4 of the bead adds
// those of the partners j = l mod 4 in ascending j, lane 0 then the bonds to
// p - 1 and p + 1, the angle terms centred at p - 1, p, p + 1 and the wall
// sites in window order, and the force is (S0 + S1) + (S2 + S3).  Without
// lists lane l < 4 takes its partners from all beads.
// Every address of the first loads comes from the arguments (nb included),
// so they do not wait for the parameter block.
__global__ __launch_bounds__(AS_WG) void k_adj_sub(Dev d, AdjBufs a, const double* __restrict__ mdt,
                                                   const double* __restrict__ upt, int nb, int s, int k,
                                                   double kT) {
  __shared__ double av[AS_BPB + 2][9], ad[AS_BPB + 2][9];
  __shared__ double bv[AS_BPB][2][3], bd[AS_BPB][2][3];
  __shared__ double tv[AS_BPB][MAXNBR][3], td[AS_BPB][MAXNBR][3];   // pair terms by list position
  __shared__ double wv[AS_BPB][ADJ_WIN][3], wd[AS_BPB][ADJ_WIN][3]; // wall-site terms by site number
  __shared__ __align__(16) int8_t tcl[AS_BPB][MAXNBR];             // j mod 4 of an entry with a term, else -1
  __shared__ __align__(16) int8_t whit[AS_BPB][ADJ_WIN];
  const Rep& R = d.reps[0];
  const MdParams P = R.mp;
  const Geom g = R.g;
  const int p0 = blockIdx.x * AS_BPB;
  const int t = threadIdx.x;
  const int wave = t / 64;
  const bool pairw = wave == 0;
  const int u = t & 63, b = u / ADJ_LANES, lane = u % ADJ_LANES, p = p0 + b;
  const bool on = p < nb, lead = pairw && on && lane == 0;
  const bool first = k == 0;
  const double* lrin = (k & 1) ? a.lr2 : a.lr;
  const double* lvin = (k & 1) ? a.lv2 : a.lv;
  double* lrout = (k & 1) ? a.lr : a.lr2;
  double* lvout = (k & 1) ? a.lv : a.lv2;
  // every bead's direction cf (lv + hh lr), written by the previous launch
  // (the first from k_adj_lcheck)
  const double* dirin = (k & 1) ? a.dirB : a.dirA;
  double* dirout = (k & 1) ? a.dirA : a.dirB;
  const double* rms = mdt + (size_t)s * nb * 6;   // [nb][6]: r_mid, v at the start of sub-step s
  const bool lists = *a.lok == 0;
  // the adding lane's own state, loaded first
  double olr[3] = {0.0, 0.0, 0.0}, olv[3] = {0.0, 0.0, 0.0}, olJ[3] = {0.0, 0.0, 0.0}, ou[3] = {0.0, 0.0, 0.0};
  double ovo[3] = {0.0, 0.0, 0.0}, oxi[3] = {0.0, 0.0, 0.0}, olu[3] = {0.0, 0.0, 0.0};
  double og = 0.0, of = 0.0;
  if (lead) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      olr[c] = lrin[3 * p + c];
      olv[c] = lvin[3 * p + c];
      olJ[c] = a.lJ[3 * p + c];
      ou[c] = upt[3 * p + c];
      ovo[c] = rms[6 * (size_t)p + 3 + c];
      if (kT != 0.0) oxi[c] = a.xi[((size_t)s * nb + p) * 3 + c];   // drawn when kT > 0 (sigma > 0)
      if (!first) olu[c] = a.lup[3 * p + c];
    }
    if (!first) { og = a.gacc[3 * p]; of = a.gacc[3 * p + 1]; }
  }
  // wave 0: the bead's own position and direction, this lane's list
  // entries (all loaded at once; those past the count are dropped, and the
  // lists are dropped when the flag says they do not hold)
  double xp[3] = {0.0, 0.0, 0.0}, dp[3] = {0.0, 0.0, 0.0};
  int jm[ADJ_PER_LANE];
#pragma unroll
  for (int m = 0; m < ADJ_PER_LANE; ++m) jm[m] = -1;
  if (pairw && on) {
    for (int c = 0; c < 3; ++c) { xp[c] = rms[6 * (size_t)p + c]; dp[c] = dirin[3 * p + c]; }
    const int cnt = d.ncnt[p];
    const int* row = d.nbr + (size_t)p * MAXNBR;
    int e[ADJ_PER_LANE];
#pragma unroll
    for (int m = 0; m < ADJ_PER_LANE; ++m) e[m] = row[lane + ADJ_LANES * m];
#pragma unroll
    for (int m = 0; m < ADJ_PER_LANE; ++m)
      if (lists && lane + ADJ_LANES * m < cnt) jm[m] = e[m];
  }
  Dd S[3] = {mkd(0.0), mkd(0.0), mkd(0.0)};
  if (wave == 1) {
    if (u < 3 * (AS_BPB + 2)) {
      // component u mod 3 of the angle centred at p0 - 1 + u / 3 (row u / 3),
      // from the three beads' positions and directions loaded here
      const int row = u / 3, cmp = u % 3, cen = p0 - 1 + row;
      if (cen >= 1 && cen <= nb - 2) {
        Dd ra[3], rb[3], rc[3], o3[3];
        bead_dual(rms, dirin, cen - 1, ra);
        bead_dual(rms, dirin, cen, rb);
        bead_dual(rms, dirin, cen + 1, rc);
        angle_dd_comp(P, ra, rb, rc, cmp, o3);
        for (int w = 0; w < 3; ++w) { av[row][3 * w + cmp] = o3[w].v; ad[row][3 * w + cmp] = o3[w].d; }
      }
    } else if (u >= 32 && u < 32 + 2 * AS_BPB) {
      // bond of bead bb to bb - 1 (side 0) or bb + 1 (side 1)
      const int bb = (u - 32) / 2, side = (u - 32) % 2;
      const int q = p0 + bb, o = side ? q + 1 : q - 1;
      if (q < nb && o >= 0 && o < nb) {
        Dd rp[3], rq[3];
        bead_dual(rms, dirin, q, rp);
        bead_dual(rms, dirin, o, rq);
        Dd T[3] = {mkd(0.0), mkd(0.0), mkd(0.0)};
        bond_dd(P, rp, rq, T);
        for (int c = 0; c < 3; ++c) { bv[bb][side][c] = T[c].v; bd[bb][side][c] = T[c].d; }
      }
    }
  } else if (wave == 2) {
    // the wall sites of bead b, numbered lane modulo ADJ_LANES
    if (on) {
      Dd rp[3];
      bead_dual(rms, dirin, p, rp);
      wall_terms(P, g, rp, lane, ADJ_LANES, wv[b], wd[b], whit[b]);
    }
  } else if (on && lists) {
    {
      // the entries' positions and directions loaded together, then the
      // dual LJ term of each entry within r_c, stored by list position
      double ej[ADJ_PER_LANE][3], dj[ADJ_PER_LANE][3];
#pragma unroll
      for (int m = 0; m < ADJ_PER_LANE; ++m) {
        const int j = jm[m] >= 0 ? jm[m] : p;
        for (int c = 0; c < 3; ++c) { ej[m][c] = rms[6 * (size_t)j + c]; dj[m][c] = dirin[3 * j + c]; }
      }
#pragma unroll
      for (int m = 0; m < ADJ_PER_LANE; ++m) {
        const int kk = lane + ADJ_LANES * m;
        bool hit = false;
        if (jm[m] >= 0) {
          const double e0 = min_image(xp[0] - ej[m][0], g.nx);
          const double e1 = min_image(xp[1] - ej[m][1], g.ny);
          const double e2 = min_image(xp[2] - ej[m][2], g.nz);
          Dd t3[3];
          hit = lj_term(P, Dd{e0, dp[0] - dj[m][0]}, Dd{e1, dp[1] - dj[m][1]}, Dd{e2, dp[2] - dj[m][2]}, t3);
          if (hit)
            for (int c = 0; c < 3; ++c) { tv[b][kk][c] = t3[c].v; td[b][kk][c] = t3[c].d; }
        }
        tcl[b][kk] = hit ? (int8_t)(jm[m] & 3) : (int8_t)-1;
      }
    }
  }
  // the pair wave's terms are read back within the wave: a wave-level
  // barrier orders its LDS stores before the loads below
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // Lane l < 4 of the bead adds the pair terms of its partners j = l mod 4
  // in ascending j (list order; without lists it takes them from all beads
  // itself) while the bonded wave works; after the barrier lane 0 adds the
  // bond to p - 1, the bond to p + 1, the angle terms centred at p - 1, p,
  // p + 1 and the wall sites in window order; the four sums are combined as
  // (S0 + S1) + (S2 + S3).
  if (pairw && on && lane < 4) {
    if (lists) {
      // the class's entries as a mask over the list, read four at a time
      uint64_t mk = 0;
#pragma unroll
      for (int q = 0; q < MAXNBR / 4; ++q) {
        const uint32_t w4 = reinterpret_cast<const uint32_t*>(tcl[b])[q];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((int8_t)(w4 >> (8 * e)) == lane) mk |= 1ull << (4 * q + e);
      }
      add_masked(S, mk, tv[b], td[b]);
    } else {
      for (int j = lane; j < nb; j += 4)
        if (j != p) {
          const double rj[3] = {rms[6 * (size_t)j], rms[6 * (size_t)j + 1], rms[6 * (size_t)j + 2]};
          const double dj[3] = {dirin[3 * j], dirin[3 * j + 1], dirin[3 * j + 2]};
          lj_pair(P, g, xp, dp, rj, dj, S);
        }
    }
  }
  __syncthreads();
  if (pairw && on && lane < 4) {
    if (lane == 0) {
      const int al = b + 1;   // row of the angle centred at p
      for (int c = 0; c < 3; ++c) {
        if (p > 0) S[c] = S[c] + Dd{bv[b][0][c], bd[b][0][c]};
        if (p < nb - 1) S[c] = S[c] + Dd{bv[b][1][c], bd[b][1][c]};
      }
      for (int c = 0; c < 3; ++c) {
        if (p - 1 >= 1 && p - 1 <= nb - 2) S[c] = S[c] + Dd{av[al - 1][6 + c], ad[al - 1][6 + c]};
        if (p >= 1 && p <= nb - 2) S[c] = S[c] + Dd{av[al][3 + c], ad[al][3 + c]};
        if (p + 1 >= 1 && p + 1 <= nb - 2) S[c] = S[c] + Dd{av[al + 1][c], ad[al + 1][c]};
      }
      const int nw = P.whi - P.wlo + 1;
      uint64_t wm = 0;
#pragma unroll
      for (int q = 0; q < ADJ_WIN / 4; ++q) {
        const uint32_t w4 = reinterpret_cast<const uint32_t*>(whit[b])[q];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * q + e < nw * nw && ((w4 >> (8 * e)) & 0xffu) != 0u) wm |= 1ull << (4 * q + e);
      }
      add_masked(S, wm, wv[b], wd[b]);
    }
  }
  // every lane of the wave takes part in the exchange; the bead's lanes 0-3
  // are lanes base .. base + 3 of the wave
  const int base = u & ~(ADJ_LANES - 1);
  double F[3], dF[3];
  for (int c = 0; c < 3; ++c) {
    double v4[4], d4[4];
    for (int l = 0; l < 4; ++l) {
      v4[l] = __shfl(S[c].v, base + l, 64);
      d4[l] = __shfl(S[c].d, base + l, 64);
    }
    F[c] = (v4[0] + v4[1]) + (v4[2] + v4[3]);
    dF[c] = (d4[0] + d4[1]) + (d4[2] + d4[3]);
  }
  if (!lead) return;
  for (int c = 0; c < 3; ++c) S[c] = Dd{F[c], dF[c]};
  double lrm[3], lvn[3], dn[3];
  bead_reverse(P, g, kT, xp, dp, S, olr, olv, olJ, ou, ovo, oxi, olu, og, of, lrm, lvn, dn);
  for (int c = 0; c < 3; ++c) {
    a.lup[3 * p + c] = olu[c];
    lrout[3 * p + c] = lrm[c];
    lvout[3 * p + c] = lvn[c];
    dirout[3 * p + c] = dn[c];
  }
  a.gacc[3 * p] = og;
  a.gacc[3 * p + 1] = of;
}

// ---------------------------------------------------------------------------
// The reversed sub-cycle of a chain of at most ADJ_CHAIN beads in two launches.
//
// The force positions of every sub-step are on the tape, and the derivative of
// the force is linear in the directions: so everything but the product with
// the directions is done for all sub-steps at once (k_adj_terms), and the
// serial part (k_adj_chain, one workgroup) is a product with a band per
// sub-step.  One launch per sub-step (k_adj_sub) evaluated the force law in
// dual numbers between two directions: 8.5 us of latency each, at 100 beads
// 0.85 of 1.5 ms per reversed step; the two launches take 14 and 125 us.  At 341
// beads, two components per thread, a gradient step takes 1.14 instead of 1.52
// ms; at 400, three per thread spill: 1.86 against 1.50.
//
// The chain's directions enter as differences of neighbours, D_q = dir_q -
// dir_{q-1}, as in the dual evaluation (a common translation of the beads then
// cancels before it is multiplied by the large stiffness terms): the band holds
// the 3 x 3 blocks of bead p for D_{p-1}, D_p, D_{p+1}, D_{p+2} -- bonds,
// angles, and pairs of beads at most two links apart -- and the block of its
// wall sites for dir_p itself.  Other pairs within r_c are kept apart, ADJ_NP
// per bead and sub-step (a bead with more evaluates them again).
// ---------------------------------------------------------------------------
constexpr int AT_BPB = 12;                   // beads per workgroup
constexpr int AT_WG = 256;
static_assert(18 * (AT_BPB + 2) <= AT_WG && ADJ_LANES * AT_BPB <= AT_WG && 3 * (AT_BPB + 1) <= AT_WG, "one pass");

struct AdjCoef {
  double* M;       // [C][12][3 nb]: blocks of the band, 3 diff + k, for component c of bead p at 3 p + c
  double* W;       // [C][3][3 nb]: walls
  double* F;       // [C][3 nb]: force
  int* np;         // [C][nb]: far pairs (-1: more than ADJ_NP), + 256 in the field
  int* pj;         // [C][ADJ_NP][nb]: partner
  double* pk;      // [C][ADJ_NP][5][nb]: coef, 2 dcoef / dr^2, separation
};
__host__ __device__ inline AdjCoef adj_coef(double* buf, int nb, int C) {
  AdjCoef k;
  const size_t n = (size_t)C * nb;
  k.M = buf;
  k.W = k.M + 36 * n;
  k.F = k.W + 9 * n;
  k.pk = k.F + 3 * n;
  k.pj = (int*)(k.pk + 5 * ADJ_NP * n);
  k.np = k.pj + ADJ_NP * n;
  return k;
}

// coef of the LJ force coef d and twice its derivative with respect to r^2.
__device__ inline void lj_coef(const MdParams& P, double r2, double& coef, double& c2) {
  const double sr2 = P.sig2 / r2, sr6 = sr2 * sr2 * sr2, sr12 = sr6 * sr6;
  coef = P.eps24 * (2.0 * sr12 - sr6) / r2;
  c2 = 2.0 * (P.eps24 * (4.0 * sr6 - 14.0 * sr12) / r2) / r2;
}

// Row blockIdx.y of the coefficients: sub-step s0 - blockIdx.y.
__global__ __launch_bounds__(AT_WG) void k_adj_terms(Dev d, const int* __restrict__ lok, AdjCoef K,
                                                     const double* __restrict__ mdt, int nb, int s0) {
  __shared__ double G[AT_BPB + 2][9][6], Gv[AT_BPB + 2][9];       // angles: columns D1, D2; forces
  __shared__ double B[AT_BPB + 1][3][3], Bv[AT_BPB + 1][3];       // bond of p0 + q to p0 + q - 1
  __shared__ double N[AT_BPB][4][6];                              // pairs with p - 2, p - 1, p + 1, p + 2
  __shared__ double W[AT_BPB][6], S[AT_BPB][3];                   // walls; pair, wall and field forces
  const Rep& R = d.reps[0];
  const MdParams P = R.mp;
  const Geom g = R.g;
  const int row = blockIdx.y, p0 = blockIdx.x * AT_BPB, t = threadIdx.x;
  const double* x = mdt + (size_t)(s0 - row) * nb * 6;
  const bool lists = *lok == 0;
  for (int k = t; k < AT_BPB * 24; k += AT_WG) (&N[0][0][0])[k] = 0.0;
  // component cmp of the angle centred at p0 - 1 + r, column k
  if (t < 18 * (AT_BPB + 2)) {
    const int r = t / 18, k = t % 18 / 3, cmp = t % 3, cen = p0 - 1 + r;
    Dd o[3] = {mkd(0.0), mkd(0.0), mkd(0.0)};
    if (cen >= 1 && cen <= nb - 2) {
      Dd ra[3], rb[3], rc[3];
      for (int c = 0; c < 3; ++c) {
        ra[c] = Dd{x[6 * (size_t)(cen - 1) + c], k == c ? -1.0 : 0.0};
        rb[c] = Dd{x[6 * (size_t)cen + c], 0.0};
        rc[c] = Dd{x[6 * (size_t)(cen + 1) + c], k == 3 + c ? 1.0 : 0.0};
      }
      angle_dd_comp(P, ra, rb, rc, cmp, o);
    }
    for (int w = 0; w < 3; ++w) {
      G[r][3 * w + cmp][k] = o[w].d;
      if (k == 0) Gv[r][3 * w + cmp] = o[w].v;
    }
  }
  if (t < 3 * (AT_BPB + 1)) {
    const int q = t / 3, k = t % 3, p = p0 + q;
    Dd T[3] = {mkd(0.0), mkd(0.0), mkd(0.0)};
    if (p > 0 && p < nb) {
      Dd rp[3], rq[3];
      for (int c = 0; c < 3; ++c) {
        rp[c] = Dd{x[6 * (size_t)p + c], k == c ? 1.0 : 0.0};
        rq[c] = Dd{x[6 * (size_t)(p - 1) + c], 0.0};
      }
      bond_dd(P, rp, rq, T);
    }
    for (int c = 0; c < 3; ++c) {
      B[q][c][k] = T[c].d;
      if (k == 0) Bv[q][c] = T[c].v;
    }
  }
  __syncthreads();
  // pairs and wall sites, ADJ_LANES lanes per bead
  const int b = t / ADJ_LANES, lane = t % ADJ_LANES, p = p0 + b;
  const bool on = b < AT_BPB && p < nb;
  double xp[3] = {0.0, 0.0, 0.0}, F[3] = {0.0, 0.0, 0.0}, w6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int cand = 0;
  if (on) {
    for (int c = 0; c < 3; ++c) xp[c] = x[6 * (size_t)p + c];
    cand = lists ? d.ncnt[p] : nb;
  }
  int far = 0;
  const uint64_t mine = ((1ull << ADJ_LANES) - 1ull) << (t & 63 & ~(ADJ_LANES - 1));
  int most = cand;                               // over the wave, so that its lanes vote together
  for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
  for (int i0 = 0; i0 < most; i0 += ADJ_LANES) {
    const int i = i0 + lane;
    bool keep = false;
    double e[3] = {0.0, 0.0, 0.0}, coef = 0.0, c2 = 0.0;
    int j = p;
    if (i < cand) j = lists ? d.nbr[(size_t)p * MAXNBR + i] : i;
    if (j != p) {
      e[0] = min_image(xp[0] - x[6 * (size_t)j], g.nx);
      e[1] = min_image(xp[1] - x[6 * (size_t)j + 1], g.ny);
      e[2] = min_image(xp[2] - x[6 * (size_t)j + 2], g.nz);
      const double r2 = e[0] * e[0] + e[1] * e[1] + e[2] * e[2];
      if (r2 < P.rc2) {
        lj_coef(P, r2, coef, c2);
        for (int c = 0; c < 3; ++c) F[c] += coef * e[c];
        const int o = j - p;
        if (o >= -2 && o <= 2) {
          double* n = N[b][o < 0 ? o + 2 : o + 1];
          n[0] = coef + c2 * e[0] * e[0]; n[1] = c2 * e[0] * e[1]; n[2] = c2 * e[0] * e[2];
          n[3] = coef + c2 * e[1] * e[1]; n[4] = c2 * e[1] * e[2]; n[5] = coef + c2 * e[2] * e[2];
        } else {
          keep = true;
        }
      }
    }
    const uint64_t m = __ballot(keep) & mine;
    const int at = far + __builtin_popcountll(m & ((1ull << (t & 63)) - 1ull));
    if (keep && at < ADJ_NP) {
      const size_t n = (size_t)row * ADJ_NP + at;
      K.pj[n * nb + p] = j;
      double* q = K.pk + n * 5 * nb + p;
      q[0] = coef; q[nb] = c2; q[2 * (size_t)nb] = e[0]; q[3 * (size_t)nb] = e[1]; q[4 * (size_t)nb] = e[2];
    }
    far += __builtin_popcountll(m);
  }
  bool field = false;
  if (on && g.wall_axis >= 0) {
    // the window of wall_terms
    const double w[3] = {wrapc(xp[0], g.nx), wrapc(xp[1], g.ny), wrapc(xp[2], g.nz)};
    const int n[3] = {g.nx, g.ny, g.nz};
    const int a = g.wall_axis, t0 = g.t0, t1 = g.t1, nw = P.whi - P.wlo + 1;
    int off = g.wall_pos - (int)floor(w[a]);
    if (off < -2) off += n[a];
    if (off > 3) off -= n[a];
    if (off >= P.wlo && off <= P.whi)
      for (int num = lane; num < nw * nw; num += ADJ_LANES) {
        const int u1 = (int)floor(w[t1]) + P.wlo + num / nw, u0 = (int)floor(w[t0]) + P.wlo + num % nw;
        const int v1 = u1 < 0 ? u1 + n[t1] : (u1 >= n[t1] ? u1 - n[t1] : u1);
        const int v0 = u0 < 0 ? u0 + n[t0] : (u0 >= n[t0] ? u0 - n[t0] : u0);
        if (v1 >= g.lo1 && v1 <= g.hi1 && v0 >= g.lo0 && v0 <= g.hi0) continue;   // pore node: fluid
        double e[3];
        e[a] = w[a] - (double)((int)floor(w[a]) + off);
        e[t0] = w[t0] - (double)u0;
        e[t1] = w[t1] - (double)u1;
        const double r2 = e[0] * e[0] + e[1] * e[1] + e[2] * e[2];
        if (!(r2 < P.rc2)) continue;
        double coef, c2;
        lj_coef(P, r2, coef, c2);
        for (int c = 0; c < 3; ++c) F[c] += coef * e[c];
        w6[0] += coef + c2 * e[0] * e[0]; w6[1] += c2 * e[0] * e[1]; w6[2] += c2 * e[0] * e[2];
        w6[3] += coef + c2 * e[1] * e[1]; w6[4] += c2 * e[1] * e[2]; w6[5] += coef + c2 * e[2] * e[2];
      }
    field = P.field_on && in_field(g, xp);
    if (field && lane == 0) F[a] += P.f_drive;
  }
  for (int o = ADJ_LANES / 2; o > 0; o >>= 1) {
    for (int c = 0; c < 3; ++c) F[c] += __shfl_xor(F[c], o, 64);
    for (int c = 0; c < 6; ++c) w6[c] += __shfl_xor(w6[c], o, 64);
  }
  if (on && lane == 0) {
    for (int c = 0; c < 3; ++c) S[b][c] = F[c];
    for (int c = 0; c < 6; ++c) W[b][c] = w6[c];
    K.np[(size_t)row * nb + p] = (far > ADJ_NP ? 255 : far) + (field ? 256 : 0);
  }
  __syncthreads();
  constexpr int sym[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
  for (int i = t; i < 16 * 3 * AT_BPB; i += AT_WG) {
    const int e = i % (3 * AT_BPB), j = i / (3 * AT_BPB), q = e / 3, c = e % 3;
    if (p0 + q >= nb) continue;
    const size_t at = (size_t)3 * nb, col = (size_t)3 * (p0 + q) + c;
    if (j < 12) {
      const int k = j % 3, z = sym[c][k];
      double v;
      if (j < 3) v = G[q][6 + c][k] + N[q][0][z];
      else if (j < 6) v = B[q][c][k] + G[q][6 + c][3 + k] + G[q + 1][3 + c][k] + N[q][0][z] + N[q][1][z];
      else if (j < 9) v = G[q + 1][3 + c][3 + k] + G[q + 2][c][k] - B[q + 1][c][k] - N[q][2][z] - N[q][3][z];
      else v = G[q + 2][c][3 + k] - N[q][3][z];
      K.M[((size_t)row * 12 + j) * at + col] = v;
    } else if (j < 15) {
      K.W[((size_t)row * 3 + (j - 12)) * at + col] = W[q][sym[c][j - 12]];
    } else {
      K.F[(size_t)row * at + col] = Bv[q][c] - Bv[q + 1][c] + Gv[q][6 + c] + Gv[q + 1][3 + c] + Gv[q + 2][c] + S[q][c];
    }
  }
}

// The serial part for rows 0 .. rows - 1 (sub-steps s0, s0 - 1, ...): thread t
// has components t, t + blockDim.x, ... (E of them) of the chain's 3 nb, in
// registers throughout; the directions are in LDS.  A row's coefficients are
// requested while the row before is worked on (two rows before for E = 1: a
// row takes less than a load).  first: the cycle starts here.
constexpr int AC_WG = 512;                   // 256 registers per thread
static_assert(3 * ADJ_CHAIN <= 2 * AC_WG, "at most two components per thread");
struct AdjRow {
  double m[12], w[3], f, vo, xi;
  int np;
};
template <int E>
__global__ __launch_bounds__(AC_WG) void k_adj_chain(Dev d, AdjBufs a, AdjCoef K, const double* __restrict__ mdt,
                                                    const double* __restrict__ upt, int nb, int s0, int rows, int first,
                                                    double kT) {
  constexpr int PAD = 6;                         // two beads beyond each end (their coefficients are 0)
  __shared__ double dir[2][3 * ADJ_CHAIN + 2 * PAD];
  const MdParams P = d.reps[0].mp;
  const Geom g = d.reps[0].g;
  const int t = threadIdx.x, n3 = 3 * nb;
  const double h = 2.0 * P.hh, gam = P.gamma, de = -h * P.e, domE = h * P.e;
  const double dcf = (h * P.e) / (P.m * gam) - P.omE / (P.m * gam * gam);
  const double dsig = P.sig > 0.0 ? ((kT / P.m) * (h * P.e * P.e)) / P.sig : 0.0;
  const bool lists = *a.lok == 0;
  double lr[E], lv[E], lJ[E], u[E], lu[E], ag[E], af[E];
  if (t < PAD)
    for (int q = 0; q < 2; ++q) dir[q][t] = dir[q][PAD + n3 + t] = 0.0;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int e = t + k * (int)blockDim.x;
    lr[k] = lv[k] = lJ[k] = u[k] = lu[k] = ag[k] = af[k] = 0.0;
    if (e >= n3) continue;
    lr[k] = a.lr[e]; lv[k] = a.lv[e]; lJ[k] = a.lJ[e]; u[k] = upt[e];
    if (!first) lu[k] = a.lup[e];
    dir[0][PAD + e] = P.cf * (lv[k] + P.hh * lr[k]);
  }
  auto fetch = [&](int r, int e, AdjRow& o) {
    o.np = 0;
    if (r >= rows || e >= n3) return;
    const size_t at = (size_t)n3;
    const int s = s0 - r, p = e / 3;
#pragma unroll
    for (int j = 0; j < 12; ++j) o.m[j] = K.M[((size_t)r * 12 + j) * at + e];
#pragma unroll
    for (int j = 0; j < 3; ++j) o.w[j] = K.W[((size_t)r * 3 + j) * at + e];
    o.f = K.F[(size_t)r * at + e];
    o.np = K.np[(size_t)r * nb + p];
    o.vo = mdt[((size_t)s * nb + p) * 6 + 3 + (e - 3 * p)];
    o.xi = kT != 0.0 ? a.xi[(size_t)s * n3 + e] : 0.0;
  };
  AdjRow c0[E], c1[E];
#pragma unroll
  for (int k = 0; k < E; ++k) {
    fetch(0, t + k * (int)blockDim.x, c0[k]);
    if (E == 1) fetch(1, t + k * (int)blockDim.x, c1[k]);
  }
  __syncthreads();
  for (int r = 0; r < rows; ++r) {
    const double* D = dir[r & 1];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = t + k * (int)blockDim.x;
      const AdjRow q = c0[k];
      if (E == 1) {
        c0[k] = c1[k];
        fetch(r + 2, e, c1[k]);
      } else {
        fetch(r + 1, e, c0[k]);
      }
      if (e >= n3) continue;
      const int p = e / 3, c = e - 3 * p;
      const double* x = D + PAD + 3 * p;         // the bead's direction
      double df = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 3; ++i) df += q.m[3 * j + i] * (x[3 * (j - 1) + i] - x[3 * (j - 2) + i]);
#pragma unroll
      for (int i = 0; i < 3; ++i) df += q.w[i] * x[i];
      const int np = q.np & 255;
      if (np == 255) {
        const double* xs = mdt + (size_t)(s0 - r) * nb * 6;
        const int cand = lists ? d.ncnt[p] : nb;
        for (int i = 0; i < cand; ++i) {
          const int j = lists ? d.nbr[(size_t)p * MAXNBR + i] : i;
          if (j >= p - 2 && j <= p + 2) continue;
          double z[3];
          z[0] = min_image(xs[6 * (size_t)p] - xs[6 * (size_t)j], g.nx);
          z[1] = min_image(xs[6 * (size_t)p + 1] - xs[6 * (size_t)j + 1], g.ny);
          z[2] = min_image(xs[6 * (size_t)p + 2] - xs[6 * (size_t)j + 2], g.nz);
          const double r2 = z[0] * z[0] + z[1] * z[1] + z[2] * z[2];
          if (!(r2 < P.rc2)) continue;
          double coef, c2;
          lj_coef(P, r2, coef, c2);
          const double* y = D + PAD + 3 * j;
          df += coef * (x[c] - y[c]) +
                c2 * (z[0] * (x[0] - y[0]) + z[1] * (x[1] - y[1]) + z[2] * (x[2] - y[2])) * (c == 0 ? z[0] : (c == 1 ? z[1] : z[2]));
        }
      } else {
        for (int i = 0; i < np; ++i) {
          const size_t n = (size_t)r * ADJ_NP + i;
          const double* z = K.pk + n * 5 * nb + p;
          const double z0 = z[2 * (size_t)nb], z1 = z[3 * (size_t)nb], z2 = z[4 * (size_t)nb];
          const double* y = D + PAD + 3 * K.pj[n * nb + p];
          df += z[0] * (x[c] - y[c]) +
                z[nb] * (z0 * (x[0] - y[0]) + z1 * (x[1] - y[1]) + z2 * (x[2] - y[2])) * (c == 0 ? z0 : (c == 1 ? z1 : z2));
        }
      }
      const double lvt = lv[k] + P.hh * lr[k];
      ag[k] += lvt * (q.vo * de + (q.f + gam * u[k]) * dcf + P.cf * u[k] + q.xi * dsig);
      ag[k] += lJ[k] * (-P.m) * ((u[k] - q.vo) * domE + q.xi * dsig);
      lu[k] = lu[k] + (P.cf * gam * lvt - P.m * P.omE * lJ[k]);
      if ((q.np & 256) && c == g.wall_axis) af[k] += x[c];
      const double lrm = lr[k] + df;
      lv[k] = P.e * lvt + P.m * P.omE * lJ[k] + P.hh * lrm;
      lr[k] = lrm;
      dir[(r & 1) ^ 1][PAD + e] = P.cf * (lv[k] + P.hh * lrm);
    }
    __syncthreads();
  }
  // per bead the parameter terms, its components in order
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int e = t + k * (int)blockDim.x;
    if (e >= n3) continue;
    a.lr[e] = lr[k]; a.lv[e] = lv[k]; a.lup[e] = lu[k];
    dir[0][e] = ag[k];
    dir[1][e] = af[k];
  }
  __syncthreads();
  for (int p = t; p < nb; p += (int)blockDim.x)
    for (int z = 0; z < 2; ++z) {
      double* o = a.gacc + 3 * p + z;
      const double* v = dir[z] + 3 * p;
      *o = (first ? 0.0 : *o) + (v[0] + v[1] + v[2]);
    }
}

// After the reversed cycle: lr, lv from the pair the last launch wrote, and
// the parameter terms added over the beads in a fixed order (beads p, p + M,
// ... summed per slot, then a tree over M = the least power of two >= nb,
// at least 128 and at most AS_FIN).
__global__ __launch_bounds__(AS_FIN) void k_adj_md_fin(AdjBufs a, int nb, int n_sub) {
  __shared__ double red[2][AS_FIN];
  const int t = threadIdx.x;
  if (n_sub & 1)
    for (int i = t; i < 3 * nb; i += AS_FIN) { a.lr[i] = a.lr2[i]; a.lv[i] = a.lv2[i]; }
  int M = 128;
  while (M < nb && M < AS_FIN) M *= 2;
  if (t < M) {
    double sg = 0.0, sf = 0.0;
    for (int p = t; p < nb; p += M) { sg += a.gacc[3 * p]; sf += a.gacc[3 * p + 1]; }
    red[0][t] = sg;
    red[1][t] = sf;
  }
  __syncthreads();
  for (int w = M / 2; w > 0; w >>= 1) {
    if (t < w) { red[0][t] += red[0][t + w]; red[1][t] += red[1][t + w]; }
    __syncthreads();
  }
  if (t == 0) {
    a.par[0] += red[0][0];
    a.par[1] += red[1][0];
  }
}

// ---------------------------------------------------------------------------
// Gather transpose, position term, eight lanes per bead as above; adds the
// spreading and gathering position terms to lam_r.
// ---------------------------------------------------------------------------
template <typename T, bool DEV>
__global__ void k_adj_gather_t(const T* __restrict__ A, Dev d, AdjBufs a, int nb) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, p = e >> 3, k = e & 7;
  if (p >= nb) return;                         // whole groups of eight lanes
  const Rep& R = d.reps[0];
  double rp[3] = {d.rs[3 * p], d.rs[3 * p + 1], d.rs[3 * p + 2]};
  Stencil st = make_stencil(R.g, rp);
  const double lu[3] = {a.lup[3 * p], a.lup[3 * p + 1], a.lup[3 * p + 2]};
  const int n = (int)corner_node(R.g, st, k);
  double u[3];
  node_velocity<T, DEV>(A, d.flags, R.lp, n, u);
  const double ul = u[0] * lu[0] + u[1] * lu[1] + u[2] * lu[2];
  for (int b = 0; b < 3; ++b) {
    const double s = corner_sum(dweight(st, k, b) * ul, true);
    if (k == b) a.lr[3 * p + b] += a.lrs[3 * p + b] + s;
  }
}

// ---------------------------------------------------------------------------
// LB transpose over the sweep's tile table: for each fluid node x the
// adjoint of its post-streaming populations, lam_f = (1 - omega) lam_B +
// omega (G0 + c.G) with G0 = sum_i w_i lam_i (1 - 4.5 (c_i.u)^2 + 1.5 u.u),
// G = sum_i w_i lam_i (3 c_i + 9 (c_i.u) c_i - 3 u) (the transpose of the
// BGK Jacobian with the second-order equilibrium), plus (c.lam_u - u.lam_u)
// / rho where a bead stencil gathered u(x); then scattered to the element of
// A it was pulled from.
// ---------------------------------------------------------------------------
template <typename T, bool DEV>
__global__ __launch_bounds__(256) void k_adj_lb(const T* __restrict__ A, const T* __restrict__ lamB,
                                                T* __restrict__ lamA, Dev d, const T* __restrict__ lamu, int ntiles,
                                                int tile_nodes) {
  using R_ = typename std::conditional<DEV, float, double>::type;
  for (int tI = blockIdx.x; tI < ntiles; tI += gridDim.x) {
    const Tile tl = d.tiles[tI];
    const Rep& Rp = d.reps[tl.rep];
    const LbParams& p = Rp.lp;
    const size_t N = (size_t)p.N;
    const size_t no = (size_t)Rp.node_off;
    const T* Ar = A + Q * no;
    const T* lBr = lamB + Q * no;
    T* lAr = lamA + Q * no;
    const T* lur = lamu + 3 * no;
    const uint8_t* fr = d.flags + no;
    const int end = min(tl.start + tile_nodes, p.N);
    for (int c = tl.start + (int)threadIdx.x; c < end; c += blockDim.x) {
      const uint8_t fl = fr[c];
      if (fl & F_SOLID) continue;
      int x = c % p.nx, yz = c / p.nx, y = yz % p.ny, z = yz / p.ny;
      Nbr nb = make_nbr(p, x, y, z);
      T fT[Q];
      pull<T>(Ar, fr, p, c, fl, nb, fT);
      R_ f[Q], lb[Q];
      for (int i = 0; i < Q; ++i) { f[i] = (R_)fT[i]; lb[i] = (R_)lBr[(size_t)i * N + c]; }
      R_ rho = 0, jx, jy, jz;
      for (int i = 0; i < Q; ++i) rho += f[i];
      jx = f[1] - f[2] + f[7] - f[8] + f[9] - f[10] + f[11] - f[12] + f[13] - f[14];
      jy = f[3] - f[4] + f[7] - f[8] - f[9] + f[10] + f[15] - f[16] + f[17] - f[18];
      jz = f[5] - f[6] + f[11] - f[12] - f[13] + f[14] + f[15] - f[16] - f[17] + f[18];
      if (DEV) rho = (R_)1 + rho;
      const R_ ux = jx / rho, uy = jy / rho, uz = jz / rho;
      const R_ usq = ux * ux + uy * uy + uz * uz;
      R_ G0 = 0, A0 = 0, G1x = 0, G1y = 0, G1z = 0, G2x = 0, G2y = 0, G2z = 0;
      for (int i = 0; i < Q; ++i) {
        const R_ wl = (R_)wgt(i) * lb[i];
        const R_ cu = cdot<R_>(i, ux, uy, uz);
        G0 += wl * ((R_)1 - (R_)4.5 * cu * cu + (R_)1.5 * usq);
        A0 += wl;
        G1x += wl * (R_)cx(i); G1y += wl * (R_)cy(i); G1z += wl * (R_)cz(i);
        G2x += wl * cu * (R_)cx(i); G2y += wl * cu * (R_)cy(i); G2z += wl * cu * (R_)cz(i);
      }
      const R_ Gx = (R_)3 * G1x + (R_)9 * G2x - (R_)3 * ux * A0;
      const R_ Gy = (R_)3 * G1y + (R_)9 * G2y - (R_)3 * uy * A0;
      const R_ Gz = (R_)3 * G1z + (R_)9 * G2z - (R_)3 * uz * A0;
      const R_ om = (R_)p.omega;
      R_ Lx = 0, Ly = 0, Lz = 0, Lu = 0, irho = 0;
      const bool forced = (fl & F_FORCED) != 0;
      if (forced) {
        Lx = (R_)lur[c]; Ly = (R_)lur[N + c]; Lz = (R_)lur[2 * N + c];
        Lu = ux * Lx + uy * Ly + uz * Lz;
        irho = (R_)1 / rho;
      }
      for (int i = 0; i < Q; ++i) {
        R_ lf = ((R_)1 - om) * lb[i] + om * (G0 + cdot<R_>(i, Gx, Gy, Gz));
        if (forced) lf += (cdot<R_>(i, Lx, Ly, Lz) - Lu) * irho;
        // element of A this population was pulled from
        const int src = c + nb.off(-cx(i), -cy(i), -cz(i));
        size_t dst = (fr[src] & F_SOLID) ? (size_t)opp(i) * N + (size_t)c : (size_t)i * N + (size_t)src;
        lAr[dst] = (T)lf;
      }
    }
  }
}

// Clear the forced bits and node lists after a reverse step (the step
// counter is not advanced).
__global__ void k_adj_cleanup(Dev d, int nslots, int maxlist) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  int nt = (int)d.ctrl->touched;
  if (k < nt && k < maxlist) {
    int2 e = d.touched[k];
    uint8_t* f = d.flags + d.reps[e.x].node_off + e.y;
    *f = *f & (uint8_t)~F_FORCED;
  }
  if (k < nslots) {
    const Rep& R = d.reps[d.slot_rep[k]];
    if (k - R.slot_off < R.mp.nb) d.head[R.node_off + d.base[k]] = -1;
  }
}
__global__ void k_adj_touched_reset(Ctrl* ctrl) { ctrl->touched = 0u; }

// grads = [dL/dgamma, dL/dF_drive, dL/dr_0 (nb x 3)]
__global__ void k_adj_finish(AdjBufs a, double* __restrict__ grads, int n3) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < 2) grads[k] = a.par[k];
  if (k < n3) grads[2 + k] = a.lr[k];
}

// ---------------------------------------------------------------------------
static inline unsigned nblk(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

void launch_adj_init(const double* dLdr, const double* dLdv, const AdjBufs& a, int nb, hipStream_t s) {
  long n = 3L * nb > 4 ? 3L * nb : 4;
  hipLaunchKernelGGL(k_adj_init, dim3(nblk(n, 256)), dim3(256), 0, s, dLdr, dLdv, a, 3 * nb);
}

template <typename T, bool DEV>
void launch_adj_reverse_step(const void* A, const void* lamB, void* lamA, const Dev& d, const Dev& dspread,
                             const AdjBufs& a, const double* mdt, const double* upt,
                             const double* Jt, uint32_t step, double kT, int ntiles, int tile_nodes, int nslots,
                             int nb, int n_sub, hipStream_t s) {
  launch_bead_prep(d, nslots, 0, s);
  hipLaunchKernelGGL((k_adj_spread_t<T>), dim3(nblk(8L * nb, 64)), dim3(64), 0, s, (const T*)lamB, d, a, Jt, nb);
  // neighbour lists at the step's start positions (d.r is the tape's r_n),
  // checked against every sub-step's force positions
  launch_nbr_build(d, nslots, 1, s);
  hipLaunchKernelGGL(k_adj_lcheck, dim3(nblk((long)nb * n_sub, 256)), dim3(256), 0, s, d, a, mdt, nb, n_sub);
  if (kT != 0.0) {   // sigma > 0 exactly when kT > 0 (gamma > 0 here)
    hipLaunchKernelGGL(k_adj_noise, dim3(nblk((long)nb * n_sub, 256)), dim3(256), 0, s, d, a.xi, step, nb, n_sub);
  }
  const int C = adj_chunk(nb, n_sub);
  if (C > 0) {
    const AdjCoef K = adj_coef(a.coef, nb, C);
    for (int r = 0; r < n_sub; r += C) {
      const int rows = n_sub - r < C ? n_sub - r : C, s0 = n_sub - 1 - r;
      hipLaunchKernelGGL(k_adj_terms, dim3(nblk(nb, AT_BPB), (unsigned)rows), dim3(AT_WG), 0, s, d, (const int*)a.lok, K,
                         mdt, nb, s0);
      const int E = (3 * nb + AC_WG - 1) / AC_WG;
      const auto chain = E == 1 ? k_adj_chain<1> : k_adj_chain<2>;
      hipLaunchKernelGGL(chain, dim3(1), dim3(64 * nblk(3 * nb, 64 * E)), 0, s, d, a, K, mdt, upt, nb, s0, rows,
                         r == 0 ? 1 : 0, kT);
    }
  } else {
    for (int k = 0; k < n_sub; ++k)
      hipLaunchKernelGGL(k_adj_sub, dim3(nblk(nb, AS_BPB)), dim3(AS_WG), 0, s, d, a, mdt, upt, nb, n_sub - 1 - k, k,
                         kT);
  }
  // k_adj_chain leaves lr, lv in place
  hipLaunchKernelGGL(k_adj_md_fin, dim3(1), dim3(AS_FIN), 0, s, a, nb, C > 0 ? 0 : n_sub);
  hipLaunchKernelGGL((k_adj_gather_t<T, DEV>), dim3(nblk(8L * nb, 64)), dim3(64), 0, s, (const T*)A, d, a, nb);
  launch_spread<T>(dspread, nslots, s);
  hipLaunchKernelGGL((k_adj_lb<T, DEV>), dim3((unsigned)ntiles), dim3(256), 0, s, (const T*)A, (const T*)lamB,
                     (T*)lamA, d, (const T*)a.lamu, ntiles, tile_nodes);
  int maxlist = 8 * nslots;
  int n = nslots > maxlist ? nslots : maxlist;
  hipLaunchKernelGGL(k_adj_cleanup, dim3(nblk(n, 256)), dim3(256), 0, s, d, nslots, maxlist);
  hipLaunchKernelGGL(k_adj_touched_reset, dim3(1), dim3(1), 0, s, d.ctrl);
}

void launch_adj_finish(const AdjBufs& a, double* grads, int nb, hipStream_t s) {
  long n = 3L * nb > 2 ? 3L * nb : 2;
  hipLaunchKernelGGL(k_adj_finish, dim3(nblk(n, 256)), dim3(256), 0, s, a, grads, 3 * nb);
}

template void launch_adj_reverse_step<double, false>(const void*, const void*, void*, const Dev&, const Dev&,
                                                     const AdjBufs&, const double*, const double*, const double*,
                                                     uint32_t, double, int, int, int, int, int, hipStream_t);
template void launch_adj_reverse_step<float, true>(const void*, const void*, void*, const Dev&, const Dev&,
                                                   const AdjBufs&, const double*, const double*, const double*,
                                                   uint32_t, double, int, int, int, int, int, hipStream_t);

}  // namespace lbmd
