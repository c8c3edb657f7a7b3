// md_kernels.hip -- the bead sub-cycle: stochastic position Verlet sub-steps
// (Sec. 2, Eq. (SPValgo)) with the fluid velocity at each bead frozen for the
// whole cycle.  One launch for the cycle where its workgroups fit on the GPU
// together (k_md_resident), else one per sub-step; the positions at which
// forces are evaluated are double buffered so that every bead reads a
// consistent snapshot.  Every replica of a context advances in the same
// launches; a workgroup never mixes replicas.
//
// Per sub-step s (h = 1/n_sub, e = exp(-gamma h)):
//   r_mid = r + h/2 v                      (written by the previous launch)
//   F     = bonds + bending + LJ + wall + field at r_mid
//   v'    = e v + (1-e)/(m gamma) (F + gamma u_p) + sig xi
//   J    -= m [(1-e)(u_p - v) + sig xi]    (friction + noise impulse)
//   r'    = r_mid + h/2 v'
// The next launch's r_mid = r' + h/2 v' is formed here as two separate
// additions, the same rounding as two half drifts.
//
// The LJ sum runs over a Verlet neighbour list (radius r_c + skin) kept in
// ascending bead order, so it adds exactly the terms of the all-pairs loop
// in the same order.  With single launches a list is rebuilt in the launch
// after any bead has moved more than skin/2 since the last build; the flag is
// carried between launches in three rotating words.
#include "lbmd_kernels.h"
#include "lbmd_tag.h"

namespace lbmd {

__global__ void k_md_begin(Dev d, int nrep) { md_begin(d, nrep, threadIdx.x, blockDim.x); }

__global__ void k_md_invalidate(uint32_t* rb, int nrep) {
  for (int r = threadIdx.x; r < nrep; r += blockDim.x) rb[4 * r + 3] = 1u;
}

// A copy of *p through the constant address space: scalar loads for a
// workgroup-uniform p, also where the compiler cannot rule out that a store
// of the kernel aliases it.  For tables that no kernel writes.
template <typename T>
__device__ inline T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  typedef const __attribute__((address_space(4))) uint32_t Word;
  Word* q = (Word*)(uintptr_t)p;
  T out;
  uint32_t* o = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
  for (size_t k = 0; k < sizeof(T) / 4; ++k) o[k] = q[k];
  return out;
}

// A pointer in a kernel's arguments, read from memory: a scalar load, and known to
// be global (else every access through it is a flat one).
template <typename T>
__device__ inline T* load_global(T* const* p) {
  typedef const __attribute__((address_space(4))) uint64_t Word;
  return (T*)(__attribute__((address_space(1))) T*)*(Word*)(uintptr_t)p;
}

// Coefficients of the sub-cycle for one replica: its own, or the
// relaxation's (no coupling, no field, no noise).
__device__ inline MdParams md_override(MdParams P, const MdOverride& ov) {
  if (ov.on) {
    P.gamma = ov.gamma; P.e = ov.e; P.omE = ov.omE;
    P.cf = ov.gamma == 0.0 ? (2.0 * P.hh) / P.m : ov.omE / (P.m * ov.gamma);
    P.sig = 0.0; P.couple = 0; P.field_on = 0;
  }
  return P;
}
__device__ inline MdParams md_params(const Rep& R, const MdOverride& ov) { return md_override(R.mp, ov); }

// Neighbour-search cells: side >= r_c + skin + CELL_MARGIN per replica; each
// cell hashes to one bucket of a power-of-two table of fixed-capacity buckets
// (colliding cells share a bucket: their beads fail the distance test).
__device__ inline uint32_t cell_bucket(int rep, int cx, int cy, int cz, uint32_t mask) {
  uint32_t h = ((uint32_t)rep * 73856093u) ^ ((uint32_t)cx * 19349663u) ^ ((uint32_t)cy * 83492791u) ^
               ((uint32_t)cz * 2654435761u);
  return h & mask;
}

__device__ inline void bead_cell(const Rep& R, const double* rp, int c[3]) {
  const int n[3] = {R.g.nx, R.g.ny, R.g.nz};
  for (int a = 0; a < 3; ++a) {
    double w = wrapc(rp[a], n[a]);
    if (!(w >= 0.0 && w < (double)n[a])) w = 0.0;   // non-finite: still a valid cell
    int k = (int)(w * (double)R.ncell[a] / (double)n[a]);
    c[a] = k < R.ncell[a] ? k : R.ncell[a] - 1;
  }
}

// r_mid of sub-step 0 (with mts: r itself, where the first slow kick
// evaluates its forces) and the displacement check that decides whether the
// first launch rebuilds the lists.
__global__ void k_md_start(Dev d, int nslots, MdOverride ov, int mts) {
  int slot = blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= nslots) return;
  const int rep = d.slot_rep[slot];
  const Rep& R = d.reps[rep];
  if (slot - R.slot_off >= R.mp.nb) return;
  const double hh = R.mp.hh;
  double d2 = 0.0, b2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double x = mts ? d.r[3 * slot + a] : d.r[3 * slot + a] + hh * d.v[3 * slot + a];
    d.rmid0[3 * slot + a] = x;
    double dd = x - d.ref[3 * slot + a];
    d2 += dd * dd;
    double db = x - d.rbin[3 * slot + a];
    b2 += db * db;
  }
  if (d2 > R.mp.halfskin2) d.rb[4 * rep] = 1u;
  if (!(b2 <= CELL_MARGIN * CELL_MARGIN)) d.cst[4 * rep] = 1u;
}

// The noise of a whole sub-cycle at once: xi[(s nslots + slot) 3 + a] for
// every sub-step s and bead (the same counter-based values the sub-step would
// draw, keyed by the replica's seed and index and the bead's chain index), so
// the transcendental functions run in one wide launch instead of on the
// critical path of every sub-step.  The step counter word is the control
// block's step plus step_offset (1: the sub-cycle of the next step).
__device__ inline void md_noise(const Dev& d, long k, int nslots, int n_sub, int step_offset) {
  if (k >= (long)n_sub * nslots) return;
  int sidx = (int)(k / nslots), slot = (int)(k - (long)sidx * nslots);
  const Rep& R = d.reps[d.slot_rep[slot]];
  const int p = slot - R.slot_off;
  if (p >= R.mp.nb || R.mp.sig == 0.0) return;
  double x[3];
  gauss3(R.mp.seed, R.mp.replica, (uint32_t)(d.ctrl->step + (uint64_t)step_offset), (uint32_t)sidx, (uint32_t)p, x);
  d.xi[3 * k] = x[0]; d.xi[3 * k + 1] = x[1]; d.xi[3 * k + 2] = x[2];
}
__global__ void k_md_noise(Dev d, int nslots, int n_sub, int step_offset) {
  md_noise(d, (long)blockIdx.x * blockDim.x + threadIdx.x, nslots, n_sub, step_offset);
}

// The bending angle at (ra, rb, rc) and what its forces need: the bond
// vectors, their cross product n, |n| = s, b1.b2 = c, phi = atan2(s, c),
// s^2 + c^2 and kappa phi.  s = 0 (straight or folded) has no unique
// gradient: its forces are exactly 0.
struct AngleCore {
  double b1[3], b2[3], n[3];
  double s, c, den, kp;
};
__device__ inline bool angle_core(const MdParams& P, const double* ra, const double* rb, const double* rc,
                                  AngleCore& A) {
  for (int a = 0; a < 3; ++a) { A.b1[a] = rb[a] - ra[a]; A.b2[a] = rc[a] - rb[a]; }
  A.n[0] = A.b1[1] * A.b2[2] - A.b1[2] * A.b2[1];
  A.n[1] = A.b1[2] * A.b2[0] - A.b1[0] * A.b2[2];
  A.n[2] = A.b1[0] * A.b2[1] - A.b1[1] * A.b2[0];
  A.s = sqrt(A.n[0] * A.n[0] + A.n[1] * A.n[1] + A.n[2] * A.n[2]);
  A.c = A.b1[0] * A.b2[0] + A.b1[1] * A.b2[1] + A.b1[2] * A.b2[2];
  if (A.s == 0.0) return false;
  const double phi = atan2(A.s, A.c);
  A.den = A.s * A.s + A.c * A.c;
  A.kp = P.kappa * phi;
  return true;
}
// Component a of the angle's forces: out[0] on the first bead, out[1] on the
// centre, out[2] on the third -- the operations of angle_component (and of
// angle_add) for that component, evaluated from one AngleCore.
__device__ inline void angle_part(const AngleCore& A, int a, double out[3]) {
  const int a1 = (a + 1) % 3, a2 = (a + 2) % 3;
  double g1 = A.b2[a1] * A.n[a2] - A.b2[a2] * A.n[a1];
  double g2 = A.n[a1] * A.b1[a2] - A.n[a2] * A.b1[a1];
  double d1 = (A.c * g1 / A.s - A.s * A.b2[a]) / A.den;
  double d2 = (A.c * g2 / A.s - A.s * A.b1[a]) / A.den;
  out[0] = 0.0 + A.kp * d1;
  out[1] = 0.0 + -(A.kp * (d1 - d2));
  out[2] = 0.0 + -(A.kp * d2);
}
__device__ inline void angle_component(const MdParams& P, const double* ra, const double* rb, const double* rc,
                                       int a, double out[3]) {
  double b1[3] = {rb[0] - ra[0], rb[1] - ra[1], rb[2] - ra[2]};
  double b2[3] = {rc[0] - rb[0], rc[1] - rb[1], rc[2] - rb[2]};
  double n[3] = {b1[1] * b2[2] - b1[2] * b2[1], b1[2] * b2[0] - b1[0] * b2[2], b1[0] * b2[1] - b1[1] * b2[0]};
  double s = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  double c = b1[0] * b2[0] + b1[1] * b2[1] + b1[2] * b2[2];
  if (s == 0.0) {
    // straight or folded: the contribution is exactly 0 (as in angle_add)
    out[0] = 0.0; out[1] = 0.0; out[2] = 0.0;
    return;
  }
  double phi = atan2(s, c);
  double den = s * s + c * c;
  const int a1 = (a + 1) % 3, a2 = (a + 2) % 3;
  double g1 = b2[a1] * n[a2] - b2[a2] * n[a1];
  double g2 = n[a1] * b1[a2] - n[a2] * b1[a1];
  double kp = P.kappa * phi;
  double d1 = (c * g1 / s - s * b2[a]) / den;
  double d2 = (c * g2 / s - s * b1[a]) / den;
  out[0] = 0.0 + kp * d1;
  out[1] = 0.0 + -(kp * (d1 - d2));
  out[2] = 0.0 + -(kp * d2);
}

// ---------------------------------------------------------------------------
// Sub-step kernel.  A workgroup holds 16 consecutive bead slots of one
// replica in three waves that work side by side: in the first, 4 lanes per
// bead evaluate its LJ pair forces; the second evaluates the bending of the
// 18 angles that touch the 16 beads, one lane per angle and component; the
// third the wall sites, one lane per bead and window row, and the bonds.  All
// go to LDS.  One lane per bead of the third wave then adds every
// contribution in the fixed order of the definition (bonds to p-1 and p+1,
// the angles centred at p-1, p, p+1, LJ in ascending partner order, wall
// sites, field), so the sum is the same as a one-thread-per-bead loop, and
// moves the bead.  Spreading the work keeps each wave's registers few, so
// that the workgroups fit on CUs beside the lattice sweep.
// ---------------------------------------------------------------------------
constexpr int MD_LANES = 4;
constexpr int MD_WG = MD_LANES * MD_BPB;     // 64
constexpr int WLO = -2, WHI = 3;             // wall-site window: offsets -2..3 from the base node (r_c <= 3)
constexpr int WSPAN = WHI - WLO + 1;         // 6
constexpr int MAXWALL = WSPAN * WSPAN;       // the 6 x 6 window of wall sites in the wall plane
constexpr int NB_PER_LANE = MAXNBR / MD_LANES;

struct MdShared {
  double ang[MD_BPB + 2][9];                 // forces of the angles centred at p0-1 .. p0+16: [0..2] on
                                             // q-1, [3..5] on q, [6..8] on q+1
  double pairF[MD_BPB][MAXNBR][3];           // LJ pair force of list entry k
  uint32_t hit[MD_BPB][MD_LANES];            // lane l, bit m: entry l + 4m is within r_c
  uint32_t wmask[MD_BPB][WSPAN];             // row o1 - WLO: which sites o0 - WLO of the row are set
  int cnt[MD_BPB];
  int lst[MD_BPB][MAXNBR];                   // the neighbour list in use (partner slots)
  // the list rebuild's scratch is dead before the wall sites are written
  union {
    struct {
      double tile[MD_WG][3];                 // rebuild: positions of 64 candidates
      uint32_t tmask[MD_BPB][MD_LANES];      // rebuild: lane l, bit e: candidate 16 l + e is close
      uint32_t bk[MD_BPB][28];               // rebuild from the cell table: the 27 buckets around a bead
    };
    double wallF[MD_BPB][MAXWALL][3];        // wall site (o1 - WLO) * WSPAN + (o0 - WLO) of each bead
  };
  int over;
};
static_assert(2 * sizeof(MdShared) <= (size_t)LDS_KEEP, "two sub-step workgroups fit in the LDS a capped sweep leaves");

// Wall sites of the bead at rp, one row of the window at a time: the sites
// at offsets P.wlo..P.whi (within -2..3) from the base node along the lower
// transverse axis (o0), for offset o1 along the higher one; offsets outside
// 1 - ceil(r_c) .. ceil(r_c) cannot reach r_c, so the window shrinks to
// -1..2 for r_c <= 2.  Each is the truncated-LJ pair force of
// one solid site within r_c; the force of offset o0 goes to out[o0 - WLO] and
// the returned mask has bit o0 - WLO set.  r_c <= 3 makes the window cover
// every candidate.  Solid sites lie in the plane a = wall_pos (minus the
// pore), so at most one offset along the wall normal can match.  Rows
// o1 = -2..3, each in o0 order, visit the sites in the order of the
// definition's sum (higher transverse axis outer).  Wrapping uses compares
// only (the window is within one period: extents are at least 6).
__device__ inline uint32_t wall_row(const MdParams& P, const Geom& g, const double* rp, int o1,
                                    double out[WSPAN][3]) {
  if (g.wall_axis < 0) return 0u;
  const double w0 = wrapc(rp[0], g.nx), w1 = wrapc(rp[1], g.ny), w2 = wrapc(rp[2], g.nz);
  const int b0 = (int)floor(w0), b1 = (int)floor(w1), b2 = (int)floor(w2);
  const int a = g.wall_axis;
  // normal-axis base and extent; transverse axes t0 < t1
  const int ba = a == 0 ? b0 : (a == 1 ? b1 : b2);
  const int na = a == 0 ? g.nx : (a == 1 ? g.ny : g.nz);
  const int bt0 = a == 0 ? b1 : b0, n0 = a == 0 ? g.ny : g.nx;
  const int bt1 = a == 2 ? b1 : b2, n1 = a == 2 ? g.ny : g.nz;
  int off = g.wall_pos - ba;                // offset along the normal reaching the plane
  if (off < WLO) off += na;
  if (off > WHI) off -= na;
  if (off < P.wlo || off > P.whi) return 0u;
  const int sa = ba + off;
  const int u1 = bt1 + o1;
  const int v1 = u1 < 0 ? u1 + n1 : (u1 >= n1 ? u1 - n1 : u1);
  const bool in1 = v1 >= g.lo1 && v1 <= g.hi1;
  uint32_t mask = 0u;
  for (int o0 = P.wlo; o0 <= P.whi; ++o0) {
    const int u0 = bt0 + o0;
    const int v0 = u0 < 0 ? u0 + n0 : (u0 >= n0 ? u0 - n0 : u0);
    const bool in0 = v0 >= g.lo0 && v0 <= g.hi0;
    if (in0 && in1) continue;               // pore node: fluid
    const int sx = a == 0 ? sa : u0;
    const int sy = a == 1 ? sa : (a == 0 ? u0 : u1);
    const int sz = a == 2 ? sa : u1;
    const double d0 = w0 - (double)sx, d1 = w1 - (double)sy, d2 = w2 - (double)sz;
    if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rc2)) continue;
    double F[3] = {0.0, 0.0, 0.0};
    lj_add(P, d0, d1, d2, F);
    out[o0 - WLO][0] = F[0]; out[o0 - WLO][1] = F[1]; out[o0 - WLO][2] = F[2];
    mask |= 1u << (o0 - WLO);
  }
  return mask;
}

// SLOW: a kick of the multiple-time-step cycle instead of a sub-step.  The
// slow forces (bead LJ, wall sites, field) are evaluated at r, which does not
// change, and `last` half kicks v += kick F are applied one after the other
// (2 between two outer steps, 1 at the ends); s is the kick's index in the
// cycle (0..M), which selects the rotating rebuild words.
template <bool SLOW>
__global__ __launch_bounds__(3 * MD_WG) void k_md_substep(Dev d, MdOverride ov, int nslots, int s, int last) {
  __shared__ MdShared sh;
  const int t = threadIdx.x;
  // wave 0 holds the neighbour lists and LJ pairs (4 lanes per bead), wave 1
  // evaluates the angles, wave 2 the wall sites and bonds and then moves the
  // beads.  Every wave takes every barrier: the branches around barriers are
  // uniform in the workgroup.
  const int wave = __builtin_amdgcn_readfirstlane(t) / MD_WG;
  const int tb = t - wave * MD_WG;           // lane within the wave
  const int bslot = tb / MD_LANES, lane = tb % MD_LANES;
  const int slot0 = blockIdx.x * MD_BPB;
  const int slot = slot0 + bslot;            // the grid covers the nslots slots exactly
  const double* rabs = (s & 1) ? d.rmid1 : d.rmid0;
  double* rout = (s & 1) ? d.rmid0 : d.rmid1;
  const double* vin = (const double*)d.xring;   // SLOW: the inner cycle's velocities
  auto clampslot = [nslots](int q) { return q < 0 ? 0 : (q >= nslots ? nslots - 1 : q); };

  // ---- first-level loads, addressed by slot alone so that they are in
  // flight before the replica's parameters arrive.  Indices are clamped into
  // the slot range; a value from outside the chain is never used.
  double rp[3] = {0.0, 0.0, 0.0};
  int* nbr_row = d.nbr + (size_t)slot * MAXNBR;
  int ncnt_in = 0;
  int pre[NB_PER_LANE];                       // list entries lane, lane + 4, ... (past the length unused)
  double vo[3], Jo[3], ul[3], xl[3], rm[3], rq[3], rbl[3], rfl[3];
  double ra[3] = {0.0, 0.0, 0.0}, rb3[3] = {0.0, 0.0, 0.0}, rc[3] = {0.0, 0.0, 0.0};
  if (wave == 0) {
    rp[0] = rabs[3 * slot]; rp[1] = rabs[3 * slot + 1]; rp[2] = rabs[3 * slot + 2];
    ncnt_in = d.ncnt[slot];
#pragma unroll
    for (int m = 0; m < NB_PER_LANE; ++m) pre[m] = nbr_row[lane + MD_LANES * m];
  } else if (wave == 1) {
    if (!SLOW && tb < 3 * (MD_BPB + 2)) {
      // positions of the angle centred at slot slot0 - 1 + tb / 3
      const int c = slot0 - 1 + tb / 3;
      const int ia = clampslot(c - 1), ib = clampslot(c), ic = clampslot(c + 1);
#pragma unroll
      for (int a = 0; a < 3; ++a) { ra[a] = rabs[3 * ia + a]; rb3[a] = rabs[3 * ib + a]; rc[a] = rabs[3 * ic + a]; }
    }
  } else {
    rp[0] = rabs[3 * slot]; rp[1] = rabs[3 * slot + 1]; rp[2] = rabs[3 * slot + 2];
  }

  // ---- the replica
  const int rep = d.slot_rep[slot0];
  const Rep& R = d.reps[rep];
  const MdParams P = md_params(R, ov);
  const Geom g = R.g;
  const int so = R.slot_off;
  const int p0 = slot0 - so;                 // chain index of the first bead here
  const int p = p0 + bslot;
  const bool active = wave == 0 && p < P.nb;
  const double* rin = rabs + 3 * (size_t)so; // chain-relative
  uint32_t* rbr = d.rb + 4 * rep;
  const uint32_t rebuild = rbr[s % 3];
  const uint32_t table_stale = d.cst[4 * rep + s % 3];
  if (t == 0) {
    if (p0 == 0) {
      rbr[(s + 2) % 3] = 0u;
      d.cst[4 * rep + (s + 2) % 3] = 0u;
      if (rebuild) atomicAdd((unsigned long long*)&d.ctrl->rebuilds, 1ull);
      if (rebuild && !table_stale) atomicAdd((unsigned long long*)&d.ctrl->cell_rebuilds, 1ull);
    }
    if (!SLOW && blockIdx.x == 0) atomicAdd((unsigned long long*)&d.ctrl->substeps, 1ull);
    sh.over = 0;
  }
  // lane 0 of each bead in wave 2 adds the contributions and moves the bead
  const bool lead = wave == 2 && lane == 0 && p < P.nb;
  const int ncnt0 = active ? ncnt_in : 0;

  // ---- neighbour list: reuse (already in registers), or rebuild -- from
  // the cell table while every bead of the chain is within CELL_MARGIN of
  // where the table binned it, else by scanning the chain in tiles of 64
  int cnt = ncnt0;
  int jl[NB_PER_LANE];
  if (!rebuild) {
#pragma unroll
    for (int m = 0; m < NB_PER_LANE; ++m) jl[m] = (lane + MD_LANES * m < cnt) ? pre[m] : -1;
  } else {
    if (wave == 0 && lane == 0) sh.cnt[bslot] = 0;
    if (!table_stale) {
      // lane l scans the distinct buckets l, l + 4, ... of the 27 cells
      // around the bead (a candidate binned within CELL_MARGIN of its
      // position lies in one of them); the lead lane then sorts
      if (active) {
        int c[3];
        bead_cell(R, rp, c);
        for (int k = lane; k < 27; k += MD_LANES) {
          const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
          sh.bk[bslot][k] = cell_bucket(rep, (c[0] + dx + R.ncell[0]) % R.ncell[0],
                                        (c[1] + dy + R.ncell[1]) % R.ncell[1], (c[2] + dz + R.ncell[2]) % R.ncell[2],
                                        d.cmask);
        }
      }
      __syncthreads();
      if (active) {
        for (int k = lane; k < 27; k += MD_LANES) {
          const uint32_t b = sh.bk[bslot][k];
          bool dup = false;
          for (int k2 = 0; k2 < k; ++k2) dup = dup || sh.bk[bslot][k2] == b;
          if (dup) continue;
          const int n = min(d.ccount[b], CELL_CAP);
          for (int e = 0; e < n; ++e) {
            const int q = d.cbuf[(size_t)b * CELL_CAP + e];
            if (d.slot_rep[q] != rep || q == slot) continue;
            double d0 = min_image(rp[0] - rabs[3 * q], g.nx);
            double d1 = min_image(rp[1] - rabs[3 * q + 1], g.ny);
            double d2 = min_image(rp[2] - rabs[3 * q + 2], g.nz);
            if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rlist2)) continue;
            const int at = atomicAdd(&sh.cnt[bslot], 1);
            if (at < MAXNBR) sh.lst[bslot][at] = q;
            else sh.over = 1;
          }
        }
      }
      __syncthreads();
      if (active && lane == 0) {
        const int c = min(sh.cnt[bslot], MAXNBR);
        int* L = sh.lst[bslot];
        for (int i = 1; i < c; ++i) {
          const int v = L[i];
          int m = i;
          while (m > 0 && L[m - 1] > v) { L[m] = L[m - 1]; --m; }
          L[m] = v;
        }
      }
    } else {
      for (int base = 0; base < P.nb; base += MD_WG) {
        __syncthreads();
        const int j = base + tb;
        if (wave == 0 && j < P.nb) {
          sh.tile[tb][0] = rin[3 * j]; sh.tile[tb][1] = rin[3 * j + 1]; sh.tile[tb][2] = rin[3 * j + 2];
        }
        __syncthreads();
        uint32_t m = 0;
        if (active) {
          for (int e = 0; e < 16; ++e) {
            int tt = 16 * lane + e;
            int jj = base + tt;
            if (jj >= P.nb || jj == p) continue;
            double d0 = min_image(rp[0] - sh.tile[tt][0], g.nx);
            double d1 = min_image(rp[1] - sh.tile[tt][1], g.ny);
            double d2 = min_image(rp[2] - sh.tile[tt][2], g.nz);
            if (d0 * d0 + d1 * d1 + d2 * d2 < P.rlist2) m |= 1u << e;
          }
        }
        if (wave == 0) sh.tmask[bslot][lane] = m;
        __syncthreads();
        if (active && lane == 0) {
          uint64_t mm = (uint64_t)sh.tmask[bslot][0] | ((uint64_t)sh.tmask[bslot][1] << 16) |
                        ((uint64_t)sh.tmask[bslot][2] << 32) | ((uint64_t)sh.tmask[bslot][3] << 48);
          int c = sh.cnt[bslot];
          while (mm) {
            int tt = __builtin_ctzll(mm);
            mm &= mm - 1;
            if (c < MAXNBR) sh.lst[bslot][c] = so + base + tt;
            else sh.over = 1;
            ++c;
          }
          sh.cnt[bslot] = c;
        }
      }
    }
    __syncthreads();
    if (active && lane == 0) {
      int c = sh.cnt[bslot];
      if (c > MAXNBR) { c = MAXNBR; sh.cnt[bslot] = c; }
      d.ncnt[slot] = c;
      d.ref[3 * slot] = rp[0]; d.ref[3 * slot + 1] = rp[1]; d.ref[3 * slot + 2] = rp[2];
    }
    __syncthreads();
    cnt = active ? sh.cnt[bslot] : 0;
    for (int k = lane; k < cnt; k += MD_LANES) nbr_row[k] = sh.lst[bslot][k];
    if (t == 0 && sh.over) atomicOr(&d.ctrl->err, E_NBRLIST);
#pragma unroll
    for (int m = 0; m < NB_PER_LANE; ++m) {
      int k = lane + MD_LANES * m;
      jl[m] = (k < cnt) ? sh.lst[bslot][k] : -1;
    }
  }

  double F[3] = {0.0, 0.0, 0.0};
  if (wave == 1) {
    // ---- the angles centred at p0 - 1 .. p0 + 16: lane 3 k + a takes
    // component a of angle k
    if (!SLOW && tb < 3 * (MD_BPB + 2)) {
      const int k = tb / 3, a = tb % 3;
      const int qc = p0 - 1 + k;
      if (qc >= 1 && qc <= P.nb - 2) {
        double f[3];
        angle_component(P, ra, rb3, rc, a, f);
        sh.ang[k][a] = f[0]; sh.ang[k][3 + a] = f[1]; sh.ang[k][6 + a] = f[2];
      }
    }
  } else if (wave == 2) {
    // the bead's own state, its chain neighbours and its list references
    // (every lane of the bead reads them; lane 0 uses them).  Loaded here,
    // not with the first loads, so that they hold no registers while the
    // other waves work; they are needed only at the end.
    if (SLOW) {
#pragma unroll
      for (int a = 0; a < 3; ++a) vo[a] = (s > 0 ? vin : d.v)[3 * slot + a];
    } else {
      const int sm = clampslot(slot - 1), sq = clampslot(slot + 1);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        rbl[a] = d.rbin[3 * slot + a];
        rfl[a] = d.ref[3 * slot + a];
        vo[a] = d.v[3 * slot + a];
        Jo[a] = d.J[3 * slot + a];
        ul[a] = d.up[3 * slot + a];
        xl[a] = ov.on ? 0.0 : d.xi[(size_t)3 * ((size_t)s * nslots + slot) + a];
        rm[a] = rabs[3 * sm + a];
        rq[a] = rabs[3 * sq + a];
      }
    }
    // ---- wall sites: rows outside wlo..whi hold no site within r_c and
    // stay empty; lane l takes the rows o1 = wlo + l, wlo + l + 4, ... (for
    // r_c <= 2 one row per lane, all lanes at once).  The clearing stores
    // precede the row stores of the same wave.
    for (int row = lane; row < WSPAN; row += MD_LANES) sh.wmask[bslot][row] = 0u;
    for (int o1 = P.wlo + lane; o1 <= P.whi; o1 += MD_LANES)
      sh.wmask[bslot][o1 - WLO] = p < P.nb ? wall_row(P, g, rp, o1, &sh.wallF[bslot][WSPAN * (o1 - WLO)]) : 0u;
    // ---- lane 0: bonds now, the rest after the barrier
    if (!SLOW && lead && !P.constrained) {
      if (p > 0) bond_add(P, rp, rm, F);
      if (p < P.nb - 1) bond_add(P, rp, rq, F);
    }
  } else {
    // ---- LJ pair forces: lane l handles list entries l, l + 4, l + 8, ...
    double q[NB_PER_LANE][3];
#pragma unroll
    for (int m = 0; m < NB_PER_LANE; ++m) {
      const int j = jl[m] >= 0 ? jl[m] : slot0;   // an unused entry reads a valid slot
      q[m][0] = rabs[3 * j]; q[m][1] = rabs[3 * j + 1]; q[m][2] = rabs[3 * j + 2];
    }
    uint32_t hit = 0;
#pragma unroll
    for (int m = 0; m < NB_PER_LANE; ++m) {
      if (jl[m] < 0) continue;
      double d0 = min_image(rp[0] - q[m][0], g.nx);
      double d1 = min_image(rp[1] - q[m][1], g.ny);
      double d2 = min_image(rp[2] - q[m][2], g.nz);
      if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rc2)) continue;
      double Fp[3] = {0.0, 0.0, 0.0};
      lj_add(P, d0, d1, d2, Fp);
      int k = lane + MD_LANES * m;
      sh.pairF[bslot][k][0] = Fp[0]; sh.pairF[bslot][k][1] = Fp[1]; sh.pairF[bslot][k][2] = Fp[2];
      hit |= 1u << m;
    }
    sh.hit[bslot][lane] = hit;
    if (lane == 0) sh.cnt[bslot] = cnt;
  }
  __syncthreads();
  if (!lead) return;
  // every contribution in the fixed order
  const int cnt_b = sh.cnt[bslot];
  const int q0 = p0 - 1;
  const int nb = P.nb;
  if (!SLOW) {
    if (p - 1 >= 1 && p - 1 <= nb - 2) { const double* A = sh.ang[p - 1 - q0]; F[0] += A[6]; F[1] += A[7]; F[2] += A[8]; }
    if (p >= 1 && p <= nb - 2) { const double* A = sh.ang[p - q0]; F[0] += A[3]; F[1] += A[4]; F[2] += A[5]; }
    if (p + 1 >= 1 && p + 1 <= nb - 2) { const double* A = sh.ang[p + 1 - q0]; F[0] += A[0]; F[1] += A[1]; F[2] += A[2]; }
  }
  // the list entries with a pair force, in list order: entry k is bit
  // k / 4 of lane k % 4's word; interleaved into one mask so that only the
  // hits are visited (lists are much longer than the pairs within r_c)
  {
    uint32_t h[MD_LANES];
#pragma unroll
    for (int l = 0; l < MD_LANES; ++l) h[l] = sh.hit[bslot][l];
    uint64_t hm = 0;
#pragma unroll
    for (int e = 0; e < NB_PER_LANE; ++e)
#pragma unroll
      for (int l = 0; l < MD_LANES; ++l) hm |= (uint64_t)((h[l] >> e) & 1u) << (MD_LANES * e + l);
    (void)cnt_b;
    while (hm) {
      const int k = __builtin_ctzll(hm);
      hm &= hm - 1;
      F[0] += sh.pairF[bslot][k][0]; F[1] += sh.pairF[bslot][k][1]; F[2] += sh.pairF[bslot][k][2];
    }
  }
  // the wall sites within r_c, in ascending site order (set bits only: most
  // beads have none)
  uint64_t wm = 0;
#pragma unroll
  for (int row = 0; row < WSPAN; ++row) wm |= (uint64_t)sh.wmask[bslot][row] << (WSPAN * row);
  while (wm) {
    const int k = __builtin_ctzll(wm);
    wm &= wm - 1;
    F[0] += sh.wallF[bslot][k][0]; F[1] += sh.wallF[bslot][k][1]; F[2] += sh.wallF[bslot][k][2];
  }
  if (P.field_on && in_field(g, rp)) F[g.wall_axis] += P.f_drive;

  if (SLOW) {
    bool fin = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double vn = vo[a] + P.kick * F[a];
      if (last == 2) vn = vn + P.kick * F[a];
      d.v[3 * slot + a] = vn;
      if (s > 0 && last == 1) d.r[3 * slot + a] = rp[a];   // the cycle's end
      fin = fin && isfinite(vn);
    }
    if (!fin) atomicOr(&d.ctrl->err, E_BEADS);
    return;
  }

  double u[3], xi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u[a] = P.couple ? ul[a] : 0.0;
    xi[a] = P.sig != 0.0 ? xl[a] : 0.0;
  }
  double vn[3];
  bool finite = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double sx = P.sig * xi[a];
    vn[a] = P.e * vo[a] + P.cf * (F[a] + P.gamma * u[a]) + sx;
    d.J[3 * slot + a] = Jo[a] - P.m * (P.omE * (u[a] - vo[a]) + sx);
    d.v[3 * slot + a] = vn[a];
    finite = finite && isfinite(vn[a]);
  }
  if (!finite) atomicOr(&d.ctrl->err, E_BEADS);
  // rigid bonds: RATTLE, the drift and the next SHAKE follow in
  // k_md_constraint, which also sets the rebuild words
  if (P.constrained) return;
  if (d.mdtape) {
    double* tp = d.mdtape + ((size_t)s * P.nb + p) * 6;
    tp[0] = rp[0]; tp[1] = rp[1]; tp[2] = rp[2];
    tp[3] = vo[0]; tp[4] = vo[1]; tp[5] = vo[2];
  }
  double re[3] = {rp[0] + P.hh * vn[0], rp[1] + P.hh * vn[1], rp[2] + P.hh * vn[2]};
  if (last) {
    d.r[3 * slot] = re[0]; d.r[3 * slot + 1] = re[1]; d.r[3 * slot + 2] = re[2];
  } else {
    double d2 = 0.0, b2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double x = re[a] + P.hh * vn[a];
      rout[3 * slot + a] = x;
      double dd = x - (rebuild ? rp[a] : rfl[a]);   // a rebuild this sub-step set ref = r_mid
      d2 += dd * dd;
      double db = x - rbl[a];
      b2 += db * db;
    }
    if (d2 > P.halfskin2) rbr[(s + 1) % 3] = 1u;
    if (!(b2 <= CELL_MARGIN * CELL_MARGIN)) d.cst[4 * rep + (s + 1) % 3] = 1u;
  }
}

__global__ void k_zero_v(double* v, int n) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) v[k] = 0.0;
}

// ---------------------------------------------------------------------------
// Inner cycle of outer step o of the multiple-time-step scheme: M_b SPV
// sub-steps with the bonded forces only (bonds, bending), the friction
// towards the frozen u_p and the noise of sub-step index o M_b + i, all in
// one launch.  The bonded force on a bead depends on the chain neighbours
// p-2 .. p+2 only, so a workgroup advances a segment of IN_WG consecutive
// slots through the whole inner cycle with its positions in LDS and one
// barrier per sub-step; the 2 M_b slots at each end are a halo computed again
// by the neighbouring workgroup (after i sub-steps the missing neighbours
// beyond the segment have corrupted at most 2 i slots at each end), so each
// workgroup stores only the IN_WG - 4 M_b slots in the middle.  Sums follow
// the definition's order: bonds to p-1 and p+1, then the angles centred at
// p-1, p, p+1.  The last lane state also gives the displacement checks of the
// slow kick that follows (index o + 1).
// A halo slot is read while the workgroup that owns it may have ended, so
// the results go to other arrays than those read: positions alternate between
// r_mid0 and r_mid1, velocities go from v to the exchange memory of the
// resident cycle (which runs instead of this kernel up to RES_MAX_WG segments),
// and the kicks bring both back.
// ---------------------------------------------------------------------------
constexpr int IN_WG = 256;

__global__ __launch_bounds__(IN_WG) void k_md_inner(Dev d, int nslots, int o, int Mb) {
  __shared__ double pos[2][IN_WG][3];
  const int j = threadIdx.x;
  const double* rin = (o & 1) ? d.rmid1 : d.rmid0;
  double* rout = (o & 1) ? d.rmid0 : d.rmid1;
  double* vout = (double*)d.xring;
  const int H = 2 * Mb, own = IN_WG - 2 * H;
  const int gslot = (int)blockIdx.x * own - H + j;
  const bool valid = gslot >= 0 && gslot < nslots;
  const int slot = valid ? gslot : 0;
  const int rep = d.slot_rep[slot];
  const Rep& R = d.reps[rep];
  const int p = slot - R.slot_off;
  const int nb = R.mp.nb;
  const bool active = valid && p < nb;
  const double hh = R.mp.hh, e = R.mp.e, cf = R.mp.cf, gam = R.mp.gamma, omE = R.mp.omE, sig = R.mp.sig;
  const double m = R.mp.m;
  double r[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, J[3] = {0.0, 0.0, 0.0}, u[3] = {0.0, 0.0, 0.0};
  if (active) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      r[a] = rin[3 * slot + a];
      v[a] = d.v[3 * slot + a];
      J[a] = d.J[3 * slot + a];
      u[a] = R.mp.couple ? d.up[3 * slot + a] : 0.0;
    }
  }
  // chain neighbour p + k is in the chain and in this segment
  auto has = [&](int k) { return p + k >= 0 && p + k < nb && j + k >= 0 && j + k < IN_WG; };
  for (int i = 0; i < Mb; ++i) {
    const int sidx = o * Mb + i;
    double xi[3] = {0.0, 0.0, 0.0};
    if (active && sig != 0.0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) xi[a] = d.xi[(size_t)3 * ((size_t)sidx * nslots + slot) + a];
    }
    double rh[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      rh[a] = r[a] + hh * v[a];
      pos[i & 1][j][a] = rh[a];
    }
    __syncthreads();
    if (active) {
      const double(*q)[3] = pos[i & 1];
      double F[3] = {0.0, 0.0, 0.0};
      if (p > 0 && has(-1)) bond_add(R.mp, rh, q[j - 1], F);
      if (p < nb - 1 && has(1)) bond_add(R.mp, rh, q[j + 1], F);
      if (p - 1 >= 1 && p - 1 <= nb - 2 && has(-2)) angle_add(R.mp, q[j - 2], q[j - 1], rh, 2, F);
      if (p >= 1 && p <= nb - 2 && has(-1) && has(1)) angle_add(R.mp, q[j - 1], rh, q[j + 1], 1, F);
      if (p + 1 >= 1 && p + 1 <= nb - 2 && has(2)) angle_add(R.mp, rh, q[j + 1], q[j + 2], 0, F);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double sx = sig * xi[a];
        const double vn = e * v[a] + cf * (F[a] + gam * u[a]) + sx;
        J[a] = J[a] - m * (omE * (u[a] - v[a]) + sx);
        v[a] = vn;
        r[a] = rh[a] + hh * vn;
      }
    }
  }
  if (j == 0 && blockIdx.x == 0) atomicAdd((unsigned long long*)&d.ctrl->substeps, (unsigned long long)Mb);
  if (!active || j < H || j >= IN_WG - H) return;
  bool fin = true;
  double d2 = 0.0, b2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    rout[3 * slot + a] = r[a];
    vout[3 * slot + a] = v[a];
    d.J[3 * slot + a] = J[a];
    fin = fin && isfinite(v[a]) && isfinite(r[a]);
    const double dd = r[a] - d.ref[3 * slot + a];
    d2 += dd * dd;
    const double db = r[a] - d.rbin[3 * slot + a];
    b2 += db * db;
  }
  if (!fin) atomicOr(&d.ctrl->err, E_BEADS);
  if (d2 > R.mp.halfskin2) d.rb[4 * rep + (o + 1) % 3] = 1u;
  if (!(b2 <= CELL_MARGIN * CELL_MARGIN)) d.cst[4 * rep + (o + 1) % 3] = 1u;
}

// ---------------------------------------------------------------------------
// Neighbour lists from the hashed cell table, once per coupled step.  Each
// bead is examined by 32 lanes, one per distinct bucket of its 27 neighbour
// cells; the lanes collect the other beads of its chain within r_c + skin,
// and one lane sorts their slots into ascending (chain) order -- the list the
// in-kernel scan would build.  A bucket that overflows leaves its replica's
// lists marked invalid (and the table unusable), so the first sub-step
// rebuilds them by the full scan: the same lists, found slower.
// ---------------------------------------------------------------------------
__global__ void k_cell_clear(int* __restrict__ ccount, int nbuckets, uint32_t* __restrict__ rb, int nrep) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nbuckets) ccount[k] = 0;
  if (k < nrep) rb[4 * k + 3] = 0u;          // valid unless a bucket overflows below
}

__device__ inline void cell_insert_slot(const Dev& d, int slot) {
  const int rep = d.slot_rep[slot];
  const Rep& R = d.reps[rep];
  if (slot - R.slot_off >= R.mp.nb) return;
  int c[3];
  bead_cell(R, &d.r[3 * slot], c);
  const uint32_t b = cell_bucket(rep, c[0], c[1], c[2], d.cmask);
  const int pos = atomicAdd(&d.ccount[b], 1);
  if (pos < CELL_CAP) d.cbuf[(size_t)b * CELL_CAP + pos] = slot;
  // a bead left out of a full bucket is "far from its binned position", so
  // the table is not used inside the sub-cycle
#pragma unroll
  for (int a = 0; a < 3; ++a) d.rbin[3 * slot + a] = pos < CELL_CAP ? d.r[3 * slot + a] : 1e300;
}

__global__ void k_cell_insert(Dev d, int nslots) {
  int slot = blockIdx.x * blockDim.x + threadIdx.x;
  if (slot < nslots) cell_insert_slot(d, slot);
}

constexpr int LB_LANES = 32;                 // lanes per bead in the list build (27 cells)
constexpr int LB_BEADS = 2;                  // beads per 64-lane workgroup
constexpr int LB_CAND = 96;                  // candidates a bead may collect

// The workgroups after the first nbuild draw the next step's noise (noise: its
// buffer, NULL for none).
__global__ __launch_bounds__(LB_LANES * LB_BEADS) void k_list_build(Dev d, int nslots, int nbuild, double* noise,
                                                                    int n_sub) {
  if ((int)blockIdx.x >= nbuild) {
    Dev dn = d;
    dn.xi = noise;
    md_noise(dn, ((long)blockIdx.x - nbuild) * (LB_LANES * LB_BEADS) + threadIdx.x, nslots, n_sub, 1);
    return;
  }
  __shared__ int cand[LB_BEADS][LB_CAND];
  __shared__ int ncand[LB_BEADS];
  __shared__ uint32_t bkt[LB_BEADS][LB_LANES];
  const int lb = threadIdx.x / LB_LANES, lane = threadIdx.x % LB_LANES;
  const int slot = blockIdx.x * LB_BEADS + lb;
  bool on = slot < nslots;
  int rep = 0, so = 0, p = 0;
  if (on) {
    rep = d.slot_rep[slot];
    so = d.reps[rep].slot_off;
    p = slot - so;
    on = p < d.reps[rep].mp.nb;
  }
  double rp[3] = {0.0, 0.0, 0.0};
  uint32_t b = 0xffffffffu;
  if (on) {
    rp[0] = d.r[3 * slot]; rp[1] = d.r[3 * slot + 1]; rp[2] = d.r[3 * slot + 2];
    if (lane < 27) {
      const Rep& R = d.reps[rep];
      int c[3];
      bead_cell(R, rp, c);
      const int dx = lane % 3 - 1, dy = (lane / 3) % 3 - 1, dz = lane / 9 - 1;
      b = cell_bucket(rep, (c[0] + dx + R.ncell[0]) % R.ncell[0], (c[1] + dy + R.ncell[1]) % R.ncell[1],
                      (c[2] + dz + R.ncell[2]) % R.ncell[2], d.cmask);
    }
  }
  bkt[lb][lane] = b;
  if (lane == 0) ncand[lb] = 0;
  __syncthreads();
  // a bucket reached from several neighbour cells (wrapped small cell counts,
  // hash collisions) is scanned by its lowest lane only: every candidate once
  bool scan = b != 0xffffffffu;
  for (int k = 0; k < lane && scan; ++k) scan = bkt[lb][k] != b;
  if (scan) {
    const Geom& g = d.reps[rep].g;
    const double rl2 = d.reps[rep].mp.rlist2;
    const int cnt = d.ccount[b];
    if (cnt > CELL_CAP) d.rb[4 * rep + 3] = 1u;   // incomplete bucket: rebuild in-kernel
    const int n = min(cnt, CELL_CAP);
    for (int k = 0; k < n; ++k) {
      const int q = d.cbuf[(size_t)b * CELL_CAP + k];
      if (d.slot_rep[q] != rep || q == slot) continue;
      double d0 = min_image(rp[0] - d.r[3 * q], g.nx);
      double d1 = min_image(rp[1] - d.r[3 * q + 1], g.ny);
      double d2 = min_image(rp[2] - d.r[3 * q + 2], g.nz);
      if (!(d0 * d0 + d1 * d1 + d2 * d2 < rl2)) continue;
      const int at = atomicAdd(&ncand[lb], 1);
      if (at < LB_CAND) cand[lb][at] = q;
    }
  }
  __syncthreads();
  if (!on || lane != 0) return;
  // ascending chain order, the MAXNBR smallest kept
  int nc = ncand[lb];
  if (nc > MAXNBR) atomicOr(&d.ctrl->err, E_NBRLIST);
  // read first: once the maximum is reached, most beads skip the atomic
  if ((uint32_t)nc > __hip_atomic_load(&d.ctrl->nbr_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(&d.ctrl->nbr_max, (uint32_t)nc);
  if (nc > LB_CAND) nc = LB_CAND;
  int* c = cand[lb];
  for (int i = 1; i < nc; ++i) {
    const int v = c[i];
    int m = i;
    while (m > 0 && c[m - 1] > v) { c[m] = c[m - 1]; --m; }
    c[m] = v;
  }
  if (nc > MAXNBR) nc = MAXNBR;
  int* row = d.nbr + (size_t)slot * MAXNBR;
  for (int i = 0; i < nc; ++i) row[i] = c[i];
  d.ncnt[slot] = nc;
  d.ref[3 * slot] = rp[0]; d.ref[3 * slot + 1] = rp[1]; d.ref[3 * slot + 2] = rp[2];
}

// k_cell_insert in the first `nins` workgroups; after them one workgroup per
// replica adds its beads' spread-on-solid shares (TAIL_SUM strided sums, then a
// fixed tree) into its ledger, and records the translocation step when every
// bead is past the wall plane for the first time.  Small workgroups, which find
// room beside the sweep.
constexpr int TAIL_WG = 256, TAIL_SUM = 1024;
__global__ __launch_bounds__(TAIL_WG) void k_tail_insert(Dev d, int nslots, int nins) {
  if ((int)blockIdx.x < nins) {                  // uniform in the workgroup
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot < nslots) cell_insert_slot(d, slot);
    return;
  }
  __shared__ double sh[TAIL_SUM];
  const int rep = blockIdx.x - nins;
  const Rep& R = d.reps[rep];
  if (R.g.wall_axis < 0 || R.mp.nb == 0) return; // uniform; nothing to add
  const int t = threadIdx.x;
  bool past = true;
  for (int p = t; p < R.mp.nb; p += TAIL_WG)
    past = past && d.r[3 * (size_t)(R.slot_off + p) + R.g.wall_axis] > (double)R.g.wall_pos;
  if (__syncthreads_and(past ? 1 : 0) && t == 0 && d.tX[rep] < 0) d.tX[rep] = (int64_t)d.ctrl->step + 1;
  for (int a = 0; a < 3; ++a) {
    for (int k = t; k < TAIL_SUM; k += TAIL_WG) {
      double s = 0.0;
      for (int p = k; p < R.mp.nb; p += TAIL_SUM) s += d.lsp[3 * (size_t)(R.slot_off + p) + a];
      sh[k] = s;
    }
    __syncthreads();
    for (int w = TAIL_SUM / 2; w > 0; w >>= 1) {
      for (int k = t; k < w; k += TAIL_WG) sh[k] += sh[k + w];
      __syncthreads();
    }
    if (t == 0) d.ledger[NLEDGER * rep + 3 + a] += sh[0];
    __syncthreads();
  }
}

void launch_step_tail(const Dev& d, int nslots, int nrep, double* noise, int n_sub, hipStream_t s) {
  if (nslots <= 0) return;
  const int nins = (nslots + TAIL_WG - 1) / TAIL_WG;
  hipLaunchKernelGGL(k_tail_insert, dim3((unsigned)(nins + nrep)), dim3(TAIL_WG), 0, s, d, nslots, nins);
  const unsigned nbuild = (unsigned)((nslots + LB_BEADS - 1) / LB_BEADS);
  const unsigned nn = noise ? (unsigned)(((long)n_sub * nslots + LB_LANES * LB_BEADS - 1) / (LB_LANES * LB_BEADS)) : 0u;
  hipLaunchKernelGGL(k_list_build, dim3(nbuild + nn), dim3(LB_LANES * LB_BEADS), 0, s, d, nslots, (int)nbuild, noise,
                     n_sub);
}

void launch_nbr_build(const Dev& d, int nslots, int nrep, hipStream_t s) {
  if (nslots <= 0) return;
  const int nb = (int)d.cmask + 1;
  const int nclr = nb > nrep ? nb : nrep;
  hipLaunchKernelGGL(k_cell_clear, dim3((nclr + 255) / 256), dim3(256), 0, s, d.ccount, nb, d.rb, nrep);
  hipLaunchKernelGGL(k_cell_insert, dim3((nslots + 255) / 256), dim3(256), 0, s, d, nslots);
  const unsigned nbuild = (unsigned)((nslots + LB_BEADS - 1) / LB_BEADS);
  hipLaunchKernelGGL(k_list_build, dim3(nbuild), dim3(LB_LANES * LB_BEADS), 0, s, d, nslots, (int)nbuild,
                     (double*)nullptr, 0);
}

void launch_md_invalidate(const Dev& d, int nrep, hipStream_t s) {
  hipLaunchKernelGGL(k_md_invalidate, dim3(1), dim3(256), 0, s, d.rb, nrep);
}

// ---------------------------------------------------------------------------
// Rigid bonds (Sec. 2, Eq. (SPValgo) with its SHAKE and RATTLE steps), one
// workgroup per chain (nb <= CON_WG).  Mode START opens the sub-cycle:
// ref = r, x = r + h/2 v (the gather's r_mid), SHAKE(x; ref), v += (x -
// x_drifted)/(h/2).  Mode STEP s follows the kick of sub-step s:
// RATTLE(v; x) at the sub-step's positions x, r = x + h/2 v, and unless it is
// the last sub-step the opening of the next: ref = r, x = r + h/2 v,
// SHAKE(x; ref), v += (x - x_drifted)/(h/2), x stored as the next r_mid.
// Both projections are tridiagonal systems in the bond multipliers: RATTLE's
// is solved once; SHAKE's linearised constraints by Newton iterations until
// the worst bond is within CON_TOL r0^2.  Each system is solved by parallel
// cyclic reduction in LDS (thread k owns bond k), or for chains of at most
// 32 beads by the Thomas algorithm on one lane; bead p adds the corrections
// of its bonds p (+) and p-1 (-) in that order.
// ---------------------------------------------------------------------------
constexpr int CON_WG = 1024;
constexpr double CON_TOL = 1e-13;
constexpr int CON_MAXIT = 50;

struct ConShared {
  double x[CON_WG][3];      // positions
  double e[CON_WG][3];      // bond vectors of the system's coefficients
  double w[CON_WG][3];      // velocities (RATTLE)
  double a[CON_WG], b[CON_WG], c[CON_WG], r[CON_WG];
  double red[CON_WG / 64];
};

// max over the workgroup (exact, any order)
__device__ inline double con_max(double x, ConShared& sh) {
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
  const int wv = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh.red[wv] = x;
  __syncthreads();
  double m = 0.0;
  for (int k = 0; k < CON_WG / 64; ++k) m = fmax(m, sh.red[k]);
  return m;
}

// Solves a[k] y[k-1] + b[k] y[k] + c[k] y[k+1] = r[k], k < n, in place
// (parallel cyclic reduction; rows beyond the ends read as identity rows);
// returns thread k's y[k].
__device__ inline double con_pcr(ConShared& sh, int n) {
  const int k = threadIdx.x;
  for (int h = 1; h < n; h <<= 1) {
    double ai = 0.0, bi = 1.0, ci = 0.0, ri = 0.0;
    double am = 0.0, bm = 1.0, cm = 0.0, rm = 0.0, ap = 0.0, bp = 1.0, cp = 0.0, rp = 0.0;
    if (k < n) {
      ai = sh.a[k]; bi = sh.b[k]; ci = sh.c[k]; ri = sh.r[k];
      if (k - h >= 0) { am = sh.a[k - h]; bm = sh.b[k - h]; cm = sh.c[k - h]; rm = sh.r[k - h]; }
      if (k + h < n) { ap = sh.a[k + h]; bp = sh.b[k + h]; cp = sh.c[k + h]; rp = sh.r[k + h]; }
    }
    __syncthreads();
    if (k < n) {
      const double k1 = ai / bm, k2 = ci / bp;
      sh.a[k] = -(am * k1);
      sh.b[k] = bi - cm * k1 - ap * k2;
      sh.c[k] = -(cp * k2);
      sh.r[k] = ri - rm * k1 - rp * k2;
    }
    __syncthreads();
  }
  return k < n ? sh.r[k] / sh.b[k] : 0.0;
}

// The same system by the Thomas algorithm on one lane (forward elimination,
// then back substitution), for short chains: n - 1 dependent rows cost less
// than the reduction's barriers, and the result rounds as the textbook
// solve does.  Returns thread k's y[k].
constexpr int CON_THOMAS_MAX = 31;
__device__ inline double con_thomas(ConShared& sh, int n) {
  const int k = threadIdx.x;
  if (k == 0 && n > 0) {
    sh.c[0] = sh.c[0] / sh.b[0];
    sh.r[0] = sh.r[0] / sh.b[0];
    for (int i = 1; i < n; ++i) {
      const double den = sh.b[i] - sh.a[i] * sh.c[i - 1];
      sh.c[i] = sh.c[i] / den;
      sh.r[i] = (sh.r[i] - sh.a[i] * sh.r[i - 1]) / den;
    }
    for (int i = n - 2; i >= 0; --i) sh.r[i] = sh.r[i] - sh.c[i] * sh.r[i + 1];
  }
  __syncthreads();
  return k < n ? sh.r[k] : 0.0;
}
__device__ inline double con_solve(ConShared& sh, int n) {
  return n <= CON_THOMAS_MAX ? con_thomas(sh, n) : con_pcr(sh, n);   // uniform in the workgroup
}

__device__ inline double dot3v(const double* u, const double* v) { return u[0] * v[0] + u[1] * v[1] + u[2] * v[2]; }

// SHAKE of the drifted positions sh.x along the bonds held in sh.e (the
// reference bonds): the correction is accumulated in sh.w (x = x_drifted +
// dx, x itself left as drifted), so that the velocity impulse dx / (h/2)
// keeps its relative precision
__device__ inline void con_shake(ConShared& sh, int nb, double d2, uint32_t* err) {
  const int k = threadIdx.x, nbond = nb - 1;
  for (int it = 0;; ++it) {
    double sv[3] = {0.0, 0.0, 0.0}, sig = 0.0;
    if (k < nbond) {
#pragma unroll
      for (int a = 0; a < 3; ++a) sv[a] = (sh.x[k][a] + sh.w[k][a]) - (sh.x[k + 1][a] + sh.w[k + 1][a]);
      sig = dot3v(sv, sv) - d2;
    }
    const double worst = con_max(fabs(sig), sh);
    if (worst <= CON_TOL * d2) return;
    if (it == CON_MAXIT) {
      if (k == 0) atomicOr(err, E_BEADS);
      return;
    }
    if (k < nbond) {
      sh.b[k] = 4.0 * dot3v(sv, sh.e[k]);
      sh.a[k] = k > 0 ? -2.0 * dot3v(sv, sh.e[k - 1]) : 0.0;
      sh.c[k] = k < nbond - 1 ? -2.0 * dot3v(sv, sh.e[k + 1]) : 0.0;
      sh.r[k] = -sig;
    }
    __syncthreads();
    const double lam = con_solve(sh, nbond);
    // every thread has read what it needs; multipliers to sh.r, then apply
    sh.r[k] = lam;
    __syncthreads();
    if (k < nb) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double y = sh.w[k][a];
        if (k < nbond) y = y + sh.r[k] * sh.e[k][a];
        if (k > 0) y = y - sh.r[k - 1] * sh.e[k - 1][a];
        sh.w[k][a] = y;                       // own entry only
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(CON_WG) void k_md_constraint(Dev d, int nslots, int mode, int s, int last) {
  __shared__ ConShared sh;
  const int rep = blockIdx.x;
  const Rep& R = d.reps[rep];
  const int nb = R.mp.nb;
  if (nb < 2 || !R.mp.constrained) return;   // uniform in the workgroup
  const int k = threadIdx.x;
  const int slot = R.slot_off + k;
  const double hh = R.mp.hh, d2 = R.mp.r0 * R.mp.r0;
  const double* rin = (s & 1) ? d.rmid1 : d.rmid0;   // this sub-step's positions (STEP)
  double* rout = (s & 1) ? d.rmid0 : d.rmid1;        // the next sub-step's
  double v[3] = {0.0, 0.0, 0.0}, r[3] = {0.0, 0.0, 0.0};
  const bool own = k < nb;
  if (own) {
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = d.v[3 * slot + a];
  }
  bool open_next = true;
  if (mode == 0) {
    // START: r is the step's start, the gather stored r_mid = r + h/2 v in rmid0
    if (own) {
#pragma unroll
      for (int a = 0; a < 3; ++a) r[a] = d.r[3 * slot + a];
    }
    rout = d.rmid0;
  } else {
    // RATTLE at the sub-step's positions
    if (own) {
#pragma unroll
      for (int a = 0; a < 3; ++a) { sh.x[k][a] = rin[3 * slot + a]; sh.w[k][a] = v[a]; }
    }
    __syncthreads();
    const int nbond = nb - 1;
    double rv[3] = {0.0, 0.0, 0.0};
    if (k < nbond) {
      double ww[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) { rv[a] = sh.x[k][a] - sh.x[k + 1][a]; ww[a] = sh.w[k][a] - sh.w[k + 1][a]; }
      sh.b[k] = 2.0 * dot3v(rv, rv);
      sh.r[k] = -dot3v(rv, ww);
#pragma unroll
      for (int a = 0; a < 3; ++a) sh.e[k][a] = rv[a];
    }
    __syncthreads();
    if (k < nbond) {
      sh.a[k] = k > 0 ? -dot3v(rv, sh.e[k - 1]) : 0.0;
      sh.c[k] = k < nbond - 1 ? -dot3v(rv, sh.e[k + 1]) : 0.0;
    }
    __syncthreads();
    const double mu = con_solve(sh, nbond);
    sh.r[k] = mu;
    __syncthreads();
    if (own) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (k < nbond) v[a] = v[a] + sh.r[k] * sh.e[k][a];
        if (k > 0) v[a] = v[a] - sh.r[k - 1] * sh.e[k - 1][a];
        r[a] = sh.x[k][a] + hh * v[a];
      }
    }
    open_next = !last;
    if (last && own) {
#pragma unroll
      for (int a = 0; a < 3; ++a) { d.r[3 * slot + a] = r[a]; d.v[3 * slot + a] = v[a]; }
    }
    __syncthreads();
  }
  if (!open_next) return;
  // the opening of the next sub-step: ref = r, x = r + h/2 v, SHAKE
  double xd[3] = {0.0, 0.0, 0.0};
  if (own) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      xd[a] = r[a] + hh * v[a];
      sh.x[k][a] = xd[a];
      sh.w[k][a] = r[a];
    }
  }
  __syncthreads();
  if (k < nb - 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) sh.e[k][a] = sh.w[k][a] - sh.w[k + 1][a];
  }
  __syncthreads();
  if (own) {
#pragma unroll
    for (int a = 0; a < 3; ++a) sh.w[k][a] = 0.0;    // the SHAKE correction
  }
  __syncthreads();
  con_shake(sh, nb, d2, &d.ctrl->err);
  if (!own) return;
  double d2r = 0.0, b2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double dx = sh.w[k][a];
    const double x = xd[a] + dx;
    v[a] = v[a] + dx / hh;
    rout[3 * slot + a] = x;
    d.v[3 * slot + a] = v[a];
    const double dd = x - d.ref[3 * slot + a];
    d2r += dd * dd;
    const double db = x - d.rbin[3 * slot + a];
    b2 += db * db;
  }
  const int w = mode == 0 ? 0 : (s + 1) % 3;
  if (d2r > R.mp.halfskin2) d.rb[4 * rep + w] = 1u;
  if (!(b2 <= CELL_MARGIN * CELL_MARGIN)) d.cst[4 * rep + w] = 1u;
}

void launch_md_begin(const Dev& d, int nrep, hipStream_t s) {
  hipLaunchKernelGGL(k_md_begin, dim3(1), dim3(256), 0, s, d, nrep);
}

void launch_md_start(const Dev& d, int nslots, const MdOverride& ov, hipStream_t s) {
  hipLaunchKernelGGL(k_md_start, dim3((nslots + 255) / 256), dim3(256), 0, s, d, nslots, ov, 0);
}

void launch_md_cycle(const Dev& d, int nslots, int nrep, int n_sub, const MdOverride& ov, hipStream_t s,
                     bool prologue, bool constrained) {
  if (nslots <= 0 || n_sub <= 0) return;
  unsigned nblk = (unsigned)(nslots / MD_BPB);
  if (prologue) {
    hipLaunchKernelGGL(k_md_begin, dim3(1), dim3(256), 0, s, d, nrep);
    hipLaunchKernelGGL(k_md_start, dim3((nslots + 255) / 256), dim3(256), 0, s, d, nslots, ov, 0);
  }
  if (constrained)
    hipLaunchKernelGGL(k_md_constraint, dim3((unsigned)nrep), dim3(CON_WG), 0, s, d, nslots, 0, 0, 0);
  for (int k = 0; k < n_sub; ++k) {
    hipLaunchKernelGGL(k_md_substep<false>, dim3(nblk), dim3(3 * MD_WG), 0, s, d, ov, nslots, k,
                       k == n_sub - 1 ? 1 : 0);
    if (constrained)
      hipLaunchKernelGGL(k_md_constraint, dim3((unsigned)nrep), dim3(CON_WG), 0, s, d, nslots, 1, k,
                         k == n_sub - 1 ? 1 : 0);
  }
}

void launch_md_cycle_mts(const Dev& d, int nslots, int n_sub, int M, hipStream_t s) {
  if (nslots <= 0 || n_sub <= 0 || M <= 0) return;
  const int Mb = n_sub / M;
  const unsigned nblk = (unsigned)(nslots / MD_BPB);
  const int own = IN_WG - 4 * Mb;
  const unsigned nin = (unsigned)((nslots + own - 1) / own);
  MdOverride none{};
  for (int o = 0; o < M; ++o) {
    hipLaunchKernelGGL(k_md_substep<true>, dim3(nblk), dim3(3 * MD_WG), 0, s, d, none, nslots, o, o == 0 ? 1 : 2);
    hipLaunchKernelGGL(k_md_inner, dim3(nin), dim3(IN_WG), 0, s, d, nslots, o, Mb);
  }
  hipLaunchKernelGGL(k_md_substep<true>, dim3(nblk), dim3(3 * MD_WG), 0, s, d, none, nslots, M, 1);
}

// ---------------------------------------------------------------------------
// Fused sub-steps: one launch advances a block of K uniform sub-steps.
//
// Workgroup w owns the chain segment [a, b) of replica rep.  Over one
// sub-step a bead's new state depends on its own state and on the positions
// of its chain neighbours p-2 .. p+2 (bonds, and the angles centred at p-1,
// p, p+1) and of its pair partners within r_c.  Give every bead its level:
// its distance from [a, b) in that dependency graph.  A bead of level k must
// be exact for the first K - k sub-steps of the block, which needs its
// dependencies (level <= k + 1) exact for one sub-step less, so the set S of
// beads of level <= K, each advanced from the positions in S, leaves [a, b)
// exact after K sub-steps even though the beads at S's rim go wrong (the halo
// argument of overlapped tiling).  S is a union of chain spans: [a, b)
// widened by 2K (level 0 inside, +1 per two chain links), and for every
// close partner j of a bead of level k < K that is not yet in S with level
// <= k + 1, a span around j of level k + 1, widened by 2 (K - k - 1).
//
// Pair partners are the entries of the neighbour lists (built at the start
// of the LB step, radius r_c + skin) within close = r_c + 2 FUSED_DELTA at
// the block's start.  Partners farther than that stay beyond r_c for the
// whole block as long as no bead moves more than FUSED_DELTA within it, so
// they contribute nothing; and a list holds every bead within close of its
// bead as long as every bead is within skin/2 - FUSED_DELTA of where the
// lists were built.  Both conditions are checked, each workgroup on the
// beads it owns: if every workgroup of the replica finds them true, no bead
// of the replica violated them and the block equals the per-sub-step
// computation bit for bit (the same operations in the same order: bonds, the
// three angles, pair partners in ascending order, wall sites in ascending
// order, field, then the kick; only pairs within r_c ever add a term, so the
// list a partner came from does not matter).  Otherwise the replica's redo
// marker is set to the block's first sub-step, later blocks of the replica
// return at once, and k_md_redo redoes the replica from there in one
// workgroup.  A block reads its start state from one set of arrays (the
// canonical r_mid0, v, J, or the shadow ones) and writes the other, so that
// the start state of a block that fails is still there.
// ---------------------------------------------------------------------------
constexpr int FU_LANES = 4;        // lanes per bead in the sub-steps
constexpr int FU_CAP = 128;        // beads of S
constexpr int FU_WG = FU_LANES * FU_CAP;
constexpr int FU_NS = 16;          // spans of S (before merging)
constexpr int FU_NC = 16;          // close partners per bead
constexpr int FU_ROUNDS = 6;       // closure rounds
constexpr int FU_LD = 16;          // list entries loaded together

struct FuSpan {
  int blo, bhi;                    // base interval (level lv inside)
  int lv;
};

struct FuShared {
  double pos[2][FU_CAP][3];        // positions at the sub-step's start / the next one
  double ang[FU_CAP][9];           // forces of the angle centred at the bead (first, centre, third)
  double bnd[FU_CAP][6];           // the bead's bond forces towards its predecessor and successor
  int lst[FU_CAP][FU_NC];          // close partners: chain indices, then local indices; ascending
  unsigned char lcnt[FU_CAP];
  unsigned char lev[FU_CAP];       // level of the bead (K + 1: not needed)
  unsigned char angok[FU_CAP];     // the angle centred at the bead is evaluated
  FuSpan span[FU_NS];
  int nspan;
  int ilo[FU_NS], ihi[FU_NS], ioff[FU_NS + 1];   // S as sorted disjoint chain intervals
  int niv;
  int nreq;
  FuSpan req[FU_NS];
  int ctl;                         // set-up state, written by thread 0 only, between barriers:
                                   // 0 go on, 1 closure complete, 2 cannot certify, 3 an earlier block failed
  int ovf;                         // a request or a partner list did not fit
  int far;                         // a bead of the segment moved too far from where the lists were built
};

// chain index of local index li, and local index of chain index q (-1 if
// not in S); S is the concatenation of the sorted disjoint intervals
__device__ inline int fu_chain(const FuShared& sh, int li) {
  for (int k = 0; k < sh.niv; ++k)
    if (li < sh.ioff[k + 1]) return sh.ilo[k] + (li - sh.ioff[k]);
  return -1;
}
__device__ inline int fu_local(const FuShared& sh, int q) {
  for (int k = 0; k < sh.niv; ++k)
    if (q >= sh.ilo[k] && q < sh.ihi[k]) return sh.ioff[k] + (q - sh.ilo[k]);
  return -1;
}
// level of chain bead q: the least over the spans of lv + ceil(distance to
// the span's base / 2), K + 1 when above K (then not in S)
__device__ inline int fu_level(const FuShared& sh, int q, int K) {
  int best = K + 1;
  for (int k = 0; k < sh.nspan; ++k) {
    const FuSpan& p = sh.span[k];
    const int dist = q < p.blo ? p.blo - q : (q >= p.bhi ? q - p.bhi + 1 : 0);
    const int l = p.lv + (dist + 1) / 2;
    best = l < best ? l : best;
  }
  return best;
}
// S from the spans (one thread): every bead of level <= K, as sorted
// disjoint chain intervals.  False when S exceeds its capacity.
__device__ inline bool fu_build(FuShared& sh, int K, int nb) {
  int lo[FU_NS], hi[FU_NS];
  const int n = sh.nspan;
  for (int k = 0; k < n; ++k) {
    const int w = 2 * (K - sh.span[k].lv);
    lo[k] = max(0, sh.span[k].blo - w);
    hi[k] = min(nb, sh.span[k].bhi + w);
  }
  for (int i = 1; i < n; ++i) {
    const int l = lo[i], h = hi[i];
    int m = i;
    while (m > 0 && lo[m - 1] > l) { lo[m] = lo[m - 1]; hi[m] = hi[m - 1]; --m; }
    lo[m] = l; hi[m] = h;
  }
  int k = 0;
  for (int i = 1; i < n; ++i) {
    if (lo[i] <= hi[k]) { hi[k] = max(hi[k], hi[i]); continue; }
    ++k;
    lo[k] = lo[i]; hi[k] = hi[i];
  }
  const int niv = k + 1;
  int tot = 0;
  for (int i = 0; i < niv; ++i) tot += hi[i] - lo[i];
  if (tot > FU_CAP) return false;
  sh.niv = niv;
  sh.ioff[0] = 0;
  for (int i = 0; i < niv; ++i) { sh.ilo[i] = lo[i]; sh.ihi[i] = hi[i]; sh.ioff[i + 1] = sh.ioff[i] + hi[i] - lo[i]; }
  return true;
}

// The beads of the replica within sqrt(r2max) of position x (any bead but
// chain index self), from the neighbour-search cell table, in ascending
// chain order: at most cap of them into out (returns their number, cap + 1
// if more).  Every bead within range is found while every bead of the
// replica lies within CELL_MARGIN of the position the table binned it at
// and sqrt(r2max) + CELL_MARGIN does not exceed the cell side.
__device__ inline int cell_partners(const Dev& d, const Rep& R, int rep, const double* pos, int self,
                                    const double* x, double r2max, int* out, int cap) {
  const Geom& g = R.g;
  const int so = R.slot_off;
  int c[3];
  bead_cell(R, x, c);
  int n = 0;
  for (int k = 0; k < 27; ++k) {
    const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
    const uint32_t b = cell_bucket(rep, (c[0] + dx + R.ncell[0]) % R.ncell[0], (c[1] + dy + R.ncell[1]) % R.ncell[1],
                                   (c[2] + dz + R.ncell[2]) % R.ncell[2], d.cmask);
    const int m = min(d.ccount[b], CELL_CAP);
    for (int e = 0; e < m; ++e) {
      const int sl = d.cbuf[(size_t)b * CELL_CAP + e];
      if (d.slot_rep[sl] != rep) continue;
      const int j = sl - so;
      if (j == self) continue;
      const double e0 = min_image(x[0] - pos[3 * sl], g.nx);
      const double e1 = min_image(x[1] - pos[3 * sl + 1], g.ny);
      const double e2 = min_image(x[2] - pos[3 * sl + 2], g.nz);
      if (!(e0 * e0 + e1 * e1 + e2 * e2 < r2max)) continue;
      // a bucket reached from two of the 27 cells (few cells per axis, or
      // hash collisions) gives its beads twice: keep each once
      int i = n;
      while (i > 0 && out[i - 1] > j) --i;
      if (i > 0 && out[i - 1] == j) continue;
      if (n == cap) return cap + 1;
      for (int m2 = n; m2 > i; --m2) out[m2] = out[m2 - 1];
      out[i] = j;
      ++n;
    }
  }
  return n;
}

// The wall sites' forces on a bead at rp, added to F in ascending site order
// (rows o1, then o0): the sites and operations of wall_row, summed as the
// sub-step kernel sums them.
__device__ inline void fu_wall(const MdParams& P, const Geom& g, const double* rp, double F[3]) {
  if (g.wall_axis < 0) return;
  const double w0 = wrapc(rp[0], g.nx), w1 = wrapc(rp[1], g.ny), w2 = wrapc(rp[2], g.nz);
  const int b0 = (int)floor(w0), b1 = (int)floor(w1), b2 = (int)floor(w2);
  const int a = g.wall_axis;
  const int ba = a == 0 ? b0 : (a == 1 ? b1 : b2);
  const int na = a == 0 ? g.nx : (a == 1 ? g.ny : g.nz);
  const int bt0 = a == 0 ? b1 : b0, n0 = a == 0 ? g.ny : g.nx;
  const int bt1 = a == 2 ? b1 : b2, n1 = a == 2 ? g.ny : g.nz;
  int off = g.wall_pos - ba;
  if (off < WLO) off += na;
  if (off > WHI) off -= na;
  if (off < P.wlo || off > P.whi) return;
  const int sa = ba + off;
  for (int o1 = P.wlo; o1 <= P.whi; ++o1) {
    const int u1 = bt1 + o1;
    const int v1 = u1 < 0 ? u1 + n1 : (u1 >= n1 ? u1 - n1 : u1);
    const bool in1 = v1 >= g.lo1 && v1 <= g.hi1;
    for (int o0 = P.wlo; o0 <= P.whi; ++o0) {
      const int u0 = bt0 + o0;
      const int v0 = u0 < 0 ? u0 + n0 : (u0 >= n0 ? u0 - n0 : u0);
      const bool in0 = v0 >= g.lo0 && v0 <= g.hi0;
      if (in0 && in1) continue;
      const int sx = a == 0 ? sa : u0;
      const int sy = a == 1 ? sa : (a == 0 ? u0 : u1);
      const int sz = a == 2 ? sa : u1;
      const double d0 = w0 - (double)sx, d1 = w1 - (double)sy, d2 = w2 - (double)sz;
      if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rc2)) continue;
      double Fs[3] = {0.0, 0.0, 0.0};
      lj_add(P, d0, d1, d2, Fs);
      F[0] += Fs[0]; F[1] += Fs[1]; F[2] += Fs[2];
    }
  }
}

// The force on chain bead q at rp in the order of the sub-step kernel: bonds
// to q-1 (at rm) and q+1 (at rq), the angles centred at q-1 (third-bead
// part a3), q (centre part ac) and q+1 (first-bead part a1) -- each NULL when
// not added --, the pair partners at base + 3 idx[0..np-1] in ascending
// chain order (terms within r_c only), the wall sites, the field.
__device__ inline void fu_force(const MdParams& P, const Geom& g, int q, const double* rp, const double* rm,
                                const double* rq, const double* a3, const double* ac, const double* a1,
                                const double* base, const int* idx, int np, double F[3], bool slow = true) {
  F[0] = 0.0; F[1] = 0.0; F[2] = 0.0;
  if (!P.constrained) {
    if (q > 0 && rm) bond_add(P, rp, rm, F);
    if (q < P.nb - 1 && rq) bond_add(P, rp, rq, F);
  }
  if (a3) { F[0] += a3[6]; F[1] += a3[7]; F[2] += a3[8]; }
  if (ac) { F[0] += ac[3]; F[1] += ac[4]; F[2] += ac[5]; }
  if (a1) { F[0] += a1[0]; F[1] += a1[1]; F[2] += a1[2]; }
  for (int k = 0; k < np; ++k) {
    const double* qp = base + 3 * (size_t)idx[k];
    const double e0 = min_image(rp[0] - qp[0], g.nx);
    const double e1 = min_image(rp[1] - qp[1], g.ny);
    const double e2 = min_image(rp[2] - qp[2], g.nz);
    if (!(e0 * e0 + e1 * e1 + e2 * e2 < P.rc2)) continue;
    double Fp[3] = {0.0, 0.0, 0.0};
    lj_add(P, e0, e1, e2, Fp);
    F[0] += Fp[0]; F[1] += Fp[1]; F[2] += Fp[2];
  }
  if (!slow) return;
  fu_wall(P, g, rp, F);
  if (P.field_on && in_field(g, rp)) F[g.wall_axis] += P.f_drive;
}

// All nine force components of the angle at (ra, rb, rc) into o (first,
// centre, third bead, each x, y, z), 0 for a straight or folded angle.
__device__ inline void fu_angle(const MdParams& P, const double* ra, const double* rb, const double* rc, double* o) {
  AngleCore A;
  if (angle_core(P, ra, rb, rc, A)) {
    for (int a = 0; a < 3; ++a) {
      double f[3];
      angle_part(A, a, f);
      o[a] = f[0]; o[3 + a] = f[1]; o[6 + a] = f[2];
    }
  } else {
    for (int k = 0; k < 9; ++k) o[k] = 0.0;
  }
}

// The SPV kick and drifts of one sub-step (as the sub-step kernel): v, J
// updated; returns r_mid of the next sub-step in x (or, when last, the end
// position).
__device__ inline bool fu_kick(const MdParams& P, const double F[3], const double* u, const double* xi, double* v,
                               double* J, const double* rp, bool last, double x[3]) {
  bool fin = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double uu = P.couple ? u[a] : 0.0;
    const double xx = P.sig != 0.0 ? xi[a] : 0.0;
    const double sx = P.sig * xx;
    const double vn = P.e * v[a] + P.cf * (F[a] + P.gamma * uu) + sx;
    J[a] = J[a] - P.m * (P.omE * (uu - v[a]) + sx);
    v[a] = vn;
    fin = fin && isfinite(vn);
    const double re = rp[a] + P.hh * vn;
    x[a] = last ? re : re + P.hh * vn;
  }
  return fin;
}

__device__ inline void fu_fail(const Dev& d, const FusedBufs& fb, int rep, int s0) {
  if (atomicCAS(&fb.redo[rep], -1, s0) == -1) atomicAdd((unsigned long long*)&d.ctrl->fused_redos, 1ull);
}

// Block j = s0 / K of the sub-cycle.  iset: the set holding the block's start
// state (0: r_mid0, v, J; 1: the shadow arrays); the other receives the end
// state (the last block writes the final positions to r).
__global__ __launch_bounds__(FU_WG) void k_md_fused(Dev d, FusedBufs fb, int nslots, int s0, int K, int last,
                                                    int iset) {
  __shared__ FuShared sh;
  const FusedSeg seg = fb.seg[blockIdx.x];
  const int rep = seg.rep;
  const Rep& R = d.reps[rep];
  const MdParams P = R.mp;
  const Geom g = R.g;
  const int so = R.slot_off, nb = P.nb;
  const int t = threadIdx.x;
  const double* rin = iset ? fb.rmS : d.rmid0;
  const double* vin = iset ? fb.vS : d.v;
  const double* Jin = iset ? fb.JS : d.J;
  double* rout = iset ? d.rmid0 : fb.rmS;
  double* vout = iset ? d.v : fb.vS;
  double* Jout = iset ? d.J : fb.JS;
  const double close = sqrt(P.rc2) + 2.0 * FUSED_DELTA + 1e-9;
  const double close2 = close * close;
  if (t == 0) {
    // an earlier block of the replica failed (another workgroup may set the
    // marker during this launch: thread 0 reads it once for the workgroup)
    sh.ctl = fb.redo[rep] >= 0 ? 3 : (d.rb[4 * rep] != 0u ? 2 : 0);   // lists not valid at the cycle's start
    if (sh.ctl == 2) atomicAdd(&d.ctrl->fused_why[0], 1u);
    sh.ovf = 0;
    sh.far = 0;
    sh.nspan = 1;
    sh.span[0] = FuSpan{seg.a, seg.b, 0};
    sh.nreq = 0;
    if (!fu_build(sh, K, nb)) sh.ctl = 2;
  }
  __syncthreads();
  if (sh.ctl == 3) return;                        // uniform
  // the lists must hold every close partner: each workgroup checks its own beads
  const double keep = sqrt(P.halfskin2) - FUSED_DELTA;
  bool held = keep > 0.0;
  for (int q = seg.a + t; q < seg.b; q += FU_WG) {
    const int sl = so + q;
    double b2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) { const double db = rin[3 * sl + a] - d.ref[3 * sl + a]; b2 += db * db; }
    held = held && b2 <= keep * keep;
  }
  if (!held) sh.far = 1;
  // ---- closure.  Every thread reads sh.ctl right after a barrier; thread
  // 0 writes it only between the two barriers of a round.
  for (int round = 0;; ++round) {
    __syncthreads();
    if (sh.ctl != 0) break;
    const int n = sh.ioff[sh.niv];
    if (t < n) {
      const int q = fu_chain(sh, t);
      const int lv = fu_level(sh, q, K);
      sh.lev[t] = (unsigned char)lv;
      sh.lcnt[t] = 0;
      if (lv < K) {
        // the list and the positions of its first entries, loads issued
        // together; entries beyond FU_LD in a slower loop
        const int sl = so + q;
        const double x[3] = {rin[3 * sl], rin[3 * sl + 1], rin[3 * sl + 2]};
        const int cnt = d.ncnt[sl];
        const int* row = d.nbr + (size_t)sl * MAXNBR;
        int e[FU_LD];
#pragma unroll
        for (int k = 0; k < FU_LD; ++k) e[k] = row[k];
        double pj[FU_LD][3];
#pragma unroll
        for (int k = 0; k < FU_LD; ++k) {
          const int js = k < cnt ? e[k] : sl;    // list entries are slots
          pj[k][0] = rin[3 * js]; pj[k][1] = rin[3 * js + 1]; pj[k][2] = rin[3 * js + 2];
        }
        int c = 0;
        bool full = false;
        // one entry: keep it if close; request a span if it needs a lower level
        auto take = [&](int j, const double* y) {
          const double e0 = min_image(x[0] - y[0], g.nx);
          const double e1 = min_image(x[1] - y[1], g.ny);
          const double e2 = min_image(x[2] - y[2], g.nz);
          if (!(e0 * e0 + e1 * e1 + e2 * e2 < close2)) return;
          if (c == FU_NC) { full = true; return; }
          sh.lst[t][c++] = j;
          if (fu_level(sh, j, K) <= lv + 1) return;
          const int at = atomicAdd(&sh.nreq, 1);
          if (at < FU_NS) sh.req[at] = FuSpan{j, j + 1, lv + 1};
          else sh.ovf = 1;
        };
#pragma unroll
        for (int k = 0; k < FU_LD; ++k)
          if (k < cnt) take(e[k] - so, pj[k]);
        for (int k = FU_LD; k < cnt; ++k) {
          const int js = row[k];
          const double y[3] = {rin[3 * js], rin[3 * js + 1], rin[3 * js + 2]};
          take(js - so, y);
        }
        if (full) sh.ovf = 1;
        sh.lcnt[t] = (unsigned char)c;
      }
    }
    __syncthreads();
    if (t == 0) {
      int c = 0, why = -1;
      if (sh.far) { c = 2; why = 0; }
      else if (sh.ovf) { c = 2; why = 1; }
      else if (sh.nreq == 0) c = 1;
      else if (sh.nspan + sh.nreq > FU_NS) { c = 2; why = 2; }
      else {
        for (int k = 0; k < sh.nreq; ++k) sh.span[sh.nspan + k] = sh.req[k];
        sh.nspan += sh.nreq;
        if (!fu_build(sh, K, nb)) { c = 2; why = 2; }
        else if (round + 1 == FU_ROUNDS) { c = 2; why = 3; }   // the closure did not settle
      }
      if (why >= 0) atomicAdd(&d.ctrl->fused_why[why], 1u);
      sh.ctl = c;
      sh.nreq = 0;
    }
  }
  if (sh.ctl != 1) {                              // uniform: read after the barrier
    if (t == 0) fu_fail(d, fb, rep, s0);
    return;
  }
  const int n = sh.ioff[sh.niv];
  // ---- sub-steps: FU_LANES lanes per bead b of S.  Lanes 0-2 evaluate
  // component l of the angle centred at the bead, lane 3 its two bond forces;
  // lane 0 (the lead) then adds every contribution in the order of the
  // sub-step kernel, kicks and drifts the bead.
  const int b = t / FU_LANES, l = t % FU_LANES;
  const bool act = b < n;
  const bool lead = act && l == 0;
  const int q = act ? fu_chain(sh, b) : 0;
  const int slot = so + q;
  const bool own = lead && q >= seg.a && q < seg.b;
  const int lm1 = act && q > 0 ? fu_local(sh, q - 1) : -1;
  const int lp1 = act && q < nb - 1 ? fu_local(sh, q + 1) : -1;
  const bool angle_here = act && q >= 1 && q <= nb - 2 && lm1 >= 0 && lp1 >= 0;
  double rp[3] = {0.0, 0.0, 0.0}, rm0[3] = {0.0, 0.0, 0.0}, vo[3] = {0.0, 0.0, 0.0}, Jo[3] = {0.0, 0.0, 0.0};
  double ul[3] = {0.0, 0.0, 0.0};
  int lc = 0;
  if (lead) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      rp[a] = rin[3 * slot + a];
      rm0[a] = rp[a];
      vo[a] = vin[3 * slot + a];
      Jo[a] = Jin[3 * slot + a];
      ul[a] = P.couple ? d.up[3 * slot + a] : 0.0;
      sh.pos[0][b][a] = rp[a];
    }
    sh.angok[b] = angle_here ? 1 : 0;
    // partners to local indices (a bead of level < K has every close
    // partner in S by the closure; one that did not would be left out rather
    // than read outside S; a bead of level K needs none)
    const int c0 = sh.lev[b] < K ? sh.lcnt[b] : 0;
    for (int k = 0; k < c0; ++k) {
      const int lj = fu_local(sh, sh.lst[b][k]);
      if (lj >= 0) sh.lst[b][lc++] = lj;
    }
  }
  bool viol = false, fin = true;
  double rfin[3] = {0.0, 0.0, 0.0};
  double xn[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) xn[a] = lead && P.sig != 0.0 ? d.xi[(size_t)3 * ((size_t)s0 * nslots + slot) + a] : 0.0;
  __syncthreads();
  for (int s = s0; s < s0 + K; ++s) {
    const int cb = (s - s0) & 1;
    double xl[3] = {xn[0], xn[1], xn[2]};
    if (lead && P.sig != 0.0 && s + 1 < s0 + K) {
#pragma unroll
      for (int a = 0; a < 3; ++a) xn[a] = d.xi[(size_t)3 * ((size_t)(s + 1) * nslots + slot) + a];
    }
    // ---- phase 1: angle components, bonds
    if (act) {
      if (l < 3) {
        if (angle_here) {
          double f[3];
          angle_component(P, sh.pos[cb][lm1], sh.pos[cb][b], sh.pos[cb][lp1], l, f);
          sh.ang[b][l] = f[0]; sh.ang[b][3 + l] = f[1]; sh.ang[b][6 + l] = f[2];
        }
      } else {
        double F1[3] = {0.0, 0.0, 0.0}, F2[3] = {0.0, 0.0, 0.0};
        if (!P.constrained) {
          if (q > 0 && lm1 >= 0) bond_add(P, sh.pos[cb][b], sh.pos[cb][lm1], F1);
          if (q < nb - 1 && lp1 >= 0) bond_add(P, sh.pos[cb][b], sh.pos[cb][lp1], F2);
        }
        for (int a = 0; a < 3; ++a) { sh.bnd[b][a] = F1[a]; sh.bnd[b][3 + a] = F2[a]; }
      }
    }
    __syncthreads();
    // ---- phase 2: the lead adds, kicks and drifts
    if (lead) {
      double F[3] = {0.0, 0.0, 0.0};
      if (!P.constrained) {
        if (q > 0 && lm1 >= 0) { F[0] += sh.bnd[b][0]; F[1] += sh.bnd[b][1]; F[2] += sh.bnd[b][2]; }
        if (q < nb - 1 && lp1 >= 0) { F[0] += sh.bnd[b][3]; F[1] += sh.bnd[b][4]; F[2] += sh.bnd[b][5]; }
      }
      if (q - 1 >= 1 && q - 1 <= nb - 2 && lm1 >= 0 && sh.angok[lm1]) {
        const double* A = sh.ang[lm1]; F[0] += A[6]; F[1] += A[7]; F[2] += A[8];
      }
      if (angle_here) { const double* A = sh.ang[b]; F[0] += A[3]; F[1] += A[4]; F[2] += A[5]; }
      if (q + 1 >= 1 && q + 1 <= nb - 2 && lp1 >= 0 && sh.angok[lp1]) {
        const double* A = sh.ang[lp1]; F[0] += A[0]; F[1] += A[1]; F[2] += A[2];
      }
      for (int k = 0; k < lc; ++k) {
        const double* qp = sh.pos[cb][sh.lst[b][k]];
        const double e0 = min_image(rp[0] - qp[0], g.nx);
        const double e1 = min_image(rp[1] - qp[1], g.ny);
        const double e2 = min_image(rp[2] - qp[2], g.nz);
        if (!(e0 * e0 + e1 * e1 + e2 * e2 < P.rc2)) continue;
        double Fp[3] = {0.0, 0.0, 0.0};
        lj_add(P, e0, e1, e2, Fp);
        F[0] += Fp[0]; F[1] += Fp[1]; F[2] += Fp[2];
      }
      fu_wall(P, g, rp, F);
      if (P.field_on && in_field(g, rp)) F[g.wall_axis] += P.f_drive;
      const bool fl = last && s == s0 + K - 1;
      double x[3];
      fin = fu_kick(P, F, ul, xl, vo, Jo, rp, fl, x) && fin;
      if (fl) {
#pragma unroll
        for (int a = 0; a < 3; ++a) rfin[a] = x[a];
      } else {
        double dd2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          rp[a] = x[a];
          sh.pos[cb ^ 1][b][a] = x[a];
          const double dm = x[a] - rm0[a];
          dd2 += dm * dm;
        }
        // the positions of the block's next sub-steps stay within the bound
        if (own && s + 1 < s0 + K && !(dd2 <= FUSED_DELTA * FUSED_DELTA)) viol = true;
      }
    }
    __syncthreads();
  }
  if (own && !fin) atomicOr(&d.ctrl->err, E_BEADS);
  if (__syncthreads_or(viol ? 1 : 0)) {
    if (t == 0) {
      atomicAdd(&d.ctrl->fused_why[4], 1u);
      fu_fail(d, fb, rep, s0);
    }
    return;
  }
  if (blockIdx.x == 0 && t == 0) atomicAdd((unsigned long long*)&d.ctrl->fused_blocks, 1ull);
  if (!own) return;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    vout[3 * slot + a] = vo[a];
    Jout[3 * slot + a] = Jo[a];
    if (last) d.r[3 * slot + a] = rfin[a];
    else rout[3 * slot + a] = rp[a];
  }
}

// After the fused blocks, one workgroup per replica (and one workgroup of a
// replica whose resident cycle waited too long).  A replica whose block
// failed at sub-step sp is redone from that block's start state to the end of
// the cycle, sub-step by sub-step, with barriers: the angles of every centre,
// then every bead's force, kick and drifts; the positions alternate between
// r_mid0 and r_mid1.  A bead's pair partners come from the neighbour lists;
// when a bead is farther than half the skin from where they were built, every
// list is built anew at the sub-step's positions -- from the cell table while
// every bead lies within CELL_MARGIN of where it was binned, else from all
// beads of the chain.  A replica whose last block wrote the shadow set gets v
// and J copied back.
constexpr int RD_WG = 1024;

// A workgroup barrier that orders LDS only: __syncthreads would also wait for
// every outstanding global access (the published positions on their way to
// memory, the next sub-step's noise), none of which another wave of the
// workgroup reads.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// ---------------------------------------------------------------------------
// Rigid bonds inside the resident cycle (and its redo): the projections of
// k_md_constraint, operation by operation, for a chain of at most RIG_MAX beads
// held in LDS; thread k of RES_WG has bead k and bond k.  A workgroup publishes
// its beads' kicked velocities instead of positions, takes those of the whole
// chain, and projects the whole chain itself: every segment does the same
// arithmetic, and one exchange per sub-step suffices.  A level of the cyclic
// reduction has one barrier (rows alternate between two buffers, a thread's own
// row stays in registers).  150 beads: 12.4 us per sub-step, 9 of them the
// projection (about five tridiagonal solves of 8 levels, 0.22 us each); as
// launches the force kernel took 5.7 and the projection 14.6 us.
// ---------------------------------------------------------------------------
constexpr int RIG_WG = 512;
static_assert(RIG_MAX <= RIG_WG, "a thread per bead");
struct RigShared {
  double x[RIG_MAX][3];        // positions of the sub-step
  double v[RIG_MAX][3];
  double e[RIG_MAX][3];        // bond vectors of the system's coefficients
  double w[RIG_MAX][3];
  double row[2][4][RIG_MAX];   // a, b, c, r of the tridiagonal rows
  double lam[RIG_MAX];
  double ref[RIG_MAX][3];      // where the lists were built (wide pass)
  double red[2][RIG_WG / 64];
};

// max over the workgroup (exact, any order); z alternates between calls
__device__ inline double rig_max(double x, RigShared& q, int z) {
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
  if ((threadIdx.x & 63) == 0) q.red[z][threadIdx.x >> 6] = x;
  lds_barrier();
  double m = 0.0;
  for (int k = 0; k < RIG_WG / 64; ++k) m = fmax(m, q.red[z][k]);
  return m;
}

// con_solve of the rows (a, b, c, r) of threads k < n; y[k] to q.lam[k], 0 beyond.
__device__ inline void rig_solve(RigShared& q, int n, double ai, double bi, double ci, double ri) {
  const int k = threadIdx.x;
  double (*row)[4][RIG_MAX] = q.row;
  if (k < n) { row[0][0][k] = ai; row[0][1][k] = bi; row[0][2][k] = ci; row[0][3][k] = ri; }
  lds_barrier();
  if (n <= CON_THOMAS_MAX) {
    if (k == 0 && n > 0) {
      double *a = row[0][0], *b = row[0][1], *c = row[0][2], *r = row[0][3];
      c[0] = c[0] / b[0];
      r[0] = r[0] / b[0];
      for (int i = 1; i < n; ++i) {
        const double den = b[i] - a[i] * c[i - 1];
        c[i] = c[i] / den;
        r[i] = (r[i] - a[i] * r[i - 1]) / den;
      }
      q.lam[n - 1] = r[n - 1];
      for (int i = n - 2; i >= 0; --i) q.lam[i] = r[i] = r[i] - c[i] * r[i + 1];
    }
    if (k >= n && k < RIG_MAX) q.lam[k] = 0.0;
    lds_barrier();
    return;
  }
  int z = 0;
  const bool busy = (k & ~63) < n;               // the wave has rows
  for (int h = 1; h < n; h <<= 1, z ^= 1) {
    if (busy) {
      const int km = max(k - h, 0), kp = min(k + h, n - 1);
      double am = row[z][0][km], bm = row[z][1][km], cm = row[z][2][km], rm = row[z][3][km];
      double ap = row[z][0][kp], bp = row[z][1][kp], cp = row[z][2][kp], rp = row[z][3][kp];
      if (k - h < 0) { am = 0.0; bm = 1.0; cm = 0.0; rm = 0.0; }
      if (k + h >= n) { ap = 0.0; bp = 1.0; cp = 0.0; rp = 0.0; }
      const double k1 = ai / bm, k2 = ci / bp;
      ai = -(am * k1);
      bi = bi - cm * k1 - ap * k2;
      ci = -(cp * k2);
      ri = ri - rm * k1 - rp * k2;
      if (k < n) { row[z ^ 1][0][k] = ai; row[z ^ 1][1][k] = bi; row[z ^ 1][2][k] = ci; row[z ^ 1][3][k] = ri; }
    }
    lds_barrier();
  }
  if (k < RIG_MAX) q.lam[k] = k < n ? ri / bi : 0.0;
  lds_barrier();
}

// The opening of a sub-step (START of k_md_constraint): r, v of thread k's bead
// to the positions x and velocities of the next sub-step, in q.x and q.v.
// False: the bonds could not be met (E_BEADS, if the result is kept).
__device__ inline bool rig_open(RigShared& q, int nb, double hh, double d2, const double* r, double* v) {
  const int k = threadIdx.x, nbond = nb - 1;
  const bool own = k < nb;
  double xd[3] = {0.0, 0.0, 0.0}, e[3] = {0.0, 0.0, 0.0};
  if (own)
    for (int a = 0; a < 3; ++a) {
      xd[a] = r[a] + hh * v[a];
      q.x[k][a] = xd[a];
      q.v[k][a] = r[a];
      q.w[k][a] = 0.0;                           // the SHAKE correction
    }
  lds_barrier();
  if (k < nbond)
    for (int a = 0; a < 3; ++a) e[a] = q.e[k][a] = q.v[k][a] - q.v[k + 1][a];
  lds_barrier();
  bool met = true;
  for (int it = 0;; ++it) {
    double sv[3] = {0.0, 0.0, 0.0}, sig = 0.0;
    if (k < nbond) {
      for (int a = 0; a < 3; ++a) sv[a] = (q.x[k][a] + q.w[k][a]) - (q.x[k + 1][a] + q.w[k + 1][a]);
      sig = dot3v(sv, sv) - d2;
    }
    const double worst = rig_max(fabs(sig), q, it & 1);
    if (worst <= CON_TOL * d2) break;
    if (it == CON_MAXIT) { met = false; break; }
    double a_ = 0.0, b_ = 1.0, c_ = 0.0;
    if (k < nbond) {
      b_ = 4.0 * dot3v(sv, e);
      a_ = k > 0 ? -2.0 * dot3v(sv, q.e[k - 1]) : 0.0;
      c_ = k < nbond - 1 ? -2.0 * dot3v(sv, q.e[k + 1]) : 0.0;
    }
    rig_solve(q, nbond, a_, b_, c_, -sig);
    if (own)
      for (int a = 0; a < 3; ++a) {
        double y = q.w[k][a];
        if (k < nbond) y = y + q.lam[k] * e[a];
        if (k > 0) y = y - q.lam[k - 1] * q.e[k - 1][a];
        q.w[k][a] = y;
      }
    lds_barrier();
  }
  if (own)
    for (int a = 0; a < 3; ++a) {
      const double dx = q.w[k][a];
      q.x[k][a] = xd[a] + dx;
      q.v[k][a] = v[a] + dx / hh;
    }
  lds_barrier();
  return met;
}

// After the kick (q.x the sub-step's positions, q.v the kicked velocities of
// every bead): RATTLE, the second half drift, and unless last the opening of
// the next sub-step; last: q.x, q.v are the step's end.
__device__ inline bool rig_step(RigShared& q, int nb, double hh, double d2, bool last) {
  const int k = threadIdx.x, nbond = nb - 1;
  double v[3] = {0.0, 0.0, 0.0}, r[3] = {0.0, 0.0, 0.0}, rv[3] = {0.0, 0.0, 0.0};
  double a_ = 0.0, b_ = 1.0, c_ = 0.0, r_ = 0.0;
  if (k < nb)
    for (int a = 0; a < 3; ++a) { v[a] = q.v[k][a]; r[a] = q.x[k][a]; }
  if (k < nbond) {
    double ww[3];
    for (int a = 0; a < 3; ++a) { rv[a] = r[a] - q.x[k + 1][a]; ww[a] = v[a] - q.v[k + 1][a]; }
    b_ = 2.0 * dot3v(rv, rv);
    r_ = -dot3v(rv, ww);
    for (int a = 0; a < 3; ++a) q.e[k][a] = rv[a];
  }
  lds_barrier();
  if (k < nbond) {
    a_ = k > 0 ? -dot3v(rv, q.e[k - 1]) : 0.0;
    c_ = k < nbond - 1 ? -dot3v(rv, q.e[k + 1]) : 0.0;
  }
  rig_solve(q, nbond, a_, b_, c_, r_);
  if (k < nb)
    for (int a = 0; a < 3; ++a) {
      if (k < nbond) v[a] = v[a] + q.lam[k] * rv[a];
      if (k > 0) v[a] = v[a] - q.lam[k - 1] * q.e[k - 1][a];
      r[a] = r[a] + hh * v[a];
    }
  if (last) {
    if (k < nb)
      for (int a = 0; a < 3; ++a) { q.x[k][a] = r[a]; q.v[k][a] = v[a]; }
    lds_barrier();
    return true;
  }
  return rig_open(q, nb, hh, d2, r, v);
}

// Sub-steps sp .. n_sub - 1 of replica rep by one workgroup of WG threads, from
// r_mid of sub-step sp in r_mid0, and v, J.  MTS: the n_sub + mts + 1 stages of
// the multiple-time-step cycle (sp = 0; see the resident cycle).
// RIGID: rigid bonds, in *rig (sp = 0; from r and v).
template <int WG, bool MTS, bool RIGID>
__device__ inline void md_redo(const Dev& d, const Rep& R, const MdParams& P, int rep, double* ang, int nslots,
                               int sp, int n_sub, int mts, RigShared* rig, int& any_far, int& any_off) {
  const Geom g = R.g;
  const int so = R.slot_off, nb = P.nb;
  const int t = threadIdx.x;
  bool fin = true, over = false, valid = d.rb[4 * rep] == 0u;   // the lists, at the cycle's start
  const int Mb = MTS ? n_sub / mts : 0, end = MTS ? n_sub + mts + 1 : n_sub;
  if (RIGID) {
    double r[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    if (t < nb)
      for (int a = 0; a < 3; ++a) { r[a] = d.r[3 * (so + t) + a]; v[a] = d.v[3 * (so + t) + a]; }
    fin = rig_open(*rig, nb, P.hh, P.r0 * P.r0, r, v);
    if (t < nb)
      for (int a = 0; a < 3; ++a) { d.rmid0[3 * (so + t) + a] = rig->x[t][a]; d.v[3 * (so + t) + a] = rig->v[t][a]; }
    __syncthreads();
  }
  for (int s = sp; s < end; ++s) {
    const bool kick = MTS && s % (Mb + 1) == 0;
    const int sub = MTS ? s - s / (Mb + 1) - 1 : s;       // index of the sub-step (no kick)
    const double* cur = ((s - sp) & 1) ? d.rmid1 : d.rmid0;
    double* nxt = ((s - sp) & 1) ? d.rmid0 : d.rmid1;
    // every bead near the position the lists were built at, the position
    // the table binned it at?
    bool near = true, held = valid;
    for (int q = t; q < nb; q += WG) {
      double b2 = 0.0, f2 = 0.0;
      for (int a = 0; a < 3; ++a) {
        const double x = cur[3 * (so + q) + a];
        const double db = x - d.rbin[3 * (so + q) + a], df = x - d.ref[3 * (so + q) + a];
        b2 += db * db;
        f2 += df * df;
      }
      near = near && b2 <= CELL_MARGIN * CELL_MARGIN;
      held = held && f2 <= P.halfskin2;
    }
    if (t == 0) { any_far = 0; any_off = 0; }
    __syncthreads();                              // also orders the previous sub-step's writes
    if (!near) any_far = 1;
    if (!held) any_off = 1;
    for (int q = t; q < nb; q += WG)
      if (!kick && q >= 1 && q <= nb - 2)
        fu_angle(P, &cur[3 * (so + q - 1)], &cur[3 * (so + q)], &cur[3 * (so + q + 1)], &ang[9 * (size_t)(so + q)]);
    __syncthreads();
    const bool lists = (MTS && !kick) || any_off == 0, table = any_far == 0;
    if (!lists) {
      // each thread builds the lists of its own beads, which it alone reads
      for (int q = t; q < nb; q += WG) {
        const int sl = so + q;
        const double rp[3] = {cur[3 * sl], cur[3 * sl + 1], cur[3 * sl + 2]};
        int L[MAXNBR];
        int n = 0;
        if (table) {
          n = cell_partners(d, R, rep, cur, q, rp, P.rlist2, L, MAXNBR);
        } else {
          for (int j = 0; j < nb && n <= MAXNBR; ++j) {
            if (j == q) continue;
            const double e0 = min_image(rp[0] - cur[3 * (so + j)], g.nx);
            const double e1 = min_image(rp[1] - cur[3 * (so + j) + 1], g.ny);
            const double e2 = min_image(rp[2] - cur[3 * (so + j) + 2], g.nz);
            if (!(e0 * e0 + e1 * e1 + e2 * e2 < P.rlist2)) continue;
            if (n < MAXNBR) L[n] = j;
            ++n;
          }
        }
        if (n > MAXNBR) { over = true; n = MAXNBR; }
        for (int k = 0; k < n; ++k) d.nbr[(size_t)sl * MAXNBR + k] = so + L[k];
        d.ncnt[sl] = n;
        for (int a = 0; a < 3; ++a) d.ref[3 * sl + a] = rp[a];
      }
      if (t == 0) {
        atomicAdd((unsigned long long*)&d.ctrl->rebuilds, 1ull);
        if (table) atomicAdd((unsigned long long*)&d.ctrl->cell_rebuilds, 1ull);
      }
      valid = true;
    }
    for (int q = t; q < nb; q += WG) {
      const int sl = so + q;
      const double rp[3] = {cur[3 * sl], cur[3 * sl + 1], cur[3 * sl + 2]};
      const int cnt = !MTS || kick ? d.ncnt[sl] : 0;
      const double* a3 = (q - 1 >= 1 && q - 1 <= nb - 2) ? &ang[9 * (size_t)(sl - 1)] : nullptr;
      const double* ac = (q >= 1 && q <= nb - 2) ? &ang[9 * (size_t)sl] : nullptr;
      const double* a1 = (q + 1 >= 1 && q + 1 <= nb - 2) ? &ang[9 * (size_t)(sl + 1)] : nullptr;
      double F[3];
      const bool fast = !kick, slow = !MTS || kick;
      fu_force(P, g, q, rp, fast && q > 0 ? &cur[3 * (sl - 1)] : nullptr,
               fast && q < nb - 1 ? &cur[3 * (sl + 1)] : nullptr, fast ? a3 : nullptr, fast ? ac : nullptr,
               fast ? a1 : nullptr, cur, d.nbr + (size_t)sl * MAXNBR, cnt, F, slow);   // list entries are slots
      double v[3] = {d.v[3 * sl], d.v[3 * sl + 1], d.v[3 * sl + 2]};
      double J[3] = {d.J[3 * sl], d.J[3 * sl + 1], d.J[3 * sl + 2]};
      double u[3] = {d.up[3 * sl], d.up[3 * sl + 1], d.up[3 * sl + 2]};
      double xi[3] = {0.0, 0.0, 0.0};
      if (P.sig != 0.0)
        for (int a = 0; a < 3; ++a) xi[a] = kick ? 0.0 : d.xi[(size_t)3 * ((size_t)sub * nslots + sl) + a];
      if (d.mdtape)
        for (int a = 0; a < 3; ++a) {
          d.mdtape[((size_t)s * nb + q) * 6 + a] = rp[a];
          d.mdtape[((size_t)s * nb + q) * 6 + 3 + a] = v[a];
        }
      const bool fl = s == end - 1;
      double x[3];
      if (kick) {
        for (int a = 0; a < 3; ++a) {
          v[a] = v[a] + P.kick * F[a];
          if (s > 0 && !fl) v[a] = v[a] + P.kick * F[a];
          x[a] = fl ? rp[a] : rp[a] + P.hh * v[a];
          fin = fin && isfinite(v[a]) && isfinite(rp[a]);
        }
      } else {
        // r itself where a kick follows
        fin = fu_kick(P, F, u, xi, v, J, rp, MTS ? (s + 1) % (Mb + 1) == 0 : fl, x) && fin;
      }
      for (int a = 0; a < 3; ++a) {
        d.v[3 * sl + a] = v[a];
        d.J[3 * sl + a] = J[a];
        if (RIGID) rig->v[q][a] = v[a];             // RIG_MAX beads: thread q has bead q
        else if (fl) d.r[3 * sl + a] = x[a];
        else nxt[3 * sl + a] = x[a];
      }
    }
    __syncthreads();                              // the angle buffer is rewritten next
    if (RIGID) {
      if (t < nb)
        for (int a = 0; a < 3; ++a) rig->x[t][a] = cur[3 * (so + t) + a];
      lds_barrier();
      fin = rig_step(*rig, nb, P.hh, P.r0 * P.r0, s == end - 1) && fin;
      if (t < nb)
        for (int a = 0; a < 3; ++a) {
          (s == end - 1 ? d.r : nxt)[3 * (so + t) + a] = rig->x[t][a];
          d.v[3 * (so + t) + a] = rig->v[t][a];
        }
      __syncthreads();
    }
  }
  if (!fin) atomicOr(&d.ctrl->err, E_BEADS);
  if (over) atomicOr(&d.ctrl->err, E_NBRLIST);
}

__global__ __launch_bounds__(RD_WG) void k_md_redo(Dev d, FusedBufs fb, double* ang, int nslots, int n_sub, int K) {
  __shared__ int any_far, any_off;
  const int rep = blockIdx.x;
  const Rep& R = d.reps[rep];
  const MdParams P = R.mp;
  const int so = R.slot_off, nb = P.nb;
  const int t = threadIdx.x;
  const int sp = fb.redo[rep];                    // constant during this launch
  const int M = n_sub / K;
  if (sp < 0) {
    if (M & 1)
      for (int q = t; q < nb; q += RD_WG)
        for (int a = 0; a < 3; ++a) {
          d.v[3 * (so + q) + a] = fb.vS[3 * (so + q) + a];
          d.J[3 * (so + q) + a] = fb.JS[3 * (so + q) + a];
        }
    return;
  }
  // the failed block's start state into r_mid0, v, J
  if ((sp / K) & 1)
    for (int q = t; q < nb; q += RD_WG)
      for (int a = 0; a < 3; ++a) {
        const int i = 3 * (so + q) + a;
        d.rmid0[i] = fb.rmS[i];
        d.v[i] = fb.vS[i];
        d.J[i] = fb.JS[i];
      }
  if (t == 0) atomicAdd((unsigned long long*)&d.ctrl->substeps, (unsigned long long)(n_sub - sp));
  md_redo<RD_WG, false, false>(d, R, P, rep, ang, nslots, sp, n_sub, 0, nullptr, any_far, any_off);
}

// ---------------------------------------------------------------------------
// The resident sub-cycle: one launch advances every chain through the whole
// uniform sub-cycle.
//
// One launch per sub-step costs 7.4 us alone and 12.5 us beside the sweep for
// 2 to 3 us of dependent arithmetic: the kernel's end writes the L2 back (full
// of the sweep's lines) and the next one's start reads everything again from
// memory.  Here workgroup w owns the chain segment [a, b) (up to RES_OWN
// beads) for the whole cycle, holds its beads' state in registers and its
// positions in LDS, and per sub-step exchanges only what its neighbours need:
// it publishes its beads' new positions and polls those of its remote beads
// (the two chain neighbours at each end, and the partners in its beads'
// neighbour lists that other segments own, usually none).
//
// The exchange has no fence and no flag (an agent-scope release would write
// the L2 back).  A position component travels as two 64-bit words, its bits and
// its bits XOR a tag that no other sub-step of any pass of any cycle uses
// (lbmd_tag.h), written and read by relaxed agent-scope atomics, which bypass the
// L2s that the XCDs do not share: a reader takes the pair when the two words
// differ by the tag, so it needs no order between them.  Two slots suffice: segments depend on each
// other symmetrically, so a segment publishes x(s + 2) over x(s) only after
// it has read x(s + 1) of a segment that has read its x(s).
//
// Workgroups on one XCD exchange through its L2: a second copy of the
// positions is written with stores of workgroup scope, which stay there, and a
// reader takes the copy that suits its owner's XCD (each workgroup publishes
// its own at the start, so nothing depends on where the hardware puts them).
// Per exchange, beside a streaming kernel, each workgroup on a CU of its own: 0.8
// to 0.95 us within an XCD, 1.4 to 1.8 through memory (alone 0.69 and 1.0 to
// 1.3).  The host orders the segments so that a short chain lands on one XCD
// (res_place).
//
// A wave issues one dependent FP64 instruction in about five cycles, so a
// sub-step's time is the longest instruction count of a wave between two
// barriers plus the exchange; eight waves split the force terms by kind so
// that each is one pass over its lanes, and the two waves that share a SIMD
// (w and w + 4) are a long and a short one.  Phase 1: waves 0 and 1 the angles
// centred at a - 1 .. b without their kappa phi factor (one lane per angle and
// component); wave 2 the factors kappa phi; wave 3 the wall sites (one lane
// per site of the beads near the plane) and the field indicator; wave 4 stages
// the noise; wave 5 the bonds and the displacement check; waves 6 and 7 the
// pair forces (four lanes per bead, each a quarter of its list).  Phase 2:
// waves 0 and 1 (one lane per bead and component) add every contribution in
// the order of the sub-step kernel, move the beads and publish, while wave 4
// polls.  32 beads per workgroup fill one pass of the lanes; three such
// workgroups fit on a CU (80 registers).  Of 3900 cycles per sub-step (400
// beads, 128^3) phase 1 takes 2000 in a segment at the pore and 1500 elsewhere,
// the sum 700 up to the publishing, the exchange the rest.
//
// The workgroups announce themselves in ctrl->placed, and the sweep starts
// only then (k_md_gate): its small workgroups would otherwise refill every gap
// they leave, and a late segment holds up its neighbours until the sweep ends.
//
// The lists hold every pair within r_c while no bead is farther than half
// the skin from where they were built.  A workgroup whose bead leaves that
// range, whose lists are not valid at the start, whose remote beads, wall sites
// or pairs exceed what the first pass keeps, or whose wait exceeds its limit sets
// the replica's failure bit; the others see it while they poll, and leave the
// pass.  The segments store their results only when all of them have finished.
// Else the wide pass takes the replica from the cycle's start; when that fails
// too, the workgroup that leaves it last advances the replica alone (md_redo).
// Every wait ends: the polled value arrives, the bit is set, or the clock runs
// out.  All of this is one launch: a second one that finds nothing to do would
// wait for room beside the sweep (0.49 ms of a 1.1 ms step).
//
// The wide pass takes any density and any displacement.  Sixteen lanes per bead
// evaluate its terms side by side, whatever their kind, and its lanes 0 to 2 add
// them in the fixed order; a segment may have WIDE_REM remote partners, each
// fetched once per stage.  Every few stages (synchronised ones: as many apart as
// no bead can use up the lists' range in at twice its present speed) each segment
// publishes a word that says whether its beads are within CELL_MARGIN of where
// the cell table binned them, whether one is beyond the lists' range, and how long
// the others hold, and takes every segment's: where some word asks for new lists,
// all segments build them there, from positions that all have published, from the
// cell table if every word allows it, else from all beads of the chain.  No
// segment passes a synchronised stage before all have left the one before, so two
// slots suffice for the words too.  ms per step in the wide pass / with single
// launches: 2000 beads folded into a cube of spacing 1.1 0.73 / 0.84, 8000 1.05 /
// 1.01 (80 registers per lane), 2000 along the wall with r_c = 2.5 1.03 / 1.28,
// 8000 of a walk that was not relaxed 2.07 / 2.34, 2000 that drift by 3 per step
// 0.94 / 1.29, 300 rigid ones by 9 2.6 / 3.3; one workgroup alone takes 14 for
// the first and 60 for the second.
//
// The multiple-time-step cycle (MTS) is the same loop over n_sub + M + 1
// stages: kicks of the slow forces (pairs, walls, field) at r, and between two
// of them Mb = n_sub / M sub-steps of the bonded forces.  Pair partners that are
// no chain neighbours exchange positions for the kicks only, so those travel in
// slots of their own (2, 3, by the kick's parity: the argument above holds
// for the kicks alone, and for every stage between chain neighbours).  The
// lists are checked at the kicks, which are the wide pass's synchronised stages.
// 2000 beads, M = 5, n_sub = 100: 0.35 ms per step; with a launch per kick and
// one for the sub-steps between (k_md_inner) 0.63.
// ---------------------------------------------------------------------------
constexpr int RES_WG = 512;
constexpr int RES_HALO = 4;                    // local indices RES_OWN + 0..3: chain beads a-2, a-1, b, b+1
constexpr int RES_REM = 144;                   // other remote beads (more: the wide pass)
constexpr int RES_IDX = RES_OWN + RES_HALO + RES_REM;
constexpr int RES_PL = 4;                      // lanes per bead of the pair waves
constexpr int RES_PH = 4;                      // pair forces kept per lane
// Wall-site forces of a segment in the first pass: no disk of radius 2 has more than
// 14 points of the unit square lattice inside (every position of the centre, in ever
// smaller squares).  r_c up to 3 reaches 32, but with so many the wide pass, which
// spreads a bead's terms over 16 lanes, is the faster one: 400 beads along the
// wall at r_c = 2.5 and 3 0.91 and 0.99 against 1.35 and 1.57 ms per step.
constexpr int RES_WH = 14 * RES_OWN;
constexpr int RES_WH_START = 12 * RES_OWN;     // at the first sub-step, for r_c > 2: they may become more
constexpr int RES_HASH = 512;
// Up to RES_ALL segments read each other's words, of more the first one reads them
// and publishes their sum: 250 segments' loads of one another's meet at the few
// channels that hold them.
constexpr uint32_t RES_ALL = 64;
constexpr uint32_t RES_FAIL = 0x80000000u;
constexpr int RES_TILE = 256;                  // beads scanned together by a full list build
static_assert(RES_IDX <= 255, "local indices fit in a byte");
static_assert(3 * (RES_OWN + 2) <= 128 && RES_OWN + 2 <= 64 && RES_PL * RES_OWN == 128, "one pass over the lanes");

struct ResShared {
  double pos[2][RES_IDX][3];                   // by parity of the sub-step and local index
  double dd[2][RES_OWN + 2][3];                // row k: d1, d2 of the angle centred at a - 1 + k (see res_angle_d)
  double kp[RES_OWN + 2];                      // its kappa phi
  double bnd[RES_OWN + 1][3];                  // row k: force on a + k of its bond to a + k - 1
  double ref[RES_OWN][3];                      // where the lists were built
  double xi[3 * RES_OWN];                      // the sub-step's noise
  uint8_t lst[RES_OWN][MAXNBR];                // the beads' lists as local indices, ascending chain order
  int lcnt[RES_OWN];
  uint8_t pcnt[RES_OWN][RES_PL];               // pair forces found (one beyond RES_PH: the sum evaluates them again)
  int wall[RES_OWN];                           // first wall-site force << 8 | their number
  double wrec[RES_OWN][3];                     // beads near the plane: distance to it, wrapped transverse coordinates
  int wbead[RES_OWN];
  int fld[RES_OWN];                            // in the pore channel
  int rslot[RES_IDX - RES_OWN];                // bead slot of remote local index RES_OWN + k, -1: none
  uint8_t rnear[RES_IDX - RES_OWN];            // its owner runs on this XCD
  uint8_t snear[RIG_MAX / RES_OWN];            // the segment does (rigid bonds)
  int links;                                   // bit 0: some owner runs on another XCD, bit 1: on this one
  int nrem;
  int dead[2];                                 // by parity of the sub-step
  int lost;                                    // a set-up failed
  int done;
  union {
    struct {
      double pairF[RES_PL][RES_PH][RES_OWN][3];   // pair forces of each lane's part of the list, in order
      double wallF[RES_WH + 3][3];             // wall-site forces, bead by bead in site order
    };
    struct {                                   // set-up
      int key[RES_HASH], val[RES_HASH];        // local index of a remote chain bead
    } h;
  };
};
// The wide pass's memory.  A list holds chain indices,
// then places: own beads' index, WIDE_FAR + the place in rem (rigid bonds: chain
// indices throughout).
constexpr int WIDE_REM = 1024;                 // remote partners of a segment
constexpr int WIDE_FAR = 64;
constexpr uint16_t WIDE_NONE = 0xffffu;
struct WideShared {
  double pos[2][RES_OWN + RES_HALO][3];        // by parity of the stage: own beads, chain beads a-2, a-1, b, b+1
  double far[WIDE_REM][3];                     // the stage's positions of the remote partners
  double ref[RES_OWN][3];                      // where the lists were built
  double v[RES_OWN][3], J[RES_OWN][3], u[RES_OWN][3];
  uint16_t rem[WIDE_REM];                      // their chain indices, ascending
  uint16_t list[RES_OWN][MAXNBR];              // WIDE_NONE beyond a list's end
  union {
    double row[RES_OWN][RES_WG / RES_OWN][3];  // force terms of a bead, in the order of the sum
    struct {                                   // new lists
      uint32_t bk[RES_OWN][27];                // the 27 buckets around a bead
      double tile[RES_TILE][3];                // positions of RES_TILE chain beads
      int ncand[RES_OWN];
    } h;
    struct {                                   // the remote partners among the chain's beads
      uint32_t set[RES_WG];                    // a bit per bead
      int pre[RES_WG];                         // set bits before this word
      int wsum[RES_WG / 64];
    } m;
  };
  int nrem;
  uint32_t bits[2], all[2];                    // by parity of the stage: this segment's word, every segment's
  int lost[2];                                 // failed before / after the barrier that opens a stage of this parity
  int done, off, near;
  MdParams P;
};
static_assert(32 * RES_WG >= RES_MAX_WG * RES_OWN, "a bit for every bead of a chain");

// The memory of a workgroup: with rigid bonds RigShared, then ResShared or
// WideShared.  Dynamic, so that the kernel and what follows a failed pass share it.
extern __shared__ __align__(16) unsigned char res_lds[];
constexpr size_t res_base(bool rigid) { return rigid ? sizeof(RigShared) : 0; }
constexpr size_t res_bytes(bool rigid) {
  return res_base(rigid) + (sizeof(ResShared) > sizeof(WideShared) ? sizeof(ResShared) : sizeof(WideShared));
}
static_assert(sizeof(RigShared) % 16 == 0 && RES_WG == RIG_WG, "ResShared follows");
static_assert(3 * res_bytes(false) <= (size_t)LDS_PER_CU && res_bytes(true) <= (size_t)LDS_PER_CU,
              "as many fit on a CU as by registers; one with rigid bonds");

// Orders one wave's LDS accesses (which the LDS executes in order) for the compiler.
__device__ inline void wave_lds() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
__device__ inline unsigned long long res_load(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void res_store(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A store that stays in this XCD's L2, where an agent-scope load of another CU
// of the XCD finds it (it misses the L1s only).
__device__ inline void res_store_near(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline uint32_t res_xcd() { return __builtin_amdgcn_s_getreg(20 | 3 << 11); }   // HW_REG_XCC_ID, 4 bits

// Bond vectors u (first) and w (second), cross product n, its length s and
// c = u.w of the angle at (ra, rb, rc): the first operations of
// angle_component.  Scalars, so that a lane's selection of a component is one
// of registers.
struct ResAngle {
  double u0, u1, u2, w0, w1, w2, n0, n1, n2, s, c;
};
__device__ inline ResAngle res_angle(const double* ra, const double* rb, const double* rc) {
  ResAngle A;
  A.u0 = rb[0] - ra[0]; A.u1 = rb[1] - ra[1]; A.u2 = rb[2] - ra[2];
  A.w0 = rc[0] - rb[0]; A.w1 = rc[1] - rb[1]; A.w2 = rc[2] - rb[2];
  A.n0 = A.u1 * A.w2 - A.u2 * A.w1;
  A.n1 = A.u2 * A.w0 - A.u0 * A.w2;
  A.n2 = A.u0 * A.w1 - A.u1 * A.w0;
  A.s = sqrt(A.n0 * A.n0 + A.n1 * A.n1 + A.n2 * A.n2);
  A.c = A.u0 * A.w0 + A.u1 * A.w1 + A.u2 * A.w2;
  return A;
}
__device__ inline double sel3(int a, double x, double y, double z) { return a == 0 ? x : (a == 1 ? y : z); }
// d1, d2 of component a (angle_component's; the forces are kp d1 on the first
// bead, -(kp (d1 - d2)) on the centre, -(kp d2) on the third).  0 for a straight
// or folded angle, whose kp is 0 too.
__device__ inline void res_angle_d(const ResAngle& A, int a, double& d1, double& d2) {
  const double wa = sel3(a, A.w1, A.w2, A.w0), wb = sel3(a, A.w2, A.w0, A.w1);
  const double ua = sel3(a, A.u1, A.u2, A.u0), ub = sel3(a, A.u2, A.u0, A.u1);
  const double na = sel3(a, A.n1, A.n2, A.n0), nb = sel3(a, A.n2, A.n0, A.n1);
  const double den = A.s * A.s + A.c * A.c;
  const double g1 = wa * nb - wb * na;
  const double g2 = na * ub - nb * ua;
  d1 = (A.c * g1 / A.s - A.s * sel3(a, A.w0, A.w1, A.w2)) / den;
  d2 = (A.c * g2 / A.s - A.s * sel3(a, A.u0, A.u1, A.u2)) / den;
  if (A.s == 0.0) d1 = d2 = 0.0;
}

// A tagged pair's value, waiting for it until the tag matches; false when the
// replica's word has the failure bit or the wait reached its limit (RES_PLACE
// while some workgroup of the launch has not started: another context's cycle
// may hold its place and wait for one that this cycle holds).
__device__ inline bool res_poll(const unsigned long long* o, uint64_t tag, const uint32_t* word, const Ctrl* ctrl,
                                uint64_t wait, int nseg, unsigned long long& val) {
  unsigned long long w1;
  val = res_load(o);
  w1 = res_load(o + 1);
  if ((val ^ w1) == tag) return true;
  const uint64_t t0 = wall_clock64();
  for (int spin = 0;; ++spin) {
    val = res_load(o);
    w1 = res_load(o + 1);
    if ((val ^ w1) == tag) return true;
    if ((spin & 15) == 15 || wait == 0) {
      const uint64_t dt = wall_clock64() - t0;
      if ((__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & RES_FAIL) || dt >= wait ||
          (dt >= RES_PLACE &&
           __hip_atomic_load(&ctrl->placed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)nseg))
        return false;
    }
  }
}

// Failure ends a pass for the whole replica.  It is decided on one word: the
// number of segments that have finished, and a failure bit that can only be set
// while that number is below ng.  True: this call set the bit.
__device__ inline bool res_give_up(uint32_t* word, uint32_t ng) {
  uint32_t w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while (w < ng) {
    const uint32_t was = atomicCAS(word, w, w | RES_FAIL);
    if (was == w) return true;
    w = was;
  }
  return false;
}
// One thread of each segment, at a pass's end: every segment of the replica, or
// none, stores its result.
__device__ inline bool res_close(uint32_t* word, uint32_t ng, bool dead, uint64_t wait) {
  if (dead) return false;
  if (atomicAdd(word, 1u) + 1u != ng) {
    const uint64_t t0 = wall_clock64();
    while (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < ng)
      if (wall_clock64() - t0 >= wait) res_give_up(word, ng);   // the word reaches ng or gets the failure bit
  }
  return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ng;
}

// The first pass of the cycle (see above); false: it failed.
template <bool MTS, bool RIGID>
__device__ __forceinline__ bool res_pass(const Dev& d, const FusedSeg seg, const Rep& R, const MdParams& P, ResShared& sh,
                                        RigShared& rig, int nslots, int nseg, int n_sub, int mts, uint64_t wait) {
  const int rep = seg.rep;
  const int Mb = MTS ? n_sub / mts : 0;          // sub-steps between two kicks
  const int end = MTS ? n_sub + mts + 1 : n_sub; // stages; MTS: stage s is a kick where Mb + 1 divides it
  const Geom g = load_uniform(&R.g);
  const int so = load_uniform(&R.slot_off), nb = P.nb;
  const int p0 = seg.a, n = seg.b - seg.a;
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t) >> 6, lane = t & 63;
  uint32_t* word = &d.rsync[3 * rep];
  const uint32_t ng = (uint32_t)((nb + RES_OWN - 1) / RES_OWN);   // the replica's segments
  auto give_up = [&]() {
    if (res_give_up(word, ng)) atomicAdd((unsigned long long*)&d.ctrl->res_second, 1ull);
  };
  auto fail = [&](int s) {
    give_up();
    sh.dead[s & 1] = 1;
  };
  auto lose = [&]() {
    give_up();
    sh.lost = 1;
  };
  const uint64_t tag0 = res_tag(load_uniform(&d.ctrl->cycles), 0, 0);

  // ---- the lanes of the sum: component c of bead i
  const int i = 16 * wave + lane / 3, c = lane % 3;
  const bool mine = wave < 2 && lane < 48 && i < n;
  const int slot = so + p0 + (mine ? i : 0), p = p0 + i;
  double x = 0.0, v = 0.0, J = 0.0, u = 0.0;
  bool fin = true;                               // of the pass; an error only if its result is kept
  if (RIGID) {
    double r3[3] = {0.0, 0.0, 0.0}, v3[3] = {0.0, 0.0, 0.0};
    if (t < nb)
      for (int a = 0; a < 3; ++a) { r3[a] = d.r[3 * (so + t) + a]; v3[a] = d.v[3 * (so + t) + a]; }
    fin = rig_open(rig, nb, P.hh, P.r0 * P.r0, r3, v3);
  }
  if (mine) {
    x = RIGID ? rig.x[p][c] : d.rmid0[3 * slot + c];
    v = RIGID ? rig.v[p][c] : d.v[3 * slot + c];
    J = d.J[3 * slot + c];
    u = P.couple ? d.up[3 * slot + c] : 0.0;
    sh.pos[0][i][c] = x;
  }
  if (t < 2) sh.dead[t] = 0;
  const int g0 = seg.id - p0 / RES_OWN;          // the replica's first segment
  if (t == 0) {
    sh.lost = 0;
    __hip_atomic_fetch_add(&d.ctrl->placed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (seg.id == 0) atomicAdd((unsigned long long*)&d.ctrl->substeps, (unsigned long long)n_sub);
    const unsigned long long w = res_xcd();
    res_store(d.xflag + 4 * (size_t)nseg + 2 * seg.id, w);
    res_store(d.xflag + 4 * (size_t)nseg + 2 * seg.id + 1, w ^ tag0);
    if (d.rb[4 * rep] != 0u) lose();             // the lists are not valid at the start
    if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & RES_FAIL) sh.lost = 1;
  }
  bool dead = false;
  do {
  // ---- set-up: the lists as local indices
  __syncthreads();                               // the positions are there
  constexpr int LL = RES_WG / RES_OWN, LE = MAXNBR / LL;   // 16 lanes per bead
  const int lb = t / LL, ll = t % LL;
  const int cnt = lb < n ? d.ncnt[so + p0 + lb] : 0;
  if (t < n)
    for (int a = 0; a < 3; ++a) sh.ref[t][a] = d.ref[3 * (so + p0 + t) + a];
  if (t == 0) { sh.nrem = 0; sh.links = 0; }
  for (int k = t; k < RES_IDX - RES_OWN; k += RES_WG) {
    // chain beads a - 2, a - 1, b, b + 1 first
    const int q = k < 2 ? p0 - 2 + k : seg.b + (k - 2);
    sh.rslot[k] = k < RES_HALO && q >= 0 && q < nb ? so + q : -1;
  }
  for (int k = t; k < RES_HASH; k += RES_WG) { sh.h.key[k] = -1; sh.h.val[k] = -1; }
  if (wave == 7) {
    // the segment as a whole will leave the lists' range within the cycle: at
    // once, not when it gets there (200 rigid beads at 0.9 per step, 2.9 against 1.9 ms)
    double m2 = 0.0;
    for (int a = 0; a < 3; ++a) {
      double y = lane < n ? d.v[3 * (so + p0 + lane) + a] : 0.0;
      for (int o = 16; o > 0; o >>= 1) y += __shfl_xor(y, o, 64);
      m2 += y * y;
    }
    const double reach = 2.0 * P.hh * n_sub;
    if (lane == 0 && m2 * reach * reach > P.halfskin2 * (double)(n * n)) lose();
  }
  __syncthreads();
  // a remote bead's first finder gives it an index
  // a full list may have lost partners: segments need not depend on each other
  if (cnt >= MAXNBR && (__hip_atomic_load(&d.ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & E_NBRLIST)) lose();
  int e[LE];
#pragma unroll
  for (int m = 0; m < LE; ++m) {
    const int k = LL * m + ll;
    e[m] = k < cnt ? d.nbr[(size_t)(so + p0 + lb) * MAXNBR + k] : -1;
  }
#pragma unroll 1
  for (int m = 0; m < LE; ++m) {
    const int em = m == 0 ? e[0] : (m == 1 ? e[1] : e[2]);
    const int q = em - so;
    if (em < 0 || (q >= p0 - 2 && q < seg.b + 2) || sh.lost) continue;
    uint32_t h = ((uint32_t)q * 2654435761u) >> 23;          // RES_HASH = 2^9
    for (int tries = 0; tries < RES_HASH; ++tries, h = (h + 1) & (RES_HASH - 1)) {
      const int was = atomicCAS(&sh.h.key[h], -1, q);
      if (was == -1) {
        const int at = atomicAdd(&sh.nrem, 1);
        if (at < RES_REM) {
          sh.h.val[h] = RES_OWN + RES_HALO + at;
          sh.rslot[RES_HALO + at] = em;
        } else {
          lose();
        }
        break;
      }
      if (was == q) break;
      if (tries == RES_HASH - 1) lose();
    }
  }
  __syncthreads();
  const int full = sh.lost;
  __syncthreads();
  if (full) { dead = true; break; }              // uniform
  if (lb < n && ll == 0) sh.lcnt[lb] = cnt;
#pragma unroll 1
  for (int m = 0; m < LE; ++m) {
    const int em = m == 0 ? e[0] : (m == 1 ? e[1] : e[2]);
    if (em < 0) continue;
    const int q = em - so;
    int li;
    if (q >= p0 && q < seg.b) li = q - p0;
    else if (q >= p0 - 2 && q < p0) li = RES_OWN + (q - p0 + 2);
    else if (q >= seg.b && q < seg.b + 2) li = RES_OWN + 2 + (q - seg.b);
    else {
      uint32_t h = ((uint32_t)q * 2654435761u) >> 23;
      for (int tries = 0; tries < RES_HASH && sh.h.key[h] != q; ++tries) h = (h + 1) & (RES_HASH - 1);
      li = sh.h.key[h] == q ? sh.h.val[h] : -1;
    }
    sh.lst[lb][LL * m + ll] = (uint8_t)(li >= 0 ? li : 0);   // -1 only when lost
  }
  // which remote beads are exchanged within this XCD
  for (int k = t; k < RES_HALO + min(sh.nrem, RES_REM); k += RES_WG) {
    const int sl = sh.rslot[k];
    unsigned long long w = 0;
    if (sl >= 0 && !res_poll(d.xflag + 4 * (size_t)nseg + 2 * (g0 + (sl - so) / RES_OWN), tag0, word, d.ctrl, wait, nseg, w))
      lose();
    const bool near = w == (unsigned long long)res_xcd();
    sh.rnear[k] = near;
    if (sl >= 0) atomicOr(&sh.links, near ? 2 : 1);
  }
  for (int k = t; k < 3 * (RES_HALO + min(sh.nrem, RES_REM)); k += RES_WG) {
    const int sl = sh.rslot[k / 3];
    sh.pos[0][RES_OWN + k / 3][k % 3] = sl < 0 ? 0.0 : (RIGID ? rig.x[sl - so][k % 3] : d.rmid0[3 * sl + k % 3]);
  }
  if (RIGID) {
    // every segment's velocities are read; the lists at the opening's positions
    for (int k = t; k < (int)ng; k += RES_WG) {
      unsigned long long w = 0;
      if (!res_poll(d.xflag + 4 * (size_t)nseg + 2 * (g0 + k), tag0, word, d.ctrl, wait, nseg, w)) lose();
      const bool near = w == (unsigned long long)res_xcd();
      sh.snear[k] = near;
      if (g0 + k != seg.id) atomicOr(&sh.links, near ? 2 : 1);
    }
    if (t < n) {
      double d2 = 0.0;
      for (int a = 0; a < 3; ++a) { const double dd = sh.pos[0][t][a] - sh.ref[t][a]; d2 += dd * dd; }
      if (d2 > P.halfskin2) lose();
    }
  }
  __syncthreads();
  if (sh.lost) { dead = true; break; }           // uniform
  const int nrem = RES_HALO + min(sh.nrem, RES_REM);

  constexpr int HL = RES_OWN, HR = RES_OWN + 2;  // local indices of a - 2 and b
  // local index of chain bead a + j, -2 <= j <= n + 1
  auto at = [&](int j) { return j < 0 ? HL + 2 + j : (j < n ? j : HR + (j - n)); };
  // no lane writes the angles and bonds beyond the chain's ends
  if (t < n + 2 && !(p0 - 1 + t >= 1 && p0 - 1 + t <= nb - 2)) {
    sh.kp[t] = 0.0;
    for (int a = 0; a < 3; ++a) sh.dd[0][t][a] = sh.dd[1][t][a] = 0.0;
  }
  if (t <= n && (P.constrained || p0 + t == 0 || p0 + t == nb))
    for (int a = 0; a < 3; ++a) sh.bnd[t][a] = 0.0;
  const int links = sh.links;                    // 0: no other segment needs this one's positions
  const size_t half = (size_t)6 * nslots;        // words of one slot of the ring
  const bool noisy = P.sig != 0.0;
  // Rigid bonds, after the sum of sub-step s: the chain's kicked velocities from
  // the other segments, its projections, and the positions of s + 1.
  auto rigid = [&](int s) {
    const int cb = s & 1;
    const uint64_t tag = tag0 + (uint64_t)(s + 1) * RES_TAG;
    const unsigned long long* from = d.xring + (cb ? 0 : half);
    for (int k = t; k < 3 * nb; k += RES_WG) {
      const int q = k / 3;
      if (q >= p0 && q < seg.b) continue;
      unsigned long long w = 0;
      if (!res_poll(from + ((size_t)so * 3 + k) * 2 + (sh.snear[q / RES_OWN] ? 4 * half : 0), tag, word, d.ctrl, wait, nseg, w)) {
        fail(s);
        break;
      }
      rig.v[q][k - 3 * q] = __longlong_as_double((long long)w);
    }
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(sh.dead[cb])) return;   // uniform: the next writes follow the barriers below
    fin = rig_step(rig, nb, P.hh, P.r0 * P.r0, s == end - 1) && fin;
    if (s < end - 1) {
      for (int k = t; k < 3 * (RES_OWN + nrem); k += RES_WG) {
        const int l = k / 3, q = l < RES_OWN ? (l < n ? p0 + l : -1) : sh.rslot[l - RES_OWN] - so;
        if (q >= 0) sh.pos[cb ^ 1][l][k - 3 * l] = rig.x[q][k - 3 * l];
      }
      if (t < n) {
        double d2 = 0.0;
        for (int a = 0; a < 3; ++a) { const double dd = rig.x[p0 + t][a] - sh.ref[t][a]; d2 += dd * dd; }
        if (d2 > P.halfskin2) fail(s);
      }
    }
    lds_barrier();
  };
  __builtin_amdgcn_s_setprio(2);
  for (int sa = 0;; ++sa) {                      // RIGID: the loops below take one sub-step at a time
  const int sb = RIGID ? sa + 1 : end;
  // Each kind of wave has a loop of its own (its registers then hold only
  // what it needs), with the same two barriers per sub-step.  A failure at
  // sub-step s is seen before the first barrier of s + 1, by all waves: s writes
  // dead[s & 1] before its second barrier, s + 2 after the first of s + 1 (the
  // load is in flight with the sub-step's others; a test after the second
  // barrier would wait for it).  q: stages since the last kick (MTS).
  if (wave < 2) {
    // ---- angles; the sum
    const int k = t / 3, ka = t % 3;             // component ka of the angle centred at a - 1 + k
    const bool ang = k < n + 2 && p0 - 1 + k >= 1 && p0 - 1 + k <= nb - 2;
    const int j0 = ang ? at(k - 2) : 0, j1 = ang ? at(k - 1) : 0, j2 = ang ? at(k) : 0;
    double* tape = mine && d.mdtape ? d.mdtape + (size_t)p * 6 + c : nullptr;
    unsigned long long* ring = d.xring + ((size_t)slot * 3 + c) * 2;
    uint64_t tag = tag0 + (uint64_t)sa * RES_TAG;
    int q = 0, o = 0;
    for (int s = sa; s < sb; ++s) {
      const int cb = s & 1, was = sh.dead[cb ^ 1];
      const bool last = s == end - 1;
      const bool kick = MTS && q == 0;
      if (MTS && q++ == Mb) { q = 0; ++o; }      // of stage s + 1
      tag += RES_TAG;                                // of sub-step s + 1
      if (ang && !kick) {
        const ResAngle A = res_angle(sh.pos[cb][j0], sh.pos[cb][j1], sh.pos[cb][j2]);
        double d1, d2;
        res_angle_d(A, ka, d1, d2);
        sh.dd[0][k][ka] = d1;
        sh.dd[1][k][ka] = d2;
      }
      if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
      // every contribution in the fixed order, the kick and the drifts
      if (mine) {
        // Absent contributions are zeros (F is never -0, which a zero would change).
        const uint32_t pc = *reinterpret_cast<const uint32_t*>(sh.pcnt[i]);
        const int wl = sh.wall[i], fl = sh.fld[i];
        const double xi = noisy ? sh.xi[3 * i + c] : 0.0;
        const double f0 = sh.pairF[0][0][i][c], f1 = sh.pairF[1][0][i][c], f2 = sh.pairF[2][0][i][c],
                     f3 = sh.pairF[3][0][i][c];
        const double kp0 = sh.kp[i], kp1 = sh.kp[i + 1], kp2 = sh.kp[i + 2];
        const double e2 = sh.dd[1][i][c], m1 = sh.dd[0][i + 1][c], m2 = sh.dd[1][i + 1][c], q1 = sh.dd[0][i + 2][c];
        const double fb0 = sh.bnd[i][c], fb1 = sh.bnd[i + 1][c];
        double F = 0.0;
        if (!kick) {
        F += fb0;
        F += -fb1;
        F += -(kp0 * e2);
        F += -(kp1 * (m1 - m2));
        F += kp2 * q1;
        }
        if (!MTS || kick) {
        if (!__any((pc & 0xfefefefeu) != 0u)) {  // at most one pair force per lane
          F += f0;
          F += f1;
          F += f2;
          F += f3;
        } else {
          bool kept = true;
          for (int l = 0; l < RES_PL; ++l) kept = kept && (int)((pc >> (8 * l)) & 0xffu) <= RES_PH;
          if (kept) {
            for (int l = 0; l < RES_PL; ++l)
              for (int m = 0; m < (int)((pc >> (8 * l)) & 0xffu); ++m) F += sh.pairF[l][m][i][c];
          } else {
            const double* rp = sh.pos[cb][i];
            for (int m = 0; m < sh.lcnt[i]; ++m) {
              const double* rq = sh.pos[cb][sh.lst[i][m]];
              const double d0 = min_image(rp[0] - rq[0], g.nx);
              const double d1 = min_image(rp[1] - rq[1], g.ny);
              const double d2 = min_image(rp[2] - rq[2], g.nz);
              if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rc2)) continue;
              double Fp[3] = {0.0, 0.0, 0.0};
              lj_add(P, d0, d1, d2, Fp);
              F += c == 0 ? Fp[0] : (c == 1 ? Fp[1] : Fp[2]);
            }
          }
        }
        if (__any((wl & 0xff) != 0))
        for (int m = wl >> 8, m1 = m + (wl & 0xff); m < m1; m += 4) {   // four loads in flight
          const double f0 = sh.wallF[m][c], f1 = sh.wallF[m + 1][c], f2 = sh.wallF[m + 2][c], f3 = sh.wallF[m + 3][c];
          F += f0;
          if (m + 1 < m1) F += f1;
          if (m + 2 < m1) F += f2;
          if (m + 3 < m1) F += f3;
        }
        if (fl && c == g.wall_axis) F += P.f_drive;
        }
        if (!MTS && tape) {
          double* tp = tape + (size_t)s * nb * 6;
          tp[0] = x;
          tp[3] = v;
        }
        if (kick) {
          v = v + P.kick * F;
          if (s > 0 && !last) v = v + P.kick * F;
          fin = fin && isfinite(v) && isfinite(x);
          if (!last) x = x + P.hh * v;
        } else {
          const double sx = P.sig * xi;
          const double vn = P.e * v + P.cf * (F + P.gamma * u) + sx;
          J = J - P.m * (P.omE * (u - v) + sx);
          v = vn;
          fin = fin && isfinite(vn);
          if (RIGID) rig.v[p][c] = vn;
          const double re = x + P.hh * vn;
          x = (MTS ? q == 0 : last) ? re : re + P.hh * vn;   // a kick takes r itself
        }
        if (RIGID || !last) {
          if (!RIGID) sh.pos[cb ^ 1][i][c] = x;
          unsigned long long* w = ring + (MTS && q == 0 ? (2 + (o & 1)) * half : (cb ? 0 : half));
          const unsigned long long bits = (unsigned long long)__double_as_longlong(RIGID ? v : x);
          if (links & 2) {
            res_store_near(w + 4 * half, bits);
            res_store_near(w + 4 * half + 1, bits ^ tag);
          }
          if (links & 1) {
            res_store(w, bits);
            res_store(w + 1, bits ^ tag);
          }
        }
      }
      lds_barrier();
    }
  } else if (wave >= 6) {
    // ---- pair forces: part [k0, k1) of bead pb's list
    const int pb = (t - 384) / RES_PL, pl = t % RES_PL;
    int k0 = 0, k1 = 0, first = 0;
    if (pb < n) {
      const int m = sh.lcnt[pb], per = (m + RES_PL - 1) / RES_PL;
      k0 = min(pl * per, m);
      k1 = min(k0 + per, m);
      first = k0 < k1 ? sh.lst[pb][k0] : 0;
    }
    int q = 0;
    for (int s = sa; s < sb; ++s) {
      const int cb = s & 1, was = sh.dead[cb ^ 1];
      const bool slow = !MTS || q == 0;
      if (MTS && q++ == Mb) q = 0;
      if (pb < n && slow) {
        const double* rp = sh.pos[cb][pb];
        const double r0 = rp[0], r1 = rp[1], r2 = rp[2];
        int hits = 0;
        for (int m = k0; m < k1; ++m) {
          const double* rq = sh.pos[cb][m == k0 ? first : sh.lst[pb][m]];
          const double d0 = min_image(r0 - rq[0], g.nx);
          const double d1 = min_image(r1 - rq[1], g.ny);
          const double d2 = min_image(r2 - rq[2], g.nz);
          if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rc2)) continue;
          double Fp[3] = {0.0, 0.0, 0.0};
          lj_add(P, d0, d1, d2, Fp);
          if (hits < RES_PH) {
            double* o = sh.pairF[pl][hits][pb];
            o[0] = Fp[0]; o[1] = Fp[1]; o[2] = Fp[2];
          }
          ++hits;
        }
        if (hits == 0) {
          double* o = sh.pairF[pl][0][pb];
          o[0] = 0.0; o[1] = 0.0; o[2] = 0.0;
        }
        sh.pcnt[pb][pl] = (uint8_t)min(hits, RES_PH + 1);
        if (s == 0 && hits > RES_PH) fail(s);    // the sum would evaluate the list again (2.3 against 0.97 ms per
                                                 // step, 400 beads along the wall, r_c = 2.5): the wide pass
      }
      if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
      lds_barrier();
    }
  } else if (wave == 2) {
    // ---- kappa phi of the angle centred at a - 1 + lane
    const bool ang = lane < n + 2 && p0 - 1 + lane >= 1 && p0 - 1 + lane <= nb - 2;
    const int j0 = ang ? at(lane - 2) : 0, j1 = ang ? at(lane - 1) : 0, j2 = ang ? at(lane) : 0;
    int q = 0;
    for (int s = sa; s < sb; ++s) {
      const int cb = s & 1, was = sh.dead[cb ^ 1];
      const bool kick = MTS && q == 0;
      if (MTS && q++ == Mb) q = 0;
      if (ang && !kick) {
        const ResAngle A = res_angle(sh.pos[cb][j0], sh.pos[cb][j1], sh.pos[cb][j2]);
        sh.kp[lane] = A.s == 0.0 ? 0.0 : P.kappa * atan2(A.s, A.c);
      }
      if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
      lds_barrier();
    }
  } else if (wave == 5) {
    // ---- bonds: the force on a + lane of its bond to a + lane - 1 (the
    // other bead takes its exact negative); the displacement check
    const bool bond = !P.constrained && lane <= n && p0 + lane > 0 && p0 + lane < nb;
    double ref[3] = {0.0, 0.0, 0.0};
    if (lane < n) {
#pragma unroll
      for (int a = 0; a < 3; ++a) ref[a] = sh.ref[lane][a];
    }
    int q = 0;
    for (int s = sa; s < sb; ++s) {
      const int cb = s & 1, was = sh.dead[cb ^ 1];
      const bool kick = MTS && q == 0;
      if (MTS && q++ == Mb) q = 0;
      if (bond && !kick) {
        double Fb[3] = {0.0, 0.0, 0.0};
        bond_add(P, sh.pos[cb][lane < n ? lane : HR], sh.pos[cb][lane ? lane - 1 : HL + 1], Fb);
        sh.bnd[lane][0] = Fb[0]; sh.bnd[lane][1] = Fb[1]; sh.bnd[lane][2] = Fb[2];
      }
      if (lane < n && s > 0 && (MTS ? kick : !RIGID)) {
        double d2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) { const double dd = sh.pos[cb][lane][a] - ref[a]; d2 += dd * dd; }
        if (d2 > P.halfskin2) fail(s);
      }
      if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
      lds_barrier();
    }
  } else if (wave == 3) {
    // ---- the wall sites of wall_row and the field indicator
    const int wa = g.wall_axis, na = wa >= 0 ? ext(g, wa) : 0;
    const int nw = P.whi - P.wlo + 1, per = nw <= 4 ? 16 : 64;
    // Three passes, each with few idle lanes: a lane per bead finds the beads
    // within r_c of the plane (the normal part of a distance alone: a sum of
    // squares rounds to no less than one of them); a lane per site of those,
    // in site order (o1 outer, o0 inner; 16 lanes per bead and 4 beads at once
    // for the 4 x 4 window, else 64 lanes), finds the sites within r_c; a lane
    // per site found evaluates its force.  With all of it in one pass a chain
    // that lies along the plane made this the longest wave: 0.37 to 0.57
    // against 0.29 ms per step (400 beads, 128^3), 0.48 to 0.62 against 0.38
    // (32 x 100 beads).
    const int num = lane % per, o1 = P.wlo + num / nw, o0 = P.wlo + num % nw;
    const int n0 = wa == 0 ? g.ny : g.nx, n1 = wa == 2 ? g.ny : g.nz;   // transverse extents
    const uint64_t below = (1ull << lane) - 1ull;
    int q = 0;
    for (int s = sa; s < sb; ++s) {
      const int cb = s & 1, was = sh.dead[cb ^ 1];
      const bool slow = !MTS || q == 0;
      if (MTS && q++ == Mb) q = 0;
      if (!slow) {
        if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
        lds_barrier();
        continue;
      }
      int fl = 0;
      bool near = false;
      double dn = 0.0, wt0 = 0.0, wt1 = 0.0;
      if (wa >= 0 && lane < n) {
        const double* rp = sh.pos[cb][lane];
        const double wn = wrapc(rp[wa], na);
        int off = g.wall_pos - (int)floor(wn);
        if (off < WLO) off += na;
        if (off > WHI) off -= na;
        if (off >= P.wlo && off <= P.whi) {      // the bead's window reaches the plane
          wt0 = wrapc(rp[g.t0], n0);
          wt1 = wrapc(rp[g.t1], n1);
          dn = wn - (double)((int)floor(wn) + off);
          near = dn * dn < P.rc2;
          fl = P.field_on && wn >= g.wall_pos - 1.5 && wn < g.wall_pos + 1.5 && wt0 >= g.lo0 - 0.5 &&
               wt0 < g.hi0 + 0.5 && wt1 >= g.lo1 - 0.5 && wt1 < g.hi1 + 0.5 ? 1 : 0;
        }
      }
      const uint64_t nm = __ballot(near);
      const int nn = __builtin_popcountll(nm);
      if (lane < n) {
        sh.fld[lane] = fl;
        sh.wall[lane] = 0;
      }
      if (near) {
        const int r = __builtin_popcountll(nm & below);
        sh.wrec[r][0] = dn; sh.wrec[r][1] = wt0; sh.wrec[r][2] = wt1;
        sh.wbead[r] = lane;
      }
      int total = 0;
      for (int r0 = 0; r0 < nn; r0 += 64 / per) {
        wave_lds();
        const int r = r0 + lane / per;
        const bool on = r < nn && num < nw * nw;
        bool hit = false;
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        if (on) {
          const double x0 = sh.wrec[r][1], x1 = sh.wrec[r][2], xn = sh.wrec[r][0];
          const int u1 = (int)floor(x1) + o1, u0 = (int)floor(x0) + o0;
          const int v1 = u1 < 0 ? u1 + n1 : (u1 >= n1 ? u1 - n1 : u1);
          const int v0 = u0 < 0 ? u0 + n0 : (u0 >= n0 ? u0 - n0 : u0);
          const bool pore = v1 >= g.lo1 && v1 <= g.hi1 && v0 >= g.lo0 && v0 <= g.hi0;
          const double dt0 = x0 - (double)u0, dt1 = x1 - (double)u1;
          d0 = wa == 0 ? xn : dt0;
          d1 = wa == 1 ? xn : (wa == 0 ? dt0 : dt1);
          d2 = wa == 2 ? xn : dt1;
          hit = !pore && d0 * d0 + d1 * d1 + d2 * d2 < P.rc2;
        }
        const uint64_t hm = __ballot(hit);
        const int o = total + __builtin_popcountll(hm & below);
        if (hit && o < RES_WH) { sh.wallF[o][0] = d0; sh.wallF[o][1] = d1; sh.wallF[o][2] = d2; }
        if (on && num == 0) {
          const uint64_t own = per == 64 ? hm : (hm >> lane) & 0xffffull;
          sh.wall[sh.wbead[r]] = (o << 8) | __builtin_popcountll(own);
        }
        total += __builtin_popcountll(hm);
      }
      wave_lds();
      if (per == 64 && total > (s == 0 ? RES_WH_START : RES_WH)) {   // too many: the wide pass takes them
        fail(s);
        if (lane < n) sh.wall[lane] = 0;         // none is read
        total = 0;
      }
      for (int o = lane; o < total; o += 64) {
        double* w = sh.wallF[o];
        double Fs[3] = {0.0, 0.0, 0.0};
        lj_add(P, w[0], w[1], w[2], Fs);
        w[0] = Fs[0]; w[1] = Fs[1]; w[2] = Fs[2];
      }
      if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
      lds_barrier();
    }
  } else {
    // ---- the noise of the workgroup's beads, one sub-step ahead (up to two
    // of its 3 n values per lane); the remote positions
    const int nx = noisy ? 3 * n : 0;
    const size_t row = (size_t)3 * nslots;
    int left = n_sub - sa;                       // sub-steps from here on
    const double* xn = d.xi + (size_t)3 * (so + p0) + (size_t)(n_sub - left) * row;
    double xa = 0.0, xc = 0.0;
    if (!MTS || left > 0) {
      xa = lane < nx ? xn[lane] : 0.0;
      xc = lane + 64 < nx ? xn[lane + 64] : 0.0;
    }
    const int rs0 = lane < 3 * nrem ? sh.rslot[lane / 3] : -1;
    const bool rn0 = lane < 3 * nrem && sh.rnear[lane / 3];
    uint64_t tag = tag0 + (uint64_t)sa * RES_TAG;
    int q = 0, o = 0;
    for (int s = sa; s < sb; ++s) {
      const int cb = s & 1, was = sh.dead[cb ^ 1];
      const bool kick = MTS && q == 0;
      if (MTS && q++ == Mb) { q = 0; ++o; }      // of stage s + 1
      tag += RES_TAG;
      if (!kick) {
        if (lane < nx) sh.xi[lane] = xa;
        if (lane + 64 < nx) sh.xi[lane + 64] = xc;
        --left;
      }
      if (__builtin_amdgcn_readfirstlane(was)) { dead = true; break; }
      lds_barrier();
      if (!RIGID && s < end - 1) {
        if (!kick && left > 0) {
          xn += row;
          if (lane < nx) xa = xn[lane];
          if (lane + 64 < nx) xc = xn[lane + 64];
        }
        const unsigned long long* from = d.xring + (MTS && q == 0 ? (2 + (o & 1)) * half : (cb ? 0 : half));
        const int m1 = 3 * (MTS && q != 0 ? RES_HALO : nrem);   // a sub-step needs the chain neighbours only
        for (int m = lane; m < m1; m += 64) {
          const int sl = m == lane ? rs0 : sh.rslot[m / 3];
          if (sl < 0) continue;
          unsigned long long w = 0;
          const size_t off = ((size_t)sl * 3 + m % 3) * 2 + ((m == lane ? rn0 : sh.rnear[m / 3] != 0) ? 4 * half : 0);
          if (!res_poll(from + off, tag, word, d.ctrl, wait, nseg, w)) {
            fail(s);
            break;
          }
          sh.pos[cb ^ 1][RES_OWN + m / 3][m % 3] = __longlong_as_double((long long)w);
        }
      }
      lds_barrier();
    }
  }
  if (!RIGID || dead) break;
  rigid(sa);
  if (mine) { x = rig.x[p][c]; v = rig.v[p][c]; }
  if (sa == end - 1) break;
  }
  if (__builtin_amdgcn_readfirstlane(sh.dead[(end - 1) & 1])) dead = true;   // the last sub-step's
  } while (false);
  __builtin_amdgcn_s_setprio(0);
  if (t == 0) sh.done = res_close(word, ng, dead, wait);
  __syncthreads();
  if (!sh.done) return false;
  if (mine) {
    d.r[3 * slot + c] = x;
    d.v[3 * slot + c] = v;
    d.J[3 * slot + c] = J;
    if (!fin) atomicOr(&d.ctrl->err, E_BEADS);
  }
  return true;
}

// As res_poll for a published vector, its words requested together.
__device__ inline bool res_poll_vec(const unsigned long long* o, uint64_t tag, const uint32_t* word, const Ctrl* ctrl,
                                    uint64_t wait, int nseg, double y[3]) {
  uint64_t t0 = 0;
  for (int spin = 0;; ++spin) {
    unsigned long long w[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) w[k] = res_load(o + k);
    for (int a = 0; a < 3; ++a) y[a] = __longlong_as_double((long long)w[2 * a]);
    if ((w[0] ^ w[1]) == tag && (w[2] ^ w[3]) == tag && (w[4] ^ w[5]) == tag) return true;
    if (spin == 0) t0 = wall_clock64();
    if ((spin & 15) == 15 || wait == 0) {
      const uint64_t dt = wall_clock64() - t0;
      if ((__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & RES_FAIL) || dt >= wait ||
          (dt >= RES_PLACE &&
           __hip_atomic_load(&ctrl->placed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)nseg))
        return false;
    }
  }
}

// The bonded terms of chain bead q, in the first five rows of its lanes: bonds to
// q - 1 and q + 1, the angles centred at q - 1 (third bead's part), q (centre) and
// q + 1 (first); zeros beyond the chain's ends.  Out of line: its constants (the
// arc tangent's) are else kept, and spilled, over the whole loop.
template <bool RIGID>
__device__ __attribute__((noinline)) void wide_bonded(int cb, int n, int q, int nb) {
  WideShared& sh = *reinterpret_cast<WideShared*>(res_lds + res_base(RIGID));
  RigShared& rig = *reinterpret_cast<RigShared*>(res_lds);
  const MdParams& P = sh.P;
  constexpr int LL = RES_WG / RES_OWN;
  const int b = threadIdx.x / LL, l = threadIdx.x % LL;
  const bool on = b < n;
  double (*const row)[3] = sh.row[b];
  // chain bead q + k, -2 <= k <= 2
  auto chain = [&](int k) -> const double* {
    if (RIGID) return rig.x[q + k];
    const int j = b + k;
    return sh.pos[cb][j < 0 ? RES_OWN + 2 + j : (j < n ? j : RES_OWN + 2 + (j - n))];
  };
  if (l < 9) {
    // component c of the angle centred at q - 1 + k
    const int k = l / 3, c = l % 3, cen = q - 1 + k;
    double y = 0.0;
    if (on && cen >= 1 && cen <= nb - 2) {
      const ResAngle A = res_angle(chain(k - 2), chain(k - 1), chain(k));
      double d1, d2;
      res_angle_d(A, c, d1, d2);
      const double kp = A.s == 0.0 ? 0.0 : P.kappa * atan2(A.s, A.c);
      y = k == 0 ? -(kp * d2) : (k == 1 ? -(kp * (d1 - d2)) : kp * d1);
    }
    row[2 + k][c] = y;
  } else if (l < 11) {
    const int k = l == 9 ? -1 : 1;
    double F[3] = {0.0, 0.0, 0.0};
    if (on && !P.constrained && q + k >= 0 && q + k < nb) bond_add(P, chain(0), chain(k), F);
    row[l - 9][0] = F[0]; row[l - 9][1] = F[1]; row[l - 9][2] = F[2];
  }
}

// The wide pass of the cycle (see above); false: it failed.
template <bool MTS, bool RIGID>
__device__ __forceinline__ bool res_wide(const Dev& d, const FusedSeg seg, const Rep& R, const MdParams& P0, WideShared& sh,
                                         RigShared& rig, int nslots, int nseg, int n_sub, int mts, uint64_t wait) {
  const int rep = seg.rep;
  const int Mb = MTS ? n_sub / mts : 0;
  const int end = MTS ? n_sub + mts + 1 : n_sub;
  const Geom g = load_uniform(&R.g);
  const int so = load_uniform(&R.slot_off), nb = P0.nb;
  const int p0 = seg.a, n = seg.b - seg.a;
  const int t = threadIdx.x;
  uint32_t* word = &d.rsync[3 * rep + 1];
  const uint32_t ng = (uint32_t)((nb + RES_OWN - 1) / RES_OWN);
  const int g0 = seg.id - p0 / RES_OWN;
  const uint64_t tag0 = res_tag(load_uniform(&d.ctrl->cycles), 1, 0);
  const size_t half = (size_t)6 * nslots;
  if (t == 0) sh.P = P0;
  __syncthreads();
  const MdParams& P = sh.P;
  // lane l of bead b's 16
  constexpr int LL = RES_WG / RES_OWN, LE = MAXNBR / LL;
  const int b = t / LL, l = t % LL, first = t & 63 & ~(LL - 1), q = p0 + b;
  const bool on = b < n;
  const int slot = so + p0 + (on ? b : 0);
  const bool star = !RIGID && ng > RES_ALL;
  auto lose = [&](int at) {
    res_give_up(word, ng);
    sh.lost[at] = 1;
  };

  bool fin = true;
  if (RIGID) {
    double r3[3] = {0.0, 0.0, 0.0}, v3[3] = {0.0, 0.0, 0.0};
    if (t < nb)
      for (int a = 0; a < 3; ++a) { r3[a] = d.r[3 * (so + t) + a]; v3[a] = d.v[3 * (so + t) + a]; }
    fin = rig_open(rig, nb, P.hh, P.r0 * P.r0, r3, v3);
  }
  // lane c < 3 has component c of the bead's state
  const bool mine = on && l < 3;
  if (mine) {
    sh.pos[0][b][l] = RIGID ? rig.x[q][l] : d.rmid0[3 * slot + l];
    sh.v[b][l] = RIGID ? rig.v[q][l] : d.v[3 * slot + l];
    sh.J[b][l] = d.J[3 * slot + l];
    sh.u[b][l] = P.couple ? d.up[3 * slot + l] : 0.0;
  }
  // where the lists were built: the bead's, with RIGID bead t's
  if (mine && !RIGID) sh.ref[b][l] = d.ref[3 * slot + l];
  if (RIGID && t < nb)
    for (int a = 0; a < 3; ++a) rig.ref[t][a] = d.ref[3 * (so + t) + a];
  const int cnt = on ? d.ncnt[slot] : 0;
  // the lists as they are do not hold: not built, or cut short
  bool stale = d.rb[4 * rep] != 0u ||
               (cnt >= MAXNBR &&
                (__hip_atomic_load(&d.ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & E_NBRLIST));
  for (int k = l; k < MAXNBR; k += LL)
    sh.list[b][k] = !stale && k < cnt ? (uint16_t)(d.nbr[(size_t)slot * MAXNBR + k] - so) : WIDE_NONE;
  if (t < 2) { sh.bits[t] = 0u; sh.all[t] = 0u; sh.lost[t] = 0; }
  __syncthreads();
  // The lists' chain indices to places, and the remote partners, each once.
  auto places = [&](int at) {
    if (RIGID) return;
    sh.m.set[t] = 0u;
    __syncthreads();
    for (int k = l; on && k < MAXNBR; k += LL) {
      const int z = sh.list[b][k];
      if (z != WIDE_NONE && !(z >= p0 && z < seg.b)) atomicOr(&sh.m.set[z >> 5], 1u << (z & 31));
    }
    __syncthreads();
    uint32_t mine32 = sh.m.set[t];
    const int n32 = __builtin_popcount(mine32);
    int pre = n32;
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(pre, o, 64);
      if ((t & 63) >= o) pre += y;
    }
    if ((t & 63) == 63) sh.m.wsum[t >> 6] = pre;
    __syncthreads();
    pre -= n32;
    for (int k = 0; k < t >> 6; ++k) pre += sh.m.wsum[k];
    sh.m.pre[t] = pre;
    if (t == RES_WG - 1) {
      sh.nrem = min(pre + n32, WIDE_REM);
      if (pre + n32 > WIDE_REM) lose(at);
    }
    for (; mine32 && pre < WIDE_REM; mine32 &= mine32 - 1u) sh.rem[pre++] = (uint16_t)(32 * t + __builtin_ctz(mine32));
    __syncthreads();
    for (int k = l; on && k < MAXNBR; k += LL) {
      const int z = sh.list[b][k];
      if (z == WIDE_NONE) continue;
      const int o = sh.m.pre[z >> 5] + __builtin_popcount(sh.m.set[z >> 5] & ((1u << (z & 31)) - 1u));
      sh.list[b][k] = (uint16_t)(z >= p0 && z < seg.b ? z - p0 : WIDE_FAR + min(o, WIDE_REM - 1));
    }
    __syncthreads();
  };
  places(0);
  bool dead = false;
  int next = 0, nsync = 0;
  __builtin_amdgcn_s_setprio(2);
  for (int s = 0; s < end; ++s) {
    const int cb = s & 1;
    const bool kick = MTS && s % (Mb + 1) == 0, slow = !MTS || kick, sync = RIGID || s == next;
    const int sub = MTS ? s - s / (Mb + 1) - 1 : s;       // index of the sub-step (no kick)
    const uint64_t tag = tag0 + (uint64_t)s * RES_TAG;
    unsigned long long* ring = d.xring + (kick ? (2 + (nsync & 1)) * half : (cb ? half : 0));
    // the positions of the remote partners
    auto remote = [&](int at) {
      for (int k = t; k < sh.nrem; k += RES_WG) {
        double y[3];
        if (!res_poll_vec(ring + (size_t)(so + sh.rem[k]) * 6, tag, word, d.ctrl, wait, nseg, y)) { lose(at); break; }
        for (int a = 0; a < 3; ++a) sh.far[k][a] = y[a];
      }
    };
    // the position of any bead of the chain
    auto position = [&](int k, double* y) {
      if (RIGID || (k >= p0 && k < seg.b)) {
        const double* o = RIGID ? rig.x[k] : sh.pos[cb][k - p0];
        y[0] = o[0]; y[1] = o[1]; y[2] = o[2];
        return true;
      }
      return res_poll_vec(ring + (size_t)(so + k) * 6, tag, word, d.ctrl, wait, nseg, y);
    };
    // Bit 0: a bead is far from where the table binned it; bit 1: beyond the range
    // of the lists; bit 8 + k: at twice its present speed it may be, k sub-steps
    // from here.
    uint32_t bits = 0u;
    if (RIGID ? t < nb : on && l == 0 && slow) {
      const double* y = RIGID ? rig.x[t] : sh.pos[cb][b];
      const double* ref = RIGID ? rig.ref[t] : sh.ref[b];
      double f2 = 0.0;
      for (int a = 0; a < 3; ++a) { const double df = y[a] - ref[a]; f2 += df * df; }
      const bool held = f2 <= P.halfskin2;
      if (sync) {
        const double* rb = d.rbin + 3 * (size_t)(RIGID ? so + t : slot);
        double b2 = 0.0, v2 = 0.0;
        for (int a = 0; a < 3; ++a) {
          const double db = y[a] - rb[a], va = RIGID ? 0.0 : sh.v[b][a];
          b2 += db * db;
          v2 += va * va;
        }
        bits = (b2 <= CELL_MARGIN * CELL_MARGIN ? 0u : 1u) | (held ? 0u : 2u);
        if (!RIGID && !MTS) {
          const double k = (0.95 * sqrt(P.halfskin2) - sqrt(f2)) / (4.0 * P.hh * sqrt(v2));
          bits |= ((0xffffu << (k >= 16.0 ? 16 : (k >= 1.0 ? (int)k : 1))) & 0xffffu) << 8;
        }
      } else if (!held) {
        lose(cb);
      }
    }
    if (stale) bits |= 2u;
    if (RIGID) {
      // every segment has the whole chain, and finds the same
      if (bits) atomicOr(&sh.all[cb], bits);
      lds_barrier();
      if (t == 0) sh.all[cb ^ 1] = 0u;           // read before this barrier, written after the next
    } else {
      if (mine) {
        const unsigned long long w = (unsigned long long)__double_as_longlong(sh.pos[cb][b][l]);
        res_store(ring + ((size_t)slot * 3 + l) * 2, w);
        res_store(ring + ((size_t)slot * 3 + l) * 2 + 1, w ^ tag);
      }
      if (bits) atomicOr(&sh.bits[cb], bits);
      lds_barrier();
      const int sp = nsync & 1;
      unsigned long long* words = d.xflag + (size_t)2 * sp * nseg;
      if (t == 0) {
        if (sync) {
          const unsigned long long w = sh.bits[cb];
          res_store(words + 2 * seg.id, w);
          res_store(words + 2 * seg.id + 1, w ^ tag);
        }
        sh.bits[cb ^ 1] = 0u;
        sh.all[cb ^ 1] = 0u;
      }
      // the partners (of lists that may be replaced: the words are on their way
      // meanwhile), every segment's word, the chain beads at the segment's ends
      if (slow) remote(cb);
      if (sync) {
        uint32_t got = 0u;
        if (!star || p0 == 0)
          for (int k = t; k < (int)ng; k += RES_WG) {
            unsigned long long w = 0;
            if (!res_poll(words + 2 * (g0 + k), tag, word, d.ctrl, wait, nseg, w)) { lose(cb); break; }
            got |= (uint32_t)w;
          }
        if (star) {
          unsigned long long* sum = d.xflag + (size_t)6 * nseg + 2 * (g0 + sp);
          if (p0 == 0) {
            if (got) atomicOr(&sh.all[cb], got);
            lds_barrier();
            if (t == 0 && !sh.lost[cb]) {
              const unsigned long long w = sh.all[cb];
              res_store(sum, w);
              res_store(sum + 1, w ^ tag);
            }
          } else if (t == RES_WG / 2) {
            unsigned long long w = 0;
            if (!res_poll(sum, tag, word, d.ctrl, wait, nseg, w)) lose(cb);
            got = (uint32_t)w;
          }
        }
        if (got) atomicOr(&sh.all[cb], got);
      }
      const int h = t - (RES_WG - RES_HALO), c = h < 2 ? p0 - 2 + h : seg.b + (h - 2);
      if (!kick && h >= 0 && c >= 0 && c < nb) {
        double y[3];
        if (!res_poll_vec(ring + (size_t)(so + c) * 6, tag, word, d.ctrl, wait, nseg, y)) lose(cb);
        for (int a = 0; a < 3; ++a) sh.pos[cb][RES_OWN + h][a] = y[a];
      }
      lds_barrier();
    }
    const uint32_t all = sync ? sh.all[cb] : 0u;
    if (sh.lost[cb]) { dead = true; break; }     // uniform: next written after the barriers of the next stage
    if (sync) {
      // after new lists at once again: a segment that is no partner of this one
      // may not replace the positions that this one searches
      next = s + (MTS ? Mb + 1 : (all & 2u ? 1 : __builtin_ctz((all >> 8) | 0x10000u)));
      ++nsync;
    }
    double x[3] = {0.0, 0.0, 0.0};
    if (on)
      for (int a = 0; a < 3; ++a) x[a] = RIGID ? rig.x[q][a] : sh.pos[cb][b][a];
    if (all & 2u) {
      // ---- new lists, from the cell table where every bead is near its bucket
      auto partner = [&](int k, const double* y) {
        if (k == q) return;
        const double d0 = min_image(x[0] - y[0], g.nx);
        const double d1 = min_image(x[1] - y[1], g.ny);
        const double d2 = min_image(x[2] - y[2], g.nz);
        if (!(d0 * d0 + d1 * d1 + d2 * d2 < P.rlist2)) return;
        const int o = atomicAdd(&sh.h.ncand[b], 1);
        if (o < MAXNBR) sh.list[b][o] = (uint16_t)k;
      };
      bool ok = true;
      if (t < RES_OWN) sh.h.ncand[t] = 0;
      if (!(all & 1u)) {
        if (on) {
          int cell[3];
          bead_cell(R, x, cell);
          for (int k = l; k < 27; k += LL) {
            const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
            sh.h.bk[b][k] = cell_bucket(rep, (cell[0] + dx + R.ncell[0]) % R.ncell[0],
                                      (cell[1] + dy + R.ncell[1]) % R.ncell[1],
                                      (cell[2] + dz + R.ncell[2]) % R.ncell[2], d.cmask);
          }
        }
        __syncthreads();
        if (on)
          for (int k = l; k < 27 && ok; k += LL) {
            const uint32_t bk = sh.h.bk[b][k];
            bool dup = false;
            for (int k2 = 0; k2 < k; ++k2) dup = dup || sh.h.bk[b][k2] == bk;
            const int m = dup ? 0 : min(d.ccount[bk], CELL_CAP);
            for (int i = 0; i < m && ok; ++i) {
              const int sl = d.cbuf[(size_t)bk * CELL_CAP + i];
              if (d.slot_rep[sl] != rep) continue;
              double y[3];
              ok = position(sl - so, y);
              if (ok) partner(sl - so, y);
            }
          }
      } else {
        for (int base = 0; base < nb; base += RES_TILE) {
          const int m = min(RES_TILE, nb - base);
          __syncthreads();
          if (t < m && ok) {
            double y[3];
            ok = position(base + t, y);
            for (int a = 0; a < 3; ++a) sh.h.tile[t][a] = y[a];
          }
          __syncthreads();
          if (on)
            for (int k = l; k < m; k += LL) partner(base + k, sh.h.tile[k]);
        }
      }
      __syncthreads();
      if (on && sh.h.ncand[b] > MAXNBR) ok = false;  // the redo says so
      if (!ok) lose(cb ^ 1);
      const int found = on ? min(sh.h.ncand[b], MAXNBR) : 0;
      if (l == 0) {                              // ascending order
        uint16_t* L = sh.list[b];
        for (int k = 1; k < found; ++k) {
          const uint16_t w = L[k];
          int m = k;
          while (m > 0 && L[m - 1] > w) { L[m] = L[m - 1]; --m; }
          L[m] = w;
        }
      }
      for (int k = l; k < MAXNBR; k += LL)
        if (k >= found) sh.list[b][k] = WIDE_NONE;
      __syncthreads();
      places(cb ^ 1);
      if (mine && !RIGID) sh.ref[b][l] = sh.pos[cb][b][l];
      if (RIGID && t < nb)
        for (int a = 0; a < 3; ++a) rig.ref[t][a] = rig.x[t][a];
      stale = false;
      if (t == 0 && p0 == 0) {
        atomicAdd((unsigned long long*)&d.ctrl->rebuilds, 1ull);
        if (!(all & 1u)) atomicAdd((unsigned long long*)&d.ctrl->cell_rebuilds, 1ull);
      }
      if (!RIGID) remote(cb ^ 1);
      __syncthreads();
    }
    // ---- the sum in the fixed order, lane c < 3 component c: the terms come by
    // rounds of one per lane, those present in consecutive rows.  An absent term
    // is a zero (F is never -0, which a zero would change).
    double F = 0.0;
    double (*const row)[3] = sh.row[b];
    if (!kick) {
      wide_bonded<RIGID>(cb, n, q, nb);
      wave_lds();
      if (l < 3)
        for (int k = 0; k < 5; ++k) F += row[k][l];
      wave_lds();
    }
    auto add = [&](bool in, double d0, double d1, double d2) {
      const uint64_t any = __ballot(in);
      if (any == 0) return;
      const uint32_t mask = (uint32_t)(any >> first) & ((1u << LL) - 1u);
      if (in) {
        double Fp[3] = {0.0, 0.0, 0.0};
        lj_add(P, d0, d1, d2, Fp);
        double* o = row[__builtin_popcount(mask & ((1u << l) - 1u))];
        o[0] = Fp[0]; o[1] = Fp[1]; o[2] = Fp[2];
      }
      wave_lds();
      const int rows = __builtin_popcount(mask);
      if (l < 3)
        for (int k = 0; k < rows; k += 4) {      // four loads in flight
          const double f0 = row[k][l], f1 = row[min(k + 1, LL - 1)][l], f2 = row[min(k + 2, LL - 1)][l],
                       f3 = row[min(k + 3, LL - 1)][l];
          F += f0;
          if (k + 1 < rows) F += f1;
          if (k + 2 < rows) F += f2;
          if (k + 3 < rows) F += f3;
        }
      wave_lds();
    };
    if (slow) {
      for (int m = 0; m < LE; ++m) {
        const int k = sh.list[b][LL * m + l];
        const bool in = on && k != WIDE_NONE;
        if (!__any(in)) break;                   // lists are filled from the front
        const int z = in ? k : 0;
        const double* y = RIGID ? rig.x[z] : (z < WIDE_FAR ? sh.pos[cb][z] : sh.far[z - WIDE_FAR]);
        const double d0 = min_image(x[0] - y[0], g.nx);
        const double d1 = min_image(x[1] - y[1], g.ny);
        const double d2 = min_image(x[2] - y[2], g.nz);
        add(in && d0 * d0 + d1 * d1 + d2 * d2 < P.rc2, d0, d1, d2);
      }
      // the sites of wall_row, a lane each, in their order
      bool near = false;
      int off = 0;
      const int wa = g.wall_axis, na = wa >= 0 ? ext(g, wa) : 0, n0 = wa == 0 ? g.ny : g.nx, n1 = wa == 2 ? g.ny : g.nz;
      double wn = 0.0, wt0 = 0.0, wt1 = 0.0;
      if (on && wa >= 0) {
        wn = wrapc(sel3(wa, x[0], x[1], x[2]), na);
        off = g.wall_pos - (int)floor(wn);
        if (off < WLO) off += na;
        if (off > WHI) off -= na;
        near = off >= P.wlo && off <= P.whi;
      }
      if (__any(near)) {
        wt0 = wrapc(wa == 0 ? x[1] : x[0], n0);
        wt1 = wrapc(wa == 2 ? x[1] : x[2], n1);
        const int nw = P.whi - P.wlo + 1;
        for (int k0 = 0; k0 < nw * nw; k0 += LL) {
          const int k = k0 + l, u1 = (int)floor(wt1) + P.wlo + k / nw, u0 = (int)floor(wt0) + P.wlo + k % nw;
          const int v1 = u1 < 0 ? u1 + n1 : (u1 >= n1 ? u1 - n1 : u1);
          const int v0 = u0 < 0 ? u0 + n0 : (u0 >= n0 ? u0 - n0 : u0);
          const bool pore = v1 >= g.lo1 && v1 <= g.hi1 && v0 >= g.lo0 && v0 <= g.hi0;
          const double dn = wn - (double)((int)floor(wn) + off), dt0 = wt0 - (double)u0, dt1 = wt1 - (double)u1;
          const double d0 = wa == 0 ? dn : dt0, d1 = wa == 1 ? dn : (wa == 0 ? dt0 : dt1), d2 = wa == 2 ? dn : dt1;
          add(near && k < nw * nw && !pore && d0 * d0 + d1 * d1 + d2 * d2 < P.rc2, d0, d1, d2);
        }
        if (near && P.field_on && l == wa && in_field(g, x)) F += P.f_drive;
      }
    }
    if (d.mdtape && mine) {
      double* tp = d.mdtape + ((size_t)s * nb + q) * 6 + l;
      tp[0] = sh.pos[cb][b][l];
      tp[3] = sh.v[b][l];
    }
    const bool last = s == end - 1;
    double xc = 0.0, v = 0.0;
    if (mine) {
      xc = RIGID ? rig.x[q][l] : sh.pos[cb][b][l];
      v = sh.v[b][l];
    }
    if (kick) {
      v = v + P.kick * F;
      if (s > 0 && !last) v = v + P.kick * F;
      fin = fin && isfinite(v) && isfinite(xc);
      if (!last) xc = xc + P.hh * v;
    } else {
      const double xi = mine && P.sig != 0.0 ? d.xi[(size_t)3 * ((size_t)sub * nslots + slot) + l] : 0.0;
      const double sx = P.sig * xi;
      const double u = mine ? sh.u[b][l] : 0.0, vn = P.e * v + P.cf * (F + P.gamma * u) + sx;
      if (mine) sh.J[b][l] = sh.J[b][l] - P.m * (P.omE * (u - v) + sx);
      v = vn;
      fin = fin && isfinite(vn);
      const double re = xc + P.hh * vn;
      xc = (MTS ? (s + 1) % (Mb + 1) == 0 : last) ? re : re + P.hh * vn;   // a kick takes r itself
    }
    if (!RIGID) {
      if (mine) { sh.pos[cb ^ 1][b][l] = xc; sh.v[b][l] = v; }
      wave_lds();                                // lane 0 looks at them before the next barrier
      continue;
    }
    // ---- rigid bonds: the chain's kicked velocities, its projections
    const uint64_t next = tag + RES_TAG;
    if (mine) {
      const unsigned long long w = (unsigned long long)__double_as_longlong(v);
      rig.v[q][l] = v;
      res_store(ring + ((size_t)slot * 3 + l) * 2, w);
      res_store(ring + ((size_t)slot * 3 + l) * 2 + 1, w ^ next);
    }
    if (t < nb && !(t >= p0 && t < seg.b)) {
      double y[3];
      if (!res_poll_vec(ring + (size_t)(so + t) * 6, next, word, d.ctrl, wait, nseg, y)) lose(cb ^ 1);
      for (int a = 0; a < 3; ++a) rig.v[t][a] = y[a];
    }
    __syncthreads();
    if (sh.lost[cb ^ 1]) { dead = true; break; }
    fin = rig_step(rig, nb, P.hh, P.r0 * P.r0, last) && fin;
    if (mine) sh.v[b][l] = rig.v[q][l];
  }
  __builtin_amdgcn_s_setprio(0);
  __syncthreads();
  if (t == 0) sh.done = res_close(word, ng, dead || sh.lost[0] || sh.lost[1], wait);
  __syncthreads();
  if (!sh.done) return false;
  if (mine) {
    d.r[3 * slot + l] = RIGID ? rig.x[q][l] : sh.pos[end & 1][b][l];
    d.v[3 * slot + l] = sh.v[b][l];
    d.J[3 * slot + l] = sh.J[b][l];
    if (!fin) atomicOr(&d.ctrl->err, E_BEADS);
  }
  return true;
}

struct ResArgs {
  Dev d;
  double* ang;
  const FusedSeg* segs;
  int nslots, nseg, n_sub, mts;
  MdOverride ov;
  uint64_t wait;
};

// What follows a failed first pass.  Out of line: inlined, its registers
// spill in the first pass (0.27 against 0.23 ms per step on 32^3).  a: the
// kernel's arguments in memory, so that none is copied for this call.
// A function's argument arrives in vector registers; this one is the same in all
// lanes, and what is read through it then too.
__device__ inline const ResArgs* res_args(const ResArgs* a) {
  const uint64_t p = (uint64_t)(uintptr_t)a;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  return (const ResArgs*)(uintptr_t)((uint64_t)hi << 32 | lo);
}
// What the wide pass uses of the arguments.
__device__ inline Dev res_dev(const Dev* a) {
  Dev d{};
  d.reps = load_global(&a->reps);
  d.r = load_global(&a->r); d.v = load_global(&a->v); d.up = load_global(&a->up); d.J = load_global(&a->J);
  d.slot_rep = load_global(&a->slot_rep);
  d.nbr = load_global(&a->nbr); d.ncnt = load_global(&a->ncnt); d.ref = load_global(&a->ref);
  d.rmid0 = load_global(&a->rmid0); d.rb = load_global(&a->rb); d.xi = load_global(&a->xi);
  d.mdtape = load_global(&a->mdtape);
  d.ccount = load_global(&a->ccount); d.cbuf = load_global(&a->cbuf); d.rbin = load_global(&a->rbin);
  d.cmask = load_uniform(&a->cmask);
  d.xring = load_global(&a->xring); d.xflag = load_global(&a->xflag); d.rsync = load_global(&a->rsync);
  d.ctrl = load_global(&a->ctrl);
  return d;
}
template <bool MTS, bool RIGID>
__device__ __attribute__((noinline)) void res_redo(const ResArgs* args) {
  const ResArgs* a = res_args(args);
  WideShared& sh = *reinterpret_cast<WideShared*>(res_lds + res_base(RIGID));
  RigShared& rig = *reinterpret_cast<RigShared*>(res_lds);   // RIGID
  const FusedSeg seg = load_uniform(&load_global(&a->segs)[blockIdx.x]);
  const Rep& R = a->d.reps[seg.rep];
  const MdParams P = md_override(load_uniform(&R.mp), a->ov);
  if (threadIdx.x == 0) atomicAdd((unsigned long long*)&a->d.ctrl->res_redone, 1ull);
  md_redo<RES_WG, MTS, RIGID>(a->d, R, P, seg.rep, a->ang, a->nslots, 0, a->n_sub, a->mts, &rig, sh.near, sh.off);
}
template <bool MTS, bool OWN, bool RIGID>
__device__ __attribute__((noinline)) void res_rescue(const ResArgs* args) {
  const ResArgs* a = res_args(args);
  WideShared& sh = *reinterpret_cast<WideShared*>(res_lds + res_base(RIGID));
  const Dev d = res_dev(&a->d);
  const FusedSeg seg = load_uniform(&load_global(&a->segs)[blockIdx.x]);
  const Rep& R = d.reps[seg.rep];
  const MdParams P = md_override(load_uniform(&R.mp), load_uniform(&a->ov));
  RigShared& rig = *reinterpret_cast<RigShared*>(res_lds);   // RIGID
  if (res_wide<MTS, RIGID>(d, seg, R, P, sh, rig, load_uniform(&a->nslots), load_uniform(&a->nseg), load_uniform(&a->n_sub),
                           load_uniform(&a->mts), load_uniform(&a->wait))) return;
  // The redo stores the state, the positions and the lists that every segment's
  // passes start from, and one of them may not have begun (it finds no room while
  // another context's cycle has its place): so the segment that leaves last
  // goes on.  Nobody waits.  The segments' stores (the adjoint's tape) are
  // released before they count themselves, so that the redo's come after them.
  const uint32_t ng = (uint32_t)((P.nb + RES_OWN - 1) / RES_OWN);
  __syncthreads();
  if (threadIdx.x == 0)
    sh.done = __hip_atomic_fetch_add(&d.rsync[3 * seg.rep + 2], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u == ng;
  __syncthreads();
  if (sh.done) res_redo<MTS, RIGID>(a);
}

// OWN: a workgroup takes the registers of a whole CU (8 waves of 256), so that
// no wave of the sweep shares it; else three fit beside each other.
template <bool MTS, bool OWN, bool RIGID>
__global__ __launch_bounds__(RES_WG, OWN ? 2 : 6) void k_md_resident(ResArgs a) {
  if (OWN) asm volatile("" ::: "v255");
  ResShared& sh = *reinterpret_cast<ResShared*>(res_lds + res_base(RIGID));
  const FusedSeg seg = load_uniform(&a.segs[blockIdx.x]);
  if (seg.rep < 0) return;                       // fills the table (see res_place)
  const Rep& R = a.d.reps[seg.rep];
  const MdParams P = md_override(load_uniform(&R.mp), a.ov);
  RigShared& rig = *reinterpret_cast<RigShared*>(res_lds);   // RIGID
  if (__builtin_expect(res_pass<MTS, RIGID>(a.d, seg, R, P, sh, rig, a.nslots, a.nseg, a.n_sub, a.mts, a.wait), 1)) return;
  __syncthreads();                               // sh.done is read
  res_rescue<MTS, OWN, RIGID>((const ResArgs*)__builtin_amdgcn_kernarg_segment_ptr());
}

void launch_md_cycle_fused(const Dev& d, const FusedBufs& fb, int nseg, int nslots, int nrep, int n_sub, int K,
                           hipStream_t s) {
  if (nslots <= 0 || n_sub <= 0 || nseg <= 0) return;
  const int M = n_sub / K;
  for (int j = 0; j < M; ++j)
    hipLaunchKernelGGL(k_md_fused, dim3((unsigned)nseg), dim3(FU_WG), 0, s, d, fb, nslots, j * K, K,
                       j == M - 1 ? 1 : 0, j & 1);
  hipLaunchKernelGGL(k_md_redo, dim3((unsigned)nrep), dim3(RD_WG), 0, s, d, fb, fb.ang, nslots, n_sub, K);
}

// Holds the stream until the resident cycle's nseg workgroups run (they never
// wait for this stream), at most RES_GATE ticks of the 100 MHz clock: 0.3 ms.
constexpr uint64_t RES_GATE = 30000;
__global__ void k_md_gate(const Ctrl* ctrl, uint32_t nseg) {
  const uint64_t t0 = wall_clock64();
  while (__hip_atomic_load(&ctrl->placed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < nseg &&
         wall_clock64() - t0 < RES_GATE)
    __builtin_amdgcn_s_sleep(8);
}
void launch_md_gate(const Dev& d, int nseg, hipStream_t s) {
  hipLaunchKernelGGL(k_md_gate, dim3(1), dim3(1), 0, s, d.ctrl, (uint32_t)nseg);
}

void launch_md_cycle_resident(const Dev& d, double* ang, const FusedSeg* seg, int ntab, int nseg, int nslots, int n_sub,
                              int mts, const MdOverride& ov, uint64_t wait, bool own, bool rigid, hipStream_t s) {
  if (nslots <= 0 || n_sub <= 0 || nseg <= 0 || ntab < nseg) return;
  const auto k = rigid ? k_md_resident<false, true, true>
                       : (mts > 0 ? (own ? k_md_resident<true, true, false> : k_md_resident<true, false, false>)
                                  : (own ? k_md_resident<false, true, false> : k_md_resident<false, false, false>));
  hipLaunchKernelGGL(k, dim3((unsigned)ntab), dim3(RES_WG), res_bytes(rigid), s,
                     (ResArgs{d, ang, seg, nslots, nseg, n_sub, mts, ov, wait}));
}

void launch_md_noise(const Dev& d, int nslots, int n_sub, int step_offset, hipStream_t s) {
  long nk = (long)n_sub * nslots;
  if (nk > 0)
    hipLaunchKernelGGL(k_md_noise, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, s, d, nslots, n_sub,
                       step_offset);
}

void launch_zero_v(const Dev& d, int nslots, hipStream_t s) {
  if (nslots > 0) hipLaunchKernelGGL(k_zero_v, dim3((3 * nslots + 255) / 256), dim3(256), 0, s, d.v, 3 * nslots);
}

}  // namespace lbmd
