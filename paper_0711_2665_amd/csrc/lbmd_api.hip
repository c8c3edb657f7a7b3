// lbmd_api.hip -- host side of liblbmd: argument checking, geometry, buffer
// layout and the sequence of kernel launches of each entry point declared in
// include/lbmd.h.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "lbmd.h"
#include "lbmd_kernels.h"

using namespace lbmd;

// Partial sums of lb_observables_static's fluid reduction (4 doubles per
// reduction tile of OBS_TILE nodes): device memory the library reserves for
// callers that cannot allocate.  Each GPU holds its own copy for the life of
// the process; its address is resolved once per device (static_scratch).
constexpr int STATIC_OBS_TILES = 16384;     // packed lattices of up to 16384 x OBS_TILE = 67,108,864 nodes
static __device__ __align__(256) double scratch[4 * STATIC_OBS_TILES];

namespace {

thread_local std::string g_last_error = "no error";

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

int take_acc(const char* where);
int check_hip(const char* where) {
  int rc = take_acc(where);
  if (rc) return rc;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "%s: %s", where, hipGetErrorString(e));
  return LB_OK;
}

// First failure among a sequence of asynchronous HIP calls.
thread_local hipError_t g_acc = hipSuccess;
inline void acc(hipError_t e) {
  if (e != hipSuccess && g_acc == hipSuccess) g_acc = e;
}
int take_acc(const char* where) {
  hipError_t e = g_acc;
  g_acc = hipSuccess;
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "%s: %s", where, hipGetErrorString(e));
  return LB_OK;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline long round_up(long x, long m) { return (x + m - 1) / m * m; }

constexpr int NODE_ALIGN = 64;      // replica node offsets are multiples of this

// Packing of R replicas into one buffer set (see lbmd_kernels.h).
struct Packing {
  std::vector<long> node_off;       // per replica
  std::vector<int> slot_off;        // per replica
  long nodes = 0;                   // total packed nodes
  int slots = 0;                    // total bead slots
  int slots_alloc = 1;              // slots, at least 1 (array sizing)
  long sweep_tiles_max = 0;         // tiles of the sweep at TILE_MIN
  long obs_tiles = 0;
  long wl_blocks_max = 0;           // wall-link list blocks (LEDGER_BLOCK entries each), upper bound
  int nseg = 0;                     // chain segments of the fused sub-cycle (FUSED_OWN beads each)
  int nrseg = 0;                    // chain segments of the resident sub-cycle (RES_OWN beads each)
};

// Fluid nodes with a solid upstream neighbour lie in the three planes around
// the wall (|c_i| <= 1 along the normal), so their count is at most three
// plane areas.
long wall_link_bound(const lb_desc& d) {
  if (d.wall_axis < 0) return 0;
  const long area = (long)d.nx * d.ny * d.nz / (d.wall_axis == 0 ? d.nx : (d.wall_axis == 1 ? d.ny : d.nz));
  return 3 * area;
}

Packing packing(const lb_desc* d, int nrep) {
  Packing pk;
  for (int r = 0; r < nrep; ++r) {
    long N = (long)d[r].nx * d[r].ny * d[r].nz;
    pk.node_off.push_back(pk.nodes);
    pk.slot_off.push_back(pk.slots);
    pk.nodes += round_up(N, NODE_ALIGN);
    pk.slots += (int)round_up(d[r].nb, MD_BPB);
    pk.sweep_tiles_max += (N + TILE_MIN - 1) / TILE_MIN;
    pk.obs_tiles += (N + OBS_TILE - 1) / OBS_TILE;
    pk.wl_blocks_max += (wall_link_bound(d[r]) + LEDGER_BLOCK - 1) / LEDGER_BLOCK;
    pk.nseg += (d[r].nb + FUSED_OWN - 1) / FUSED_OWN;
    pk.nrseg += (d[r].nb + RES_OWN - 1) / RES_OWN;
  }
  pk.slots_alloc = pk.slots > 0 ? pk.slots : 1;
  return pk;
}

// slots of the exchange memory (without a resident cycle its first holds velocities)
int xring_slots(const Packing& pk) { return pk.nrseg <= RES_MAX_WG ? XRING : 1; }

struct WorkLayout {
  size_t ctrl, reps, tiles, otiles, slot_rep, head, next, base, touched, nbr, ncnt, rb, rmid0, rmid1, ref, part, xi,
      tX, ccount, cbuf, rbin, cst, wlinks, ledger, lpart, lcount, lsp, fseg, rmS, vS, JS, fang, redo, rseg, xring, xflag, rsync;
  size_t nbuckets;
  size_t total;
};

// The table of the resident sub-cycle: entry b is the segment of workgroup b, or
// one with rep = -1.  Workgroups go to the XCDs in turn, so entries b with the
// same b % XCDS share one: chains of up to RES_XCD segments take one XCD
// (the least loaded, from one that depends on the seed, so that contexts side
// by side choose different ones), longer ones every XCD in runs of neighbours.
std::vector<FusedSeg> res_place(const lb_desc* d, int nrep, const Packing& pk) {
  std::vector<FusedSeg> out;
  if (pk.nrseg <= 0 || pk.nrseg > RES_MAX_WG) return out;
  std::vector<FusedSeg> bin[XCDS];
  std::vector<int> order(nrep), first(nrep);
  for (int r = 0, id = 0; r < nrep; ++r) {
    order[r] = r;
    first[r] = id;
    id += (d[r].nb + RES_OWN - 1) / RES_OWN;
  }
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return d[a].nb > d[b].nb; });
  const int start = pk.nrseg > 1 ? (int)(((uint32_t)d[0].seed * 2654435761u) >> 29) : 0;
  for (int r : order) {
    const int ng = (d[r].nb + RES_OWN - 1) / RES_OWN;
    int least = start;
    for (int k = 1; k < XCDS; ++k)
      if (bin[(start + k) % XCDS].size() < bin[least].size()) least = (start + k) % XCDS;
    for (int g = 0; g < ng; ++g)
      bin[ng > RES_XCD ? (int)((long)g * XCDS / ng) : least].push_back(
          FusedSeg{r, g * RES_OWN, std::min((g + 1) * RES_OWN, (int)d[r].nb), first[r] + g});
  }
  size_t rows = 0;
  for (const auto& b : bin) rows = std::max(rows, b.size());
  out.assign(rows * XCDS, FusedSeg{-1, 0, 0, 0});
  for (int x = 0; x < XCDS; ++x)
    for (size_t k = 0; k < bin[x].size(); ++k) out[k * XCDS + x] = bin[x][k];
  while (out.back().rep < 0) out.pop_back();
  return out;
}

WorkLayout work_layout(const lb_desc* d, int nrep, const Packing& pk) {
  WorkLayout w;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += align256(bytes); return at; };
  const size_t ns = (size_t)pk.slots_alloc;
  const size_t R = (size_t)nrep;
  w.ctrl = take(sizeof(Ctrl));
  w.reps = take(sizeof(Rep) * R);
  w.tiles = take(sizeof(Tile) * (size_t)pk.sweep_tiles_max);
  w.otiles = take(sizeof(Tile) * (size_t)pk.obs_tiles);
  w.slot_rep = take(sizeof(int) * ns);
  w.head = take(sizeof(int) * (size_t)pk.nodes);
  w.next = take(sizeof(int) * ns);
  w.base = take(sizeof(int) * ns);
  w.touched = take(sizeof(int2) * 8 * ns);
  w.nbr = take(sizeof(int) * MAXNBR * ns);
  w.ncnt = take(sizeof(int) * ns);
  w.rb = take(sizeof(uint32_t) * 4 * R);
  w.rmid0 = take(sizeof(double) * 3 * ns);
  w.rmid1 = take(sizeof(double) * 3 * ns);
  w.ref = take(sizeof(double) * 3 * ns);
  w.part = take(sizeof(double) * 4 * (size_t)pk.obs_tiles);
  w.xi = take(sizeof(double) * 3 * ns * (size_t)d[0].n_sub * 2);   // two sub-cycles: this step's and the next
  w.tX = take(sizeof(int64_t) * R);
  w.nbuckets = 64;
  while (w.nbuckets < 2 * ns) w.nbuckets *= 2;
  w.ccount = take(sizeof(int) * w.nbuckets);
  w.cbuf = take(sizeof(int) * CELL_CAP * w.nbuckets);
  w.rbin = take(sizeof(double) * 3 * ns);
  w.cst = take(sizeof(uint32_t) * 4 * R);
  w.wlinks = take(sizeof(WallLink) * LEDGER_BLOCK * (size_t)pk.wl_blocks_max);
  w.ledger = take(sizeof(double) * NLEDGER * R);
  w.lpart = take(sizeof(double) * 3 * (size_t)(pk.wl_blocks_max > 0 ? pk.wl_blocks_max : 1));
  w.lcount = take(sizeof(uint32_t) * R);
  w.lsp = take(sizeof(double) * 3 * ns);
  w.fseg = take(sizeof(FusedSeg) * (size_t)(pk.nseg > 0 ? pk.nseg : 1));
  w.rmS = take(sizeof(double) * 3 * ns);
  w.vS = take(sizeof(double) * 3 * ns);
  w.JS = take(sizeof(double) * 3 * ns);
  w.fang = take(sizeof(double) * 9 * ns);
  w.redo = take(sizeof(int) * R);
  w.rsync = take(sizeof(uint32_t) * 3 * R);
  w.rseg = take(sizeof(FusedSeg) * std::max<size_t>(res_place(d, nrep, pk).size(), 1));
  w.xring = take(sizeof(uint64_t) * xring_slots(pk) * 2 * 3 * ns);
  w.xflag = take(sizeof(uint64_t) * XFLAG * 2 * (size_t)(pk.nrseg > 0 ? pk.nrseg : 1));
  w.total = o;
  return w;
}

size_t elem_size(const lb_desc* d) { return d->precision == LB_FP64 ? sizeof(double) : sizeof(float); }

// Byte layout of the state buffer: populations, then r and v of every slot,
// then the step counter, then the per-replica translocation steps.
struct StateLayout {
  size_t pops, r, v, step, tX, ledger, total;
};
StateLayout state_layout(const lb_desc* d, int nrep, const Packing& pk) {
  StateLayout s;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += align256(bytes); return at; };
  s.pops = take(elem_size(d) * Q * (size_t)pk.nodes);
  s.r = take(sizeof(double) * 3 * (size_t)pk.slots_alloc);
  s.v = take(sizeof(double) * 3 * (size_t)pk.slots_alloc);
  s.step = take(sizeof(uint64_t));
  s.tX = take(sizeof(int64_t) * (size_t)nrep);
  s.ledger = take(sizeof(double) * NLEDGER * (size_t)nrep);
  s.total = o;
  return s;
}

int validate_one(const lb_desc* d, int r) {
  if (d->nx <= 0 || d->ny <= 0 || d->nz <= 0) return fail(LB_ERR_ARG, "replica %d: extents must be positive", r);
  long N = (long)d->nx * d->ny * d->nz;
  if (N * (long)Q > 2147483647L) return fail(LB_ERR_ARG, "replica %d: lattice too large: 19 N must fit in 31 bits", r);
  if (d->precision != LB_FP64 && d->precision != LB_FP32_DEV)
    return fail(LB_ERR_ARG, "replica %d: unknown precision %d", r, d->precision);
  if (!(d->tau > 0.5)) return fail(LB_ERR_ARG, "replica %d: tau must exceed 1/2 (got %g)", r, d->tau);
  for (int a = 0; a < 3; ++a)
    if (!std::isfinite(d->g[a])) return fail(LB_ERR_ARG, "replica %d: body force must be finite", r);
  if (d->wall_axis < -1 || d->wall_axis > 2) return fail(LB_ERR_ARG, "replica %d: wall_axis must be -1, 0, 1 or 2", r);
  if (d->wall_axis >= 0) {
    int n = d->wall_axis == 0 ? d->nx : (d->wall_axis == 1 ? d->ny : d->nz);
    if (d->wall_pos < 2 || d->wall_pos > n - 3) return fail(LB_ERR_ARG, "replica %d: wall plane must lie in [2, n-3]", r);
    int t0 = d->wall_axis == 0 ? d->ny : d->nx;
    int t1 = d->wall_axis == 2 ? d->ny : d->nz;
    if (d->pore_h < 0 || d->pore_h > t0 || d->pore_h > t1) return fail(LB_ERR_ARG, "replica %d: pore wider than the wall", r);
  }
  if (!(d->fluid_kT >= 0.0) || !std::isfinite(d->fluid_kT))
    return fail(LB_ERR_ARG, "replica %d: fluid_kT must be finite and >= 0", r);
  if (d->nb < 0) return fail(LB_ERR_ARG, "replica %d: negative bead count", r);
  if (d->n_sub < 1) return fail(LB_ERR_ARG, "replica %d: n_sub must be >= 1", r);
  if (d->mts_outer < 0) return fail(LB_ERR_ARG, "replica %d: mts_outer must be >= 0", r);
  if (d->coupling != LB_COUPLING_TRILINEAR && d->coupling != LB_COUPLING_NGP)
    return fail(LB_ERR_ARG, "replica %d: unknown coupling %d", r, d->coupling);
  if (d->constraints != 0 && d->constraints != 1)
    return fail(LB_ERR_ARG, "replica %d: constraints must be 0 or 1", r);
  if (d->constraints == 1 && (d->mts_outer != 0 || d->nb > MAX_CONSTRAINED_BEADS))
    return fail(LB_ERR_ARG, "replica %d: rigid bonds need the uniform sub-cycle and at most %d beads", r,
                MAX_CONSTRAINED_BEADS);
  if (d->mts_outer > 0 && (d->n_sub % d->mts_outer != 0 || d->n_sub / d->mts_outer > MTS_MAX_INNER))
    return fail(LB_ERR_ARG, "replica %d: mts_outer must divide n_sub into at most %d sub-steps per outer step", r,
                MTS_MAX_INNER);
  if (d->nb > 0) {
    if (!(d->mass > 0.0)) return fail(LB_ERR_ARG, "replica %d: bead mass must be positive", r);
    if (!(d->gamma >= 0.0) || !(d->kT >= 0.0)) return fail(LB_ERR_ARG, "replica %d: gamma and kT must be >= 0", r);
    if (d->gamma > 0.0 && d->mass != 1.0)
      return fail(LB_ERR_ARG, "replica %d: a chain coupled with gamma > 0 needs mass 1 (the kick's drift towards the "
                              "fluid is (1 - e) u / m, while the impulse the fluid takes is m (1 - e)(u - v))", r);
    if (!(d->rc > 0.0) || d->rc > 3.0) return fail(LB_ERR_ARG, "replica %d: rc must lie in (0, 3]", r);
    if (!(d->sigma > 0.0)) return fail(LB_ERR_ARG, "replica %d: sigma must be positive", r);
    if ((long)d->nb > (1L << 24)) return fail(LB_ERR_ARG, "replica %d: too many beads", r);
    if (d->wall_axis >= 0 && (d->nx < 6 || d->ny < 6 || d->nz < 6))
      return fail(LB_ERR_ARG, "replica %d: a wall with beads needs extents >= 6", r);
  }
  return LB_OK;
}

int validate(const lb_desc* d, int nrep) {
  if (!d) return fail(LB_ERR_ARG, "null description");
  if (nrep < 1 || nrep > MAX_REPLICAS) return fail(LB_ERR_ARG, "replica count must lie in [1, %d]", MAX_REPLICAS);
  long nodes = 0, slots = 0;
  for (int r = 0; r < nrep; ++r) {
    int rc = validate_one(&d[r], r);
    if (rc) return rc;
    if (d[r].precision != d[0].precision) return fail(LB_ERR_ARG, "replica %d: all replicas need one precision", r);
    if (d[r].n_sub != d[0].n_sub) return fail(LB_ERR_ARG, "replica %d: all replicas need one n_sub", r);
    if (d[r].mts_outer != d[0].mts_outer) return fail(LB_ERR_ARG, "replica %d: all replicas need one mts_outer", r);
    nodes += round_up((long)d[r].nx * d[r].ny * d[r].nz, NODE_ALIGN);
    slots += round_up(d[r].nb, MD_BPB);
  }
  if (nodes * (long)Q > 2147483647L * 8L) return fail(LB_ERR_ARG, "ensemble too large");
  if (slots * 8L > 2147483647L / 8) return fail(LB_ERR_ARG, "too many beads in the ensemble");
  return LB_OK;
}

Geom make_geom(const lb_desc* d) {
  Geom g;
  g.nx = d->nx; g.ny = d->ny; g.nz = d->nz;
  g.nxy = d->nx * d->ny;
  g.N = (long)d->nx * d->ny * d->nz;
  g.wall_axis = d->wall_axis;
  g.wall_pos = d->wall_pos;
  g.t0 = d->wall_axis == 0 ? 1 : 0;
  g.t1 = d->wall_axis == 2 ? 1 : 2;
  if (d->wall_axis < 0) { g.t0 = 0; g.t1 = 1; }
  g.ngp = d->coupling == LB_COUPLING_NGP ? 1 : 0;
  int n0 = ext(g, g.t0), n1 = ext(g, g.t1);
  g.lo0 = n0 / 2 - d->pore_h / 2; g.hi0 = g.lo0 + d->pore_h - 1;
  g.lo1 = n1 / 2 - d->pore_h / 2; g.hi1 = g.lo1 + d->pore_h - 1;
  return g;
}

// SPV coefficients for friction rate gamma and thermal energy kT.
void spv_coefficients(MdParams& P, double gamma, double kT, double h) {
  P.gamma = gamma;
  if (gamma == 0.0) {
    P.e = 1.0; P.omE = 0.0; P.cf = h / P.m; P.sig = 0.0;
    return;
  }
  P.e = std::exp(-(gamma * h));
  P.omE = 1.0 - P.e;
  P.cf = P.omE / (P.m * gamma);
  double var = (kT / P.m) * (1.0 - P.e * P.e);
  P.sig = kT > 0.0 ? std::sqrt(var) : 0.0;
}

MdParams make_md(const lb_desc* d, double skin) {
  MdParams P;
  std::memset(&P, 0, sizeof(P));
  P.nb = d->nb;
  P.n_sub = d->n_sub;
  double h = 1.0 / (double)d->n_sub;
  P.hh = 0.5 * h;
  P.m = d->nb > 0 ? d->mass : 1.0;
  P.k_bond = d->k_bond; P.r0 = d->r0; P.kappa = d->kappa;
  P.eps24 = 24.0 * d->eps; P.sig2 = d->sigma * d->sigma; P.rc2 = d->rc * d->rc;
  P.f_drive = d->f_drive;
  P.couple = 1; P.field_on = 1;
  P.seed = d->seed; P.replica = d->replica;
  P.rlist2 = (d->rc + skin) * (d->rc + skin);
  P.halfskin2 = (0.5 * skin) * (0.5 * skin);
  spv_coefficients(P, d->gamma, d->kT, h);
  P.kick = d->mts_outer > 0 ? 0.5 * (1.0 / (double)d->mts_outer) / P.m : 0.0;
  const int cr = d->rc > 2.0 ? 3 : 2;       // ceil(rc) for 1 < rc <= 3 (rc <= 1: the 2-window still covers it)
  P.wlo = 1 - cr;
  P.whi = cr;
  P.constrained = d->constraints == 1 ? 1 : 0;
  return P;
}

// Noise amplitudes of the fluctuating fluid: mode k (4..18) receives
// sqrt(rho mu_k) r with mu_k = 3 kT (1 - (1 - omega)^2) / b_k, b_k =
// sum_i w_i e_ki^2 (fluctuation-dissipation for a mode relaxed by the
// factor 1 - omega each step, at c_s^2 = 1/3).
void fluid_noise_params(LbParams& lp, const lb_desc& d) {
  lp.fluct = d.fluid_kT > 0.0 ? 1 : 0;
  lp.fseed = d.seed;
  lp.frep = d.replica;
  const double keep = 1.0 - lp.omega;
  for (int k = 4; k < Q; ++k) {
    double b = 0.0;
    for (int i = 0; i < Q; ++i) b += wgt(i) * (double)(mode_coef(k, i) * mode_coef(k, i));
    const double a = lp.fluct ? std::sqrt(3.0 * d.fluid_kT * (1.0 - keep * keep) / b) : 0.0;
    lp.famp[k - 4] = a;
    lp.famp32[k - 4] = (float)a;
  }
}

// Solid / near-wall flags of one replica (Sec. 4: wall plane with a square
// pore); returns the number of fluid nodes.  Appends the replica's fluid
// nodes with solid upstream neighbours, in node order, to links.
long build_flags(const Geom& g, uint8_t* fl, int rep, std::vector<WallLink>& links) {
  long nfluid = 0;
  for (int z = 0; z < g.nz; ++z)
    for (int y = 0; y < g.ny; ++y)
      for (int x = 0; x < g.nx; ++x)
        fl[(size_t)x + (size_t)g.nx * ((size_t)y + (size_t)g.ny * z)] = site_solid(g, x, y, z) ? F_SOLID : 0;
  for (int z = 0; z < g.nz; ++z)
    for (int y = 0; y < g.ny; ++y)
      for (int x = 0; x < g.nx; ++x) {
        size_t cidx = (size_t)x + (size_t)g.nx * ((size_t)y + (size_t)g.ny * z);
        if (fl[cidx] & F_SOLID) continue;
        ++nfluid;
        uint32_t mask = 0u;
        for (int i = 1; i < Q; ++i)
          if (site_solid(g, x - cx(i), y - cy(i), z - cz(i))) mask |= 1u << i;
        if (mask) {
          fl[cidx] |= F_NEAR;
          links.push_back(WallLink{rep, (int)cidx, mask, 0});
        }
      }
  return nfluid;
}

}  // namespace

// Sweep configuration: tile size, tile order and grid of the K1 launch.
struct SweepCfg {
  int tile_nodes = TILE_MIN;
  int order = 0;      // 0: replica-major; 1: XCD-chunked (see tile_table)
  int grid = 0;       // 0: one workgroup per tile; else persistent grid-stride
  int cap = 0;        // 0, or at most this many sweep workgroups per CU (LDS reserved)
};

// A wait inside the resident sub-cycle normally lasts microseconds; longer
// ones mean that the GPU is shared.
constexpr uint64_t RES_WAIT = 10000000;   // 0.1 s
constexpr uint64_t RES_WAIT_MOST = 1000000000;   // 10 s

// The limit that LBMD_MD_WAIT_TICKS asks for, in *ticks (as it is without it).
int wait_limit(uint64_t* ticks) {
  const char* e = std::getenv("LBMD_MD_WAIT_TICKS");
  if (!e) return LB_OK;
  uint64_t v = 0;
  const char* p = e;
  for (; *p >= '0' && *p <= '9' && v <= RES_WAIT_MOST; ++p) v = 10 * v + (uint64_t)(*p - '0');
  if (p == e || *p || v > RES_WAIT_MOST)
    return fail(LB_ERR_ARG, "LBMD_MD_WAIT_TICKS is not a whole number from 0 to %llu: \"%.40s\"",
                (unsigned long long)RES_WAIT_MOST, e);
  *ticks = v;
  return LB_OK;
}

struct lb_ctx {
  std::vector<lb_desc> d;
  int nrep = 1;
  int device = 0;            // HIP device current at creation
  double* scratch_dev = nullptr;  // that device's address of the static scratch array
  lb_buffers b;
  hipStream_t s;
  int cur;          // 0: pops_a holds the current populations
  bool dev;
  int n_sub;
  Packing pk;
  WorkLayout wl;
  StateLayout sl;
  std::vector<Rep> reps;
  Dev D;
  int nslots = 0;
  bool step_lists = false;   // neighbour lists built from a cell list at every coupled step
  bool lists_stale = true;   // the positions changed outside a coupled step since the last build
  bool any_noise = false;
  bool any_fluct = false;    // some replica has a fluctuating fluid
  int mts = 0;               // outer steps of the multiple-time-step sub-cycle (0: uniform sub-steps)
  bool any_constrained = false;  // some replica has rigid bonds
  bool noise_ready = false;  // the noise slot of the current population parity holds this step's noise
  SweepCfg sweep;
  int ntiles = 0;
  int wl_blocks = 0;         // blocks of the wall-link list (bounce-back ledger)
  int fusedK = 0;            // sub-steps per fused block of the uniform sub-cycle (0: not in blocks)
  int fusedK_max = 0;        // the block length the context supports (0: none)
  FusedBufs fb{};
  bool resident = false;     // the sub-cycle runs in one launch of co-resident workgroups
  bool resident_own = false; // each on a CU of its own
  const FusedSeg* rseg = nullptr;
  int nrtab = 0;             // its entries
  uint64_t md_wait = RES_WAIT;   // longest wait inside it, ticks of the 100 MHz clock
  int64_t steps = 0;
  int nchain = 0;            // replicas with beads
  int64_t res_cycles = 0;    // replica cycles enqueued as resident ones
  // second stream for the sweep over the nodes without bead force, which
  // runs concurrently with the bead phase on the caller's; fork/join events
  hipStream_t s2 = nullptr;
  hipEvent_t prep = nullptr, join = nullptr;
  // graph of two coupled steps, starting at population parity graph_cur
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
  int graph_cur = -1;
  bool capturing = false;
  // the capture each step event was last recorded in (0: outside any): a
  // wait inside a capture must use a record of the same capture, else the
  // graph would depend on nodes of another (possibly destroyed) graph
  uint64_t cap_gen = 0;
  std::map<hipEvent_t, uint64_t> ev_gen;
  bool stale_wait = false;
  // adjoint: the forward pass recorded by lb_adjoint_forward
  int adj_n = 0, adj_K = 0;
  bool adj_taped = false;   // the forward pass recorded the whole horizon's tape
  int64_t adj_step0 = 0;
  char* adj_ws = nullptr;
  // kernel timing (lb_profile_start / lb_profile_stop)
  std::vector<hipEvent_t> ev;   // 4 per recorded step: bead start/end, LB start/end
  int prof_max = 0;
  int prof_n = 0;
  bool prof_on = false;
};

namespace {

void* cur_pops(lb_ctx* c) { return c->cur == 0 ? c->b.pops_a : c->b.pops_b; }

// Device address of the static scratch array on device dev (the current
// device), resolved once per device under a lock.  In host code the array's
// name only stands in for the symbol; the kernels get this address.
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_addr[MAX_DEVICES] = {};
int static_scratch(int dev, double** out) {
  if (dev < 0 || dev >= MAX_DEVICES) return fail(LB_ERR_DEVICE, "device %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(LB_ERR_DEVICE, "static scratch: %s", hipGetErrorString(e));
    g_scratch_addr[dev] = (double*)p;
  }
  *out = g_scratch_addr[dev];
  return LB_OK;
}
void* other_pops(lb_ctx* c) { return c->cur == 0 ? c->b.pops_b : c->b.pops_a; }

// Sweep tiles in launch order.  Order 0 lists each replica's tiles in node
// order.  Order 1 deals the same list into 8 contiguous chunks and
// interleaves them, so that workgroup b (which the dispatcher places on XCD
// b mod 8) takes chunk b mod 8: neighbouring tiles then run on one XCD and
// share its L2.
std::vector<Tile> tile_table(const lb_ctx* c, const SweepCfg& sc) {
  std::vector<Tile> t;
  for (int r = 0; r < c->nrep; ++r) {
    const int N = c->reps[r].lp.N;
    for (int st = 0; st < N; st += sc.tile_nodes) t.push_back(Tile{r, st});
  }
  if (sc.order == 1 && t.size() >= 16) {
    const size_t n = t.size(), nch = 8, per = (n + nch - 1) / nch;
    std::vector<Tile> o;
    o.reserve(n);
    for (size_t k = 0; k < per; ++k)
      for (size_t ch = 0; ch < nch; ++ch) {
        size_t i = ch * per + k;
        if (i < n) o.push_back(t[i]);
      }
    t.swap(o);
  }
  return t;
}

int upload_tiles(lb_ctx* c, const SweepCfg& sc) {
  if (sc.tile_nodes < TILE_MIN || sc.tile_nodes % TILE_MIN) return fail(LB_ERR_ARG, "tile size must be a multiple of %d", TILE_MIN);
  std::vector<Tile> t = tile_table(c, sc);
  if ((long)t.size() > c->pk.sweep_tiles_max) return fail(LB_ERR_ARG, "tile table overflow");
  hipError_t e = hipMemcpyAsync((char*)c->b.work + c->wl.tiles, t.data(), sizeof(Tile) * t.size(),
                                hipMemcpyHostToDevice, c->s);
  if (e == hipSuccess) e = hipStreamSynchronize(c->s);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "tile upload: %s", hipGetErrorString(e));
  c->sweep = sc;
  c->ntiles = (int)t.size();
  return LB_OK;
}

// Event slot k of the current recorded step (0, 1: bead phase; 2, 3: sweep),
// recorded on stream st.
void prof_mark(lb_ctx* c, int k, hipStream_t st) {
  if (c->capturing || !c->prof_on || c->prof_n >= c->prof_max) return;
  acc(hipEventRecord(c->ev[4 * (size_t)c->prof_n + k], st));
}
void prof_next(lb_ctx* c) {
  if (!c->capturing && c->prof_on && c->prof_n < c->prof_max) ++c->prof_n;
}

// Event record and wait of the step's fork/join structure, with the capture
// the record belongs to kept on the host (see lb_ctx::ev_gen).
void ev_record(lb_ctx* c, hipEvent_t e, hipStream_t st) {
  acc(hipEventRecord(e, st));
  c->ev_gen[e] = c->capturing ? c->cap_gen : 0;
}
void ev_wait(lb_ctx* c, hipStream_t st, hipEvent_t e) {
  if (c->capturing) {
    auto it = c->ev_gen.find(e);
    if (it == c->ev_gen.end() || it->second != c->cap_gen) c->stale_wait = true;
  }
  acc(hipStreamWaitEvent(st, e, 0));
}

// The sweep from A to B; ledger: with the wall's bounce-back momentum (which
// reads A); tick: it also counts the step.
void sweep_ab(lb_ctx* c, const void* A, void* B, int skip_forced, bool ledger, int tick, hipStream_t st) {
  const SweepCfg& w = c->sweep;
  const int nlb = ledger ? c->wl_blocks : 0;
  if (c->dev)
    launch_lb<float, true>(A, B, c->D, c->ntiles, w.tile_nodes, w.grid, w.cap, skip_forced, c->any_fluct, nlb, tick,
                           st);
  else
    launch_lb<double, false>(A, B, c->D, c->ntiles, w.tile_nodes, w.grid, w.cap, skip_forced, c->any_fluct, nlb, tick,
                             st);
}

// The device view with d.xi at noise slot k (two sub-cycles of noise, one
// per population parity).
Dev with_noise_slot(const lb_ctx* c, int k) {
  Dev D = c->D;
  D.xi = c->D.xi + (size_t)k * 3 * (size_t)c->pk.slots_alloc * (size_t)c->n_sub;
  return D;
}

// Draws the current step's noise on st unless it was drawn during the
// previous coupled step.
void ensure_noise(lb_ctx* c, hipStream_t st) {
  if (!c->any_noise || c->noise_ready || c->nslots == 0) return;
  launch_md_noise(with_noise_slot(c, c->cur), c->nslots, c->n_sub, 0, st);
  c->noise_ready = true;
}

// Builds the neighbour lists of long chains on st if the positions changed
// outside a coupled step (a step would otherwise build them first).
void ensure_lists(lb_ctx* c, hipStream_t st) {
  if (!c->step_lists || !c->lists_stale) return;
  launch_nbr_build(c->D, c->nslots, c->nrep, st);
  c->lists_stale = false;
}

// One fluid-only step on stream st.
void enqueue_lb_step(lb_ctx* c, hipStream_t st) {
  c->noise_ready = false;
  prof_mark(c, 0, st);
  prof_mark(c, 1, st);
  prof_mark(c, 2, st);
  // the fluid noise's workgroups read the step counter
  sweep_ab(c, cur_pops(c), other_pops(c), 0, true, c->any_fluct ? 0 : 1, st);
  prof_mark(c, 3, st);
  if (c->any_fluct) launch_step_end(c->D, 0, st);
  c->cur ^= 1;
  prof_next(c);
}

// One coupled step on stream st: the stencil nodes of r(n) are marked first;
// the sweep over all other nodes then runs on the second stream while the
// beads move; the marked nodes are updated once the bead force is spread.
// The bead phase and what follows from it (the next step's lists and noise)
// stay on st, which waits for the sweep only at the step's last launch: a step
// bound by the sweep then has nothing but that launch after it.
void enqueue_coupled_step_ab(lb_ctx* c, const void* A, void* B, hipStream_t st) {
  ensure_noise(c, st);
  const Dev D = with_noise_slot(c, c->cur);
  prof_mark(c, 0, st);
  // the lists of this step were built at the end of the previous one, unless
  // the positions changed since; their validity flags are read when the
  // preparation opens the sub-cycle
  if (c->step_lists && c->lists_stale) launch_nbr_build(D, c->nslots, c->nrep, st);
  launch_bead_prep(D, c->nslots, c->nrep, st);
  ev_record(c, c->prep, st);
  const bool resident = c->resident && (c->fusedK == 0 || D.mdtape);
  auto sweep_side = [&]() {
    ev_wait(c, c->s2, c->prep);
    if (resident) launch_md_gate(D, c->pk.nrseg, c->s2);
    prof_mark(c, 2, c->s2);
    sweep_ab(c, A, B, 1, true, 0, c->s2);
    prof_mark(c, 3, c->s2);
    ev_record(c, c->join, c->s2);
  };
  // enqueued before the sub-cycle's many launches, but after the resident
  // cycle: where both streams share a hardware queue, the gate before the
  // sweep then follows the workgroups it waits for
  if (!resident) sweep_side();
  // the gather also opens the sub-cycle
  const int start = c->mts > 0 ? 2 : 1;
  if (c->dev) launch_gather<float, true>(A, D, c->nslots, start, st);
  else launch_gather<double, false>(A, D, c->nslots, start, st);
  MdOverride none{};
  if (c->fusedK > 0 && !D.mdtape)
    launch_md_cycle_fused(D, c->fb, c->pk.nseg, c->nslots, c->nrep, c->n_sub, c->fusedK, st);
  else if (resident) {
    if (!c->capturing) c->res_cycles += c->nchain;
    launch_md_cycle_resident(D, c->fb.ang, c->rseg, c->nrtab, c->pk.nrseg, c->nslots, c->n_sub, c->mts, none, c->md_wait,
                             c->resident_own, c->any_constrained, st);
  } else if (c->mts > 0) {
    launch_md_cycle_mts(D, c->nslots, c->n_sub, c->mts, st);
  } else {
    launch_md_cycle(D, c->nslots, c->nrep, c->n_sub, none, st, false, c->any_constrained);
  }
  if (resident) sweep_side();
  if (c->dev) launch_spread_lb<float, true>(A, B, D, c->nslots, c->nrep, st);
  else launch_spread_lb<double, false>(A, B, D, c->nslots, c->nrep, st);
  prof_mark(c, 1, st);
  // the next step's lists from r(n+1) and, into the other slot, its noise
  launch_step_tail(D, c->nslots, c->nrep, c->any_noise ? with_noise_slot(c, c->cur ^ 1).xi : nullptr, c->n_sub, st);
  c->lists_stale = false;
  ev_wait(c, st, c->join);
  launch_step_end(D, c->nslots, st);
  c->noise_ready = c->any_noise;
  prof_next(c);
}
void enqueue_coupled_step(lb_ctx* c, hipStream_t st) {
  if (c->nslots == 0) {
    enqueue_lb_step(c, st);
    return;
  }
  enqueue_coupled_step_ab(c, cur_pops(c), other_pops(c), st);
  c->cur ^= 1;
}

void drop_graph(lb_ctx* c) {
  if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
  if (c->graph) (void)hipGraphDestroy(c->graph);
  c->gexec = nullptr;
  c->graph = nullptr;
  c->graph_cur = -1;
}

// Captures two coupled steps (so that the population parity returns to the
// start) into a graph.  Every per-step quantity the kernels need (step
// counter, forced-node count) lives in device memory, and no memset is
// recorded, so replays are equivalent to eager steps.
int build_graph(lb_ctx* c) {
  drop_graph(c);
  // the graph starts from a step whose noise is drawn and whose lists are built
  ensure_noise(c, c->s);
  ensure_lists(c, c->s);
  const int cur0 = c->cur;
  // a stream for the capture alone: one that lived on would hold a place among
  // the few hardware queues, which the streams of other contexts then share
  hipStream_t scap = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&scap, hipStreamNonBlocking);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "graph capture: %s", hipGetErrorString(e));
  c->capturing = true;
  ++c->cap_gen;
  c->stale_wait = false;
  e = hipStreamBeginCapture(scap, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) {
    c->capturing = false;
    (void)hipStreamDestroy(scap);
    return fail(LB_ERR_DEVICE, "graph capture: %s", hipGetErrorString(e));
  }
  enqueue_coupled_step(c, scap);
  enqueue_coupled_step(c, scap);
  hipGraph_t g = nullptr;
  hipError_t e2 = hipStreamEndCapture(scap, &g);
  c->capturing = false;
  (void)hipStreamDestroy(scap);
  c->cur = cur0;
  int rc = take_acc("graph capture");
  // every wait inside the capture used a record made inside it
  if (!rc && c->stale_wait)
    rc = fail(LB_ERR_DEVICE, "graph capture: a stream waited on an event recorded outside the capture");
  // the stream the steps forked joined back before the end of the capture:
  // it may not still be capturing (work enqueued on it later would otherwise
  // belong to a graph that no longer exists)
  if (!rc && e2 == hipSuccess) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    hipError_t e3 = hipStreamIsCapturing(c->s2, &cs);
    if (e3 != hipSuccess || cs != hipStreamCaptureStatusNone)
      rc = fail(LB_ERR_DEVICE, "graph capture: the forked stream is still capturing (%s)",
                e3 != hipSuccess ? hipGetErrorString(e3) : "status not none");
  }
  if (e2 != hipSuccess || rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc ? rc : fail(LB_ERR_DEVICE, "graph capture: %s", hipGetErrorString(e2));
  }
  hipGraphExec_t x = nullptr;
  e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(g);
    return fail(LB_ERR_DEVICE, "graph instantiate: %s", hipGetErrorString(e));
  }
  c->graph = g;
  c->gexec = x;
  c->graph_cur = cur0;
  return LB_OK;
}

// Workspace of the adjoint: checkpoints every K steps (and the final state),
// the per-step tape of one segment, adjoint fields.
struct AdjLayout {
  size_t ckpt, tape_pops, tape_beads, lamA, lamB, lamu, lbead, mdtape, xi, coef, par, total;
  size_t pops_slot, bead_arr, md_arr;
  size_t upj_arr;      // u_p and J of every slot, one block (they lie together in the bead buffer)
  size_t tape_entry;   // one step's bead tape: r, then u_p and J
  int nseg;
};

AdjLayout adj_layout(const lb_ctx* c, int nsteps, int K) {
  AdjLayout L;
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  L.nseg = (nsteps + K - 1) / K;
  L.pops_slot = align256(es * Q * (size_t)c->pk.nodes);
  L.bead_arr = align256(sizeof(double) * 3 * (size_t)c->pk.slots_alloc);
  L.md_arr = align256(sizeof(double) * 6 * (size_t)c->d[0].nb * (size_t)c->n_sub);
  L.upj_arr = align256(sizeof(double) * 6 * (size_t)c->pk.slots_alloc);
  L.tape_entry = L.bead_arr + L.upj_arr;
  size_t o = 0;
  L.ckpt = o; o += (size_t)(L.nseg + 1) * c->sl.total;
  L.tape_pops = o; o += (size_t)K * L.pops_slot;
  L.tape_beads = o; o += (size_t)K * L.tape_entry;
  L.lamA = o; o += L.pops_slot;
  L.lamB = o; o += L.pops_slot;
  L.lamu = o; o += align256(es * 3 * (size_t)c->pk.nodes);
  L.lbead = o; o += 10 * L.bead_arr;
  L.mdtape = o; o += (size_t)K * L.md_arr;
  L.xi = o; o += align256(sizeof(double) * 3 * (size_t)c->d[0].nb * (size_t)c->n_sub);
  L.coef = o; o += align256(adj_row_bytes(c->d[0].nb) * (size_t)adj_chunk(c->d[0].nb, c->n_sub));
  L.par = o; o += 256;
  L.total = o;
  return L;
}

int adj_check(const lb_ctx* c, int nsteps, int K) {
  if (c->nrep != 1) return fail(LB_ERR_UNSUPPORTED, "the adjoint runs on one-replica contexts");
  const lb_desc& d = c->d[0];
  if (d.nb < 1 || d.nb > MAX_ADJ_BEADS)
    return fail(LB_ERR_UNSUPPORTED, "the adjoint needs 1 <= nb <= %d (got %d)", MAX_ADJ_BEADS, d.nb);
  if (!(c->reps[0].mp.gamma > 0.0)) return fail(LB_ERR_ARG, "the adjoint needs gamma > 0");
  if (c->reps[0].lp.fluct) return fail(LB_ERR_UNSUPPORTED, "the adjoint needs an athermal fluid (fluid_kT = 0)");
  if (c->mts > 0) return fail(LB_ERR_UNSUPPORTED, "the adjoint needs the uniform sub-cycle (mts_outer = 0)");
  if (c->any_constrained) return fail(LB_ERR_UNSUPPORTED, "the adjoint needs harmonic bonds (constraints = 0)");
  if (c->d[0].coupling != LB_COUPLING_TRILINEAR)
    return fail(LB_ERR_UNSUPPORTED, "the adjoint needs the trilinear transfer (the nearest-grid-point one is not "
                                    "differentiable in the positions)");
  if (nsteps < 1 || K < 1) return fail(LB_ERR_ARG, "nsteps and K must be >= 1");
  if (c->prof_on) return fail(LB_ERR_ARG, "profiling is active");
  return LB_OK;
}

// Copies a state buffer (lb_get_state layout) into the context: populations
// to dst_pops, r, v, step counter, translocation steps.
void restore_state(lb_ctx* c, const char* st, void* dst_pops) {
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  acc(hipMemcpyAsync(dst_pops, st + c->sl.pops, es * Q * (size_t)c->pk.nodes, hipMemcpyDeviceToDevice, c->s));
  const size_t nb3 = sizeof(double) * 3 * (size_t)c->pk.slots_alloc;
  acc(hipMemcpyAsync(c->D.r, st + c->sl.r, nb3, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->D.v, st + c->sl.v, nb3, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(&c->D.ctrl->step, st + c->sl.step, sizeof(uint64_t), hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->D.tX, st + c->sl.tX, sizeof(int64_t) * c->nrep, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->D.ledger, st + c->sl.ledger, sizeof(double) * NLEDGER * c->nrep, hipMemcpyDeviceToDevice,
                     c->s));
  launch_md_invalidate(c->D, c->nrep, c->s);
  c->lists_stale = true;
  c->noise_ready = false;
}

// Runs steps n0 .. n0 + len - 1 from the checkpoint of that segment (the
// state at n0, already in the context's arrays or in `ckpt`), writing the
// tape the reverse steps read: populations before each step, r, v, u_p, J
// of each step and the sub-steps' r_mid, v.  The last step's populations go
// to other_pops(c).
void record_segment(lb_ctx* c, const AdjLayout& L, char* w, const char* ckpt, int len) {
  auto tape_pops = [&](int j) { return (void*)(w + L.tape_pops + (size_t)j * L.pops_slot); };
  // the step's start positions r, and after the step u_p and J (adjacent in
  // the bead buffer, so one copy takes both)
  auto tape_r = [&](int j) { return (double*)(w + L.tape_beads + (size_t)j * L.tape_entry); };
  auto tape_upj = [&](int j) { return (double*)(w + L.tape_beads + (size_t)j * L.tape_entry + L.bead_arr); };
  const size_t nb3 = sizeof(double) * 3 * (size_t)c->pk.slots_alloc;
  restore_state(c, ckpt, tape_pops(0));
  for (int j = 0; j < len; ++j) {
    acc(hipMemcpyAsync(tape_r(j), c->D.r, nb3, hipMemcpyDeviceToDevice, c->s));
    void* B = j + 1 < len ? tape_pops(j + 1) : other_pops(c);
    c->D.mdtape = (double*)(w + L.mdtape + (size_t)j * L.md_arr);
    // these steps keep the population parity, so the noise slot does not
    // alternate: every step draws its own noise
    c->noise_ready = false;
    enqueue_coupled_step_ab(c, tape_pops(j), B, c->s);
    c->D.mdtape = nullptr;
    acc(hipMemcpyAsync(tape_upj(j), c->D.up, 2 * nb3, hipMemcpyDeviceToDevice, c->s));
  }
}

}  // namespace

extern "C" {

const char* lb_last_error(void) { return g_last_error.c_str(); }
void lb_destroy(lb_ctx* ctx);

int lb_ensemble_sizes(const lb_desc* d, int nrep, lb_sizes* out) {
  int rc = validate(d, nrep);
  if (rc) return rc;
  if (!out) return fail(LB_ERR_ARG, "null output");
  Packing pk = packing(d, nrep);
  size_t es = elem_size(d);
  out->pops_bytes = align256(es * Q * (size_t)pk.nodes);
  out->flags_bytes = align256((size_t)pk.nodes);
  out->force_bytes = align256(es * 3 * (size_t)pk.nodes);
  out->beads_bytes = align256(sizeof(double) * 15 * (size_t)pk.slots_alloc);
  out->work_bytes = work_layout(d, nrep, pk).total;
  out->state_bytes = state_layout(d, nrep, pk).total;
  out->snapshot_bytes = out->pops_bytes + out->force_bytes + out->beads_bytes + align256(out->work_bytes);
  out->nodes = (size_t)pk.nodes;
  out->bead_slots = (size_t)pk.slots_alloc;
  return LB_OK;
}

int lb_buffer_sizes(const lb_desc* d, lb_sizes* out) { return lb_ensemble_sizes(d, 1, out); }

int lb_ensemble_init(const lb_desc* d, int nrep, const lb_buffers* b, const double* r0_host, const double* v0_host,
                     void* stream, lb_ctx** out) {
  int rc = validate(d, nrep);
  if (rc) return rc;
  if (!b || !out) return fail(LB_ERR_ARG, "null buffers or output");
  const void* ptrs[6] = {b->pops_a, b->pops_b, b->flags, b->force, b->beads, b->work};
  for (int k = 0; k < 6; ++k) {
    if (!ptrs[k]) return fail(LB_ERR_ARG, "buffer %d is NULL", k);
    if (((uintptr_t)ptrs[k]) & 255) return fail(LB_ERR_ARG, "buffer %d is not 256-byte aligned", k);
  }
  long nb_total = 0;
  for (int r = 0; r < nrep; ++r) nb_total += d[r].nb;
  if (nb_total > 0 && !r0_host) return fail(LB_ERR_ARG, "bead positions required");
  for (long k = 0; k < 3 * nb_total; ++k) {
    if (!std::isfinite(r0_host[k]) || (v0_host && !std::isfinite(v0_host[k])))
      return fail(LB_ERR_ARG, "non-finite bead state");
  }
  uint64_t wait_ticks = RES_WAIT;
  if (int rc2 = wait_limit(&wait_ticks)) return rc2;
  lb_ctx* c = new lb_ctx();
  c->d.assign(d, d + nrep);
  c->nrep = nrep;
  {
    hipError_t e = hipGetDevice(&c->device);
    int rcs = e == hipSuccess ? static_scratch(c->device, &c->scratch_dev) : fail(LB_ERR_DEVICE, "hipGetDevice: %s",
                                                                                     hipGetErrorString(e));
    if (rcs) { delete c; return rcs; }
  }
  c->b = *b;
  c->s = (hipStream_t)stream;
  {
    hipError_t e1 = hipStreamCreateWithFlags(&c->s2, hipStreamNonBlocking);
    hipError_t e3 = hipEventCreateWithFlags(&c->join, hipEventDisableTiming);
    hipError_t e6 = hipEventCreateWithFlags(&c->prep, hipEventDisableTiming);
    if (e1 != hipSuccess || e3 != hipSuccess || e6 != hipSuccess) {
      lb_destroy(c);
      return fail(LB_ERR_DEVICE, "stream/event creation failed");
    }
  }
  c->cur = 0;
  c->dev = d[0].precision == LB_FP32_DEV;
  c->n_sub = d[0].n_sub;
  c->mts = d[0].mts_outer;
  c->pk = packing(d, nrep);
  c->wl = work_layout(d, nrep, c->pk);
  c->sl = state_layout(d, nrep, c->pk);
  c->nslots = c->pk.slots;
  for (int r = 0; r < nrep; ++r) c->nchain += d[r].nb > 0 ? 1 : 0;
  // every chain's neighbour lists are built from the cell table at every
  // coupled step, beside the spreading, with a skin wide enough that a
  // step's motion rarely forces a rebuild inside the sub-cycle
  c->step_lists = c->nslots > 0;
  std::vector<FusedSeg> rsegs;
  // the fused sub-cycle (uniform sub-steps, harmonic bonds) is available in
  // blocks of up to FUSED_K sub-steps; it is off until asked for
  {
    bool rigid = false;
    for (int r = 0; r < nrep; ++r) rigid = rigid || (d[r].constraints == 1 && d[r].nb >= 2);
    if (d[0].mts_outer == 0 && !rigid && c->pk.nseg > 0)
      for (int K = FUSED_K; K >= 2; --K)
        if (d[0].n_sub % K == 0) { c->fusedK_max = K; break; }
    c->fusedK = 0;
    c->resident = c->pk.nrseg > 0 && c->pk.nrseg <= RES_MAX_WG &&
                  c->n_sub >= RES_MIN_SUB;
    // the sweep reads and writes every population once
    rsegs = res_place(d, nrep, c->pk);
    c->nrtab = (int)rsegs.size();
    c->resident_own = c->pk.nrseg <= RES_OWN_WG && c->nrtab <= RES_OWN_XCD * XCDS &&
                      2.0 * Q * (double)elem_size(d) * (double)c->pk.nodes <= RES_OWN_BYTES * (c->n_sub + c->mts);
    if (rigid) {
      // every chain rigid and of a length that a workgroup projects, on a CU of
      // its own (the launches take 20 us per sub-step: more than any sweep's loss)
      for (int r = 0; r < nrep; ++r)
        c->resident = c->resident && (d[r].nb == 0 || (d[r].constraints == 1 && d[r].nb >= 2 && d[r].nb <= RIG_MAX));
      c->resident = c->resident && c->pk.nrseg <= RES_OWN_WG && c->nrtab <= RES_OWN_XCD * XCDS;
      c->resident_own = true;
    }
    c->md_wait = wait_ticks;
  }
  const double skin = SKIN_STEP;
  const size_t ns = (size_t)c->pk.slots_alloc;
  const long nodes = c->pk.nodes;

  // replica table, flags, slot map
  std::vector<uint8_t> fl((size_t)nodes, F_SOLID);   // alignment padding is solid
  std::vector<int> slot_rep(ns, 0);
  std::vector<Tile> ot;
  std::vector<WallLink> links;
  c->reps.resize(nrep);
  for (int r = 0; r < nrep; ++r) {
    Rep& R = c->reps[r];
    std::memset(&R, 0, sizeof(Rep));
    R.g = make_geom(&d[r]);
    R.lp.nx = d[r].nx; R.lp.ny = d[r].ny; R.lp.nz = d[r].nz; R.lp.nxy = d[r].nx * d[r].ny;
    R.lp.N = (int)R.g.N;
    R.lp.omega = 1.0 / d[r].tau;
    for (int a = 0; a < 3; ++a) R.lp.g[a] = d[r].g[a];
    R.lp.has_g = (d[r].g[0] != 0.0 || d[r].g[1] != 0.0 || d[r].g[2] != 0.0) ? 1 : 0;
    fluid_noise_params(R.lp, d[r]);
    R.mp = make_md(&d[r], skin);
    if (R.mp.nb > 0 && R.mp.sig != 0.0) c->any_noise = true;
    if (R.lp.fluct) c->any_fluct = true;
    if (R.mp.constrained && R.mp.nb >= 2) c->any_constrained = true;
    R.node_off = c->pk.node_off[r];
    R.slot_off = c->pk.slot_off[r];
    R.nslot = (int)round_up(d[r].nb, MD_BPB);
    for (int k = 0; k < R.nslot; ++k) slot_rep[(size_t)R.slot_off + k] = r;
    R.wl_begin = (int)(links.size() / LEDGER_BLOCK);
    R.nfluid = (double)build_flags(R.g, fl.data() + R.node_off, r, links);
    while (links.size() % LEDGER_BLOCK) links.push_back(WallLink{r, 0, 0u, 0});
    R.wl_end = (int)(links.size() / LEDGER_BLOCK);
    {
      const int n[3] = {d[r].nx, d[r].ny, d[r].nz};
      const double side = d[r].rc + skin + CELL_MARGIN;
      for (int a = 0; a < 3; ++a) {
        int k = (int)std::floor((double)n[a] / side);
        R.ncell[a] = k < 1 ? 1 : k;
      }
    }
    R.tile_begin = (int)ot.size();
    for (int st = 0; st < R.lp.N; st += OBS_TILE) ot.push_back(Tile{r, st});
    R.tile_end = (int)ot.size();
  }

  char* w = (char*)b->work;
  Dev& D = c->D;
  std::memset(&D, 0, sizeof(Dev));
  D.reps = (const Rep*)(w + c->wl.reps);
  D.tiles = (const Tile*)(w + c->wl.tiles);
  D.otiles = (const Tile*)(w + c->wl.otiles);
  D.flags = (uint8_t*)b->flags;
  D.force = b->force;
  double* beads = (double*)b->beads;
  D.r = beads; D.v = beads + 3 * ns; D.up = beads + 6 * ns; D.J = beads + 9 * ns; D.rs = beads + 12 * ns;
  D.slot_rep = (const int*)(w + c->wl.slot_rep);
  D.head = (int*)(w + c->wl.head);
  D.next = (int*)(w + c->wl.next);
  D.base = (int*)(w + c->wl.base);
  D.touched = (int2*)(w + c->wl.touched);
  D.nbr = (int*)(w + c->wl.nbr);
  D.ncnt = (int*)(w + c->wl.ncnt);
  D.ref = (double*)(w + c->wl.ref);
  D.rmid0 = (double*)(w + c->wl.rmid0);
  D.rmid1 = (double*)(w + c->wl.rmid1);
  D.rb = (uint32_t*)(w + c->wl.rb);
  D.xi = (double*)(w + c->wl.xi);
  D.part = (double*)(w + c->wl.part);
  D.tX = (int64_t*)(w + c->wl.tX);
  D.ccount = (int*)(w + c->wl.ccount);
  D.cbuf = (int*)(w + c->wl.cbuf);
  D.rbin = (double*)(w + c->wl.rbin);
  D.cst = (uint32_t*)(w + c->wl.cst);
  D.cmask = (uint32_t)(c->wl.nbuckets - 1);
  D.ctrl = (Ctrl*)(w + c->wl.ctrl);
  D.wlinks = (const WallLink*)(w + c->wl.wlinks);
  D.ledger = (double*)(w + c->wl.ledger);
  D.lpart = (double*)(w + c->wl.lpart);
  D.lcount = (uint32_t*)(w + c->wl.lcount);
  D.lsp = (double*)(w + c->wl.lsp);
  D.redo = (int*)(w + c->wl.redo);
  D.xring = (unsigned long long*)(w + c->wl.xring);
  D.xflag = (unsigned long long*)(w + c->wl.xflag);
  D.rsync = (uint32_t*)(w + c->wl.rsync);
  c->rseg = (const FusedSeg*)(w + c->wl.rseg);
  c->fb.seg = (const FusedSeg*)(w + c->wl.fseg);
  c->fb.rmS = (double*)(w + c->wl.rmS);
  c->fb.vS = (double*)(w + c->wl.vS);
  c->fb.JS = (double*)(w + c->wl.JS);
  c->fb.ang = (double*)(w + c->wl.fang);
  c->fb.redo = D.redo;
  c->wl_blocks = (int)(links.size() / LEDGER_BLOCK);
  if ((long)c->wl_blocks > c->pk.wl_blocks_max) {
    lb_destroy(c);
    return fail(LB_ERR_ARG, "internal: wall-link list exceeds its bound");
  }

  hipStream_t s = c->s;
  acc(hipMemcpyAsync(b->flags, fl.data(), (size_t)nodes, hipMemcpyHostToDevice, s));
  acc(hipMemcpyAsync(w + c->wl.reps, c->reps.data(), sizeof(Rep) * nrep, hipMemcpyHostToDevice, s));
  acc(hipMemcpyAsync(w + c->wl.otiles, ot.data(), sizeof(Tile) * ot.size(), hipMemcpyHostToDevice, s));
  acc(hipMemcpyAsync(w + c->wl.slot_rep, slot_rep.data(), sizeof(int) * ns, hipMemcpyHostToDevice, s));
  if (!links.empty())
    acc(hipMemcpyAsync(w + c->wl.wlinks, links.data(), sizeof(WallLink) * links.size(), hipMemcpyHostToDevice, s));
  std::vector<FusedSeg> segs;
  for (int r = 0; r < nrep; ++r)
    for (int a = 0; a < d[r].nb; a += FUSED_OWN) segs.push_back(FusedSeg{r, a, std::min(a + FUSED_OWN, d[r].nb), 0});
  if (!segs.empty())
    acc(hipMemcpyAsync(w + c->wl.fseg, segs.data(), sizeof(FusedSeg) * segs.size(), hipMemcpyHostToDevice, s));
  if (!rsegs.empty())
    acc(hipMemcpyAsync(w + c->wl.rseg, rsegs.data(), sizeof(FusedSeg) * rsegs.size(), hipMemcpyHostToDevice, s));
  launch_fill_i32(D.redo, nrep, -1, s);
  launch_fill_f64(D.ledger, (long)NLEDGER * nrep, 0.0, s);
  launch_fill_i32((int*)D.lcount, nrep, 0, s);
  // rest populations, replica by replica ([19][N_r] from element 19 node_off)
  for (int r = 0; r < nrep; ++r) {
    const size_t off = elem_size(d) * Q * (size_t)c->reps[r].node_off;
    const long N = c->reps[r].lp.N;
    for (void* p : {b->pops_a, b->pops_b}) {
      if (c->dev) launch_fill_rest<float, true>((char*)p + off, N, s);
      else launch_fill_rest<double, false>((char*)p + off, N, s);
    }
  }
  acc(hipMemsetAsync(b->force, 0, elem_size(d) * 3 * (size_t)nodes, s));
  acc(hipMemsetAsync(b->beads, 0, sizeof(double) * 15 * ns, s));
  acc(hipMemsetAsync(D.ctrl, 0, sizeof(Ctrl), s));
  // no tag of this context: the memory may hold the exchanges of an earlier one
  acc(hipMemsetAsync(D.xring, 0, sizeof(uint64_t) * xring_slots(c->pk) * 2 * 3 * ns, s));
  acc(hipMemsetAsync(D.xflag, 0, sizeof(uint64_t) * XFLAG * 2 * (size_t)std::max<long>(c->pk.nrseg, 1), s));
  launch_fill_i32(D.head, nodes, -1, s);
  launch_fill_f64(D.ref, 3L * (long)ns, 1e300, s);
  launch_fill_f64(D.rbin, 3L * (long)ns, 1e300, s);
  acc(hipMemsetAsync(D.cst, 0, sizeof(uint32_t) * 4 * nrep, s));
  acc(hipMemsetAsync(D.ncnt, 0, sizeof(int) * ns, s));
  acc(hipMemsetAsync(D.rb, 0, sizeof(uint32_t) * 4 * nrep, s));
  {
    std::vector<int64_t> tx((size_t)nrep, -1);
    acc(hipMemcpyAsync(D.tX, tx.data(), sizeof(int64_t) * nrep, hipMemcpyHostToDevice, s));
    launch_md_invalidate(D, nrep, s);
    // bead state, replica by replica into its slots
    long k = 0;
    for (int r = 0; r < nrep; ++r) {
      int nb = d[r].nb;
      if (nb == 0) continue;
      acc(hipMemcpyAsync(D.r + 3 * (size_t)c->reps[r].slot_off, r0_host + 3 * k, sizeof(double) * 3 * nb,
                         hipMemcpyHostToDevice, s));
      if (v0_host)
        acc(hipMemcpyAsync(D.v + 3 * (size_t)c->reps[r].slot_off, v0_host + 3 * k, sizeof(double) * 3 * nb,
                           hipMemcpyHostToDevice, s));
      k += nb;
    }
    hipError_t e = hipStreamSynchronize(s);   // the host vectors above must outlive the copies
    if (e != hipSuccess) { lb_destroy(c); return fail(LB_ERR_DEVICE, "init: %s", hipGetErrorString(e)); }
  }
  rc = take_acc("init");
  if (rc) { lb_destroy(c); return rc; }
  rc = upload_tiles(c, SweepCfg{});
  if (rc) { lb_destroy(c); return rc; }
  rc = check_hip("init");
  if (rc) { lb_destroy(c); return rc; }
  *out = c;
  return LB_OK;
}

int lb_init(const lb_desc* d, const lb_buffers* b, const double* r0_host, const double* v0_host, void* stream,
            lb_ctx** out) {
  return lb_ensemble_init(d, 1, b, r0_host, v0_host, stream, out);
}

void lb_destroy(lb_ctx* ctx) {
  if (!ctx) return;
  if (ctx->s) (void)hipStreamSynchronize(ctx->s);
  if (ctx->s2) (void)hipStreamSynchronize(ctx->s2);
  drop_graph(ctx);
  for (hipEvent_t e : ctx->ev) (void)hipEventDestroy(e);
  if (ctx->prep) (void)hipEventDestroy(ctx->prep);
  if (ctx->join) (void)hipEventDestroy(ctx->join);
  if (ctx->s2) (void)hipStreamDestroy(ctx->s2);
  delete ctx;
}

int lb_ensemble_layout(lb_ctx* c, int64_t* node_off, int64_t* slot_off) {
  if (!c || !node_off || !slot_off) return fail(LB_ERR_ARG, "bad arguments");
  for (int r = 0; r < c->nrep; ++r) {
    node_off[r] = c->reps[r].node_off;
    slot_off[r] = c->reps[r].slot_off;
  }
  return LB_OK;
}

int lb_profile_start(lb_ctx* c, int max_steps) {
  if (!c || max_steps < 1) return fail(LB_ERR_ARG, "bad arguments");
  if (c->prof_on) return fail(LB_ERR_ARG, "profiling already active");
  size_t need = 4 * (size_t)max_steps;
  while (c->ev.size() < need) {
    hipEvent_t e;
    hipError_t r = hipEventCreate(&e);
    if (r != hipSuccess) return fail(LB_ERR_DEVICE, "hipEventCreate: %s", hipGetErrorString(r));
    c->ev.push_back(e);
  }
  c->prof_max = max_steps;
  c->prof_n = 0;
  c->prof_on = true;
  return LB_OK;
}

int lb_profile_stop(lb_ctx* c, double* mean_lb_ms, double* mean_bead_ms, int* nsteps) {
  if (!c) return fail(LB_ERR_ARG, "null context");
  if (!c->prof_on) return fail(LB_ERR_ARG, "profiling not active");
  c->prof_on = false;
  hipError_t r = hipStreamSynchronize(c->s);
  if (r == hipSuccess) r = hipStreamSynchronize(c->s2);
  if (r != hipSuccess) return fail(LB_ERR_DEVICE, "stream: %s", hipGetErrorString(r));
  double tl = 0.0, tb = 0.0;
  for (int k = 0; k < c->prof_n; ++k) {
    float a = 0.f, b = 0.f;
    r = hipEventElapsedTime(&b, c->ev[4 * (size_t)k], c->ev[4 * (size_t)k + 1]);
    if (r != hipSuccess) return fail(LB_ERR_DEVICE, "event time: %s", hipGetErrorString(r));
    r = hipEventElapsedTime(&a, c->ev[4 * (size_t)k + 2], c->ev[4 * (size_t)k + 3]);
    if (r != hipSuccess) return fail(LB_ERR_DEVICE, "event time: %s", hipGetErrorString(r));
    tl += a;
    tb += b;
  }
  int n = c->prof_n;
  if (mean_lb_ms) *mean_lb_ms = n ? tl / n : 0.0;
  if (mean_bead_ms) *mean_bead_ms = n ? tb / n : 0.0;
  if (nsteps) *nsteps = n;
  return take_acc("lb_profile_stop");
}

int lb_step(lb_ctx* c, int nsteps) {
  if (!c || nsteps < 0) return fail(LB_ERR_ARG, "bad arguments");
  for (int k = 0; k < nsteps; ++k) enqueue_lb_step(c, c->s);
  c->steps += nsteps;
  return check_hip("lb_step");
}

int md_couple_step(lb_ctx* c, int nsteps) {
  if (!c || nsteps < 0) return fail(LB_ERR_ARG, "bad arguments");
  for (int k = 0; k < nsteps; ++k) enqueue_coupled_step(c, c->s);
  c->steps += nsteps;
  return check_hip("md_couple_step");
}

int lb_ensemble_run(lb_ctx* c, int nsteps, int use_graph) {
  if (!c || nsteps < 0) return fail(LB_ERR_ARG, "bad arguments");
  if (!use_graph || c->prof_on) return md_couple_step(c, nsteps);
  int left = nsteps;
  if (left >= 2) {
    if (!c->gexec || (c->graph_cur != c->cur && c->graph_cur != (c->cur ^ 1))) {
      int rc = build_graph(c);
      if (rc) return rc;
    }
    if (c->graph_cur != c->cur) {   // one eager step to reach the graph's parity
      enqueue_coupled_step(c, c->s);
      --left;
    }
    if (left >= 2) {
      ensure_noise(c, c->s);
      ensure_lists(c, c->s);
    }
    if (c->resident && c->fusedK == 0) c->res_cycles += (int64_t)(left / 2) * 2 * c->nchain;
    for (; left >= 2; left -= 2) acc(hipGraphLaunch(c->gexec, c->s));
  }
  for (; left > 0; --left) enqueue_coupled_step(c, c->s);
  c->steps += nsteps;
  return check_hip("lb_ensemble_run");
}

int md_relax(lb_ctx* c, int nsub_total, double gamma_relax) {
  if (!c || nsub_total < 0 || !(gamma_relax >= 0.0)) return fail(LB_ERR_ARG, "bad arguments");
  if (c->nslots == 0) return LB_OK;
  MdOverride ov;
  ov.on = 1;
  ov.gamma = gamma_relax;
  const double h = 1.0 / (double)c->n_sub;
  if (gamma_relax == 0.0) {
    ov.e = 1.0; ov.omE = 0.0;
  } else {
    ov.e = std::exp(-(gamma_relax * h));
    ov.omE = 1.0 - ov.e;
  }
  ov.cf = 0.0;   // per replica: omE / (m gamma), or h / m without friction
  int left = nsub_total;
  while (left > 0) {
    int n = left < c->n_sub ? left : c->n_sub;
    if (c->resident && n >= RES_MIN_SUB) {
      c->res_cycles += c->nchain;
      launch_nbr_build(c->D, c->nslots, c->nrep, c->s);
      launch_md_begin(c->D, c->nrep, c->s);
      launch_md_start(c->D, c->nslots, ov, c->s);
      launch_md_cycle_resident(c->D, c->fb.ang, c->rseg, c->nrtab, c->pk.nrseg, c->nslots, n, 0, ov, c->md_wait,
                               c->resident_own, c->any_constrained, c->s);
    } else {
      launch_md_cycle(c->D, c->nslots, c->nrep, n, ov, c->s, true, c->any_constrained);
    }
    left -= n;
  }
  launch_zero_v(c->D, c->nslots, c->s);
  c->lists_stale = true;
  return check_hip("md_relax");
}

int lb_observables(lb_ctx* c, double* out_dev, int which_mask) {
  if (!c || !out_dev) return fail(LB_ERR_ARG, "bad arguments");
  if (which_mask & ~LB_OBS_ALL) return fail(LB_ERR_ARG, "unknown observable group in the mask 0x%x", which_mask);
  if (!which_mask) return LB_OK;
  const int no = (int)c->pk.obs_tiles;
  if (c->dev) launch_observables<float, true>(cur_pops(c), c->D, no, c->nrep, out_dev, which_mask, c->D.part, c->s);
  else launch_observables<double, false>(cur_pops(c), c->D, no, c->nrep, out_dev, which_mask, c->D.part, c->s);
  return check_hip("lb_observables");
}

int lb_observables_static(lb_ctx* c, double* out_dev, int which_mask) {
  if (!c || !out_dev) return fail(LB_ERR_ARG, "bad arguments");
  if (which_mask & ~LB_OBS_ALL) return fail(LB_ERR_ARG, "unknown observable group in the mask 0x%x", which_mask);
  const long no = c->pk.obs_tiles;
  if ((which_mask & LB_OBS_FLUID) && no > STATIC_OBS_TILES)
    return fail(LB_ERR_ARG, "lattice too large for the static scratch: %ld reduction tiles of %d nodes > %d", no,
                OBS_TILE, STATIC_OBS_TILES);
  if (!which_mask) return LB_OK;
  if (c->dev)
    launch_observables<float, true>(cur_pops(c), c->D, (int)no, c->nrep, out_dev, which_mask, c->scratch_dev, c->s);
  else
    launch_observables<double, false>(cur_pops(c), c->D, (int)no, c->nrep, out_dev, which_mask, c->scratch_dev, c->s);
  return check_hip("lb_observables_static");
}

int lb_get_state(lb_ctx* c, void* dst) {
  if (!c || !dst) return fail(LB_ERR_ARG, "bad arguments");
  char* o = (char*)dst;
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  acc(hipMemcpyAsync(o + c->sl.pops, cur_pops(c), es * Q * (size_t)c->pk.nodes, hipMemcpyDeviceToDevice, c->s));
  const size_t nb3 = sizeof(double) * 3 * (size_t)c->pk.slots_alloc;
  acc(hipMemcpyAsync(o + c->sl.r, c->D.r, nb3, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + c->sl.v, c->D.v, nb3, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + c->sl.step, &c->D.ctrl->step, sizeof(uint64_t), hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + c->sl.tX, c->D.tX, sizeof(int64_t) * c->nrep, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + c->sl.ledger, c->D.ledger, sizeof(double) * NLEDGER * c->nrep, hipMemcpyDeviceToDevice,
                     c->s));
  return check_hip("lb_get_state");
}

int lb_set_state(lb_ctx* c, const void* src) {
  if (!c || !src) return fail(LB_ERR_ARG, "bad arguments");
  const char* o = (const char*)src;
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  acc(hipMemcpyAsync(cur_pops(c), o + c->sl.pops, es * Q * (size_t)c->pk.nodes, hipMemcpyDeviceToDevice, c->s));
  const size_t nb3 = sizeof(double) * 3 * (size_t)c->pk.slots_alloc;
  acc(hipMemcpyAsync(c->D.r, o + c->sl.r, nb3, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->D.v, o + c->sl.v, nb3, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(&c->D.ctrl->step, o + c->sl.step, sizeof(uint64_t), hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->D.tX, o + c->sl.tX, sizeof(int64_t) * c->nrep, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->D.ledger, o + c->sl.ledger, sizeof(double) * NLEDGER * c->nrep, hipMemcpyDeviceToDevice,
                     c->s));
  launch_md_invalidate(c->D, c->nrep, c->s);
  c->lists_stale = true;
  c->noise_ready = false;
  uint64_t st = 0;
  acc(hipMemcpyAsync(&st, o + c->sl.step, sizeof(uint64_t), hipMemcpyDeviceToHost, c->s));
  hipError_t e = hipStreamSynchronize(c->s);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "lb_set_state: %s", hipGetErrorString(e));
  c->steps = (int64_t)st;
  return check_hip("lb_set_state");
}

void* lb_current_pops(lb_ctx* c) { return c ? cur_pops(c) : nullptr; }

int lb_check(lb_ctx* c) {
  if (!c) return fail(LB_ERR_ARG, "null context");
  hipError_t e = hipStreamSynchronize(c->s);
  if (e == hipSuccess) e = hipStreamSynchronize(c->s2);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "stream: %s", hipGetErrorString(e));
  uint32_t err = 0;
  e = hipMemcpy(&err, &c->D.ctrl->err, sizeof(err), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "watchdog read: %s", hipGetErrorString(e));
  if (err) {
    std::string why;
    if (err & E_DENSITY) why += "non-positive or non-finite density; ";
    if (err & E_BEADS) why += "non-finite bead velocity; ";
    if (err & E_NBRLIST) why += "neighbour list overflow; ";
    if (err & E_SPREAD) why += "too many beads on one node stencil; ";
    return fail(LB_ERR_UNSTABLE, "watchdog: %s", why.c_str());
  }
  return LB_OK;
}

int64_t lb_step_count(lb_ctx* c) { return c ? c->steps : -1; }

// The control block, once the stream is done.
static int read_ctrl(lb_ctx* c, Ctrl& h) {
  hipError_t e = hipStreamSynchronize(c->s);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "stream: %s", hipGetErrorString(e));
  e = hipMemcpy(&h, c->D.ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "diagnostics read: %s", hipGetErrorString(e));
  return LB_OK;
}

int lb_md_passes(lb_ctx* c, int64_t* out) {
  if (!c || !out) return fail(LB_ERR_ARG, "bad arguments");
  Ctrl h;
  if (int rc = read_ctrl(c, h)) return rc;
  out[0] = c->res_cycles;
  out[1] = (int64_t)h.res_second;
  out[2] = (int64_t)h.res_redone;
  return LB_OK;
}

int lb_diagnostics(lb_ctx* c, int64_t* out) {
  if (!c || !out) return fail(LB_ERR_ARG, "bad arguments");
  Ctrl h;
  if (int rc = read_ctrl(c, h)) return rc;
  out[0] = (int64_t)h.rebuilds;
  out[1] = (int64_t)h.substeps;
  out[2] = (int64_t)c->ntiles;
  out[3] = (int64_t)h.err;
  out[4] = (int64_t)h.step;
  out[5] = (int64_t)h.forced_total;
  out[6] = (int64_t)h.cell_rebuilds;
  out[7] = (int64_t)h.fused_blocks;
  out[8] = (int64_t)h.fused_redos;
  for (int k = 0; k < 5; ++k) out[9 + k] = (int64_t)h.fused_why[k];
  out[14] = (int64_t)h.nbr_max;
  return LB_OK;
}

int lb_ensemble_translocation(lb_ctx* c, int64_t* out_host) {
  if (!c || !out_host) return fail(LB_ERR_ARG, "bad arguments");
  hipError_t e = hipStreamSynchronize(c->s);
  if (e == hipSuccess) e = hipMemcpy(out_host, c->D.tX, sizeof(int64_t) * c->nrep, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "translocation read: %s", hipGetErrorString(e));
  return LB_OK;
}

int lb_md_fused(lb_ctx* c, int K) {
  if (!c || K < 0) return fail(LB_ERR_ARG, "bad arguments");
  if (K > 0 && c->fusedK_max == 0)
    return fail(LB_ERR_UNSUPPORTED, "the fused sub-cycle needs the uniform sub-cycle, harmonic bonds and a chain");
  if (K > 0 && (K < 2 || K > c->fusedK_max || c->n_sub % K != 0))
    return fail(LB_ERR_ARG, "block length must divide n_sub and lie in [2, %d]", c->fusedK_max);
  if (K != c->fusedK) drop_graph(c);
  c->fusedK = K;
  return LB_OK;
}

int lb_sweep_config(lb_ctx* c, int tile_nodes, int order, int grid, int cap) {
  if (!c || order < 0 || order > 1 || grid < 0 || !(cap == 0 || (cap >= SWEEP_CAP_MIN && cap <= SWEEP_CAP_MAX)))
    return fail(LB_ERR_ARG, "bad arguments");
  SweepCfg sc;
  sc.tile_nodes = tile_nodes;
  sc.order = order;
  sc.grid = grid;
  sc.cap = cap;
  int rc = upload_tiles(c, sc);
  if (rc) return rc;
  drop_graph(c);
  return LB_OK;
}

}  // extern "C"

namespace {

// Candidate sweep layouts: tile sizes 256..2048 in both orders; persistent
// grids of 256..2048 workgroups over tiles of 256 and 512 nodes; and one
// workgroup per tile of 256..1024 nodes with at most 2, 3 or 4 sweep
// workgroups per CU.
std::vector<SweepCfg> sweep_candidates() {
  std::vector<SweepCfg> cand;
  for (int tn : {256, 512, 1024, 2048})
    for (int order : {0, 1}) cand.push_back(SweepCfg{tn, order, 0, 0});
  for (int tn : {256, 512})
    for (int g : {256, 384, 512, 768, 1024, 2048}) cand.push_back(SweepCfg{tn, 0, g, 0});
  for (int tn : {256, 512, 1024})
    for (int cap : {2, 3, 4}) cand.push_back(SweepCfg{tn, 0, 0, cap});
  return cand;
}

// Device copy of everything a coupled step reads or writes (current
// populations, beads, work area, force field), in a buffer of the caller,
// and the host fields that follow it, so that timed trial steps leave no
// trace.
struct Snapshot {
  char* mem = nullptr;
  size_t pops = 0, beads = 0, work = 0, force = 0;
  int cur = 0;
  int64_t steps = 0, res_cycles = 0;
  bool lists_stale = true;
  bool noise_ready = false;
};

size_t snapshot_bytes(const lb_ctx* c) {
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  return align256(es * Q * (size_t)c->pk.nodes) + align256(sizeof(double) * 15 * (size_t)c->pk.slots_alloc) +
         align256(c->wl.total) + align256(es * 3 * (size_t)c->pk.nodes);
}

int snapshot_take(lb_ctx* c, Snapshot& S, char* mem) {
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  S.pops = align256(es * Q * (size_t)c->pk.nodes);
  S.beads = align256(sizeof(double) * 15 * (size_t)c->pk.slots_alloc);
  S.work = align256(c->wl.total);
  S.force = align256(es * 3 * (size_t)c->pk.nodes);
  S.mem = mem;
  char* o = S.mem;
  acc(hipMemcpyAsync(o, cur_pops(c), S.pops, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + S.pops, c->b.beads, S.beads, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + S.pops + S.beads, c->b.work, c->wl.total, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(o + S.pops + S.beads + S.work, c->b.force, es * 3 * (size_t)c->pk.nodes,
                     hipMemcpyDeviceToDevice, c->s));
  S.cur = c->cur;
  S.steps = c->steps;
  S.res_cycles = c->res_cycles;
  S.lists_stale = c->lists_stale;
  S.noise_ready = c->noise_ready;
  return take_acc("snapshot");
}

void snapshot_restore(lb_ctx* c, const Snapshot& S) {
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  c->cur = S.cur;
  c->steps = S.steps;
  c->res_cycles = S.res_cycles;
  c->lists_stale = S.lists_stale;
  c->noise_ready = S.noise_ready;
  const char* o = S.mem;
  acc(hipMemcpyAsync(cur_pops(c), o, es * Q * (size_t)c->pk.nodes, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->b.beads, o + S.pops, sizeof(double) * 15 * (size_t)c->pk.slots_alloc,
                     hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->b.work, o + S.pops + S.beads, c->wl.total, hipMemcpyDeviceToDevice, c->s));
  acc(hipMemcpyAsync(c->b.force, o + S.pops + S.beads + S.work, es * 3 * (size_t)c->pk.nodes,
                     hipMemcpyDeviceToDevice, c->s));
}

// Times every candidate layout: `reps` sweeps from the current populations
// into the other array, or (coupled) `reps` coupled steps replayed from the
// two-step graph, from a snapshot restored after each candidate.  Keeps the
// first candidate within 1% of the fastest (timing noise then does not flip
// the choice between layouts that perform alike) and caches it, with its
// time, per packing, precision, sweep variant (athermal or fluctuating fluid)
// and mode.
int tune_layout(lb_ctx* c, int reps, bool coupled, char* snap, size_t snap_bytes, int* out_cfg, double* out_ms) {
  if (!c || reps < 1) return fail(LB_ERR_ARG, "bad arguments");
  static std::map<std::string, std::pair<SweepCfg, double>> cache;
  std::string key = coupled ? "step:" : "sweep:";
  key += c->dev ? "f32:" : "f64:";
  key += c->any_fluct ? "thermal:" : "athermal:";
  for (const lb_desc& x : c->d) {
    char buf[160];
    snprintf(buf, sizeof(buf), "%d,%d,%d,%d,%d,%d,%d,%d,%d,%.17g;", x.nx, x.ny, x.nz, x.wall_axis, x.wall_pos,
             x.pore_h, x.nb, x.n_sub, x.mts_outer, x.rc);
    key += buf;
  }
  auto it = cache.find(key);
  SweepCfg best;
  double best_ms = -1.0;
  if (it != cache.end()) {
    best = it->second.first;
    best_ms = it->second.second;
  } else {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
      if (e0) (void)hipEventDestroy(e0);
      return fail(LB_ERR_DEVICE, "hipEventCreate failed");
    }
    const std::vector<SweepCfg> cand = sweep_candidates();
    const bool prof = c->prof_on;
    c->prof_on = false;
    Snapshot S;
    int rc = LB_OK;
    if (coupled) {
      if (!snap || snap_bytes < snapshot_bytes(c) || ((uintptr_t)snap & 255))
        rc = fail(LB_ERR_ARG, "snapshot buffer: need %zu bytes, 256-byte aligned (got %zu)", snapshot_bytes(c),
                  snap_bytes);
      else
        rc = snapshot_take(c, S, snap);
    }
    std::vector<double> times;
    for (size_t k = 0; k < cand.size() && !rc; ++k) {
      rc = upload_tiles(c, cand[k]);
      if (rc) break;
      drop_graph(c);
      if (coupled) {
        rc = lb_ensemble_run(c, 2, 1);   // capture and a first replay
        if (rc) break;
        acc(hipEventRecord(e0, c->s));
        rc = lb_ensemble_run(c, 2 * ((reps + 1) / 2), 1);
        if (rc) break;
        acc(hipEventRecord(e1, c->s));
      } else {
        // into the other array, which the next step overwrites: the state
        // is unchanged
        for (int j = 0; j < 2; ++j) sweep_ab(c, cur_pops(c), other_pops(c), 0, false, 0, c->s);
        acc(hipEventRecord(e0, c->s));
        for (int j = 0; j < reps; ++j) sweep_ab(c, cur_pops(c), other_pops(c), 0, false, 0, c->s);
        acc(hipEventRecord(e1, c->s));
      }
      hipError_t e = hipEventSynchronize(e1);
      float ms = 0.f;
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
      if (e != hipSuccess) { rc = fail(LB_ERR_DEVICE, "autotune: %s", hipGetErrorString(e)); break; }
      times.push_back(ms / (coupled ? 2 * ((reps + 1) / 2) : reps));
      if (coupled) snapshot_restore(c, S);
    }
    if (S.mem) {
      if (rc) snapshot_restore(c, S);
      hipError_t e = hipStreamSynchronize(c->s);
      if (!rc && e != hipSuccess) rc = fail(LB_ERR_DEVICE, "autotune: %s", hipGetErrorString(e));
    }
    drop_graph(c);
    c->prof_on = prof;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    rc = take_acc("autotune");
    if (rc) return rc;
    if (std::getenv("LBMD_AUTOTUNE_LOG"))
      for (size_t k = 0; k < cand.size(); ++k)
        fprintf(stderr, "lb_autotune %s: tile %d order %d grid %d cap %d: %.4f ms\n", coupled ? "step" : "sweep",
                cand[k].tile_nodes, cand[k].order, cand[k].grid, cand[k].cap, times[k]);
    double tmin = times[0];
    for (double t : times) tmin = t < tmin ? t : tmin;
    for (size_t k = 0; k < cand.size(); ++k)
      if (times[k] <= 1.01 * tmin) { best = cand[k]; best_ms = times[k]; break; }
    cache[key] = std::make_pair(best, best_ms);
  }
  int rc = upload_tiles(c, best);
  if (rc) return rc;
  drop_graph(c);
  if (out_cfg) { out_cfg[0] = best.tile_nodes; out_cfg[1] = best.order; out_cfg[2] = best.grid; out_cfg[3] = best.cap; }
  if (out_ms) *out_ms = best_ms;
  return check_hip("lb_autotune");
}

}  // namespace

extern "C" {

int lb_autotune(lb_ctx* c, int reps, int* out_cfg, double* out_ms) {
  return tune_layout(c, reps, false, nullptr, 0, out_cfg, out_ms);
}

int lb_autotune_step(lb_ctx* c, int reps, void* snap_dev, size_t snap_bytes, int* out_cfg, double* out_ms) {
  return tune_layout(c, reps, true, (char*)snap_dev, snap_bytes, out_cfg, out_ms);
}

int lb_set_coupling(lb_ctx* c, int rep, double gamma, double f_drive) {
  if (!c || rep < 0 || rep >= c->nrep || !(gamma >= 0.0) || !std::isfinite(gamma) || !std::isfinite(f_drive))
    return fail(LB_ERR_ARG, "bad arguments");
  if (gamma > 0.0 && c->d[rep].nb > 0 && c->d[rep].mass != 1.0)
    return fail(LB_ERR_ARG, "a chain coupled with gamma > 0 needs mass 1");
  Rep& R = c->reps[rep];
  R.mp.f_drive = f_drive;
  spv_coefficients(R.mp, gamma, c->d[rep].kT, 1.0 / (double)c->n_sub);
  c->d[rep].gamma = gamma;
  c->d[rep].f_drive = f_drive;
  bool noise = false;
  for (const Rep& x : c->reps) noise = noise || (x.mp.nb > 0 && x.mp.sig != 0.0);
  if (noise != c->any_noise) drop_graph(c);
  c->any_noise = noise;
  c->noise_ready = false;
  hipError_t e = hipMemcpyAsync((char*)c->b.work + c->wl.reps + sizeof(Rep) * (size_t)rep, &R, sizeof(Rep),
                                hipMemcpyHostToDevice, c->s);
  if (e == hipSuccess) e = hipStreamSynchronize(c->s);   // R is read from host memory
  if (e != hipSuccess) return fail(LB_ERR_DEVICE, "lb_set_coupling: %s", hipGetErrorString(e));
  return LB_OK;
}

int lb_adjoint_sizes(lb_ctx* c, int nsteps, int K, size_t* bytes) {
  if (!c || !bytes) return fail(LB_ERR_ARG, "bad arguments");
  int rc = adj_check(c, nsteps, K);
  if (rc) return rc;
  *bytes = adj_layout(c, nsteps, K).total;
  return LB_OK;
}

int lb_adjoint_forward(lb_ctx* c, int nsteps, int K, void* ws, size_t ws_bytes) {
  if (!c || !ws) return fail(LB_ERR_ARG, "bad arguments");
  int rc = adj_check(c, nsteps, K);
  if (rc) return rc;
  AdjLayout L = adj_layout(c, nsteps, K);
  if (ws_bytes < L.total) return fail(LB_ERR_ARG, "workspace too small (%zu < %zu bytes)", ws_bytes, L.total);
  if (((uintptr_t)ws) & 255) return fail(LB_ERR_ARG, "workspace is not 256-byte aligned");
  char* w = (char*)ws;
  c->adj_ws = nullptr;
  c->adj_step0 = c->steps;
  rc = lb_get_state(c, w + L.ckpt);
  if (rc) return rc;
  if (L.nseg == 1) {
    // one segment: the forward pass writes the tape itself, and the
    // backward pass reverses it without recomputing the horizon
    record_segment(c, L, w, w + L.ckpt, nsteps);
    c->cur ^= 1;   // the last step wrote other_pops
    c->steps += nsteps;
    rc = lb_get_state(c, w + L.ckpt + c->sl.total);
    if (rc) return rc;
  } else {
    for (int seg = 0; seg < L.nseg; ++seg) {
      int len = std::min(K, nsteps - seg * K);
      for (int k = 0; k < len; ++k) enqueue_coupled_step(c, c->s);
      c->steps += len;
      rc = lb_get_state(c, w + L.ckpt + (size_t)(seg + 1) * c->sl.total);
      if (rc) return rc;
    }
  }
  c->adj_n = nsteps;
  c->adj_K = K;
  c->adj_ws = w;
  c->adj_taped = L.nseg == 1;
  return check_hip("lb_adjoint_forward");
}

int lb_adjoint_backward(lb_ctx* c, const double* dLdr, const double* dLdv, double* grads) {
  if (!c || !dLdr || !grads) return fail(LB_ERR_ARG, "bad arguments");
  if (!c->adj_ws) return fail(LB_ERR_ARG, "no recorded forward pass (call lb_adjoint_forward first)");
  const int nsteps = c->adj_n, K = c->adj_K;
  int rc = adj_check(c, nsteps, K);
  if (rc) return rc;
  AdjLayout L = adj_layout(c, nsteps, K);
  char* w = c->adj_ws;
  const int nb = c->d[0].nb;
  const size_t es = c->dev ? sizeof(float) : sizeof(double);
  AdjBufs a;
  a.lr = (double*)(w + L.lbead);
  a.lv = (double*)(w + L.lbead + L.bead_arr);
  a.lJ = (double*)(w + L.lbead + 2 * L.bead_arr);
  a.lup = (double*)(w + L.lbead + 3 * L.bead_arr);
  a.lrs = (double*)(w + L.lbead + 4 * L.bead_arr);
  a.lr2 = (double*)(w + L.lbead + 5 * L.bead_arr);
  a.lv2 = (double*)(w + L.lbead + 6 * L.bead_arr);
  a.gacc = (double*)(w + L.lbead + 7 * L.bead_arr);
  a.dirA = (double*)(w + L.lbead + 8 * L.bead_arr);
  a.dirB = (double*)(w + L.lbead + 9 * L.bead_arr);
  a.lamu = w + L.lamu;
  a.par = (double*)(w + L.par);
  a.lok = (int*)(w + L.par + 128);
  a.xi = (double*)(w + L.xi);
  a.coef = (double*)(w + L.coef);
  void* lamB = w + L.lamB;   // adjoint of the populations after the step being reversed
  void* lamA = w + L.lamA;
  acc(hipMemsetAsync(lamB, 0, L.pops_slot, c->s));
  acc(hipMemsetAsync(lamA, 0, L.pops_slot, c->s));
  acc(hipMemsetAsync(a.lamu, 0, es * 3 * (size_t)c->pk.nodes, c->s));
  launch_adj_init(dLdr, dLdv, a, nb, c->s);
  auto tape_pops = [&](int j) { return (void*)(w + L.tape_pops + (size_t)j * L.pops_slot); };
  auto tape_r = [&](int j) { return (double*)(w + L.tape_beads + (size_t)j * L.tape_entry); };
  auto tape_up = [&](int j) { return (double*)(w + L.tape_beads + (size_t)j * L.tape_entry + L.bead_arr); };
  auto tape_J = [&](int j) { return tape_up(j) + 3 * (size_t)c->pk.slots_alloc; };
  const double kT = c->d[0].kT;
  for (int seg = L.nseg - 1; seg >= 0; --seg) {
    const int n0 = seg * K;
    const int len = std::min(K, nsteps - n0);
    // recompute the segment from its checkpoint, writing the tape (a
    // one-segment horizon was taped by the forward pass)
    if (!c->adj_taped) record_segment(c, L, w, w + L.ckpt + (size_t)seg * c->sl.total, len);
    // reverse the segment's steps
    for (int j = len - 1; j >= 0; --j) {
      Dev da = c->D;
      da.r = tape_r(j);
      Dev ds = da;
      ds.J = a.lup;
      ds.force = a.lamu;
      const uint32_t step = (uint32_t)(c->adj_step0 + n0 + j);
      const double* mdt = (const double*)(w + L.mdtape + (size_t)j * L.md_arr);
      if (c->dev)
        launch_adj_reverse_step<float, true>(tape_pops(j), lamB, lamA, da, ds, a, mdt, tape_up(j),
                                             tape_J(j), step, kT, c->ntiles, c->sweep.tile_nodes, c->nslots,
                                             nb, c->n_sub, c->s);
      else
        launch_adj_reverse_step<double, false>(tape_pops(j), lamB, lamA, da, ds, a, mdt, tape_up(j),
                                               tape_J(j), step, kT, c->ntiles, c->sweep.tile_nodes,
                                               c->nslots, nb, c->n_sub, c->s);
      std::swap(lamA, lamB);
    }
  }
  // the context returns to the state after the forward pass
  restore_state(c, w + L.ckpt + (size_t)L.nseg * c->sl.total, cur_pops(c));
  launch_adj_finish(a, grads, nb, c->s);
  return check_hip("lb_adjoint_backward");
}

int lb_adjoint_run(lb_ctx* c, int nsteps, int K, void* ws, size_t ws_bytes, const double* dLdr, double* grads) {
  int rc = lb_adjoint_forward(c, nsteps, K, ws, ws_bytes);
  if (rc) return rc;
  return lb_adjoint_backward(c, dLdr, nullptr, grads);
}

}  // extern "C"
