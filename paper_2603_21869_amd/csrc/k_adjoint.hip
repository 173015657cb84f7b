// Reverse mode of the explicit stage and of the destruction step.
//
// Explicit stage (Sec. 2.3, Algorithms 2 and 4, eqs. ko_mom, ko_temp, ko_k,
// ko_o; the solver's differentiability, Sec. 1 and 4):
// the adjoints of the stage's inputs u, v, w, p, T, k, omega from those of its
// outputs u, v, w, T, k, omega, at a given input state, with nu_t the closure
// of the input k and omega (eqs. a_star, ko_turb_diff), so that its adjoint
// is folded into theirs.
//
// The stage updates every fluid cell by dt times a sum of face fluxes, each a
// function of the two cells of the face (a boundary face's outer values being
// affine ghost rules of the inner cell, Sec. 2.7), plus cell sources that
// read the central velocity gradient.  The transposed Jacobian at a cell is
//   - the weights of each output cell: dt * ybar of the outputs that the
//     fluxes feed (zero where an output is not updated or is clamped at eps),
//     the factor by which each output passes its own input (1, or 0 where k
//     or omega is clamped), and 4 Lambda S_ab with Lambda = W_k nu_t +
//     W_omega alpha, the weight of the strain-rate sources;
//   - gathered per input cell: its own pass terms, then each face's flux
//     derivatives with respect to this cell's values times the difference of
//     the two cells' weights, the production terms of its own and of its
//     neighbours' strain rates, buoyancy, and the closure chain rule.
// The destruction step's is of the same form (below).  Arithmetic in FP64
// throughout.
//
// Each reverse mode is one kernel that reads every input once and writes every
// output once: the weights live in registers and LDS only.  A workgroup of
// 64 x RY threads walks the planes of a column tile, one column per
// thread.  Lanes 1 .. 62 and every row form weights, lanes 2 .. 61 and rows
// 1 .. RY - 2 have results: a tile is 60 x (RY - 2) columns and the
// rest recompute the weights its results read (1.4 times the weight
// arithmetic, no memory traffic beyond the caches).  The x neighbours come
// from the adjacent lanes of the wave (DPP shifts), the y neighbours from LDS
// rows, the z neighbours from the walk: the weights are formed one plane
// ahead, and a cell's result is stored once the plane above has been
// weighed.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "nfvm_device.hpp"

namespace nfvm {

namespace {
constexpr int ABX = 64, ABY = 4;
// Rows of a workgroup: as many waves as its registers leave room for on one
// CU (explicit stage 235 VGPRs: 8 waves; destruction 158: 12, with 10 rows of
// results in 12 instead of 6 in 8: 965 -> 780 us on the 512 x 256 x 128 room).
constexpr int EX_RY = 8, DS_RY = 12;
constexpr int ADJ_TX = 60;           // columns of a tile along x

// transported fields in flux order and their ghost-rule codes
constexpr int NF = 6;  // u v w theta k omega
__device__ __forceinline__ int ghost_code(int f) {
  return f < 3 ? G_U + f : (f == 3 ? G_T : (f == 4 ? G_K : G_OM));
}

// What the kernels read of the grid and its physics; the reciprocals are
// formed once on the host (a division costs a thread a dozen instructions).
struct AdjParams {
  int nx, ny, nz, d3, sx, sxy, off;
  int ntx, nty, cz, total;  // column tiles, planes per chunk, tiles in all
  double ih[3], ih2[3];     // 1 / h, 1 / (2 h)
  double nu, inu, alpha_T, is3, is4, is5, dt, T_ref, bg[3];
  int komega, energy, buoyancy;
};

// Chunks of planes per column tile.  A chunk of cz planes takes cz + 2 steps
// of its workgroup (the planes of weights on both sides) and about one more
// to start and end, and the 256 CUs hold one workgroup each at a time (its
// registers): the count that makes the rounds times the steps shortest.
constexpr int ADJ_CUS = 256;
int adj_chunks(int cols, int nz) {
  long long best = -1;
  int chunks = 1;
  // (more chunks than this leave every CU busy whatever the tail)
  const int most = std::min(nz, 64 * ADJ_CUS / std::min(cols, 64 * ADJ_CUS) + 1);
  for (int c = 1; c <= most; ++c) {
    const int cz = (nz + c - 1) / c;
    if ((nz + cz - 1) / cz != c) continue;  // (the same cz as a smaller count)
    const long long t = ((long long)cols * c + ADJ_CUS - 1) / ADJ_CUS * (cz + 3);
    if (best < 0 || t < best) {
      best = t;
      chunks = c;
    }
  }
  return chunks;
}

AdjParams adj_params(const Geom& g, const Phys& ph, int rows) {
  AdjParams p;
  p.nx = g.nx;
  p.ny = g.ny;
  p.nz = g.nz;
  p.d3 = g.dim == 3;
  p.sx = g.sx;
  p.sxy = g.sxy;
  p.off = g.off;
  p.ntx = (g.nx + ADJ_TX - 1) / ADJ_TX;
  p.nty = (g.ny + rows - 3) / (rows - 2);
  const int cols = p.ntx * p.nty;
  const int chunks = adj_chunks(cols, g.nz);
  p.cz = (g.nz + chunks - 1) / chunks;
  p.total = cols * ((g.nz + p.cz - 1) / p.cz);
  const double h[3] = {g.hx, g.hy, g.hz};
  for (int d = 0; d < 3; ++d) {
    p.ih[d] = 1.0 / h[d];
    p.ih2[d] = 0.5 / h[d];
    p.bg[d] = -ph.beta_T * ph.g[d];
  }
  p.nu = ph.nu;
  p.inu = 1.0 / ph.nu;
  p.alpha_T = ph.alpha_T;
  p.is3 = ph.inv_Pr_t;
  p.is4 = ph.inv_sigma_k;
  p.is5 = ph.inv_sigma_w;
  p.dt = ph.dt;
  p.T_ref = ph.T_ref;
  p.komega = ph.komega;
  p.energy = ph.energy;
  p.buoyancy = ph.buoyancy;
  return p;
}
inline dim3 adj_grid(const AdjParams& p) { return dim3((unsigned)((p.total + 7) / 8 * 8)); }

// The tile of this workgroup; workgroup b runs on XCD b % 8, and each XCD
// takes a contiguous range of tiles (x fastest), whose halos overlap in its L2.
__device__ __forceinline__ bool adj_tile(const AdjParams& p, int& tx, int& ty, int& tz) {
  const int per = gridDim.x >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (t >= p.total) return false;
  tx = t % p.ntx;
  const int r = t / p.ntx;
  ty = r % p.nty;
  tz = r / p.nty;
  return true;
}

// Element at byte offset vi of a row given by a scalar pointer (kept opaque,
// so that the access takes a scalar base and a 32-bit lane offset rather than
// a 64-bit address per lane and array).
#define ADJ_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ ADJ_GLOBAL T* row_at(T* row, unsigned vi) {
  ADJ_GLOBAL char* q = (ADJ_GLOBAL char*)(ADJ_GLOBAL T*)row;
  asm("" : "+s"(q), "+v"(vi));
  return (ADJ_GLOBAL T*)(q + vi);
}

// Type byte of cell (i, r, m) (vt: i + 1, clamped to the padded row; pi: i
// was in it), solid past the padded array.
__device__ __forceinline__ int adj_type(const AdjParams& p, const uint8_t* type, unsigned vt,
                                        bool pi, int r, int m) {
  const int gz = p.d3 ? 1 : 0;
  const int rq = min(max(r, -1), p.ny), mq = min(max(m, -gz), p.nz - 1 + gz);
  const int t = *row_at(type + (p.off + mq * p.sxy + rq * p.sx - 1), vt);
  return pi && r == rq && m == mq ? t : PID_SOLID;
}

// The value of the next lower (higher) lane of the wave; every lane of the
// wave must take part, and lane 0 (63) gets 0.
template <int CTRL>
__device__ __forceinline__ int lane_shift(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  return __hiloint2double(lane_shift<CTRL>(__double2hiint(v)),
                          lane_shift<CTRL>(__double2loint(v)));
}
constexpr int WAVE_SHR1 = 0x138, WAVE_SHL1 = 0x130;
template <class T>
__device__ __forceinline__ T lane_below(T v) {
  return lane_shift<WAVE_SHR1>(v);
}
template <class T>
__device__ __forceinline__ T lane_above(T v) {
  return lane_shift<WAVE_SHL1>(v);
}

// d(ghost value) / d(own value) across a boundary face
__device__ __forceinline__ double slope(const DevPatch& pp, int code, int komega) {
  return ghost<double>(pp, code, 1.0, komega) - ghost<double>(pp, code, 0.0, komega);
}

struct ExplicitIo {
  const double *u, *v, *w, *T, *k, *om;        // state, dense (T absolute)
  const double *ybu, *ybv, *ybw, *ybT, *ybk, *ybo;  // adjoints of the outputs, dense
  double *xu, *xv, *xw, *xp, *xT, *xk, *xo;    // adjoints of the inputs, dense
};

struct ExplicitArgs {
  ExplicitIo io;  // (first: read again from the kernel arguments where used)
  AdjParams p;
  const uint8_t* type;
  const DevPatch* pt;
};

// The array pointers, loaded from the kernel-argument segment (through the
// scalar cache) at each use: with the parameters they are more than the
// scalar registers hold, and kept ones are spilled to vector lanes.
__device__ __forceinline__ const __attribute__((address_space(4))) ExplicitIo* explicit_io() {
  auto q = (const __attribute__((address_space(4))) ExplicitIo*)
      __builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(q));
  return q;
}

// One cell of the walk: u v w theta k omega, nu_t and the type byte.
struct AdjCell {
  double v[NF], nu;
  int t;
};

// The closures of one fluid cell: nu_t with its derivatives in k and omega
// (eqs. a_star, Re_t), and alpha of the omega production (eq. a) with its own.
struct AdjClosure {
  double nt, dk, dw, al, ak, aw;
};

// Partial result of one cell.
struct AdjAcc {
  double x[NF], nb, pb;  // adjoints of the six fields, of nu_t and of p
};

__device__ __forceinline__ void field_coef(const AdjParams& p, double (&g0)[NF],
                                           double (&is)[NF]) {
  g0[0] = g0[1] = g0[2] = g0[4] = g0[5] = p.nu;
  g0[3] = p.alpha_T;
  is[0] = is[1] = is[2] = 1.0;
  is[3] = p.is3;
  is[4] = p.is4;
  is[5] = p.is5;
}

// The face between the fluid cells lo and up along D: the flux derivatives
// with respect to both cells' values times g = (W_lo - W_up) / h, the weight
// of the flux in the outputs, added to L and U.
template <int D>
__device__ __forceinline__ void face_adj(const AdjParams& p, const double (&lo)[NF], double nlo,
                                         const double (&Wl)[NF], const double (&up)[NF],
                                         double nup, const double (&Wu)[NF], AdjAcc& L,
                                         AdjAcc& U) {
  double g0[NF], is[NF];
  field_coef(p, g0, is);
  const double ihd = p.ih[D];
  const double Uf = 0.5 * (lo[D] + up[D]);
  const double nutf = 0.5 * (nlo + nup);
  // the upwind value is the lower cell's for Uf >= 0
  const bool pos = Uf >= 0.0;
  const double Up = pos ? Uf : 0.0, Un = pos ? 0.0 : Uf;
  double dU = 0.0, dn = 0.0;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const double g = ihd * (Wl[f] - Wu[f]);
    const double df = (g0[f] + nutf * is[f]) * ihd;
    L.x[f] -= g * (Up + df);
    U.x[f] += g * (df - Un);
    dU -= g * ((pos ? lo[f] : up[f]) + (f == 3 ? p.T_ref : 0.0));
    dn += g * is[f] * (up[f] - lo[f]);
    if (f == D) {
      // -(p + 2/3 k)_f on the faces normal to momentum component D
      L.pb -= 0.5 * g;
      U.pb -= 0.5 * g;
      if (p.komega) {
        L.x[4] -= g * (1.0 / 3.0);
        U.x[4] -= g * (1.0 / 3.0);
      }
    }
  }
  dU *= 0.5;
  dn *= 0.5 * ihd;
  L.x[D] += dU;
  U.x[D] += dU;
  L.nb += dn;
  U.nb += dn;
}

// The boundary face of fluid cell c on side s (0: -, 1: +) along d, whose
// outer values are ghosts of c: the flux derivatives through both sides, and
// this cell's own strain rate through the ghost velocities (lam: 4 Lambda
// S_ad of the cell, a = 0 .. 2).
__device__ __forceinline__ void ghost_face_adj(const AdjParams& p, const DevPatch& pp, int d,
                                               int s, const AdjCell& c, const double (&Wc)[NF],
                                               const double (&lam)[3], AdjAcc& A) {
  double g0[NF], is[NF];
  field_coef(p, g0, is);
  const int komega = p.komega;
  const double sg = s ? 1.0 : -1.0;
  const double ihd = d == 0 ? p.ih[0] : (d == 1 ? p.ih[1] : p.ih[2]);
  double n[NF], gs[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    n[f] = ghost<double>(pp, ghost_code(f), c.v[f], komega);
    gs[f] = slope(pp, ghost_code(f), komega);
  }
  const double nn = ghost<double>(pp, G_NUT, c.nu, komega);
  const double gp = slope(pp, G_P, komega), gn = slope(pp, G_NUT, komega);
  auto at = [&](const double (&a)[NF]) { return d == 0 ? a[0] : (d == 1 ? a[1] : a[2]); };
  const double Uf = 0.5 * (at(c.v) + at(n));
  const double nutf = 0.5 * (c.nu + nn);
  const bool own_up = (Uf >= 0.0) == (s == 1);
  double dU = 0.0, dn = 0.0;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const double wf = sg * ihd * Wc[f];
    const double lower = s ? c.v[f] : n[f], upper = s ? n[f] : c.v[f];
    const double up = Uf >= 0.0 ? lower : upper;
    const double gam = g0[f] + nutf * is[f];
    const double dup = own_up ? 1.0 : gs[f];
    A.x[f] += wf * (-Uf * dup + gam * sg * (gs[f] - 1.0) * ihd);
    dU += wf * (-up - (f == 3 ? p.T_ref : 0.0));
    dn += wf * is[f] * (upper - lower) * ihd;
  }
  const double dUo = dU * 0.5 * (1.0 + at(gs));
  const double wd = sg * ihd * at(Wc);
  const double f2 = sg * (d == 0 ? p.ih2[0] : (d == 1 ? p.ih2[1] : p.ih2[2]));
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (a == d) A.x[a] += dUo;
    if (komega && (a < 2 || p.d3)) A.x[a] += lam[a] * f2 * gs[a];
  }
  A.nb += dn * 0.5 * (1.0 + gn);
  A.pb += wd * -0.5 * (1.0 + gp);
  if (komega) A.x[4] += wd * (-1.0 / 3.0) * (1.0 + gs[4]);
}

// alpha* = (a0 + x) / (1 + x), x = Re_t / R_k; alpha = a_inf (A0 + y) / (1 + y),
// y = Re_t / R_w; Re_t = k / (nu omega-hat).
__device__ __forceinline__ void adj_closure(const AdjParams& p, double k, double w,
                                            AdjClosure& c) {
  const bool live = w > C_EPS;
  const double ioh = 1.0 / (live ? w : C_EPS);
  const double ki = k * ioh, ret = ki * p.inu, ri = ret * ioh;
  const double a0 = C_BETA_I / 3.0;
  const double x = ret * (1.0 / C_R_K), y = ret * (1.0 / C_R_W);
  const double ix = 1.0 / (1.0 + x), iy = 1.0 / (1.0 + y);
  const double as = (a0 + x) * ix;
  const double das = (1.0 - a0) * (1.0 / C_R_K) * ix * ix;  // d as / d Re_t
  const double da = C_A_INF * (1.0 - C_A0) * (1.0 / C_R_W) * iy * iy;
  c.nt = as * ki;
  c.dk = das * (p.inu * ioh) * ki + as * ioh;
  c.dw = live ? -(das * ri) * ki - as * ki * ioh : 0.0;
  c.al = C_A_INF * (C_A0 + y) * iy;
  c.ak = da * p.inu * ioh;
  c.aw = live ? -(da * ri) : 0.0;
}

__device__ __forceinline__ double adj_nut(const AdjParams& p, const AdjCell& c) {
  AdjClosure q;
  q.nt = 0.0;
  if (p.komega && is_fluid((uint8_t)c.t)) adj_closure(p, c.v[4], c.v[5], q);
  return q.nt;
}
}  // namespace

// The explicit stage's reverse mode: 153 bytes per cell (twelve dense arrays
// in and seven out, with the type byte: it was 603 with the state packed and
// the weights of every cell stored by one pass and gathered by another).
// Bound by latency at the two waves per SIMD that its live values leave (235
// VGPRs; about 900 vector instructions per cell and plane keep the vector
// units busy 45 % of the time): on the 512 x 256 x 128 room 1.52 ms per call,
// 1.7 TB/s of those bytes, from 3.65 ms for the two passes.  Measured and slower
// or no faster: predicated loads with zeroed defaults (1.88 ms, spills), 6 rows
// (2.03), 64-bit lane addresses (1.61), all array pointers kept in scalar
// registers (1.58).
__global__ __launch_bounds__(ABX* EX_RY, 2) void k_adj_explicit(ExplicitArgs a) {
  const AdjParams& p = a.p;
  const uint8_t* __restrict__ type = a.type;
  const DevPatch* __restrict__ pt = a.pt;
  // a plane's state (rows b + 1; rows 0 and EX_RY + 1: the rows past the
  // workgroup's sides), the weights of u, v, w, T, and those of k and omega
  // with the strain weights of the y differences.  The state and the first
  // weights alternate between two buffers, so two barriers per plane suffice:
  // a wave that stages plane m + 1 has passed the second barrier of plane m,
  // and the buffer it writes was last read before that wave's slowest
  // companion passed the first barrier of plane m.
  __shared__ double ls[2][7][EX_RY + 2][ABX];
  __shared__ double lw[2][4][EX_RY][ABX];
  __shared__ double lb[5][EX_RY][ABX];
  __shared__ uint8_t lt[2][EX_RY + 2][ABX];
  int tx, ty, tz;
  if (!adj_tile(p, tx, ty, tz)) return;  // (whole workgroup)
  // (a wave is one row: its index, and with it every row and plane offset,
  // is kept in scalar registers)
  const int lane = threadIdx.x, b = __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int i = tx * ADJ_TX - 2 + lane, j = ty * (EX_RY - 2) - 1 + b;
  // byte offsets in a dense row and a padded row of types, clamped
  const unsigned vi = 8u * (unsigned)min(max(i, 0), p.nx - 1);
  const unsigned vt = (unsigned)(min(max(i, -1), p.nx) + 1);
  const bool pi = i >= -1 && i <= p.nx, bi = i >= 0 && i < p.nx;
  const bool d3 = p.d3 != 0;
  const int k0 = tz * p.cz, k1 = min(p.nz, k0 + p.cz);
  const bool inner = b >= 1 && b <= (EX_RY - 2);  // rows with results (wave uniform)
  const bool res = inner && lane >= 2 && lane < 2 + ADJ_TX && bi && j < p.ny;
  const bool edge = b == 0 || b == EX_RY - 1;
  const int je = b == 0 ? j - 1 : j + 1, re = b == 0 ? 0 : EX_RY + 1;
  const size_t plane = (size_t)p.nx * p.ny;
  // Cell (i, r, m), every load unconditional at indices clamped into the
  // arrays: past the padded array the type reads as solid, and the values of
  // a cell that is not fluid are never used.
  auto load = [&](int r, int m, AdjCell& c) {
    const int rq = min(max(r, 0), p.ny - 1), mq = min(max(m, 0), p.nz - 1);
    const size_t D = mq * plane + (size_t)rq * p.nx;
    const auto io = explicit_io();
    c.v[0] = *row_at(io->u + D, vi);
    c.v[1] = *row_at(io->v + D, vi);
    c.v[2] = *row_at(io->w + D, vi);
    c.v[3] = *row_at(io->T + D, vi);
    c.v[4] = *row_at(io->k + D, vi);
    c.v[5] = *row_at(io->om + D, vi);
    c.t = adj_type(p, type, vt, pi, r, m);
    c.nu = 0.0;
  };
  auto load_bar = [&](int m, double (&y)[NF]) {
    const int rq = min(max(j, 0), p.ny - 1), mq = min(max(m, 0), p.nz - 1);
    const size_t D = mq * plane + (size_t)rq * p.nx;
    const auto io = explicit_io();
    y[0] = *row_at(io->ybu + D, vi);
    y[1] = *row_at(io->ybv + D, vi);
    y[2] = *row_at(io->ybw + D, vi);
    y[3] = *row_at(io->ybT + D, vi);
    y[4] = *row_at(io->ybk + D, vi);
    y[5] = *row_at(io->ybo + D, vi);
  };
  double g0[NF], is[NF];
  field_coef(p, g0, is);
  const int m0 = d3 ? k0 - 1 : 0, m1 = d3 ? k1 : 0;  // planes weighed
  // cc: the plane weighed, cp: the one above, ce: the plane's row past the
  // side; the plane below stays in the other LDS buffer
  AdjCell cc, cp, ce;
  load(j, m0 - 1, cc);
  cc.v[3] -= p.T_ref;
  cc.nu = adj_nut(p, cc);
#pragma unroll
  for (int f = 0; f < NF; ++f) ls[1][f][b + 1][lane] = cc.v[f];
  ls[1][6][b + 1][lane] = cc.nu;
  lt[1][b + 1][lane] = (uint8_t)cc.t;
  load(j, m0, cc);
  load(j, m0 + 1, cp);
  if (edge) load(je, m0, ce);
  double y[NF];
  load_bar(m0, y);
  cc.v[3] -= p.T_ref;
  cc.nu = adj_nut(p, cc);
  // the plane below: its weights, strain weights of the z differences,
  // closure derivatives and partial result
  double Wp4 = 0, Wp5 = 0, Lzp[3] = {0, 0, 0}, dkp = 0, dwp = 0;
  AdjAcc ap;
#pragma unroll
  for (int f = 0; f < NF; ++f) ap.x[f] = 0.0;
  ap.nb = ap.pb = 0.0;
  bool fp = false;  // the cell below is fluid
  auto store = [&](int m) {
    if (fp && p.komega) {
      // nu_t is the closure of this cell's k and omega
      ap.x[4] += ap.nb * dkp;
      ap.x[5] += ap.nb * dwp;
    }
    if (res) {
      const size_t D = m * plane + (size_t)j * p.nx;
      const auto io = explicit_io();
      *row_at(io->xu + D, vi) = ap.x[0];
      *row_at(io->xv + D, vi) = ap.x[1];
      *row_at(io->xw + D, vi) = ap.x[2];
      *row_at(io->xp + D, vi) = ap.pb;
      *row_at(io->xT + D, vi) = ap.x[3];
      *row_at(io->xk + D, vi) = ap.x[4];
      *row_at(io->xo + D, vi) = ap.x[5];
    }
  };
  for (int m = m0, buf = 0; m <= m1; ++m, buf ^= 1) {
    const bool fc = is_fluid((uint8_t)cc.t);
    // ---- stage the plane
#pragma unroll
    for (int f = 0; f < NF; ++f) ls[buf][f][b + 1][lane] = cc.v[f];
    ls[buf][6][b + 1][lane] = cc.nu;
    lt[buf][b + 1][lane] = (uint8_t)cc.t;
    if (edge) {
      ce.v[3] -= p.T_ref;
      ce.nu = adj_nut(p, ce);
#pragma unroll
      for (int f = 0; f < NF; ++f) ls[buf][f][re][lane] = ce.v[f];
      ls[buf][6][re][lane] = ce.nu;
      lt[buf][re][lane] = (uint8_t)ce.t;
    }
    double W[NF];
#pragma unroll
    for (int a = 0; a < 3; ++a) W[a] = fc && (a < 2 || d3) ? p.dt * y[a] : 0.0;
    W[3] = fc && p.energy ? p.dt * y[3] : 0.0;
    W[4] = W[5] = 0.0;
#pragma unroll
    for (int f = 0; f < 4; ++f) lw[buf][f][b][lane] = W[f];
    __syncthreads();
    cp.v[3] -= p.T_ref;
    cp.nu = adj_nut(p, cp);
    const int tzl = lt[buf ^ 1][b + 1][lane];
    // ---- weights of this plane's outputs
    AdjCell xl, xh;  // the x neighbours
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      xl.v[f] = lane_below(cc.v[f]);
      xh.v[f] = lane_above(cc.v[f]);
    }
    xl.nu = lane_below(cc.nu);
    xh.nu = lane_above(cc.nu);
    xl.t = lane_below(cc.t);
    xh.t = lane_above(cc.t);
    const int tyl = lt[buf][b][lane], tyh = lt[buf][b + 2][lane];
    AdjAcc A;
#pragma unroll
    for (int f = 0; f < NF; ++f) A.x[f] = y[f];
    A.nb = A.pb = 0.0;
    double L4[6] = {0, 0, 0, 0, 0, 0}, dkc = 0.0, dwc = 0.0;  // S00 S11 S22 S01 S02 S12
    if (fc && p.komega) {
      double rk = 0.0, rw = 0.0;
      double G[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          if (d == 2 && !d3) continue;
          double nv[3], nk, nw, nn;  // velocity, k, omega, nu_t across the face
          int tn;
          if (d == 1 || (d == 2 && s == 0)) {
            const int r = d == 2 ? b + 1 : (s ? b + 2 : b), bf = d == 2 ? buf ^ 1 : buf;
            nv[0] = ls[bf][0][r][lane];
            nv[1] = ls[bf][1][r][lane];
            nv[2] = ls[bf][2][r][lane];
            nk = ls[bf][4][r][lane];
            nw = ls[bf][5][r][lane];
            nn = ls[bf][6][r][lane];
            tn = d == 2 ? tzl : (s ? tyh : tyl);
          } else {
            const AdjCell& q = d == 0 ? (s ? xh : xl) : cp;
            nv[0] = q.v[0];
            nv[1] = q.v[1];
            nv[2] = q.v[2];
            nk = q.v[4];
            nw = q.v[5];
            nn = q.nu;
            tn = q.t;
          }
          if (!is_fluid((uint8_t)tn)) {
            const DevPatch& pp = pt[tn & 0x7f];
#pragma unroll
            for (int a = 0; a < 3; ++a) nv[a] = ghost<double>(pp, G_U + a, cc.v[a], p.komega);
            nk = ghost<double>(pp, G_K, cc.v[4], p.komega);
            nw = ghost<double>(pp, G_OM, cc.v[5], p.komega);
            nn = ghost<double>(pp, G_NUT, cc.nu, p.komega);
          }
          const double sg = s ? 1.0 : -1.0;
          const double Uf = 0.5 * (cc.v[d] + nv[d]);
          const double nutf = 0.5 * (cc.nu + nn);
          const bool own = (Uf >= 0.0) == (s == 1);
          rk += p.ih[d] * (-sg * Uf * (own ? cc.v[4] : nk) +
                           (p.nu + nutf * p.is4) * (nk - cc.v[4]) * p.ih[d]);
          rw += p.ih[d] * (-sg * Uf * (own ? cc.v[5] : nw) +
                           (p.nu + nutf * p.is5) * (nw - cc.v[5]) * p.ih[d]);
#pragma unroll
          for (int a = 0; a < 3; ++a)
            if (a < 2 || d3) G[a][d] += sg * p.ih2[d] * nv[a];
        }
      const double S[6] = {G[0][0],
                           G[1][1],
                           G[2][2],
                           0.5 * (G[0][1] + G[1][0]),
                           0.5 * (G[0][2] + G[2][0]),
                           0.5 * (G[1][2] + G[2][1])};
      const double S2 = 2.0 * (S[0] * S[0] + S[1] * S[1] + S[2] * S[2] +
                               2.0 * (S[3] * S[3] + S[4] * S[4] + S[5] * S[5]));
      AdjClosure q;
      adj_closure(p, cc.v[4], cc.v[5], q);
      dkc = q.dk;
      dwc = q.dw;
      const double kn = cc.v[4] + p.dt * (rk + cc.nu * S2);
      const double wn = cc.v[5] + p.dt * (rw + q.al * S2);
      const bool pk = kn > C_EPS;
      const bool fixed = (cc.t & FIXED_BIT) != 0;
      const bool pw = fixed || wn > C_EPS;
      W[4] = pk ? p.dt * y[4] : 0.0;
      W[5] = (!fixed && pw) ? p.dt * y[5] : 0.0;
      A.x[4] = pk ? y[4] : 0.0;
      A.x[5] = pw ? y[5] : 0.0;
      const double lam4 = 4.0 * (W[4] * cc.nu + W[5] * q.al);
#pragma unroll
      for (int r = 0; r < 6; ++r) L4[r] = lam4 * S[r];
      // production nu_t S^2 and alpha S^2 at this cell
      A.nb = W[4] * S2;
      A.x[4] += W[5] * S2 * q.ak;
      A.x[5] += W[5] * S2 * q.aw;
    }
    lb[0][b][lane] = W[4];
    lb[1][b][lane] = W[5];
    lb[2][b][lane] = L4[3];
    lb[3][b][lane] = L4[1];
    lb[4][b][lane] = L4[5];
    __syncthreads();
    // loads of the next plane weighed (its upper neighbour, adjoints and the
    // row past the side), used after the next barriers
    AdjCell cn;
    double yn[NF];
    load(j, m + 2, cn);
    load_bar(m + 1, yn);
    if (edge) load(je, m + 1, ce);
    if (inner) {
      // ---- the face and the strain rates between the plane below and this one
      if (d3 && m > k0 - 1) {
        if (fp && fc) {
          double nv[NF], Wn[NF];
#pragma unroll
          for (int f = 0; f < NF; ++f) nv[f] = ls[buf ^ 1][f][b + 1][lane];
#pragma unroll
          for (int f = 0; f < 4; ++f) Wn[f] = lw[buf ^ 1][f][b][lane];
          Wn[4] = Wp4;
          Wn[5] = Wp5;
          face_adj<2>(p, nv, ls[buf ^ 1][6][b + 1][lane], Wn, cc.v, cc.nu, W, ap, A);
        }
        if (fp) {
          ap.x[0] -= L4[4] * p.ih2[2];
          ap.x[1] -= L4[5] * p.ih2[2];
          ap.x[2] -= L4[2] * p.ih2[2];
        }
        if (fc) {
          A.x[0] += Lzp[0] * p.ih2[2];
          A.x[1] += Lzp[1] * p.ih2[2];
          A.x[2] += Lzp[2] * p.ih2[2];
        }
        if (m > k0) store(m - 1);
      }
      // ---- within the plane
      if (m >= k0 && m < k1) {
        // x faces: each lane takes its lower face and hands the lower cell's
        // part to the lane below
        {
          double Wl[NF];
#pragma unroll
          for (int f = 0; f < NF; ++f) Wl[f] = lane_below(W[f]);
          AdjAcc lo;
#pragma unroll
          for (int f = 0; f < NF; ++f) lo.x[f] = 0.0;
          lo.nb = lo.pb = 0.0;
          if (fc && is_fluid((uint8_t)xl.t))
            face_adj<0>(p, xl.v, xl.nu, Wl, cc.v, cc.nu, W, lo, A);
#pragma unroll
          for (int f = 0; f < NF; ++f) A.x[f] += lane_above(lo.x[f]);
          A.nb += lane_above(lo.nb);
          A.pb += lane_above(lo.pb);
        }
        // strain rates of the x neighbours (0 where they are not fluid)
        const double sx0 = lane_below(L4[0]) - lane_above(L4[0]);
        const double sx1 = lane_below(L4[3]) - lane_above(L4[3]);
        const double sx2 = lane_below(L4[4]) - lane_above(L4[4]);
        if (fc) {
          A.x[0] += sx0 * p.ih2[0];
          A.x[1] += sx1 * p.ih2[0];
          A.x[2] += sx2 * p.ih2[0];
          // y faces and the y neighbours' strain rates
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int r = s ? b + 2 : b, q = s ? b + 1 : b - 1;
            if (is_fluid((uint8_t)(s ? tyh : tyl))) {
              double nv[NF], Wn[NF];
#pragma unroll
              for (int f = 0; f < NF; ++f) nv[f] = ls[buf][f][r][lane];
              const double nn = ls[buf][6][r][lane];
#pragma unroll
              for (int f = 0; f < 4; ++f) Wn[f] = lw[buf][f][q][lane];
              Wn[4] = lb[0][q][lane];
              Wn[5] = lb[1][q][lane];
              AdjAcc other;
#pragma unroll
              for (int f = 0; f < NF; ++f) other.x[f] = 0.0;
              other.nb = other.pb = 0.0;
              if (s)
                face_adj<1>(p, cc.v, cc.nu, W, nv, nn, Wn, A, other);
              else
                face_adj<1>(p, nv, nn, Wn, cc.v, cc.nu, W, other, A);
              const double f2 = s ? -p.ih2[1] : p.ih2[1];
              A.x[0] += lb[2][q][lane] * f2;
              A.x[1] += lb[3][q][lane] * f2;
              A.x[2] += lb[4][q][lane] * f2;
            }
          }
          // boundary faces
          unsigned gm = (!is_fluid((uint8_t)xl.t) ? 1u : 0u) | (!is_fluid((uint8_t)xh.t) ? 2u : 0u) |
                        (!is_fluid((uint8_t)tyl) ? 4u : 0u) | (!is_fluid((uint8_t)tyh) ? 8u : 0u);
          if (d3)
            gm |= (!is_fluid((uint8_t)tzl) ? 16u : 0u) | (!is_fluid((uint8_t)cp.t) ? 32u : 0u);
          while (gm) {
            const int q = __ffs(gm) - 1;
            gm &= gm - 1;
            const int d = q >> 1, s = q & 1;
            const int tn = q == 0 ? xl.t : (q == 1 ? xh.t : (q == 2 ? tyl : (q == 3 ? tyh : (q == 4 ? tzl : cp.t))));
            const double lam[3] = {d == 0 ? L4[0] : (d == 1 ? L4[3] : L4[4]),
                                   d == 0 ? L4[3] : (d == 1 ? L4[1] : L4[5]),
                                   d == 0 ? L4[4] : (d == 1 ? L4[5] : L4[2])};
            ghost_face_adj(p, pt[tn & 0x7f], d, s, cc, W, lam, A);
          }
          // buoyancy -beta_T theta g_a
          if (p.buoyancy) A.x[3] += W[0] * p.bg[0] + W[1] * p.bg[1] + W[2] * p.bg[2];
        }
      }
    }
    // ---- this plane becomes the one below
    Wp4 = W[4];
    Wp5 = W[5];
#pragma unroll
    for (int f = 0; f < NF; ++f) y[f] = yn[f];
    Lzp[0] = L4[4];
    Lzp[1] = L4[5];
    Lzp[2] = L4[2];
    dkp = dkc;
    dwp = dwc;
    ap = A;
    fp = fc;
    cc = cp;
    cp = cn;
  }
  if (!d3 && inner) store(0);
}

void launch_explicit_adjoint(const Geom& g, const Phys& ph, const uint8_t* type,
                             const DevPatch* pt, const double* const st[6],
                             const double* const yb[6], double* const xb[7], hipStream_t s) {
  const ExplicitArgs a{{st[0], st[1], st[2], st[3], st[4], st[5], yb[0], yb[1], yb[2], yb[3],
                        yb[4], yb[5], xb[0], xb[1], xb[2], xb[3], xb[4], xb[5], xb[6]},
                       adj_params(g, ph, EX_RY),
                       type,
                       pt};
  hipLaunchKernelGGL(k_adj_explicit, adj_grid(a.p), dim3(ABX, EX_RY), 0, s, a);
}

// ---- destruction step (Sec. 2.5, Algorithm 3, eqs. k_des_step, o_des_step,
// beta_star, o_des) ------------------------------------------------------------
// k' = k / Dk, Dk = 1 + tau beta*(Re_t) f_beta*(chi_k) omega, chi_k = (grad k .
// grad omega) / omega-hat^3; omega' = omega / Dw, Dw = 1 + tau beta_i
// f_beta(chi_omega) omega, chi_omega = |X| / (beta*_inf omega-hat)^3 with X
// the vortex stretching a^T S a - |a|^2 tr S (a the axial vector of the
// antisymmetric part of the velocity gradient, S its symmetric part); fixed
// cells keep omega, non-fluid cells keep both.  The weights of an output cell
// are the adjoints of its gradients: of grad k and grad omega (E, six values)
// and of the velocity gradient G (M, nine values); an input cell gathers its
// own terms and those of the gradients that read it.
namespace {
struct DesLocal {
  double dkn_k, dkn_w;     // d k' / d (own k, own omega), gradients held
  double dwn_w;            // d omega' / d own omega, gradient held
  double lam_k;            // d k' / d (grad k . grad omega)
  double lam_w;            // d omega' / d X
};

// The destruction at one fluid cell from its k, omega, the gradients of k
// and omega and the velocity gradient: the partial derivatives the reverse
// mode needs.
__device__ __forceinline__ DesLocal des_local(double inu, double tau, double kP, double wP,
                                              const double (&gk)[3], const double (&gw)[3],
                                              const double (&G)[3][3], bool fixed) {
  DesLocal r;
  const bool live = wP > C_EPS;
  const double oh = live ? wP : C_EPS;
  const double ioh = 1.0 / oh, ioh3 = ioh * ioh * ioh;
  const double dkdw = gk[0] * gw[0] + gk[1] * gw[1] + gk[2] * gw[2];
  const double chik = dkdw * ioh3;
  const double iq = 1.0 / (1.0 + 400.0 * chik * chik);
  const double fbs = chik <= 0.0 ? 1.0 : (1.0 + 680.0 * chik * chik) * iq;
  const double dfbs = chik <= 0.0 ? 0.0 : 560.0 * chik * iq * iq;  // d fbs / d chi_k
  const double ret = kP * ioh * inu;
  const double x = ret * (1.0 / C_R_BETA);
  const double x4 = x * x * x * x;
  const double i4 = 1.0 / (1.0 + x4);
  const double bst = C_BSTAR * (1.0 - (11.0 / 15.0) * i4);
  const double dbst = C_BSTAR * (11.0 / 15.0) * i4 * i4 * 4.0 * x * x * x *
                      (1.0 / C_R_BETA);  // d bst / d ret
  const double iDk = 1.0 / (1.0 + tau * bst * fbs * wP);
  const double dDk = -kP * iDk * iDk;  // d k' / d Dk
  const double dret_k = ioh * inu, dret_w = live ? -ret * ioh : 0.0;
  const double dchik_w = live ? -3.0 * chik * ioh : 0.0;
  r.dkn_k = iDk + dDk * tau * fbs * wP * dbst * dret_k;
  r.dkn_w = dDk * tau * (bst * fbs + fbs * wP * dbst * dret_w + bst * wP * dfbs * dchik_w);
  r.lam_k = dDk * tau * bst * wP * dfbs * ioh3;
  r.dwn_w = 1.0;
  r.lam_w = 0.0;
  if (!fixed) {
    const double a0 = 0.5 * (G[2][1] - G[1][2]), a1 = 0.5 * (G[0][2] - G[2][0]),
                 a2 = 0.5 * (G[1][0] - G[0][1]);
    const double s01 = 0.5 * (G[0][1] + G[1][0]), s02 = 0.5 * (G[0][2] + G[2][0]),
                 s12 = 0.5 * (G[1][2] + G[2][1]);
    const double aSa = a0 * a0 * G[0][0] + a1 * a1 * G[1][1] + a2 * a2 * G[2][2] +
                       2.0 * (a0 * a1 * s01 + a0 * a2 * s02 + a1 * a2 * s12);
    const double X = aSa - (a0 * a0 + a1 * a1 + a2 * a2) * (G[0][0] + G[1][1] + G[2][2]);
    const double c3 = 1.0 / (C_BSTAR * C_BSTAR * C_BSTAR);
    const double chiw = fabs(X) * ioh3 * c3;
    const double i8 = 1.0 / (1.0 + 80.0 * chiw);
    const double fb = (1.0 + 70.0 * chiw) * i8;
    const double dfb = -10.0 * i8 * i8;
    const double iDw = 1.0 / (1.0 + tau * C_BETA_I * fb * wP);
    const double dfbw = -tau * C_BETA_I * wP * wP * iDw * iDw;  // d omega' / d fb
    r.dwn_w = iDw * iDw + dfbw * dfb * (live ? -3.0 * chiw * ioh : 0.0);
    const double sgn = X > 0.0 ? 1.0 : (X < 0.0 ? -1.0 : 0.0);
    r.lam_w = dfbw * dfb * sgn * ioh3 * c3;
  }
  return r;
}

// d X / d G_pq = a_p a_q - |a|^2 delta_pq + the part through a (the axial
// vector), with dX/da = 2 S a - 2 a tr S
__device__ __forceinline__ void stretch_grad(const double (&G)[3][3], double (&dX)[3][3]) {
  const double a[3] = {0.5 * (G[2][1] - G[1][2]), 0.5 * (G[0][2] - G[2][0]),
                       0.5 * (G[1][0] - G[0][1])};
  double S[3][3];
  for (int p = 0; p < 3; ++p)
    for (int q = 0; q < 3; ++q) S[p][q] = 0.5 * (G[p][q] + G[q][p]);
  const double tr = S[0][0] + S[1][1] + S[2][2];
  const double aa = a[0] * a[0] + a[1] * a[1] + a[2] * a[2];
  double ga[3];
  for (int p = 0; p < 3; ++p)
    ga[p] = 2.0 * (S[p][0] * a[0] + S[p][1] * a[1] + S[p][2] * a[2]) - 2.0 * a[p] * tr;
  for (int p = 0; p < 3; ++p)
    for (int q = 0; q < 3; ++q) dX[p][q] = a[p] * a[q] - (p == q ? aa : 0.0);
  dX[2][1] += 0.5 * ga[0];
  dX[1][2] -= 0.5 * ga[0];
  dX[0][2] += 0.5 * ga[1];
  dX[2][0] -= 0.5 * ga[1];
  dX[1][0] += 0.5 * ga[2];
  dX[0][1] -= 0.5 * ga[2];
}

constexpr int ND = 5;  // u v w k omega
__device__ __forceinline__ int des_code(int f) {
  return f < 3 ? G_U + f : (f == 3 ? G_K : G_OM);
}
struct DesIo {
  const double* s[ND];        // state u v w k omega, dense
  const double *kb, *wb;      // adjoints of k' and omega', dense
  double* x[ND];              // adjoints of the inputs, dense
};
struct DesCell {
  double v[ND];
  int t;
};
}  // namespace

// The destruction step's reverse mode: 97 bytes per cell (it was 474 with the
// fifteen weights of every cell stored and gathered).  Bound by latency at
// three waves per SIMD (vector units busy 44 % of the time): 0.78 ms per call on
// the 512 x 256 x 128 room, from 2.71 ms for the two passes.  Four waves per
// SIMD (128 VGPRs) spill 130 registers: 2.16 ms.
__global__ __launch_bounds__(ABX* DS_RY, 3) void k_adj_destroy(AdjParams p,
                                                            const uint8_t* __restrict__ type,
                                                            const DevPatch* __restrict__ pt,
                                                            double tau, DesIo io) {
  // a plane's state (rows b + 1; rows 0 and DS_RY + 1: the rows past the
  // workgroup's sides) and the weights of its y differences.  The state
  // alternates between two buffers, the other one holding the plane below.
  // It is read between the two barriers of a plane and the weights after the
  // second, so each is overwritten only after a barrier that follows its
  // last reader.
  __shared__ double ls[2][ND][DS_RY + 2][ABX];
  __shared__ double ly[ND][DS_RY][ABX];
  __shared__ uint8_t lt[2][DS_RY + 2][ABX];
  int tx, ty, tz;
  if (!adj_tile(p, tx, ty, tz)) return;  // (whole workgroup)
  const int lane = threadIdx.x, b = __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int i = tx * ADJ_TX - 2 + lane, j = ty * (DS_RY - 2) - 1 + b;
  // byte offsets in a dense row and a padded row of types, clamped
  const unsigned vi = 8u * (unsigned)min(max(i, 0), p.nx - 1);
  const unsigned vt = (unsigned)(min(max(i, -1), p.nx) + 1);
  const bool pi = i >= -1 && i <= p.nx, bi = i >= 0 && i < p.nx;
  const bool d3 = p.d3 != 0;
  const int k0 = tz * p.cz, k1 = min(p.nz, k0 + p.cz);
  const bool inner = b >= 1 && b <= (DS_RY - 2);  // rows with results (wave uniform)
  const bool res = inner && lane >= 2 && lane < 2 + ADJ_TX && bi && j < p.ny;
  const bool edge = b == 0 || b == DS_RY - 1;
  const int je = b == 0 ? j - 1 : j + 1, re = b == 0 ? 0 : DS_RY + 1;
  const size_t plane = (size_t)p.nx * p.ny;
  // (loads as in k_adj_explicit)
  auto load = [&](int r, int m, DesCell& c) {
    const int rq = min(max(r, 0), p.ny - 1), mq = min(max(m, 0), p.nz - 1);
    const size_t D = mq * plane + (size_t)rq * p.nx;
#pragma unroll
    for (int f = 0; f < ND; ++f) c.v[f] = *row_at(io.s[f] + D, vi);
    c.t = adj_type(p, type, vt, pi, r, m);
  };
  const int m0 = d3 ? k0 - 1 : 0, m1 = d3 ? k1 : 0;  // planes weighed
  // cc: the plane weighed, cp: the one above, ce: the plane's row past the
  // side; the plane below stays in the other LDS buffer
  DesCell cc, cp, ce;
  load(j, m0 - 1, cc);
#pragma unroll
  for (int f = 0; f < ND; ++f) ls[1][f][b + 1][lane] = cc.v[f];
  lt[1][b + 1][lane] = (uint8_t)cc.t;
  load(j, m0, cc);
  load(j, m0 + 1, cp);
  if (edge) load(je, m0, ce);
  double kb, wb;
  auto load_bar = [&](int m, double& a, double& c) {
    const int rq = min(max(j, 0), p.ny - 1), mq = min(max(m, 0), p.nz - 1);
    const size_t D = mq * plane + (size_t)rq * p.nx;
    a = *row_at(io.kb + D, vi);
    c = *row_at(io.wb + D, vi);
  };
  load_bar(m0, kb, wb);
  // the plane below: partial result and weights of its z differences
  double xp[ND] = {0, 0, 0, 0, 0}, zp[ND] = {0, 0, 0, 0, 0};
  bool fp = false;
  auto store = [&](int m) {
    const size_t D = m * plane + (size_t)j * p.nx;
    if (res)
#pragma unroll
      for (int f = 0; f < ND; ++f) *row_at(io.x[f] + D, vi) = xp[f];
  };
  for (int m = m0, buf = 0; m <= m1; ++m, buf ^= 1) {
    const bool fc = is_fluid((uint8_t)cc.t);
#pragma unroll
    for (int f = 0; f < ND; ++f) ls[buf][f][b + 1][lane] = cc.v[f];
    lt[buf][b + 1][lane] = (uint8_t)cc.t;
    if (edge) {
#pragma unroll
      for (int f = 0; f < ND; ++f) ls[buf][f][re][lane] = ce.v[f];
      lt[buf][re][lane] = (uint8_t)ce.t;
    }
    __syncthreads();
    const int tzl = lt[buf ^ 1][b + 1][lane];
    // ---- weights of this plane's outputs
    DesCell xl, xh;
#pragma unroll
    for (int f = 0; f < ND; ++f) {
      xl.v[f] = lane_below(cc.v[f]);
      xh.v[f] = lane_above(cc.v[f]);
    }
    xl.t = lane_below(cc.t);
    xh.t = lane_above(cc.t);
    const int tyl = lt[buf][b][lane], tyh = lt[buf][b + 2][lane];
    double x[ND] = {0.0, 0.0, 0.0, kb, wb};
    // weights by direction of the difference: u, v, w (M), k, omega (E)
    double wx[ND] = {0, 0, 0, 0, 0}, wy[ND] = {0, 0, 0, 0, 0}, wz[ND] = {0, 0, 0, 0, 0};
    if (fc) {
      double gk[3] = {0, 0, 0}, gw[3] = {0, 0, 0};
      double G[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (d == 2 && !d3) continue;
        double n[2][ND];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          int tn;
          if (d == 1 || (d == 2 && s == 0)) {
            const int r = d == 2 ? b + 1 : (s ? b + 2 : b), bf = d == 2 ? buf ^ 1 : buf;
#pragma unroll
            for (int f = 0; f < ND; ++f) n[s][f] = ls[bf][f][r][lane];
            tn = d == 2 ? tzl : (s ? tyh : tyl);
          } else {
            const DesCell& q = d == 0 ? (s ? xh : xl) : cp;
#pragma unroll
            for (int f = 0; f < ND; ++f) n[s][f] = q.v[f];
            tn = q.t;
          }
          if (!is_fluid((uint8_t)tn)) {
            const DevPatch& pp = pt[tn & 0x7f];
#pragma unroll
            for (int f = 0; f < ND; ++f)
              n[s][f] = ghost<double>(pp, des_code(f), cc.v[f], p.komega);
          }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a)
          if (a < 2 || d3) G[a][d] = (n[1][a] - n[0][a]) * p.ih2[d];
        gk[d] = (n[1][3] - n[0][3]) * p.ih2[d];
        gw[d] = (n[1][4] - n[0][4]) * p.ih2[d];
      }
      const DesLocal r =
          des_local(p.inu, tau, cc.v[3], cc.v[4], gk, gw, G, (cc.t & FIXED_BIT) != 0);
      x[3] = kb * r.dkn_k;
      x[4] = kb * r.dkn_w + wb * r.dwn_w;
      const double lk = kb * r.lam_k;
      wx[3] = lk * gw[0];
      wy[3] = lk * gw[1];
      wz[3] = lk * gw[2];
      wx[4] = lk * gk[0];
      wy[4] = lk * gk[1];
      wz[4] = lk * gk[2];
      if (r.lam_w != 0.0) {
        double dX[3][3];
        stretch_grad(G, dX);
        const double lw = wb * r.lam_w;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          if (a == 2 && !d3) continue;
          wx[a] = lw * dX[a][0];
          wy[a] = lw * dX[a][1];
          wz[a] = lw * dX[a][2];
        }
      }
    }
#pragma unroll
    for (int f = 0; f < ND; ++f) ly[f][b][lane] = wy[f];
    __syncthreads();
    // loads of the next plane weighed (its upper neighbour, adjoints and the
    // row past the side), used after the next barrier
    DesCell cn;
    double kbn, wbn;
    load(j, m + 2, cn);
    load_bar(m + 1, kbn, wbn);
    if (edge) load(je, m + 1, ce);
    if (inner) {
      if (d3 && m > k0) {
        // the cell below reads this plane's differences
        if (fp)
#pragma unroll
          for (int f = 0; f < ND; ++f) xp[f] -= wz[f] * p.ih2[2];
        store(m - 1);
      }
      if (m >= k0 && m < k1) {
        // (every neighbour that is not fluid has weight 0)
        double gx[ND];
#pragma unroll
        for (int f = 0; f < ND; ++f)
          gx[f] = (lane_below(wx[f]) - lane_above(wx[f])) * p.ih2[0];
        if (fc) {
#pragma unroll
          for (int f = 0; f < ND; ++f) {
            x[f] += gx[f];
            x[f] += (ly[f][b - 1][lane] - ly[f][b + 1][lane]) * p.ih2[1];
            if (d3) x[f] += zp[f] * p.ih2[2];
          }
          // this cell's own gradients read it through the ghosts
          unsigned gm = (!is_fluid((uint8_t)xl.t) ? 1u : 0u) | (!is_fluid((uint8_t)xh.t) ? 2u : 0u) |
                        (!is_fluid((uint8_t)tyl) ? 4u : 0u) | (!is_fluid((uint8_t)tyh) ? 8u : 0u);
          if (d3)
            gm |= (!is_fluid((uint8_t)tzl) ? 16u : 0u) | (!is_fluid((uint8_t)cp.t) ? 32u : 0u);
          while (gm) {
            const int q = __ffs(gm) - 1;
            gm &= gm - 1;
            const int d = q >> 1;
            const int tn = q == 0 ? xl.t : (q == 1 ? xh.t : (q == 2 ? tyl : (q == 3 ? tyh : (q == 4 ? tzl : cp.t))));
            const DevPatch& pp = pt[tn & 0x7f];
            const double i2 = d == 0 ? p.ih2[0] : (d == 1 ? p.ih2[1] : p.ih2[2]);
            const double f2 = (q & 1) ? i2 : -i2;
#pragma unroll
            for (int f = 0; f < ND; ++f) {
              const double wo = d == 0 ? wx[f] : (d == 1 ? wy[f] : wz[f]);
              x[f] += wo * f2 * slope(pp, des_code(f), p.komega);
            }
          }
        }
      }
    }
#pragma unroll
    for (int f = 0; f < ND; ++f) {
      xp[f] = x[f];
      zp[f] = wz[f];
    }
    fp = fc;
    kb = kbn;
    wb = wbn;
    cc = cp;
    cp = cn;
  }
  if (!d3 && inner) store(0);
}

void launch_destroy_adjoint(const Geom& g, const Phys& ph, const uint8_t* type,
                            const DevPatch* pt, const double* const st[5], double tau,
                            const double* kb, const double* wb, double* const xb[5],
                            hipStream_t s) {
  const AdjParams p = adj_params(g, ph, DS_RY);
  DesIo io;
  for (int f = 0; f < ND; ++f) {
    io.s[f] = st[f];
    io.x[f] = xb[f];
  }
  io.kb = kb;
  io.wb = wb;
  hipLaunchKernelGGL(k_adj_destroy, adj_grid(p), dim3(ABX, DS_RY), 0, s, p, type, pt, tau, io);
}

// ---- helpers of the whole step's reverse mode ------------------------------------
__global__ void k_dense_add(size_t n, const double* __restrict__ a, const double* __restrict__ b,
                            double* __restrict__ out, double scale) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) out[q] = scale * (a[q] + b[q]);
}
// out = scale (a + b) over n dense values (scale 1 leaves the sum as formed)
void launch_dense_add(size_t n, const double* a, const double* b, double* out, hipStream_t s,
                      double scale) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_dense_add, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, a, b,
                     out, scale);
}

__global__ void k_zero_held(Geom g, const uint8_t* __restrict__ type, double* __restrict__ a) {
  const int i = blockIdx.x * ABX + threadIdx.x, j = blockIdx.y * ABY + threadIdx.y,
            k = blockIdx.z;
  if (i >= g.nx || j >= g.ny) return;
  const uint8_t t = type[g.idx(i, j, k)];
  if (is_fluid(t) && (t & FIXED_BIT)) a[((size_t)k * g.ny + j) * g.nx + i] = 0.0;
}
// zero the dense adjoint a on the wall-adjacent cells whose omega is held
void launch_zero_held(const Geom& g, const uint8_t* type, double* a, hipStream_t s) {
  const dim3 G((g.nx + ABX - 1) / ABX, (g.ny + ABY - 1) / ABY, g.nz), B(ABX, ABY);
  hipLaunchKernelGGL(k_zero_held, G, B, 0, s, g, type, a);
}

}  // namespace nfvm
