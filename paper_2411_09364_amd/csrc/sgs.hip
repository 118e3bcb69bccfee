// Eddy viscosity (Sec. 2.1, Eqs. smag, dsmag, cs, lij, mij; Sec. 2.2 SGS paragraph).
//
// Every Smagorinsky variant is stored as nu_t = coef[k] * S(k, j, i) where S = |S| at the
// cell centre and coef a per-plane factor:
//   static         coef = (C_s Delta_k)^2
//   van Driest     coef = (C_s Delta_k D_k)^2, D_k = 1 - exp(-y*/25) from the plane-mean
//                  wall stress of the nearer wall
//   dynamic        coef = c_s(k) Delta_k^2 with c_s from the plane-averaged Germano-Lilly
//                  identity (clipped at zero)
// so the predictor reads one field plus an nz-long vector.
//
// Strain ghosts: with the wall model, wall-parallel velocity ghosts for the strain are the
// linear extrapolation in z of the first two interior values (one-sided wall-normal
// derivative in the first layer, Sec. 2.2), and in a duct those of u and w in y as well;
// otherwise the stored ghosts are used.
//
// Ducts (walls in y too, Sec. 4.4): the van Driest factor takes y* as the smallest of
// d_w u_tau,w / nu over the four walls and is folded into the stored field (|S| D^2), so
// the plane coefficient stays (C_s Delta_k)^2.
#include "les_internal.h"
#include "mlp_core.h"

#include <algorithm>

namespace les {

template <typename T>
struct VelView {
  const T* u;
  const T* v;
  const T* w;
};

// u or v at (k, j, i) with the z strain ghost rule.
template <typename T>
__device__ inline T sval(const GridP& g, const T* f, int k, int j, int i) {
  if (g.zbc == LES_ZBC_WALLMODEL) {
    if (k == 0) {
      const T a1 = f[idx3(g, 1, j, i)], a2 = f[idx3(g, 2, j, i)];
      return a1 - (T)g.dzc[0] * ((a2 - a1) / (T)g.dzc[1]);
    }
    if (k == g.nz + 1) {
      const int n = g.nz;
      const T a1 = f[idx3(g, n, j, i)], a0 = f[idx3(g, n - 1, j, i)];
      return a1 + (T)g.dzc[n] * ((a1 - a0) / (T)g.dzc[n - 1]);
    }
  }
  return f[idx3(g, k, j, i)];
}

// u or w of a duct with the wall model on a y ghost row: the linear extrapolation in y of the
// first two interior rows (uniform dy), taken after the z rule (zr: apply it, for u).
template <typename T>
__device__ inline T sval_y(const GridP& g, const T* f, int k, int j, int i, bool zr) {
  auto at = [&](int jj) { return zr ? sval(g, f, k, jj, i) : f[idx3(g, k, jj, i)]; };
  if (g.ywall && g.zbc == LES_ZBC_WALLMODEL && j >= g.ny) {
    if (j == g.ny + 1) {
      const T a0 = at(0), a1 = at(1);
      return a0 - (a1 - a0);
    }
    const T a0 = at(g.ny - 1), a1 = at(g.ny - 2);
    return a0 + (a0 - a1);
  }
  return at(j);
}

// Strain rate at the centre of cell (k, j, i): s[0..5] = S11 S22 S33 S12 S13 S23.
template <typename T>
__device__ inline void centre_strain(const GridP& g, const T* u, const T* v, const T* w, int k, int j, int i, T s[6]) {
  const int ip = wrap_p(i, g.nx), im = wrap_m(i, g.nx), jp = wrap_p(j, g.nys), jm = wrap_m(j, g.nys);
  const T rdx = (T)g.rdx, rdy = (T)g.rdy, h = (T)0.5, q = (T)0.25;
  const T rdzc = (T)g.rdzc[k], rdzcm = (T)g.rdzc[k - 1];
#define US(kk, jj, ii) sval_y(g, u, kk, jj, ii, true)
#define VS(kk, jj, ii) sval(g, v, kk, jj, ii)
#define W(kk, jj, ii) sval_y(g, w, kk, jj, ii, false)
  const T u0 = US(k, j, i), uim = US(k, j, im), ujp = US(k, jp, i), ujm = US(k, jm, i);
  const T ujp_im = US(k, jp, im), ujm_im = US(k, jm, im);
  const T v0 = VS(k, j, i), vjm = VS(k, jm, i), vip = VS(k, j, ip), vim = VS(k, j, im);
  const T vjm_ip = VS(k, jm, ip), vjm_im = VS(k, jm, im);
  s[0] = (u0 - uim) * rdx;
  s[1] = (v0 - vjm) * rdy;
  s[2] = (W(k, j, i) - W(k - 1, j, i)) * (T)g.rdzf[k];
  const T e_a = h * ((ujp - u0) * rdy + (vip - v0) * rdx);           // (j, i)
  const T e_b = h * ((ujp_im - uim) * rdy + (v0 - vim) * rdx);       // (j, i-1)
  const T e_c = h * ((u0 - ujm) * rdy + (vjm_ip - vjm) * rdx);       // (j-1, i)
  const T e_d = h * ((uim - ujm_im) * rdy + (vjm - vjm_im) * rdx);   // (j-1, i-1)
  s[3] = q * (e_a + e_b + e_c + e_d);
  const T ukp = US(k + 1, j, i), ukm = US(k - 1, j, i), ukp_im = US(k + 1, j, im), ukm_im = US(k - 1, j, im);
  const T f_a = h * ((ukp - u0) * rdzc + (W(k, j, ip) - W(k, j, i)) * rdx);
  const T f_b = h * ((ukp_im - uim) * rdzc + (W(k, j, i) - W(k, j, im)) * rdx);
  const T f_c = h * ((u0 - ukm) * rdzcm + (W(k - 1, j, ip) - W(k - 1, j, i)) * rdx);
  const T f_d = h * ((uim - ukm_im) * rdzcm + (W(k - 1, j, i) - W(k - 1, j, im)) * rdx);
  s[4] = q * (f_a + f_b + f_c + f_d);
  const T vkp = VS(k + 1, j, i), vkm = VS(k - 1, j, i), vkp_jm = VS(k + 1, jm, i), vkm_jm = VS(k - 1, jm, i);
  const T g_a = h * ((vkp - v0) * rdzc + (W(k, jp, i) - W(k, j, i)) * rdy);
  const T g_b = h * ((vkp_jm - vjm) * rdzc + (W(k, j, i) - W(k, jm, i)) * rdy);
  const T g_c = h * ((v0 - vkm) * rdzcm + (W(k - 1, jp, i) - W(k - 1, j, i)) * rdy);
  const T g_d = h * ((vjm - vkm_jm) * rdzcm + (W(k - 1, j, i) - W(k - 1, jm, i)) * rdy);
  s[5] = q * (g_a + g_b + g_c + g_d);
#undef US
#undef VS
#undef W
}

template <typename T>
__device__ inline T strain_mag(const T s[6]) {
  return sqrt((T)2 * (s[0] * s[0] + s[1] * s[1] + s[2] * s[2]) + (T)4 * (s[3] * s[3] + s[4] * s[4] + s[5] * s[5]));
}

// Writes a cell-centred value and, on the first/last plane, the ghost plane of the
// eddy-viscosity field (odd about walls, R12; periodic copy otherwise).
template <typename T>
__device__ inline void store_nut(const GridP& g, T* nut, int k, int j, int i, T val) {
  nut[idx3(g, k, j, i)] = val;
  const int n = g.nz;
  if (g.zbc == LES_ZBC_PERIODIC) {
    if (k == n) nut[idx3(g, 0, j, i)] = val;
    if (k == 1) nut[idx3(g, n + 1, j, i)] = val;
  } else {
    if (k == 1) nut[idx3(g, 0, j, i)] = -val;
    if (k == n) nut[idx3(g, n + 1, j, i)] = -val;
  }
}

// ============================================================================ |S|
// One thread per (j, i) column of STRAIN_KZ planes, marching up: the differences across a plane
// face and an x-y edge are read by the cells on both sides, so 17 loads a cell instead of 30, with
// 32-bit offsets into the plane (row, row above and below, each at i - 1, i, i + 1).  Bound by the
// load and index instructions, not by its bytes: with a thread per cell and every ghost rule
// checked at every point a duct of 512 x 80 x 80 in FP64 took 62 us, now 42, 240 x 120 x 75 in
// FP32 27, now 18 (2 and 8 planes a thread: 47 and 43, 20 and 18).  The values that
// the wall model extrapolates follow from the ones at hand.  Sums of two products name their fused
// multiply-adds (the first product into the rounded second one): left to the compiler, the choice may
// change with the code around, and a batch and a single context have to agree to the last bit.
constexpr int STRAIN_KZ = 4;

template <typename T>
__device__ __forceinline__ void strain_column(const GridP& g, const T* __restrict__ u, const T* __restrict__ v,
                                              const T* __restrict__ w, T* __restrict__ nut,
                                              const double* fac, int j, int i, int k0, int kn) {
  const int nx = g.nx, jp = wrap_p(j, g.nys), jm = wrap_m(j, g.nys);
  const int ip = wrap_p(i, nx), im = wrap_m(i, nx);
  const int r0 = j * nx, rp = jp * nx, rm = jm * nx;
  const T rdx = (T)g.rdx, rdy = (T)g.rdy, h = (T)0.5, q = (T)0.25;
  auto edge = [&](T a, T ra, T b, T rb) { return h * fma(a, ra, b * rb); };
  const bool wm = g.zbc == LES_ZBC_WALLMODEL;
  // wall model in a duct: the ghost rows of u and w continue their first two rows (sval_y)
  const bool ylo = wm && g.ywall && j == 0, yhi = wm && g.ywall && j == g.ny - 1;
  auto rows = [&](T a, T& up, T& dn) {
    if (ylo) dn = a - (up - a);
    if (yhi) up = a + (a - dn);
  };
  int64_t pk = (int64_t)(k0 - 1) * g.sxy;
  // plane k0 - 1: w, u and v below; plane k0: u and v of the column's own rows
  const T *ub = u + pk, *vb = v + pk, *wb = w + pk;
  T ukm = ub[r0 + i], ukm_im = ub[r0 + im], vkm = vb[r0 + i], vkm_jm = vb[rm + i];
  T wk = wb[r0 + i], wx = wb[r0 + ip], wxm = wb[r0 + im], wy = wb[rp + i], wym = wb[rm + i];
  T u0 = ub[g.sxy + r0 + i], uim = ub[g.sxy + r0 + im], v0 = vb[g.sxy + r0 + i], vjm = vb[g.sxy + rm + i];
  rows(wk, wy, wym);
  if (wm && k0 == 1) {
    // wall model: u and v on the ghost planes continue their first two planes (sval)
    const T *u2 = u + 2 * g.sxy, *v2 = v + 2 * g.sxy, c = (T)g.dzc[0], e = (T)g.dzc[1];
    ukm = u0 - c * ((u2[r0 + i] - u0) / e), ukm_im = uim - c * ((u2[r0 + im] - uim) / e);
    vkm = v0 - c * ((v2[r0 + i] - v0) / e), vkm_jm = vjm - c * ((v2[rm + i] - vjm) / e);
  }
  for (int k = k0; k < kn; ++k) {
    pk += g.sxy;
    const T *uk = u + pk, *vk = v + pk, *wn = w + pk, *uu = uk + g.sxy, *vv = vk + g.sxy;
    T ukp = uu[r0 + i], ukp_im = uu[r0 + im], vkp = vv[r0 + i], vkp_jm = vv[rm + i];
    T ujp = uk[rp + i], ujp_im = uk[rp + im], ujm = uk[rm + i], ujm_im = uk[rm + im];
    const T vip = vk[r0 + ip], vim = vk[r0 + im], vjm_ip = vk[rm + ip], vjm_im = vk[rm + im];
    const T w0 = wn[r0 + i], wip = wn[r0 + ip], wim = wn[r0 + im];
    T wjp = wn[rp + i], wjm = wn[rm + i];
    rows(u0, ujp, ujm);
    rows(uim, ujp_im, ujm_im);
    rows(w0, wjp, wjm);
    if (wm && k == g.nz) {
      const T c = (T)g.dzc[k], e = (T)g.dzc[k - 1];
      ukp = u0 + c * ((u0 - ukm) / e), ukp_im = uim + c * ((uim - ukm_im) / e);
      vkp = v0 + c * ((v0 - vkm) / e), vkp_jm = vjm + c * ((vjm - vkm_jm) / e);
    }
    const T rdzc = (T)g.rdzc[k], rdzcm = (T)g.rdzc[k - 1];
    const T s0 = (u0 - uim) * rdx, s1 = (v0 - vjm) * rdy, s2 = (w0 - wk) * (T)g.rdzf[k];
    const T e_a = edge(ujp - u0, rdy, vip - v0, rdx), e_b = edge(ujp_im - uim, rdy, v0 - vim, rdx);
    const T e_c = edge(u0 - ujm, rdy, vjm_ip - vjm, rdx), e_d = edge(uim - ujm_im, rdy, vjm - vjm_im, rdx);
    const T s3 = q * (e_a + e_b + e_c + e_d);
    const T f_a = edge(ukp - u0, rdzc, wip - w0, rdx), f_b = edge(ukp_im - uim, rdzc, w0 - wim, rdx);
    const T f_c = edge(u0 - ukm, rdzcm, wx - wk, rdx), f_d = edge(uim - ukm_im, rdzcm, wk - wxm, rdx);
    const T s4 = q * (f_a + f_b + f_c + f_d);
    const T g_a = edge(vkp - v0, rdzc, wjp - w0, rdy), g_b = edge(vkp_jm - vjm, rdzc, w0 - wjm, rdy);
    const T g_c = edge(v0 - vkm, rdzcm, wy - wk, rdy), g_d = edge(vjm - vkm_jm, rdzcm, wk - wym, rdy);
    const T s5 = q * (g_a + g_b + g_c + g_d);
    T val = sqrt((T)2 * fma(s2, s2, fma(s0, s0, s1 * s1)) + (T)4 * fma(s5, s5, fma(s3, s3, s4 * s4)));
    if (fac != nullptr) val = (T)((double)val * fac[k - k0]);
    store_nut(g, nut, k, j, i, val);
    ukm = u0, ukm_im = uim, vkm = v0, vkm_jm = vjm;
    u0 = ukp, uim = ukp_im, v0 = vkp, vjm = vkp_jm;
    wk = w0, wx = wip, wxm = wim, wy = wjp, wym = wjm;
  }
}

// blocks of 32 x 8 columns, kz <= STRAIN_KZ planes
template <typename T>
__global__ void __launch_bounds__(256) k_strain_mag(GridP g, const T* __restrict__ u, const T* __restrict__ v,
                                                    const T* __restrict__ w, T* __restrict__ nut,
                                                    const double* __restrict__ vd4, double ly, int kz) {
  __shared__ double vdf[8][STRAIN_KZ];
  const int i = blockIdx.x * 32 + threadIdx.x, j = blockIdx.y * 8 + threadIdx.y;
  const int k0 = blockIdx.z * kz + 1, kn = min(k0 + kz, g.nz + 1);
  if (vd4 != nullptr) {
    // duct van Driest factors (four walls) of the block's rows and planes: y* the smallest d_w
    // u_tau,w / nu
    const int t = threadIdx.y * 32 + threadIdx.x;
    if (t < 8 * STRAIN_KZ) {
      const double zc = g.zc[min(k0 + t % STRAIN_KZ, g.nz)], yc = (blockIdx.y * 8 + t / STRAIN_KZ + 0.5) * g.dy;
      const double ys = fmin(fmin(zc * vd4[0], (g.lz - zc) * vd4[1]), fmin(yc * vd4[2], (ly - yc) * vd4[3])) / g.nu;
      const double d = 1.0 - exp(-ys / 25.0);
      vdf[t / STRAIN_KZ][t % STRAIN_KZ] = d * d;
    }
    __syncthreads();
  }
  if (i >= g.nx || j >= g.ny) return;
  const double* fac = vd4 != nullptr ? vdf[threadIdx.y] : nullptr;
  strain_column(g, u, v, w, nut, fac, j, i, k0, kn);
}

// Friction velocities of the four duct walls for the van Driest factor: sqrt(|(<tau_1>,
// <tau_2>)|) per wall, each component averaged over its own points on that wall that are not
// wall faces (z walls: rows j < ny, the v stress over j < ny - 1; y walls: planes 1..nz, the w
// stress over faces 1..nz-1).  Stresses from the wall models, or nu times the wall-normal
// difference across the no-slip ghosts.  Stage 1: VD_BLOCKS blocks, each a fixed-order tree
// of its strided share into 8 partials (part[b][8]); stage 2: one block sums them in block
// order and writes vd4 = (z bottom, z top, y = 0, y = ly).
constexpr int VD_BLOCKS = 64;

template <typename T>
__global__ void __launch_bounds__(256) k_vd_duct_partial(GridP g, const T* u, const T* v, const T* w,
                                                         const double* tau, const double* tauy, int wallmodel,
                                                         double* part) {
  __shared__ double sm[8][256];
  double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int n = g.nz, ny = g.ny, nx = g.nx;
  const int64_t s = g.sxy, sy = (int64_t)(n + 2) * nx;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t c = t0; c < (int64_t)nx * ny; c += stride) {
    const bool vrow = c < (int64_t)nx * (ny - 1);   // v rows off the wall face y = ly
    if (wallmodel) {
      a[0] += tau[c];
      a[2] += tau[2 * s + c];
      if (vrow) {
        a[1] += tau[s + c];
        a[3] += tau[3 * s + c];
      }
    } else {
      a[0] += g.nu * ((double)u[s + c] - (double)u[c]) / g.dzc[0];
      a[2] += g.nu * ((double)u[(int64_t)n * s + c] - (double)u[(int64_t)(n + 1) * s + c]) / g.dzc[n];
      if (vrow) {
        a[1] += g.nu * ((double)v[s + c] - (double)v[c]) / g.dzc[0];
        a[3] += g.nu * ((double)v[(int64_t)n * s + c] - (double)v[(int64_t)(n + 1) * s + c]) / g.dzc[n];
      }
    }
  }
  for (int64_t e = t0; e < (int64_t)nx * n; e += stride) {
    const int k = (int)(e / nx) + 1, i = (int)(e % nx);
    const bool wface = k < n;   // w faces off the wall face k = nz
    if (wallmodel) {
      const int64_t o = (int64_t)k * nx + i;
      a[4] += tauy[o];
      a[6] += tauy[2 * sy + o];
      if (wface) {
        a[5] += tauy[sy + o];
        a[7] += tauy[3 * sy + o];
      }
    } else {
      a[4] += g.nu * ((double)u[idx3(g, k, 0, i)] - (double)u[idx3(g, k, ny + 1, i)]) / g.dy;
      a[6] += g.nu * ((double)u[idx3(g, k, ny - 1, i)] - (double)u[idx3(g, k, ny, i)]) / g.dy;
      if (wface) {
        a[5] += g.nu * ((double)w[idx3(g, k, 0, i)] - (double)w[idx3(g, k, ny + 1, i)]) / g.dy;
        a[7] += g.nu * ((double)w[idx3(g, k, ny - 1, i)] - (double)w[idx3(g, k, ny, i)]) / g.dy;
      }
    }
  }
  for (int q = 0; q < 8; ++q) sm[q][threadIdx.x] = a[q];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int q = 0; q < 8; ++q) sm[q][threadIdx.x] += sm[q][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 8) part[blockIdx.x * 8 + threadIdx.x] = sm[threadIdx.x][0];
}

// sums of q-strided block partials (nq per block, VD_BLOCKS = 64 blocks: one lane each) by a
// fixed-order shuffle tree within one wave; lane 0 holds the totals
__device__ inline void wave_block_sums(const double* part, int nq, double* a) {
  const int lane = threadIdx.x & 63;
  for (int q = 0; q < nq; ++q) {
    double x = lane < VD_BLOCKS ? part[lane * nq + q] : 0.0;
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    a[q] = x;
  }
}

// cnt (learned closure, may be null): the fallback counters are cleared here, ahead of the
// inference kernel that adds to them.
__global__ void k_vd_duct_final(GridP g, const double* part, double* vd4, int* cnt) {
  static_assert(VD_BLOCKS <= 64, "one lane per block partial");
  double a[8];
  wave_block_sums(part, 8, a);
  if (threadIdx.x != 0) return;
  if (cnt != nullptr) {
    cnt[0] = 0;
    cnt[1] = 0;
  }
  const double nx = g.nx, ny = g.ny, n = g.nz;
  const double cz = nx * ny, cv = nx * (ny - 1), cy = nx * n, cw = nx * (n - 1);
  vd4[0] = sqrt(hypot(a[0] / cz, a[1] / cv));
  vd4[1] = sqrt(hypot(a[2] / cz, a[3] / cv));
  vd4[2] = sqrt(hypot(a[4] / cy, a[5] / cw));
  vd4[3] = sqrt(hypot(a[6] / cy, a[7] / cw));
}

// van Driest coefficient: plane-mean wall stresses -> u_tau per wall -> coef[k].
// tau = wall-model stresses, or (no-slip) nu (u_1 - u_0)/dzc_0 from the ghosts.  Stage 1:
// VD_BLOCKS blocks of fixed-order partials of the four plane sums (part[b][4]); stage 2, one
// block: the sums in block order, u_tau per wall, then coef[k] for every plane.
template <typename T>
__global__ void __launch_bounds__(256) k_vd_coef_partial(GridP g, const T* u, const T* v, const double* tau,
                                                         int wallmodel, double* part) {
  __shared__ double sm[4][256];
  double a[4] = {0, 0, 0, 0};
  const int64_t s = g.sxy;
  const int n = g.nz;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < s; c += stride) {
    if (wallmodel) {
      for (int q = 0; q < 4; ++q) a[q] += tau[q * s + c];
    } else {
      a[0] += g.nu * ((double)u[s + c] - (double)u[c]) / g.dzc[0];
      a[1] += g.nu * ((double)v[s + c] - (double)v[c]) / g.dzc[0];
      a[2] += g.nu * ((double)u[(int64_t)n * s + c] - (double)u[(int64_t)(n + 1) * s + c]) / g.dzc[n];
      a[3] += g.nu * ((double)v[(int64_t)n * s + c] - (double)v[(int64_t)(n + 1) * s + c]) / g.dzc[n];
    }
  }
  for (int q = 0; q < 4; ++q) sm[q][threadIdx.x] = a[q];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int q = 0; q < 4; ++q) sm[q][threadIdx.x] += sm[q][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = sm[threadIdx.x][0];
}

__global__ void __launch_bounds__(256) k_vd_coef_final(GridP g, const double* part, double cs,
                                                       double* coef) {
  __shared__ double ut[2];
  const int n = g.nz;
  double a[4];
  if (threadIdx.x < 64) wave_block_sums(part, 4, a);
  if (threadIdx.x == 0) {
    const double s = (double)g.sxy;
    ut[0] = sqrt(hypot(a[0] / s, a[1] / s));
    ut[1] = sqrt(hypot(a[2] / s, a[3] / s));
  }
  __syncthreads();
  for (int k = threadIdx.x + 1; k <= n; k += blockDim.x) {
    const double zc = g.zc[k];
    const bool lower = zc <= 0.5 * g.lz;
    const double d = lower ? zc : g.lz - zc;
    const double utk = lower ? ut[0] : ut[1];
    const double damp = 1.0 - exp(-d * utk / g.nu / 25.0);
    const double f = cs * sqrt(g.delta2[k]) * damp;
    coef[k] = f * f;
    if (k == 1) coef[0] = f * f;
    if (k == n) coef[n + 1] = f * f;
  }
}

// ============================================================================ dynamic model
// Plane sums in a fixed order -> c_s(k) = max(0, <LM>/<MM>) (0 if <MM> = 0), whole box
// when z is periodic; coef[k] = c_s Delta_k^2 with ghost copies.  One block per plane:
// strided partial sums over the tiles, then a fixed-order tree.  With periodic z every block
// forms the total over all planes itself (same order in every block).
template <typename T>
__device__ __forceinline__ void dsm_reduce_body(int k, GridP g, const double* part, int ntile, double* cs,
                                                double* coef, const int* gate, T* fnut) {
  if (gate != nullptr && gate[0] == 0) return;
  __shared__ double sm[2][256];
  const int n = g.nz;
  const bool per = g.zbc == LES_ZBC_PERIODIC;
  double a = 0.0, b = 0.0;
  if (per) {
    for (int64_t e = threadIdx.x; e < (int64_t)n * ntile; e += 256) {
      a += part[2 * e];
      b += part[2 * e + 1];
    }
  } else {
    for (int t = threadIdx.x; t < ntile; t += 256) {
      a += part[((int64_t)k * ntile + t) * 2];
      b += part[((int64_t)k * ntile + t) * 2 + 1];
    }
  }
  sm[0][threadIdx.x] = a;
  sm[1][threadIdx.x] = b;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      sm[0][threadIdx.x] += sm[0][threadIdx.x + st];
      sm[1][threadIdx.x] += sm[1][threadIdx.x + st];
    }
    __syncthreads();
  }
  const double sa = sm[0][0], sb = sm[1][0];
  const double c = sb > 0.0 ? fmax(sa / sb, 0.0) : 0.0;
  if (threadIdx.x == 0) {
    cs[k] = c;
    if (coef != nullptr) {
      coef[k + 1] = c * g.delta2[k + 1];
      if (k == 0) coef[per ? n + 1 : 0] = c * g.delta2[1];
      if (k == n - 1) coef[per ? 0 : n + 1] = c * g.delta2[n];
    }
  }
  if (fnut != nullptr) {
    // learned closure: the cells of this plane that the network left to the dynamic model
    // (stored -|S|) take c |S|
    const int64_t nxy = (int64_t)g.nx * g.ny;
    for (int64_t r = threadIdx.x; r < nxy; r += blockDim.x) {
      const int j = (int)(r / g.nx), i = (int)(r % g.nx);
      const T val = fnut[idx3(g, k + 1, j, i)];
      if (val < (T)0) store_nut(g, fnut, k + 1, j, i, (T)c * -val);
    }
  }
}

// fnut (learned closure, may be null): also the fallback of the plane's flagged cells
template <typename T>
__global__ void __launch_bounds__(256) k_dsm_reduce(GridP g, const double* part, int ntile, double* cs,
                                                    double* coef, const int* gate, T* fnut) {
  dsm_reduce_body<T>(blockIdx.x, g, part, ntile, cs, coef, gate, fnut);
}

// ============================================================================ fused dynamic model
// One z-marching pass per (32-wide tile, chunk of planes) computing |S| and the plane sums
// of L_ij M_ij and M_ij M_ij, reading u, v, w once (halo 2) and writing |S| once.
//   LDS: velocity of one plane on the tile + 2 halo, the 12 filter inputs (u_i u_j, |S| S_ij at
//        cell centres) of one plane on the tile + 1 halo, their x sums on the tile + 1 halo in y,
//        and the test-filtered staggered velocity of one plane on the tile + 1 halo.
//   Registers: at the thread's cell what the plane above needs of this one (Strain below) and the
//        running z sums of the test filter.  The first threads have one halo point as well, whose
//        march is kept in LDS: in registers every thread would hold room for it.
// Iteration q reads the 3 x 3 neighbourhood of velocity plane q once per point, for the
// in-plane strain terms of plane q and the x-y test filter together; with the z differences that
// it completes it finishes the strain and filter inputs of plane p = q - 1, the filtered velocity
// of plane p and, from that, the strain of the filtered velocity, L and M of plane k = q - 2.
// The test filter runs unnormalised, (1, 2, 1) per direction (exact powers of two, folded into the
// final sums), x first and then y: two of the three x (y) values come from LDS.
// The filtered centre velocities are the two-point means of the filtered staggered ones (both
// are linear), except where the two filters differ: w next to the z walls (the z pass of a centred
// quantity is the identity there) and v next to the y walls of a duct.
// Wall rules: on the first off-wall layers the z pass of the filter is the identity (the index-space
// extrapolation of the neighbour reduces to it), alpha^2 = 4^(2/3) there; the strain ghost rule
// of either velocity makes the z difference across the wall that of the next edge inward (wall
// model, linear extrapolation) or twice the cell's own value (no-slip, odd).
// Bound by latency at two waves per SIMD in FP64 (156 KB of LDS and 256 registers: one block of 32 x 16
// cells per CU; the VALU busy 36 % of the time, a wave waiting for 44 % of its own and ready but not issued for
// 22 %) and by VALU issue at three in FP32 (32 x 8 cells, three blocks per CU; VALU busy 69 to 73 %).
// 512x256x128 FP64 with the wall model: 601 -> 505 us, against 596 us for 15 inputs through a 9-point filter with
// all four edges of a cell worked out; 256x128x96: 127 -> 112; 64 boxes of 32^3 to 96^3 in FP32: 4614 -> 3909 us a
// step; 512x80x80 duct: 217 -> 147.  Measured and dropped in FP64: 32 x 8 tiles at two blocks per CU (572: the
// halo's share), x sums by lane shifts in place of LDS (508), separate waves for halo points on 32 x 12 tiles
// (612) or for the model on 16 waves (884, spills), the halo points after the first barrier (586).
namespace fused {
constexpr int TX = 32;
constexpr int NQ = 12;   // filter inputs per cell
template <typename T>
struct Tile {
  static constexpr int TY = dsm_tile_rows(sizeof(T) == 8), NT = TX * TY, WV = NT / 64;
  static constexpr int RX2 = TX + 4, RY2 = TY + 4, N2 = RX2 * RY2;  // halo 2
  static constexpr int RX1 = TX + 2, RY1 = TY + 2, N1 = RX1 * RY1;  // halo 1
  static constexpr int NROW = 2 * TX, NHALO = NROW + 2 * RY1;        // halo-1 points around the tile
  static constexpr int WEU = sizeof(T) == 8 ? 2 : 3;                 // waves per SIMD
};
// inputs per 16-byte LDS access
template <typename T>
struct alignas(16) Pack {
  static constexpr int N = 16 / sizeof(T);
  T x[N];
};
}  // namespace fused

// Terms of one point that a z march of the strain carries (edge terms scaled by 1/8: the mean of
// four edge values of half sums): of plane q - 1 the in-plane strain, U = u_i + u_{i-1},
// V = v_j + v_{j-1}, w on its upper face and the x and y differences of w there; of plane q - 2
// the upper z-edge terms (ex, ey) and w.  The two-point sums replace the four edges of a cell:
// (u_{j+1} - u_j) + (u_j - u_{j-1}) and the like telescope.
template <typename T>
struct Strain {
  static constexpr int N = 11;
  T s11, s22, s12, U, V, w, wx, wy, ex, ey, wl;
};
// In-plane terms of a plane at one point, component by component, from the 3 x 3 neighbourhoods
// ([row][column]); s12 takes u's share first, then v's.
template <typename T>
__device__ __forceinline__ void strain_inplane(int c, const T (&a)[3][3], T rdx, T rdy, Strain<T>& n) {
#pragma clang fp contract(on)
  const T rdx8 = (T)0.125 * rdx, rdy8 = (T)0.125 * rdy;
  if (c == 0) {
    n.U = a[1][1] + a[1][0];
    n.s11 = (a[1][1] - a[1][0]) * rdx;
    n.s12 = ((a[2][1] + a[2][0]) - (a[0][1] + a[0][0])) * rdy8;
  } else if (c == 1) {
    n.V = a[1][1] + a[0][1];
    n.s22 = (a[1][1] - a[0][1]) * rdy;
    n.s12 = ((a[1][2] + a[0][2]) - (a[1][0] + a[0][0])) * rdx8 + n.s12;
  } else {
    n.w = a[1][1];
    n.wx = (a[1][2] - a[1][0]) * rdx8;
    n.wy = (a[2][1] - a[0][1]) * rdy8;
  }
}

// Upper z-edge terms of plane q - 1 from plane q (n) and the march up to plane q - 1 (c)
template <typename T>
__device__ __forceinline__ void strain_edges(const Strain<T>& c, const Strain<T>& n, T rdzc8, T& ex, T& ey) {
#pragma clang fp contract(on)
  ex = (n.U - c.U) * rdzc8 + c.wx;
  ey = (n.V - c.V) * rdzc8 + c.wy;
}

// x of another lane of the same row of 16 lanes, by a DPP lane pattern
template <int CTRL>
__device__ inline double dpp_f64(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, false));
}
// sum over each row of 16 lanes, a 4-level tree (partners at lane distance 1 and 2 in a quad,
// then the mirrored half-row and row): every lane of a row holds the same bits
__device__ inline double row_sum(double x) {
  x = x + dpp_f64<0xB1>(x);    // quad permutation 1 0 3 2
  x = x + dpp_f64<0x4E>(x);    // quad permutation 2 3 0 1
  x = x + dpp_f64<0x141>(x);   // half-row mirror
  x = x + dpp_f64<0x140>(x);   // row mirror
  return x;
}
// lane L's value of x, uniform across the wave
__device__ inline double lane_f64(double x, int L) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), L),
                          __builtin_amdgcn_readlane(__double2loint(x), L));
}
// Both sums over each half wave (32 lanes) with one row tree: rows 0 and 2 of a take what rows
// 1 and 3 hold, rows 1 and 3 the same of b, then row_sum.  The result in rows 0..3: a of the
// lower half, b of the lower half, a of the upper half, b of the upper half.
__device__ inline double half_sums(double a, double b) {
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  const v2u lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const v2u hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return row_sum(__hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]));
}

template <typename T>
__device__ inline T strain_norm(const T s[6]) {
#pragma clang fp contract(on)
  const T d = s[0] * s[0] + s[1] * s[1] + s[2] * s[2];
  const T e = s[3] * s[3] + s[4] * s[4] + s[5] * s[5];
  return sqrt((T)2 * d + (T)4 * e);
}

// YW (ducts, walls in y too): the y pass of the test filter is the identity on the first and
// last rows for y-centred quantities (u, w and the cell quantities), v~ vanishes on and
// beyond the y wall faces, the y ghost rows of u~ and w~ follow the strain ghost rule, alpha^2
// counts the filter's dimensions per cell, and the partial sums are per x line (one per row
// of each wave: 32 lanes) instead of per wave.
template <typename T, bool YW, int ZBC>
__device__ __forceinline__ void dsm_fused_body(dim3 bid, int gdx, int gdy, GridP g, const T* __restrict__ u,
                                               const T* __restrict__ v, const T* __restrict__ w,
                                               T* __restrict__ nut, double* __restrict__ part, int kc,
                                               const int* __restrict__ gate) {
#pragma clang fp contract(on)
  using TL = fused::Tile<T>;
  using Pack = fused::Pack<T>;
  constexpr int TX = fused::TX, TY = TL::TY, NT = TL::NT, WV = TL::WV, NQ = fused::NQ, PN = Pack::N, NP = NQ / PN;
  constexpr int RX2 = TL::RX2, N2 = TL::N2, RX1 = TL::RX1, RY1 = TL::RY1, N1 = TL::N1, NROW = TL::NROW,
                NHALO = TL::NHALO;
  if (gate != nullptr && gate[0] == 0) return;   // learned closure: no point fell back
  __shared__ __align__(16) T vel[3][N2];   // velocity plane q
  static_assert(__alignof__(vel) >= 16 && sizeof(vel[0]) % 16 == 0, "16-byte parts of a plane, straight from memory");
  __shared__ Pack qb[NP][N1];        // filter inputs of plane p
  __shared__ Pack xb[NP][RY1 * TX];  // their x sums
  __shared__ T ut[3][N1];            // filtered velocity of plane p (times 64)
  __shared__ T hst[Strain<T>::N + 6][NHALO];   // march of the halo points
  int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
  const int i0 = bid.x * TX, j0 = bid.y * TY;
  const int nz = g.nz;
  const int kb = 1 + bid.z * kc;
  const int ke = min(nz, kb + kc - 1);
  constexpr bool per = ZBC == LES_ZBC_PERIODIC;
  constexpr bool wm = ZBC == LES_ZBC_WALLMODEL;
  const int ntile = gdx * gdy;
  const int tile = bid.y * gdx + bid.x;
  const T rdx = (T)g.rdx, rdy = (T)g.rdy;
  const int64_t sxy = g.sxy;
  auto phys = [&](int q) {  // logical plane -> stored plane (periodic wrap of interior planes)
    if (!per) return q;
    int m = (q - 1) % nz;
    if (m < 0) m += nz;
    return m + 1;
  };
  // The velocity plane under way.  FP64: straight from memory to LDS (DIRECT), into the one buffer, issued when
  // the block has done with the plane before; no registers hold it, where the compiler would spill just those
  // and so wait for the loads at once.  16 bytes per lane, a pair of columns: the tile's first column i0 - 2 and
  // nx are even, so pairs stay whole and aligned across the wrap.  FP32: in registers between its fetch and its
  // commit to LDS, a whole iteration, with one element per lane.
  // lofs: byte offset in a plane of the thread's parts of the tile + 2 halo (tiles may exceed the grid: wrap);
  // threads past the halo load nothing (DIRECT), or offset 0 and commit nothing.
  constexpr bool DIRECT = sizeof(T) == 8;
  constexpr int LC = DIRECT ? 2 : 1;                    // columns per lane
  constexpr int NPART = N2 / LC, NL = (NPART + NT - 1) / NT;
  int lofs[NL];
  T ra[3][DIRECT ? 1 : NL];
  for (int r = 0; r < NL; ++r) {
    const int e = (tid + r * NT) * LC;
    int i = (i0 - 2 + e % RX2) % g.nx, j = (j0 - 2 + e / RX2) % g.nys;
    if (i < 0) i += g.nx;
    if (j < 0) j += g.nys;
    lofs[r] = e < N2 ? (j * g.nx + i) * (int)sizeof(T) : 0;
  }
  auto fetch = [&](int q) {
    const int pq = phys(q);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const PlaneLoader<T> ld(c == 0 ? u : (c == 1 ? v : w), pq, sxy);
#pragma unroll
      for (int r = 0; r < NL; ++r) {
        if constexpr (DIRECT) {
          const int first = __builtin_amdgcn_readfirstlane(tid) + r * NT;
          if (tid + r * NT < NPART) ld.to_lds(&vel[c][first * LC], lofs[r]);
        } else {
          ra[c][r] = ld(lofs[r] / (int)sizeof(T));
        }
      }
    }
  };
  auto commit = [&]() {
#pragma unroll
    for (int r = 0; r < NL; ++r)
      if (tid + r * NT < N2)
#pragma unroll
        for (int c = 0; c < 3; ++c) vel[c][tid + r * NT] = ra[c][r];
  };
  // ducts with the wall model: u and w on the y ghost rows of the committed plane, extrapolated
  // from the two rows inward (strain ghosts); only blocks at a y wall hold such rows
  const bool ywall_block = YW && wm && (j0 == 0 || j0 + TY + 1 >= g.ny);
  auto extrapolate_rows = [&]() {
    for (int e = tid; e < 4 * RX2; e += NT) {
      const int c = e / (2 * RX2) * 2, x = e % RX2;
      const bool low = e / RX2 % 2 == 0;
      const int row = low ? 1 : g.ny - j0 + 2, d = low ? RX2 : -RX2;   // R2 rows of j = -1, ny
      if (low ? j0 != 0 : j0 + TY + 1 < g.ny) continue;
      const int o = row * RX2 + x;
      const T a0 = vel[c][o + d];
      vel[c][o] = a0 - (vel[c][o + 2 * d] - a0);
    }
  };
  // |S| of the own cell on plane k; the first and last planes also fill the ghost plane (odd about
  // walls, periodic copy otherwise)
  auto store_plane = [&](int k, T val) {
    const int o = (j0 + ty) * g.nx + i0 + tx;
    PlaneLoader<T>(nut, k, sxy).store(o, val);
    if (k == 1) PlaneLoader<T>(nut, per ? nz + 1 : 0, sxy).store(o, per ? val : -val);
    if (k == nz) PlaneLoader<T>(nut, per ? 0 : nz + 1, sxy).store(o, per ? val : -val);
  };
  // z weights (lower, centre, upper) of the unnormalised test filter: (1, 2, 1), the identity
  // (0, 4, 0) for z-centred quantities on the first off-wall layers, 0 for w on the top wall face
  auto zw = [&](int q, bool centred, int which) -> T {
    if (!per && !centred && q == nz) return (T)0;
    if (!per && centred && (q == 1 || q == nz)) return which == 1 ? (T)4 : (T)0;
    return which == 1 ? (T)2 : (T)1;
  };
  // planes of the march: filter inputs on pstart..pend, velocity from qstart
  const int pstart = per ? kb - 1 : max(kb - 1, 1);
  const int pend = per ? ke + 1 : min(ke + 1, nz);
  const bool from_wall = !per && pstart == 1;
  const int qstart = from_wall ? 1 : pstart - 1;
  const int qlast = per ? pend + 1 : min(pend + 1, nz);   // last velocity plane read
  auto inside = [&]() { return i0 + tx < g.nx && j0 + ty < g.ny; };
  T fwb = (T)0, fwt = (T)0;   // x-y filtered w of planes 1 and nz - 1 at the own cell (z walls)
  // ducts: filtered V of the first and last rows (z sums of its own; fv: plane p, fvk: plane k)
  T V1 = (T)0, V2 = (T)0, fv = (T)0, fvk = (T)0;
  auto yedge = [&]() { return YW && (j0 + ty == 0 || j0 + ty == g.ny - 1); };   // duct: first or last row
  // reciprocal spacing (over 8) of the z difference between planes q - 1 and q: twice the cell's
  // own value across a bottom wall with no-slip, nothing beyond the top wall (the march prepares it)
  auto rz8 = [&](int q) -> T {
    if (!per && q > nz) return (T)0;
    return ((from_wall && q == 1) ? (T)0.25 : (T)0.125) * (T)ro_load(g.rdzc, phys(q - 1));
  };
  // planes next to the z walls: C is the point's march at plane q - 1, n plane q; lx, ly the lower
  // edge terms of plane q - 1.  Edge on the bottom wall, wall model: the z difference of the edge
  // above it; edge on the top wall, prepared in n.wx, n.wy: that of the edge below it, or twice
  // the cell's own value (no-slip)
  auto wall_edges = [&](int q, const Strain<T>& C, Strain<T>& n, T ex, T ey, T& lx, T& ly, T plw, bool mine) {
    if (mine && q == 1) fwb = plw;
    if (mine && q == nz - 1) fwt = plw;
    if (wm && from_wall && q == 2) {
      lx = ex - C.wx;
      ly = ey - C.wy;
    }
    if (q == nz) {
      const T r8 = (T)0.25 * (T)ro_load(g.rdzc, nz);
      n.wx = wm ? ex - C.wx : -r8 * n.U;
      n.wy = wm ? ey - C.wy : -r8 * n.V;
    }
  };
  // ---- plane q at one point: filtered velocity of plane q - 1, strain and filter inputs of plane
  // q - 1; x, y in R1 coordinates.  Beyond the top wall (q = nz + 1) the LDS plane is stale and all
  // of it is multiplied by zero.  Straight-line code but for the planes next to the walls.
  auto point = [&](int q, int x, int y, Strain<T>& C, T (&G1)[3], T (&G2)[3], bool mine) {
    const int e = y * RX1 + x;
    const int o = (y + 1) * RX2 + x + 1;
    Strain<T> n;
    const int jr = j0 - 1 + y;
    const bool edge = YW && (jr == 0 || jr == g.ny - 1);
    T pl[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      T nb[3][3], r[3];
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) nb[dy][dx] = vel[c][o + (dy - 1) * RX2 + dx - 1];
      strain_inplane<T>(c, nb, rdx, rdy, n);
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) r[dy] = (T)2 * nb[dy][1] + (nb[dy][0] + nb[dy][2]);
      if (YW && c != 1)
        pl[c] = edge ? (T)4 * r[1] : (T)2 * r[1] + (r[0] + r[2]);
      else
        pl[c] = (T)2 * r[1] + (r[0] + r[2]);
      if (YW && c == 1) {
        if (mine) {
          const T vr = (T)4 * (jr == 0 ? r[1] : r[0]);
          fv = V1 + zw(q - 1, true, 2) * vr;
          V1 = V2 + zw(q, true, 1) * vr;
          V2 = zw(q + 1, true, 0) * vr;
        }
        if (jr >= g.ny - 1 || jr < 0) pl[c] = (T)0;   // v~ on and beyond the y walls
      }
      ut[c][e] = G1[c] + zw(q - 1, c < 2, 2) * pl[c];
      G1[c] = G2[c] + zw(q, c < 2, 1) * pl[c];
      G2[c] = zw(q + 1, c < 2, 0) * pl[c];
    }
    T lx = C.ex, ly = C.ey;
    strain_edges<T>(C, n, rz8(q), n.ex, n.ey);
    if (!per && (q <= 2 || q >= nz - 1)) wall_edges(q, C, n, n.ex, n.ey, lx, ly, pl[2], mine);
    const T s[6] = {C.s11, C.s22, (C.w - C.wl) * (T)ro_load(g.rdzf, phys(q - 1)), C.s12, n.ex + lx, n.ey + ly};
    const T sm_ = strain_norm<T>(s);
    const T U = C.U, V = C.V, W = C.w + C.wl;
    const T in[NQ] = {U * U, V * V, W * W, U * V, U * W, V * W,
                      sm_ * s[0], sm_ * s[1], sm_ * s[2], sm_ * s[3], sm_ * s[4], sm_ * s[5]};
#pragma unroll
    for (int a = 0; a < NP; ++a) {
      Pack t;
#pragma unroll
      for (int b = 0; b < PN; ++b) t.x[b] = in[a * PN + b];
      qb[a][e] = t;
    }
    if (mine && nut != nullptr && q - 1 >= kb && q - 1 <= ke && inside()) store_plane(q - 1, sm_);
    n.wl = C.w;
    C = n;
  };
  // x sums of the inputs at R1 point (x, y)
  auto xsums = [&](int x, int y) {
    const int e = y * RX1 + x;
#pragma unroll
    for (int a = 0; a < NP; ++a) {
      const Pack l = qb[a][e - 1], m = qb[a][e], r = qb[a][e + 1];
      Pack t;
#pragma unroll
      for (int b = 0; b < PN; ++b) t.x[b] = (T)2 * m.x[b] + (l.x[b] + r.x[b]);
      xb[a][y * TX + x - 1] = t;
    }
  };
  // running sums of the z pass of the test filter over the thread's cell: S1 holds
  // plane p's sum without its upper neighbour, S2 plane p + 1's lower-neighbour term
  T S1[NQ] = {}, S2[NQ] = {};
  // y sums of the inputs of plane p, folded into the z sums; F: the filtered inputs of plane p - 1
  auto filter = [&](int p, T (&F)[NQ]) {
    const T zu = zw(p - 1, true, 2), zc = zw(p, true, 1), zl = zw(p + 1, true, 0);
    const T ws = yedge() ? (T)0 : (T)1, wc = yedge() ? (T)4 : (T)2;
#pragma unroll
    for (int a = 0; a < NP; ++a) {
      const Pack lo = xb[a][tid], m = xb[a][tid + TX], hi = xb[a][tid + 2 * TX];
#pragma unroll
      for (int b = 0; b < PN; ++b) {
        const int c = a * PN + b;
        const T q = YW ? wc * m.x[b] + ws * (lo.x[b] + hi.x[b]) : (T)2 * m.x[b] + (lo.x[b] + hi.x[b]);
        F[c] = S1[c] + zu * q;
        S1[c] = S2[c] + zc * q;
        S2[c] = zl * q;
      }
    }
  };
  // ducts: the y ghost rows of u~ and w~ by the strain ghost rule (extrapolated with the wall
  // model, odd with no-slip), from the completed rows next to them
  auto fix_rows = [&]() {
    for (int e = tid; e < N1; e += NT) {
      const int jr = j0 - 1 + e / RX1;
      if (jr != -1 && jr != g.ny) continue;
      const int d = jr < 0 ? RX1 : -RX1;   // one row inward
      for (int c = 0; c < 3; c += 2) {
        const T a0 = ut[c][e + d];
        ut[c][e] = wm ? a0 - (ut[c][e + 2 * d] - a0) : -a0;
      }
    }
  };
  // ---- output plane k from F, the test-filtered inputs of its cell (times 64, the products
  // times 4 more), the strain march CT of the filtered velocity (times 64), its upper edge terms
  // (ex, ey) and lower ones (lx, ly) of plane k
  Strain<T> CT = {};
  double hs = 0.0;   // plane sums of the cells (half_sums)
  auto output = [&](int k, const T (&F)[NQ], T ex, T ey, T lx, T ly) {
    const int pk = phys(k);
    const T st[6] = {CT.s11, CT.s22, (CT.w - CT.wl) * (T)ro_load(g.rdzf, pk), CT.s12, ex + lx, ey + ly};
    const bool wall_layer = !per && (k == 1 || k == nz);
    // 3-D, 2-D or (duct corners) 1-D test filter: 4, 4^(2/3), 2^(2/3)
    const T alpha2 = (wall_layer && yedge()) ? (T)1.5874010519681994
                                           : ((wall_layer || yedge()) ? (T)2.5198420997897464 : (T)4);
    const T am = (alpha2 * (T)0.015625) * strain_norm<T>(st);
    T fv_ = CT.V, fw = CT.w + CT.wl;
    if (!per && k == 1) fw = (T)4 * fwb;
    if (!per && k == nz) fw = (T)4 * fwt;
    if (YW && yedge()) fv_ = fvk;
    const T q64 = (T)0.015625, gu = q64 * CT.U, gv = q64 * fv_, gw = q64 * fw;
    const T Fa[6] = {CT.U, fv_, fw, CT.U, CT.U, fv_}, Fb[6] = {gu, gv, gw, gv, gw, gw};
    double la = 0.0, lo = 0.0, ma = 0.0, mo = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const T Lc = F[c] - Fa[c] * Fb[c], Mc = F[6 + c] - am * st[c];
      const double L = (double)Lc, m = (double)Mc;
      if (c < 3) {
        la += L * m;
        ma += m * m;
      } else {
        lo += L * m;
        mo += m * m;
      }
    }
    const double d2 = ro_load(g.delta2, pk) * (1.0 / 32.0);   // 2 Delta^2 / 64
    const double lm = inside() ? (la + 2.0 * lo) * (d2 * (1.0 / 256.0)) : 0.0;
    const double mm = inside() ? (ma + 2.0 * mo) * (d2 * d2) : 0.0;
    hs = half_sums(lm, mm);
  };
  // sums of plane k to memory: called one iteration later, so that no store is young when the loads
  // of a plane are waited for
  auto put_sums = [&](int k) {
    if (k < kb || k > ke) return;
    if (YW) {
      // x-line sums: a row of the tile is 32 lanes of one wave; partials [k][j][tile x]
      const int jrow = j0 + ty;
      if (tx % 16 == 0 && jrow < g.ny) part[(((int64_t)(k - 1) * g.ny + jrow) * gdx + bid.x) * 2 + tx / 16] = hs;
      return;
    }
    // the waves' partials go out per plane and are summed over (tile, wave) in a fixed order by
    // the plane reduction
    const double lm = lane_f64(hs, 0) + lane_f64(hs, 32);
    const double mm = lane_f64(hs, 16) + lane_f64(hs, 48);
    if (tid % 64 == 0) {
      double* pk2 = part + (((int64_t)(k - 1) * ntile + tile) * WV + __builtin_amdgcn_readfirstlane(tid / 64)) * 2;
      pk2[0] = lm;
      pk2[1] = mm;
    }
  };
  // start of an iteration: plane q has arrived
  auto arrive = [&](int q) {
    if constexpr (DIRECT)
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the thread's loads to LDS
    else if (q <= qlast)
      commit();
    lds_barrier();
    if (ywall_block && q <= qlast) {
      extrapolate_rows();
      lds_barrier();
    }
    if (!DIRECT && q < qlast) fetch(q + 1);
  };
  fetch(qstart);
  // ---- march.  Threads exchange data through LDS only (the stored |S| and partial sums are read
  // by later launches): the barriers leave global loads in flight.
  Strain<T> C = {};
  T G1[3] = {}, G2[3] = {};
  if (tid < NHALO)
    for (int a = 0; a < Strain<T>::N + 6; ++a) hst[a][tid] = (T)0;
#pragma unroll 1
  for (int q = qstart; q <= pend + 1; ++q) {
    const int p = q - 1, k = q - 2;
    if constexpr (YW || per) {
      // LDS addresses from here are worked out anew on each plane: where registers would hold them between
      // planes, some are spilled, and a reload waits for the loads and stores under way
      asm volatile("" : "+v"(tid));
      tx = tid % TX;
      ty = tid / TX;
    }
    arrive(q);
    put_sums(q - 3);
    point(q, tx + 1, ty + 1, C, G1, G2, true);
    // the thread's halo-1 point (R1 coordinates), if it has one: the rows below and above the tile, then
    // the columns beside it
    const int hc = tid - NROW;
    const int hx = hc < 0 ? tx + 1 : (hc < RY1 ? 0 : RX1 - 1), hy = hc < 0 ? (tid < TX ? 0 : RY1 - 1) : hc % RY1;
    if (tid < NHALO) {
      struct {
        Strain<T> m;
        T G1[3], G2[3];
      } H;
      T h[Strain<T>::N + 6];
#pragma unroll
      for (int a = 0; a < Strain<T>::N + 6; ++a) h[a] = hst[a][tid];
      static_assert(sizeof(H) == sizeof(h), "all of it T");
      __builtin_memcpy(&H, h, sizeof(h));
      point(q, hx, hy, H.m, H.G1, H.G2, false);
      __builtin_memcpy(h, &H, sizeof(h));
#pragma unroll
      for (int a = 0; a < Strain<T>::N + 6; ++a) hst[a][tid] = h[a];
    }
    lds_barrier();
    if (DIRECT && q < qlast) fetch(q + 1);
    if (p < pstart) continue;
    xsums(tx + 1, ty + 1);
    if (tid < NROW) xsums(hx, hy);
    if (YW) fix_rows();
    lds_barrier();
    // filtered velocity of plane p at the own cell, and the upper edge terms of plane k
    Strain<T> n;
    T ex, ey;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      T nb[3][3];
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) nb[dy][dx] = ut[c][(ty + dy) * RX1 + tx + dx];
      strain_inplane<T>(c, nb, rdx, rdy, n);
    }
    strain_edges<T>(CT, n, rz8(p), ex, ey);
    T lx = CT.ex, ly = CT.ey;
    if (!per && (p <= 2 || p == nz)) wall_edges(p, CT, n, ex, ey, lx, ly, (T)0, false);
    T F[NQ];
    filter(p, F);
    output(k, F, ex, ey, lx, ly);
    n.wl = CT.w;
    n.ex = ex;
    n.ey = ey;
    CT = n;
    if (YW) fvk = fv;
  }
  put_sums(pend - 1);
  if (!per && ke == nz) {   // the z pass is the identity on the top layer
    output(nz, S1, CT.wx, CT.wy, CT.ex, CT.ey);
    put_sums(nz);
  }
}

template <typename T, bool YW, int ZBC>
__global__ void __launch_bounds__(fused::Tile<T>::NT, fused::Tile<T>::WEU) k_dsm_fused(GridP g, const T* u, const T* v,
                                                                                    const T* w, T* nut, double* part,
                                                                                    int kc, const int* gate) {
  dsm_fused_body<T, YW, ZBC>(xcd_tile(blockIdx, gridDim), gridDim.x, gridDim.y, g, u, v, w, nut, part, kc, gate);
}

// ---------------------------------------------------------------- FP32 with walls or Crank-Nicolson
// The same model with every value rounded where an FP32 run has always rounded it: the four edges of a cell
// apart, 15 inputs (the centre velocities among them) through the 9-point filter term by term.  L is a
// difference of nearly equal FP32 values, so either kernel's c_s is off by some 1e-7 (between walls up to 5e-4),
// and the pressure of an FP32 run answers the last bits of the eddy viscosity: by 3e-4 of itself in a channel
// (1024x512x256) and 3e-5 in a 256^3 box with Crank-Nicolson in all directions, as much as its distance from a
// 64-bit solution, but by 1.3e-6 in periodic boxes with explicit viscous terms (32^3 to 256^3).  The kernel above is
// faster (3217 -> 2223 us on that channel) and not closer (2.9e-4 against 2.2e-4), so in FP32 only the last take it.
//   LDS: velocity of planes p, p + 1 on the tile + 2 halo (strain ghosts substituted), the 15 filter inputs (u_i,
//        u_i u_j, |S| S_ij at cell centres) of plane p on the tile + 1 halo in pairs, the test-filtered
//        staggered velocity of two planes on the tile + 1 halo.
//   Registers: the z pass of the test filter as running sums over the thread's cell; the upper z-edge terms of the
//        off-diagonal strain and w of the previous plane at the thread's points, the lower terms of the plane
//        above.
// The stage of plane p forms the filter inputs of plane p from velocity planes p, p + 1 and completes the
// filtered velocity of plane p - 1; then the cell values of plane p - 1 are final.
namespace fused32 {
constexpr int TX = 32;
constexpr int NQ = 15;   // filter inputs per cell
template <typename T, bool YW>
struct Tile {
  static constexpr int TY = dsm_tile_rows(false), NT = TX * TY, WV = NT / 64;
  static constexpr int RX2 = TX + 4, RY2 = TY + 4, N2 = RX2 * RY2;  // halo 2
  static constexpr int RX1 = TX + 2, RY1 = TY + 2, N1 = RX1 * RY1;  // halo 1
  static constexpr int NHALO = 2 * (RX1 + TY);                       // halo-1 points around the tile
};
}  // namespace fused32

// Upper z-edge terms at a cell of plane k: (du/dz + dw/dx) / 2 on the x-z edges of the cell's
// two x faces (fa: the face of u_i, fb: of u_{i-1}), (dv/dz + dw/dy) / 2 on the y-z edges of
// its two y faces (ga, gb), all on the face between planes k and k + 1, and w on that face.
// They are the lower edge terms of the cell above.
template <typename T>
struct ZEdges {
  T fa, fb, ga, gb, w;
};

// from an accessor A(c, dz, o): component c (0 u, 1 v, 2 w) of plane k + dz (dz in {0, 1}) at
// plane offset o; sy is one step in y, rdzc the reciprocal centre spacing above plane k
template <typename T, typename Acc>
__device__ inline ZEdges<T> zedges(const Acc& A, int o, int sy, T rdx, T rdy, T rdzc) {
  const T h = (T)0.5;
  ZEdges<T> E;
  const T w0 = A(2, 0, o);
  E.fa = h * ((A(0, 1, o) - A(0, 0, o)) * rdzc + (A(2, 0, o + 1) - w0) * rdx);
  E.fb = h * ((A(0, 1, o - 1) - A(0, 0, o - 1)) * rdzc + (w0 - A(2, 0, o - 1)) * rdx);
  E.ga = h * ((A(1, 1, o) - A(1, 0, o)) * rdzc + (A(2, 0, o + sy) - w0) * rdy);
  E.gb = h * ((A(1, 1, o - sy) - A(1, 0, o - sy)) * rdzc + (w0 - A(2, 0, o - sy)) * rdy);
  E.w = w0;
  return E;
}

// strain at a cell of plane k (Sec. 2.2: diagonal terms from face differences, off-diagonal
// terms as means of four edge values) from the accessor over plane k, the lower edge terms P
// (the upper terms of plane k - 1) and the cell's own upper terms E
template <typename T, typename Acc>
__device__ inline void strain_zm(const Acc& A, int o, int sy, T rdx, T rdy, T rdzf, const ZEdges<T>& P,
                                 const ZEdges<T>& E, T s[6]) {
  const T h = (T)0.5, q = (T)0.25;
  const T u0 = A(0, 0, o), uim = A(0, 0, o - 1), ujp = A(0, 0, o + sy), ujm = A(0, 0, o - sy);
  const T ujp_im = A(0, 0, o + sy - 1), ujm_im = A(0, 0, o - sy - 1);
  const T v0 = A(1, 0, o), vjm = A(1, 0, o - sy), vip = A(1, 0, o + 1), vim = A(1, 0, o - 1);
  const T vjm_ip = A(1, 0, o - sy + 1), vjm_im = A(1, 0, o - sy - 1);
  s[0] = (u0 - uim) * rdx;
  s[1] = (v0 - vjm) * rdy;
  s[2] = (E.w - P.w) * rdzf;
  const T e_a = h * ((ujp - u0) * rdy + (vip - v0) * rdx);
  const T e_b = h * ((ujp_im - uim) * rdy + (v0 - vim) * rdx);
  const T e_c = h * ((u0 - ujm) * rdy + (vjm_ip - vjm) * rdx);
  const T e_d = h * ((uim - ujm_im) * rdy + (vjm - vjm_im) * rdx);
  s[3] = q * (e_a + e_b + e_c + e_d);
  s[4] = q * (E.fa + E.fb + P.fa + P.fb);
  s[5] = q * (E.ga + E.gb + P.ga + P.gb);
}

template <typename T>
__device__ inline T strain_norm32(const T s[6]) {
  return sqrt((T)2 * (s[0] * s[0] + s[1] * s[1] + s[2] * s[2]) + (T)4 * (s[3] * s[3] + s[4] * s[4] + s[5] * s[5]));
}

template <typename T, bool YW>
__device__ __forceinline__ void dsm_fused32_body(dim3 bid, int gdx, int gdy, GridP g, const T* __restrict__ u,
                                               const T* __restrict__ v, const T* __restrict__ w,
                                               T* __restrict__ nut, double* __restrict__ part, int kc,
                                               const int* __restrict__ gate) {
  using TL = fused32::Tile<T, YW>;
  constexpr int TX = fused32::TX, TY = TL::TY, NT = TL::NT, WV = TL::WV, NQ = fused32::NQ;
  constexpr int RX2 = TL::RX2, N2 = TL::N2, RX1 = TL::RX1, RY1 = TL::RY1, N1 = TL::N1, NHALO = TL::NHALO;
  if (gate != nullptr && gate[0] == 0) return;   // learned closure: no point fell back
  constexpr int NL = (N2 + NT - 1) / NT;          // halo-2 points per thread (loads)
  constexpr int NH = (N1 + NT - 1) / NT;          // halo-1 points per thread (velocity filter)
  __shared__ T vel[2][3][N2];   // [plane & 1][component][R2]
  typedef HIP_vector_type<T, 2> T2;
  __shared__ T2 qb[(NQ + 1) / 2][N1];   // filter inputs of the current stage plane, in pairs
  __shared__ T ut[2][3][N1];    // filtered velocity [plane & 1][component][R1]
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * TX + tx;
  const int i0 = bid.x * TX, j0 = bid.y * TY;
  const int nz = g.nz;
  const int kb = 1 + bid.z * kc;
  const int ke = min(nz, kb + kc - 1);
  const int zbc = g.zbc;
  const bool per = zbc == LES_ZBC_PERIODIC;
  const bool wm = zbc == LES_ZBC_WALLMODEL;
  const int ntile = gdx * gdy;
  const int tile = bid.y * gdx + bid.x;
  const T rdx = (T)g.rdx, rdy = (T)g.rdy;
  const T W0 = (T)0.25, W1 = (T)0.5;
  const int64_t sxy = g.sxy;
  auto phys = [&](int q) {  // logical plane -> stored plane (periodic wrap of interior planes)
    if (!per) return q;
    int m = (q - 1) % nz;
    if (m < 0) m += nz;
    return m + 1;
  };
  // the z spacing above plane q as the plane above sees it (they differ only across the
  // periodic wrap, where the stored spacings at both ends are separately rounded)
  auto rdzc_above = [&](int q) { return (T)ro_load(g.rdzc, phys(q + 1) - 1); };
  // in-plane offsets of the thread's halo-2 load points (tiles may exceed the grid: wrap)
  int lofs[NL];
  for (int r = 0; r < NL; ++r) {
    const int e = tid + r * NT;
    const int rx = e % RX2, ry = e / RX2;
    int i = (i0 - 2 + rx) % g.nx, j = (j0 - 2 + ry) % g.nys;
    if (i < 0) i += g.nx;
    if (j < 0) j += g.nys;
    lofs[r] = e < N2 ? j * g.nx + i : 0;
  }
  // global row of a load point before the wrap (ducts)
  auto lrow = [&](int r) { return j0 - 2 + (tid + r * NT) / RX2; };
  // velocity of one plane held in registers between its fetch and its commit to LDS, so that
  // the global loads of plane p + 2 overlap the work on plane p: the loads are raw and
  // unconditional (points past the halo read offset 0 and are not committed)
  T ra[NL], rb[NL], rc[NL];
  auto fetch = [&](int q) {
    const int pq = phys(q);
    const PlaneLoader<T> lu(u, pq, sxy), lv(v, pq, sxy), lw(w, pq, sxy);
    for (int r = 0; r < NL; ++r) {
      ra[r] = lu(lofs[r]);
      rb[r] = lv(lofs[r]);
      rc[r] = lw(lofs[r]);
    }
    if (YW && wm) {
      const int64_t bw = (int64_t)pq * sxy;
      for (int r = 0; r < NL; ++r) {
        if (tid + r * NT < N2 && (lrow(r) == -1 || lrow(r) == g.ny)) {
          // duct: strain ghosts of u and w on the y ghost rows, extrapolated in y
          const int64_t o0 = bw + (lofs[r] % g.nx) + (int64_t)(lrow(r) < 0 ? 0 : g.ny - 1) * g.nx;
          const int64_t o1 = o0 + (lrow(r) < 0 ? g.nx : -g.nx);
          const T a0 = u[o0], a1 = u[o1], c0 = w[o0], c1 = w[o1];
          ra[r] = a0 - (a1 - a0);
          rc[r] = c0 - (c1 - c0);
        }
      }
    }
  };
  auto yghost = [&](int r) { return YW && (lrow(r) == -1 || lrow(r) == g.ny); };
  // commit plane q to its ring slot; with the wall model the top ghost plane's u, v are the
  // linear extrapolation in z of planes nz and nz - 1 (the thread's own entries; plane nz - 1
  // sits in the slot being replaced, read before it is overwritten)
  auto commit = [&](int q) {
    const int sl = q & 1;
    if (wm && phys(q) == nz + 1) {
      const int s1 = (q - 1) & 1;
      const T ca = (T)ro_load(g.dzc, nz), cb = (T)ro_load(g.dzc, nz - 1);
      for (int r = 0; r < NL; ++r) {
        const int e = tid + r * NT;
        if (e < N2) {
          const T b1 = vel[s1][1][e], b2 = vel[sl][1][e];
          rb[r] = b1 + ca * ((b1 - b2) / cb);
          // ducts: u on a y ghost row keeps its y extrapolation of the stored plane (corner rule)
          if (!yghost(r)) {
            const T a1 = vel[s1][0][e], a2 = vel[sl][0][e];
            ra[r] = a1 + ca * ((a1 - a2) / cb);
          }
        }
      }
    }
    for (int r = 0; r < NL; ++r) {
      const int e = tid + r * NT;
      if (e < N2) {
        vel[sl][0][e] = ra[r];
        vel[sl][1][e] = rb[r];
        vel[sl][2][e] = rc[r];
      }
    }
  };
  // z pass of the velocity filter by partial sums: G1 holds plane p's sum without its upper
  // neighbour, G2 plane p + 1's lower-neighbour term; z weights per plane (lower, centre,
  // upper) are (0, 1, 0) for u, v on the first off-wall layers and 0 for w on the top wall face
  T G1[NH][3], G2[NH][3];
  auto zw = [&](int q, int c, int which) -> T {
    if (!per && c == 2 && q == nz) return (T)0;
    if (!per && c < 2 && (q == 1 || q == nz)) return which == 1 ? (T)1 : (T)0;
    return which == 1 ? W1 : W0;
  };
  // x-y filter of velocity plane q at the thread's halo-1 points, folded into the z sums;
  // completes the filtered velocity of plane q - 1 (written to its ring slot when put != 0)
  auto filter_xy = [&](int q, bool put) {
    const int sl = q & 1, so = (q - 1) & 1;
    for (int r = 0; r < NH; ++r) {
      const int e = tid + r * NT;
      if (e < N1) {
        // the thread's halo-1 points for the velocity filter (R2 coordinates)
        const int hx = e % RX1 + 1, hy = e / RX1 + 1;
        const int jr = j0 - 2 + hy;   // global row of the point
        const bool yedge = YW && (jr == 0 || jr == g.ny - 1);
        for (int c = 0; c < 3; ++c) {
          T pl = (T)0;
          for (int dy = -1; dy <= 1; ++dy) {
            const T* rr = &vel[sl][c][(hy + dy) * RX2 + hx];
            const T row = W0 * rr[-1] + W1 * rr[0] + W0 * rr[1];
            const T wy = (yedge && c != 1) ? (dy == 0 ? (T)1 : (T)0) : (dy == 0 ? W1 : W0);
            pl = pl + wy * row;
          }
          if (YW && c == 1 && (jr >= g.ny - 1 || jr < 0)) pl = (T)0;   // v~ on and beyond the y walls
          if (put) ut[so][c][e] = G1[r][c] + zw(q - 1, c, 2) * pl;
          G1[r][c] = G2[r][c] + zw(q, c, 1) * pl;
          G2[r][c] = zw(q + 1, c, 0) * pl;
        }
      }
    }
  };
  // ducts: the y ghost rows of u~ and w~ of plane q by the strain ghost rule (extrapolated
  // with the wall model, odd with no-slip), from the completed rows next to them
  auto fix_rows = [&](int q) {
    const int sl = q & 1;
    for (int e = tid; e < N1; e += NT) {
      const int jr = j0 - 1 + e / RX1;
      if (jr != -1 && jr != g.ny) continue;
      const int d = jr < 0 ? RX1 : -RX1;   // one row inward
      for (int c = 0; c < 3; c += 2) {
        const T a0 = ut[sl][c][e + d];
        ut[sl][c][e] = wm ? a0 - (ut[sl][c][e + 2 * d] - a0) : -a0;
      }
    }
  };
  // the thread's stage points: its own cell and, on the first NHALO threads, one halo-1 point
  // (R2 coordinates); each carries the upper z-edge terms of the previous plane
  const int ox = tx + 2, oy = ty + 2;
  const bool has_halo = tid < NHALO;
  int bx = 1, by = 1;
  if (has_halo) {
    const int h = tid;
    if (h < 2 * RX1) {
      bx = h % RX1 + 1;
      by = h < RX1 ? 1 : RY1;
    } else {
      bx = (h - 2 * RX1) < TY ? 1 : RX1;
      by = (h - 2 * RX1) % TY + 2;
    }
  }
  ZEdges<T> P0, P1;   // velocity: own cell, halo point
  ZEdges<T> PT;       // filtered velocity: own cell
  auto vacc = [](int s0, int s1) {
    return [=](int c, int dz, int o) -> T { return vel[dz ? s1 : s0][c][o]; };
  };
  // running sums of the z pass of the test filter over the thread's cell: S1 holds plane p's
  // sum without its upper neighbour, S2 plane p + 1's lower-neighbour term
  T S1[NQ], S2[NQ], qx[NQ];
  auto zq = [&](int q, int which) -> T {
    if (!per && (q == 1 || q == nz)) return which == 1 ? (T)1 : (T)0;
    return which == 1 ? W1 : W0;
  };
  // ---- stage p: filter inputs of plane p at the tile + 1 halo, then their x-y filter at the
  // thread's cell (into qx)
  auto stage = [&](int p) {
    const int pq = phys(p);
    const int s0 = p & 1, s1 = (p + 1) & 1;
    const T rdzf = (T)ro_load(g.rdzf, pq), rdzc = (T)ro_load(g.rdzc, pq);
    const T rdzn = rdzc_above(p);
    const bool wrap = phys(p + 1) - 1 != pq;
    const bool own = p >= kb && p <= ke;
    const auto A = vacc(s0, s1);
    auto point = [&](int x, int y, ZEdges<T>& P, bool store) {
      const int o = y * RX2 + x;
      const ZEdges<T> E = zedges<T>(A, o, RX2, rdx, rdy, rdzc);
      T s[6];
      strain_zm<T>(A, o, RX2, rdx, rdy, rdzf, P, E, s);
      const T sm_ = strain_norm32<T>(s);
      const int e = (y - 1) * RX1 + x - 1;
      const T uc = (T)0.5 * (A(0, 0, o) + A(0, 0, o - 1));
      const T vc = (T)0.5 * (A(1, 0, o) + A(1, 0, o - RX2));
      const T wc = (T)0.5 * (E.w + P.w);
      qb[0][e] = T2(uc, vc);
      qb[1][e] = T2(wc, uc * uc);
      qb[2][e] = T2(vc * vc, wc * wc);
      qb[3][e] = T2(uc * vc, uc * wc);
      qb[4][e] = T2(vc * wc, sm_ * s[0]);
      qb[5][e] = T2(sm_ * s[1], sm_ * s[2]);
      qb[6][e] = T2(sm_ * s[3], sm_ * s[4]);
      qb[7][e] = T2(sm_ * s[5], (T)0);
      if (store && nut != nullptr && own) {
        const int i = i0 + tx, j = j0 + ty;
        if (i < g.nx && j < g.ny) store_nut(g, nut, p, j, i, sm_);
      }
      if (wrap)
        P = zedges<T>(A, o, RX2, rdx, rdy, rdzn);
      else
        P = E;
    };
    point(ox, oy, P0, true);
    if (has_halo) point(bx, by, P1, false);
    lds_barrier();
    // x-y filter of the 15 inputs at the thread's own cell (R1 coords tx+1, ty+1)
    for (int a = 0; a < NQ; ++a) qx[a] = (T)0;
    const bool yedge = YW && (j0 + ty == 0 || j0 + ty == g.ny - 1);
#pragma unroll 1
    for (int dy = -1; dy <= 1; ++dy)
#pragma unroll 1
      for (int dx = -1; dx <= 1; ++dx) {
        const T wy = yedge ? (dy == 0 ? (T)1 : (T)0) : (dy == 0 ? W1 : W0);
        const T wxy = wy * (dx == 0 ? W1 : W0);
        const int e = (ty + 1 + dy) * RX1 + tx + 1 + dx;
#pragma unroll
        for (int a = 0; a < NQ; ++a) {
          const T2 pr = qb[a / 2][e];
          qx[a] = qx[a] + wxy * (a % 2 ? pr.y : pr.x);
        }
      }
  };
  // ---- output plane k: F holds the test-filtered inputs of its cell; the filtered velocity of
  // planes k and k + 1 is in the ring (the top ghost plane is formed on the fly), PT holds the
  // upper edge terms of plane k - 1
  auto output = [&](int k, const T* F) {
    const int pk = phys(k);
    double lm = 0.0, mm = 0.0;
    const int i = i0 + tx, j = j0 + ty;
    const int o = (ty + 1) * RX1 + tx + 1;   // own cell in R1
    const int sA = k & 1, sB = (k + 1) & 1;
    const bool top = !per && k == nz;
    const T rdzc = (T)ro_load(g.rdzc, pk), rdzf = (T)ro_load(g.rdzf, pk);
    T st[6];
    if (top) {
      // strain ghost rule above the top wall, from planes nz (slot sA) and nz - 1 (slot sB)
      const T ca = (T)ro_load(g.dzc, nz), cb = (T)ro_load(g.dzc, nz - 1);
      const auto A = [&](int c, int dz, int oo) -> T {
        const T a1 = ut[sA][c][oo];
        if (dz == 0) return a1;
        const T a2 = ut[sB][c][oo];
        return wm ? a1 + ca * ((a1 - a2) / cb) : -a1;
      };
      strain_zm<T>(A, o, RX1, rdx, rdy, rdzf, PT, zedges<T>(A, o, RX1, rdx, rdy, rdzc), st);
    } else {
      const auto A = [&](int c, int dz, int oo) -> T { return ut[dz ? sB : sA][c][oo]; };
      const ZEdges<T> E = zedges<T>(A, o, RX1, rdx, rdy, rdzc);
      strain_zm<T>(A, o, RX1, rdx, rdy, rdzf, PT, E, st);
      if (phys(k + 1) - 1 != pk)
        PT = zedges<T>(A, o, RX1, rdx, rdy, rdzc_above(k));
      else
        PT = E;
    }
    if (i < g.nx && j < g.ny) {
      const T stm = strain_norm32<T>(st);
      const bool wall_layer = !per && (k == 1 || k == nz);
      const bool wall_row = YW && (j == 0 || j == g.ny - 1);
      // 3-D, 2-D or (duct corners) 1-D test filter: 4, 4^(2/3), 2^(2/3)
      const T alpha2 = (wall_layer && wall_row) ? (T)1.5874010519681994
                                                : ((wall_layer || wall_row) ? (T)2.5198420997897464 : (T)4);
      const T d2 = (T)ro_load(g.delta2, pk);
      const T Fa[6] = {F[0], F[1], F[2], F[0], F[0], F[1]}, Fb[6] = {F[0], F[1], F[2], F[1], F[2], F[2]};
      for (int c = 0; c < 6; ++c) {
        const T L = F[3 + c] - Fa[c] * Fb[c];
        const T M = (T)2 * d2 * (F[9 + c] - alpha2 * stm * st[c]);
        const double wgt2 = c < 3 ? 1.0 : 2.0;
        lm += wgt2 * (double)L * (double)M;
        mm += wgt2 * (double)M * (double)M;
      }
    }
    lm = row_sum(lm);
    mm = row_sum(mm);
    if (YW) {
      // x-line sums: a row of the tile is 32 lanes (two rows of 16) of one wave; partials
      // [k][j][tile x]
      const bool lo = (tid & 63) < 32;
      lm = lo ? lane_f64(lm, 0) + lane_f64(lm, 16) : lane_f64(lm, 32) + lane_f64(lm, 48);
      mm = lo ? lane_f64(mm, 0) + lane_f64(mm, 16) : lane_f64(mm, 32) + lane_f64(mm, 48);
      const int jrow = j0 + ty;
      if (tx == 0 && jrow < g.ny) {
        const int64_t oo = (((int64_t)(k - 1) * g.ny + jrow) * gdx + bid.x) * 2;
        part[oo] = lm;
        part[oo + 1] = mm;
      }
      return;
    }
    // wave sums in a fixed order (row trees, then the four rows in turn); the waves' partials
    // go out per plane and are summed over (tile, wave) in a fixed order by the plane reduction
    lm = ((lane_f64(lm, 0) + lane_f64(lm, 16)) + lane_f64(lm, 32)) + lane_f64(lm, 48);
    mm = ((lane_f64(mm, 0) + lane_f64(mm, 16)) + lane_f64(mm, 32)) + lane_f64(mm, 48);
    if (tid % 64 == 0) {
      const int64_t oo = ((int64_t)(k - 1) * ntile * WV + tile * WV + tid / 64) * 2;
      part[oo] = lm;
      part[oo + 1] = mm;
    }
  };
  // ---- prologue: planes pstart - 1 and pstart in the ring, pstart + 1 in flight
  const int pstart = per ? kb - 1 : max(kb - 1, 1);
  const int pend = per ? ke + 1 : min(ke + 1, nz);
  if (wm && pstart == 1) {
    // the bottom ghost plane: u, v extrapolated linearly in z from planes 1 (in the ring) and
    // 2 (held in registers), w and the duct's y-ghost u as stored
    fetch(1);
    commit(1);
    fetch(2);
    T xa[NL], xb[NL];
    for (int r = 0; r < NL; ++r) {
      xa[r] = ra[r];
      xb[r] = rb[r];
    }
    fetch(0);
    const T ca = (T)ro_load(g.dzc, 0), cb = (T)ro_load(g.dzc, 1);
    for (int r = 0; r < NL; ++r) {
      const int e = tid + r * NT;
      if (e < N2) {
        const T b1 = vel[1][1][e];
        rb[r] = b1 - ca * ((xb[r] - b1) / cb);
        if (!yghost(r)) {
          const T a1 = vel[1][0][e];
          ra[r] = a1 - ca * ((xa[r] - a1) / cb);
        }
      }
    }
    commit(0);
    fetch(2);
  } else {
    fetch(pstart - 1);
    commit(pstart - 1);
    fetch(pstart);
    commit(pstart);
    fetch(pstart + 1);
  }
  lds_barrier();
  for (int r = 0; r < NH; ++r)
    for (int c = 0; c < 3; ++c) G2[r][c] = (T)0;
  filter_xy(pstart - 1, false);
  filter_xy(pstart, false);
  {
    const auto A = vacc((pstart - 1) & 1, pstart & 1);
    const T rdzn = rdzc_above(pstart - 1);
    P0 = zedges<T>(A, oy * RX2 + ox, RX2, rdx, rdy, rdzn);
    if (has_halo) P1 = zedges<T>(A, by * RX2 + bx, RX2, rdx, rdy, rdzn);
  }
  for (int a = 0; a < NQ; ++a) S2[a] = (T)0;
  lds_barrier();   // the first commit replaces plane pstart - 1
  // ---- march: velocity plane p + 1 is committed to LDS at the top of iteration p, the loads
  // of plane p + 2 are issued right after and complete under the work on plane p.  Threads
  // exchange data through LDS only (the stored |S| and partial sums are read by later
  // launches): the barriers leave global loads in flight.
  for (int p = pstart; p <= pend; ++p) {
    commit(p + 1);
    lds_barrier();
    fetch(min(p + 2, pend + 1));   // the last one reloads plane pend + 1 and is not committed
    filter_xy(p + 1, true);
    stage(p);
    if (YW) {
      fix_rows(p);
      lds_barrier();
    }
    const int k = p - 1;
    if (k == kb - 1 && (per || kb > 1)) {
      // upper edge terms of the filtered velocity below the first output plane
      const auto A = [&](int c, int dz, int oo) -> T { return ut[dz ? (p & 1) : (k & 1)][c][oo]; };
      PT = zedges<T>(A, (ty + 1) * RX1 + tx + 1, RX1, rdx, rdy, rdzc_above(k));
    }
    if (k >= kb && k <= ke) {
      if (!per && k == 1) {
        // below the bottom wall: the strain ghost rule from planes 1 and 2, w~ = 0 on the wall
        const T ca = (T)ro_load(g.dzc, 0), cb = (T)ro_load(g.dzc, 1);
        const auto A = [&](int c, int dz, int oo) -> T {
          if (dz) return ut[1][c][oo];
          if (c == 2) return (T)0;
          const T a1 = ut[1][c][oo], a2 = ut[0][c][oo];
          return wm ? a1 - ca * ((a2 - a1) / cb) : -a1;
        };
        PT = zedges<T>(A, (ty + 1) * RX1 + tx + 1, RX1, rdx, rdy, (T)ro_load(g.rdzc, 0));
      }
      for (int a = 0; a < NQ; ++a) S1[a] = S1[a] + zq(k, 2) * qx[a];
      output(k, S1);
    }
    for (int a = 0; a < NQ; ++a) {
      S1[a] = S2[a] + zq(p, 1) * qx[a];
      S2[a] = zq(p + 1, 0) * qx[a];
    }
  }
  if (!per && ke == nz) output(nz, S1);   // the z pass is the identity on the top layer
}

template <typename T, bool YW>
__global__ void __launch_bounds__((fused32::Tile<T, YW>::NT), dsm_blocks_per_cu(false))
    k_dsm_fused32(GridP g, const T* u, const T* v, const T* w, T* nut, double* part, int kc, const int* gate) {
  dsm_fused32_body<T, YW>(xcd_tile(blockIdx, gridDim), gridDim.x, gridDim.y, g, u, v, w, nut, part, kc, gate);
}

// Ducts: c_s per x line (j, k) from the tile partials [k][j][tile x], summed in tile order,
// clipped at zero (0 where <M M> = 0); one thread per line.  gate: as in k_dsm_fused.
__global__ void __launch_bounds__(256) k_dsm_reduce_lines(GridP g, const double* part, int ntx, double* cs,
                                                          const int* gate) {
  if (gate != nullptr && gate[0] == 0) return;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= g.nz * g.ny) return;
  double a = 0.0, b = 0.0;
  for (int t = 0; t < ntx; ++t) {
    a += part[((int64_t)e * ntx + t) * 2];
    b += part[((int64_t)e * ntx + t) * 2 + 1];
  }
  cs[e] = b > 0.0 ? fmax(a / b, 0.0) : 0.0;
}

// Ducts: the stored field becomes c_s(j, k) |S| (the plane factor coef[k] = Delta_k^2), the
// ghost planes taking the coefficient of their neighbour plane; one thread per stored cell
// of the interior rows (the ghost rows are refilled afterwards).
template <typename T>
__global__ void __launch_bounds__(256) k_nut_lines(GridP g, T* nut, const double* cs) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nxy = (int64_t)g.nx * g.ny;
  if (e >= (int64_t)(g.nz + 2) * nxy) return;
  const int k = (int)(e / nxy);
  const int64_t r = e % nxy;
  const int j = (int)(r / g.nx);
  const int kk = k < 1 ? 1 : (k > g.nz ? g.nz : k);
  const int64_t c = (int64_t)k * g.sxy + r;
  nut[c] = (T)((double)nut[c] * cs[(int64_t)(kk - 1) * g.ny + j]);
}

// Batched dynamic model (and its plane / volume reduction) over all boxes of a batch (periodic boxes).
template <typename T>
__global__ void __launch_bounds__(fused::Tile<T>::NT, fused::Tile<T>::WEU) kb_dsm_fused(BatchMap m) {
  int box;
  const dim3 bid = batch_bid(m, BK_DSM, blockIdx.x, box);
  const BoxDesc& d = m.desc[box];
  dsm_fused_body<T, false, LES_ZBC_PERIODIC>(bid, d.gdim[BK_DSM][0], d.gdim[BK_DSM][1], d.g, (const T*)d.u, (const T*)d.v,
                                             (const T*)d.w, (T*)d.nut, d.dsm_part, d.kc, nullptr);
}

template <typename T>
__global__ void __launch_bounds__(256) kb_dsm_reduce(BatchMap m) {
  int box;
  const dim3 bid = batch_bid(m, BK_DSMRED, blockIdx.x, box);
  const BoxDesc& d = m.desc[box];
  dsm_reduce_body<T>(bid.x, d.g, d.dsm_part, d.gdim[BK_DSM][0] * d.gdim[BK_DSM][1] * fused::Tile<T>::WV, d.cs, d.coef,
                     nullptr, (T*)nullptr);
}

// One plane of a box per thread, by the single context's code: batch and single context agree to the last bit.
template <typename T>
__global__ void __launch_bounds__(256) kb_strain_mag(BatchMap m) {
  int box;
  const dim3 bid = batch_bid(m, BK_POINT, blockIdx.x, box);
  const BoxDesc& d = m.desc[box];
  const int i = bid.x * blockDim.x + threadIdx.x;
  const int j = bid.y * blockDim.y + threadIdx.y;
  const int k = bid.z + 1;
  if (i >= d.g.nx || j >= d.g.ny) return;
  strain_column(d.g, (const T*)d.u, (const T*)d.v, (const T*)d.w, (T*)d.nut, nullptr, j, i, k, k + 1);
}

// ============================================================================ learned closure
// Plane sums of the four wall-stress components (bottom x, bottom y, top x, top y) from the
// wall-model stresses or the no-slip viscous flux, WM_BLOCKS blocks over contiguous chunks of
// the plane, each a fixed-order tree; the last block to finish (a ticket counter, cleared
// again by that block) sums the partials by a fixed-order tree and stores the friction velocity of
// each wall, u_tau = sqrt(|(<tau_x>, <tau_y>)|), in dt[2] (bottom) and dt[3] (top).  cnt
// (learned closure, may be null): that block also clears the fallback counters, ahead of the
// inference kernel that adds to them.
constexpr int WM_BLOCKS = 64;

template <typename T>
__global__ void __launch_bounds__(256) k_wall_mean(GridP g, const T* u, const T* v, const double* tau, int wallmodel,
                                                   double* part, double* dtp, int* cnt, unsigned* ticket) {
  __shared__ double sm[4][256];
  __shared__ bool last;
  double a[4] = {0, 0, 0, 0};
  const int64_t s = g.sxy;
  const int n = g.nz;
  const int64_t chunk = (s + WM_BLOCKS - 1) / WM_BLOCKS;
  const int64_t c0 = blockIdx.x * chunk, c1 = c0 + chunk < s ? c0 + chunk : s;
  if (g.zbc != LES_ZBC_PERIODIC)
    for (int64_t c = c0 + threadIdx.x; c < c1; c += 256) {
      if (wallmodel) {
        for (int q = 0; q < 4; ++q) a[q] += tau[q * s + c];
      } else {
        a[0] += g.nu * ((double)u[s + c] - (double)u[c]) / g.dzc[0];
        a[1] += g.nu * ((double)v[s + c] - (double)v[c]) / g.dzc[0];
        a[2] += g.nu * ((double)u[(int64_t)n * s + c] - (double)u[(int64_t)(n + 1) * s + c]) / g.dzc[n];
        a[3] += g.nu * ((double)v[(int64_t)n * s + c] - (double)v[(int64_t)(n + 1) * s + c]) / g.dzc[n];
      }
    }
  for (int q = 0; q < 4; ++q) sm[q][threadIdx.x] = a[q];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int q = 0; q < 4; ++q) sm[q][threadIdx.x] += sm[q][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 4) {
    part[blockIdx.x * 4 + threadIdx.x] = sm[threadIdx.x][0];
    __threadfence();   // the partial is visible device-wide before the ticket is taken
  }
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(ticket, 1u) == WM_BLOCKS - 1;
  __syncthreads();
  if (!last || threadIdx.x >= 64) return;
  __threadfence();   // the other blocks' partials, published before their tickets
  static_assert(WM_BLOCKS <= 64, "one lane per block partial");
  double w[4];
  for (int q = 0; q < 4; ++q) {   // a fixed-order shuffle tree over the block partials
    double x = threadIdx.x < WM_BLOCKS ? part[threadIdx.x * 4 + q] : 0.0;
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    w[q] = x;
  }
  if (threadIdx.x != 0) return;
  const double area = (double)s;
  dtp[2] = sqrt(hypot(w[0] / area, w[1] / area));
  dtp[3] = sqrt(hypot(w[2] / area, w[3] / area));
  if (cnt != nullptr) {
    cnt[0] = 0;
    cnt[1] = 0;
  }
  *ticket = 0u;
}

// Rotation tensor at the cell centre (edges, then the four-edge mean, like the strain),
// with the strain ghost rules (z, and y in a duct): o[0..2] = O12, O13, O23.
template <typename T>
__device__ inline void centre_rotation(const GridP& g, const T* u, const T* v, const T* w, int k, int j, int i,
                                       double o[3]) {
  const int ip = wrap_p(i, g.nx), im = wrap_m(i, g.nx), jp = wrap_p(j, g.nys), jm = wrap_m(j, g.nys);
  const double rdx = g.rdx, rdy = g.rdy, rdzc = 1.0 / g.dzc[k], rdzcm = 1.0 / g.dzc[k - 1];
  auto U = [&](int kk, int jj, int ii) { return (double)sval_y(g, u, kk, jj, ii, true); };
  auto V = [&](int kk, int jj, int ii) { return (double)sval(g, v, kk, jj, ii); };
  auto W = [&](int kk, int jj, int ii) { return (double)sval_y(g, w, kk, jj, ii, false); };
  auto r12 = [&](int jj, int ii) {
    return 0.5 * ((U(k, wrap_p(jj, g.nys), ii) - U(k, jj, ii)) * rdy - (V(k, jj, wrap_p(ii, g.nx)) - V(k, jj, ii)) * rdx);
  };
  o[0] = 0.25 * (r12(j, i) + r12(j, im) + r12(jm, i) + r12(jm, im));
  auto r13 = [&](int kk, int ii, double rz) {
    return 0.5 * ((U(kk + 1, j, ii) - U(kk, j, ii)) * rz - (W(kk, j, wrap_p(ii, g.nx)) - W(kk, j, ii)) * rdx);
  };
  o[1] = 0.25 * (r13(k, i, rdzc) + r13(k, im, rdzc) + r13(k - 1, i, rdzcm) + r13(k - 1, im, rdzcm));
  auto r23 = [&](int kk, int jj, double rz) {
    return 0.5 * ((V(kk + 1, jj, i) - V(kk, jj, i)) * rz - (W(kk, wrap_p(jj, g.nys), i) - W(kk, jj, i)) * rdy);
  };
  o[2] = 0.25 * (r23(k, j, rdzc) + r23(k, jm, rdzc) + r23(k - 1, j, rdzcm) + r23(k - 1, jm, rdzcm));
  (void)ip;
  (void)jp;
}

// The seven raw inputs of the network at a cell (see les.h): invariants of S/n and O/n,
// n = sqrt(S_ij S_ij + O_ij O_ij), then y+ and Delta/delta (delta = 1).
__device__ inline void raw_features(const double s[6], const double o[3], double yplus, double delta, double f[7]) {
  // closed forms for a symmetric S = (s11 s22 s33 s12 s13 s23) and an antisymmetric O with
  // upper entries (o12 o13 o23): P = O^2 (symmetric), Q = S^2 (symmetric)
  const double s11 = s[0], s22 = s[1], s33 = s[2], s12 = s[3], s13 = s[4], s23 = s[5];
  const double o1 = o[0], o2 = o[1], o3 = o[2];
  const double ss = s11 * s11 + s22 * s22 + s33 * s33 + 2.0 * (s12 * s12 + s13 * s13 + s23 * s23);
  const double oo = 2.0 * (o1 * o1 + o2 * o2 + o3 * o3);
  const double nrm = sqrt(ss + oo);
  const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
  const double i2 = inv * inv, i3 = i2 * inv, i4 = i2 * i2;
  const double p00 = -(o1 * o1 + o2 * o2), p11 = -(o1 * o1 + o3 * o3), p22 = -(o2 * o2 + o3 * o3);
  const double p01 = -o2 * o3, p02 = o1 * o3, p12 = -o1 * o2;
  const double q00 = s11 * s11 + s12 * s12 + s13 * s13, q11 = s12 * s12 + s22 * s22 + s23 * s23;
  const double q22 = s13 * s13 + s23 * s23 + s33 * s33;
  const double q01 = s11 * s12 + s12 * s22 + s13 * s23, q02 = s11 * s13 + s12 * s23 + s13 * s33;
  const double q12 = s12 * s13 + s22 * s23 + s23 * s33;
  const double s3 = q00 * s11 + q11 * s22 + q22 * s33 + 2.0 * (q01 * s12 + q02 * s13 + q12 * s23);   // tr S^3
  const double ps = p00 * s11 + p11 * s22 + p22 * s33 + 2.0 * (p01 * s12 + p02 * s13 + p12 * s23);   // tr O^2 S
  const double pq = p00 * q00 + p11 * q11 + p22 * q22 + 2.0 * (p01 * q01 + p02 * q02 + p12 * q12);   // tr O^2 S^2
  f[0] = ss * i2;
  f[1] = -oo * i2;
  f[2] = s3 * i3;
  f[3] = ps * i3;
  f[4] = pq * i4;
  f[5] = yplus;
  f[6] = delta;
}

struct MlpNorm {
  double lo[7], inv[7];   // scaled input = (raw - lo) * inv, inv = 1 / (hi - lo)
};

// y+ of cell (k, j): the distance to the nearer z wall in that wall's units (ut[0] bottom,
// ut[1] top); in a duct the smallest d_w u_tau,w over the four walls (ut[2] at y = 0, ut[3]
// at y = ly), the van Driest rule; 0 with periodic z.
__device__ inline double cell_yplus(const GridP& g, int k, int j, const double* ut, double ly) {
  if (g.zbc == LES_ZBC_PERIODIC) return 0.0;
  const double zc = g.zc[k];
  if (g.ywall) {
    const double yc = (j + 0.5) * g.dy;
    return fmin(fmin(zc * ut[0], (g.lz - zc) * ut[1]), fmin(yc * ut[2], (ly - yc) * ut[3])) / g.nu;
  }
  const bool lower = zc <= 0.5 * g.lz;
  return (lower ? zc : g.lz - zc) * (lower ? ut[0] : ut[1]) / g.nu;
}

template <typename T>
__device__ inline void cell_features(const GridP& g, const T* u, const T* v, const T* w, int k, int j, int i,
                                     const double* ut, double ly, double f[7], T s6[6]) {
  centre_strain(g, u, v, w, k, j, i, s6);
  double s[6];
  for (int a = 0; a < 6; ++a) s[a] = (double)s6[a];
  double o[3];
  centre_rotation(g, u, v, w, k, j, i, o);
  raw_features(s, o, cell_yplus(g, k, j, ut, ly), sqrt(g.delta2[k]), f);
}

// Fused inference, z-marching over a chunk of planes per 32 x 8 tile (like the dynamic
// model): the velocity ring of 3 planes on the tile + 1 halo sits in LDS (strain ghost rule
// applied on wall ghost planes).  Per plane each thread forms the velocity-gradient tensor
// of its cell (diagonal at the centre, off-diagonal terms as four-edge means, so S and O are
// its symmetric and antisymmetric parts), the seven scaled inputs, and each wave of 64 cells
// runs the network on the matrix cores.  Stores c |S| with c = max(0, MLP); a cell whose
// scaled inputs leave [-0.05, 1.05] is counted and stores -|S| instead, a mark that
// k_mlp_fallback replaces by the dynamic coefficient of its plane (of its x line in a duct,
// YW) times |S| once the dynamic model of the same state has run (c |S| >= 0 elsewhere).
namespace tiled {
constexpr int TX = 32, TY = 8, NT = TX * TY;
constexpr int RX = TX + 2, RY = TY + 2, N1 = RX * RY;
}  // namespace tiled

template <typename T, bool YW, int ZBC = -1>
__global__ void __launch_bounds__(256, 4) k_mlp_nut(GridP g, const T* __restrict__ u, const T* __restrict__ v,
                                                 const T* __restrict__ w, T* __restrict__ nut,
                                                 const float* __restrict__ P, MlpNorm nm,
                                                 const double* __restrict__ ut, double ly, int* __restrict__ cnt,
                                                 int kc) {
  using namespace mlp;
  using tiled::TX;
  using tiled::TY;
  using tiled::RX;
  using tiled::RY;
  using tiled::N1;
  __shared__ Weights Wt;
  constexpr int XS = 8;   // stored features per cell (7 and a zero): four blocks per CU in FP64
  __shared__ __align__(16) unsigned short xs[WAVES][64 * XS];
  __shared__ T vel[3][3][N1];
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * TX + tx;
  const int wave = tid / 64, lane = tid % 64;
  const dim3 bid = xcd_tile(blockIdx, gridDim);
  const int i0 = bid.x * TX, j0 = bid.y * TY;
  const int nz = g.nz;
  const int kb = 1 + bid.z * kc;
  const int ke = min(nz, kb + kc - 1);
  const int zbc = ZBC < 0 ? g.zbc : ZBC;
  const bool per = zbc == LES_ZBC_PERIODIC;
  const bool wm = zbc == LES_ZBC_WALLMODEL;
  load_weights(P, Wt, tid, tiled::NT);
  auto phys = [&](int q) {
    if (!per) return q;
    int m = (q - 1) % nz;
    if (m < 0) m += nz;
    return m + 1;
  };
  auto slot = [](int q) { return ((q % 3) + 3) % 3; };
  // in-plane offsets of the thread's halo points (tiles may exceed the grid: wrap), and the
  // velocity of one plane held in registers from its fetch to its commit to LDS, so that the
  // loads of plane k + 2 overlap the work on plane k (strain ghost rule applied at fetch)
  constexpr int NL = (N1 + tiled::NT - 1) / tiled::NT;
  int lofs[NL];
  int yg[NL];   // ducts: 0, or the offset to the first interior row next to a y ghost row (+-nx)
  for (int r = 0; r < NL; ++r) {
    const int e = tid + r * tiled::NT;
    const int lrow = j0 - 1 + e / RX;
    int ii = (i0 - 1 + e % RX) % g.nx, jj = lrow % g.nys;
    if (ii < 0) ii += g.nx;
    if (jj < 0) jj += g.nys;
    lofs[r] = e < N1 ? jj * g.nx + ii : 0;
    yg[r] = 0;
    if (YW && wm && e < N1 && (lrow == -1 || lrow == g.ny)) {
      // strain ghost of u and w on a y ghost row: 2 a0 - a1 from the two rows next to it
      lofs[r] = (lrow < 0 ? 0 : g.ny - 1) * g.nx + ii;
      yg[r] = lrow < 0 ? g.nx : -g.nx;
    }
  }
  const int64_t sxy = g.sxy;
  // raw unconditional loads (points past the halo read offset 0 and are not committed), so
  // that nothing waits for them before their commit one plane later; the wall model's strain
  // ghosts on the wall ghost planes are formed at the commit from the thread's own LDS entries
  // of the two planes next to the wall
  T ra[NL], rb[NL], rc[NL];
  auto fetch = [&](int q) {
    const int pq = phys(q);
    const PlaneLoader<T> lu(u, pq, sxy), lv(v, pq, sxy), lw(w, pq, sxy);
    for (int r = 0; r < NL; ++r) {
      ra[r] = lu(lofs[r]);
      rb[r] = lv(lofs[r]);
      rc[r] = lw(lofs[r]);
    }
    if (YW) {
      for (int r = 0; r < NL; ++r) {
        if (yg[r] != 0) {
          // lofs points at the interior row next to the ghost row: u and w extrapolated in y
          // (in the z ghost planes these corner values are not used); v is 0 on the wall face
          const T a1 = lu(lofs[r] + yg[r]), c1 = lw(lofs[r] + yg[r]);
          ra[r] = ra[r] - (a1 - ra[r]);
          rc[r] = rc[r] - (c1 - rc[r]);
          rb[r] = (T)0;
        }
      }
    }
  };
  auto commit = [&](int q) {
    const int sl = slot(q);
    const int pq = phys(q);
    if (wm && (pq == 0 || pq == nz + 1)) {
      const bool bot = pq == 0;
      const int s1 = slot(bot ? q + 1 : q - 1), s2 = slot(bot ? q + 2 : q - 2);
      const T ca = (T)ro_load(g.dzc, bot ? 0 : nz), cb = (T)ro_load(g.dzc, bot ? 1 : nz - 1);
      for (int r = 0; r < NL; ++r) {
        const int e = tid + r * tiled::NT;
        if (e < N1 && !(YW && yg[r] != 0)) {
          const T a1 = vel[s1][0][e], a2 = vel[s2][0][e];
          const T b1 = vel[s1][1][e], b2 = vel[s2][1][e];
          ra[r] = bot ? a1 - ca * ((a2 - a1) / cb) : a1 + ca * ((a1 - a2) / cb);
          rb[r] = bot ? b1 - ca * ((b2 - b1) / cb) : b1 + ca * ((b1 - b2) / cb);
        }
      }
    }
    for (int r = 0; r < NL; ++r) {
      const int e = tid + r * tiled::NT;
      if (e < N1) {
        vel[sl][0][e] = ra[r];
        vel[sl][1][e] = rb[r];
        vel[sl][2][e] = rc[r];
      }
    }
  };
  if (wm && kb == 1) {
    // the bottom ghost plane is formed from planes 1 and 2: those are committed first (plane 2
    // is fetched again for the loop's first commit)
    fetch(1);
    commit(1);
    fetch(2);
    commit(2);
    fetch(0);
    commit(0);
    fetch(2);
  } else {
    fetch(kb - 1);
    commit(kb - 1);
    fetch(kb);
    commit(kb);
    fetch(kb + 1);
  }
  int flagged = 0;
  const int i = i0 + tx, j = j0 + ty;
  const bool inside = i < g.nx && j < g.ny;
  // threads exchange data through LDS only: the barriers leave global loads in flight
  for (int k = kb; k <= ke; ++k) {
    commit(k + 1);
    lds_barrier();
    fetch(min(k + 2, ke + 1));   // the last one reloads plane ke + 1 and is not committed
    const int pk = phys(k);
    const int sm = slot(k - 1), s0 = slot(k), sp = slot(k + 1);
    const int x = tx + 1, y = ty + 1;
    auto A = [&](int c, int dz, int dy, int dx) -> T {
      const int sl = dz < 0 ? sm : (dz > 0 ? sp : s0);
      return vel[sl][c][(y + dy) * RX + x + dx];
    };
    const T rdx = (T)g.rdx, rdy = (T)g.rdy, rdzf = (T)ro_load(g.rdzf, pk);
    const T rdzc = (T)ro_load(g.rdzc, pk), rdzcm = (T)ro_load(g.rdzc, pk - 1);
    const T q4 = (T)0.25, h = (T)0.5;
    // velocity-gradient tensor at the centre
    const T a11 = (A(0, 0, 0, 0) - A(0, 0, 0, -1)) * rdx;
    const T a22 = (A(1, 0, 0, 0) - A(1, 0, -1, 0)) * rdy;
    const T a33 = (A(2, 0, 0, 0) - A(2, -1, 0, 0)) * rdzf;
    const T dudy = q4 * (((A(0, 0, 1, 0) - A(0, 0, 0, 0)) + (A(0, 0, 1, -1) - A(0, 0, 0, -1)) +
                          (A(0, 0, 0, 0) - A(0, 0, -1, 0)) + (A(0, 0, 0, -1) - A(0, 0, -1, -1))) * rdy);
    const T dvdx = q4 * (((A(1, 0, 0, 1) - A(1, 0, 0, 0)) + (A(1, 0, 0, 0) - A(1, 0, 0, -1)) +
                          (A(1, 0, -1, 1) - A(1, 0, -1, 0)) + (A(1, 0, -1, 0) - A(1, 0, -1, -1))) * rdx);
    const T dudz = q4 * ((A(0, 1, 0, 0) - A(0, 0, 0, 0)) * rdzc + (A(0, 1, 0, -1) - A(0, 0, 0, -1)) * rdzc +
                         (A(0, 0, 0, 0) - A(0, -1, 0, 0)) * rdzcm + (A(0, 0, 0, -1) - A(0, -1, 0, -1)) * rdzcm);
    const T dwdx = q4 * (((A(2, 0, 0, 1) - A(2, 0, 0, 0)) + (A(2, 0, 0, 0) - A(2, 0, 0, -1)) +
                          (A(2, -1, 0, 1) - A(2, -1, 0, 0)) + (A(2, -1, 0, 0) - A(2, -1, 0, -1))) * rdx);
    const T dvdz = q4 * ((A(1, 1, 0, 0) - A(1, 0, 0, 0)) * rdzc + (A(1, 1, -1, 0) - A(1, 0, -1, 0)) * rdzc +
                         (A(1, 0, 0, 0) - A(1, -1, 0, 0)) * rdzcm + (A(1, 0, -1, 0) - A(1, -1, -1, 0)) * rdzcm);
    const T dwdy = q4 * (((A(2, 0, 1, 0) - A(2, 0, 0, 0)) + (A(2, 0, 0, 0) - A(2, 0, -1, 0)) +
                          (A(2, -1, 1, 0) - A(2, -1, 0, 0)) + (A(2, -1, 0, 0) - A(2, -1, -1, 0))) * rdy);
    T s6[6] = {a11, a22, a33, h * (dudy + dvdx), h * (dudz + dwdx), h * (dvdz + dwdy)};
    const double s[6] = {(double)s6[0], (double)s6[1], (double)s6[2], (double)s6[3], (double)s6[4], (double)s6[5]};
    const double o[3] = {0.5 * ((double)dudy - (double)dvdx), 0.5 * ((double)dudz - (double)dwdx),
                         0.5 * ((double)dvdz - (double)dwdy)};
    double yplus = 0.0;
    if (!per) {
      const double zc = ro_load(g.zc, pk);
      if (YW) {
        const double yc = (j + 0.5) * g.dy;
        yplus = fmin(fmin(zc * ro_load(ut, 0), (g.lz - zc) * ro_load(ut, 1)),
                     fmin(yc * ro_load(ut, 2), (ly - yc) * ro_load(ut, 3))) / g.nu;
      } else {
        const bool lower = zc <= 0.5 * g.lz;
        yplus = (lower ? zc : g.lz - zc) * (lower ? ro_load(ut, 0) : ro_load(ut, 1)) / g.nu;
      }
    }
    double f[7];
    raw_features(s, o, yplus, sqrt(ro_load(g.delta2, pk)), f);
    bool flag = false;
    for (int a = 0; a < 7; ++a) {
      const double xn = (f[a] - nm.lo[a]) * nm.inv[a];
      flag = flag || xn < -0.05 || xn > 1.05;
      f[a] = xn;
    }
    {
      // seven bf16 inputs and a zero as one 16-byte LDS store
      auto pk = [&](int a) -> unsigned int {
        if (!inside) return 0u;
        const fl2 pr = {(float)f[a], a + 1 < F ? (float)f[a + 1] : 0.0f};
        return __builtin_bit_cast(unsigned int, __builtin_convertvector(pr, bf2));
      };
      uint4* dst = reinterpret_cast<uint4*>(&xs[wave][lane * XS]);
      dst[0] = make_uint4(pk(0), pk(2), pk(4), pk(6));
    }
    // each wave reads only its own inputs: LDS operations of a wave complete in order
    __builtin_amdgcn_wave_barrier();
    Fwd out;
    forward_wave<false, XS>(Wt, xs[wave], lane, out);
    const int qq = lane >> 4;
    const float yv = qq == 0 ? out.y[0] : (qq == 1 ? out.y[1] : (qq == 2 ? out.y[2] : out.y[3]));
    if (inside) {
      const T smag = strain_mag(s6);
      const T c = yv > 0.0f ? (T)yv : (T)0;
      if (flag) ++flagged;
      store_nut(g, nut, pk, j, i, flag ? -smag : c * smag);
    }
    lds_barrier();   // the ring slot of plane k - 1 is refilled next
  }
  if (cnt != nullptr) {
    for (int off = 32; off > 0; off >>= 1) flagged += __shfl_down(flagged, off, 64);
    if (lane == 0 && flagged) atomicAdd(&cnt[1], flagged);
  }
}

// Fallback of the learned closure: the cells k_mlp_nut marked (negative stored value -|S|)
// take the dynamic coefficient of their plane (of their x line in a duct) computed from the
// same velocity, c_s |S|, ghost planes included.  Runs only when the current evaluation
// flagged a cell (gate = its counter); one thread per interior cell.
template <typename T>
__global__ void __launch_bounds__(256) k_mlp_fallback(GridP g, T* __restrict__ nut, const double* __restrict__ cs,
                                                      const int* __restrict__ gate) {
  if (gate[0] == 0) return;
  const int64_t nxy = (int64_t)g.nx * g.ny;
  const int64_t ncell = (int64_t)g.nz * nxy;
  // grid-stride: the launch is small, so that it costs little when no cell fell back
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < ncell; e += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(e / nxy) + 1;
    const int64_t r = e % nxy;
    const int j = (int)(r / g.nx), i = (int)(r % g.nx);
    const T val = nut[idx3(g, k, j, i)];
    if (!(val < (T)0)) continue;
    const double c = g.ywall ? cs[(int64_t)(k - 1) * g.ny + j] : cs[k - 1];
    store_nut(g, nut, k, j, i, (T)c * -val);
  }
}

// Training pairs: sample s sits at the interior cell hashed from (seed, s) (SplitMix64); x
// gets its seven raw features, y the dynamic coefficient of its plane (of its x line in a
// duct).
__device__ inline uint64_t splitmix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <typename T>
__global__ void k_mlp_sample(GridP g, const T* u, const T* v, const T* w, const double* cs, const double* ut,
                             double ly, uint64_t seed, int64_t n, float* x, float* y) {
  const int64_t sidx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (sidx >= n) return;
  const uint64_t nxy = (uint64_t)g.nx * (uint64_t)g.ny;
  const uint64_t ncell = (uint64_t)g.nz * nxy;
  const uint64_t e = splitmix64(seed ^ splitmix64((uint64_t)sidx)) % ncell;
  const int k = (int)(e / nxy) + 1;
  const int64_t r = (int64_t)(e % nxy);
  const int j = (int)(r / g.nx), i = (int)(r % g.nx);
  double f[7];
  T s6[6];
  cell_features(g, u, v, w, k, j, i, ut, ly, f, s6);
  for (int a = 0; a < 7; ++a) x[sidx * 7 + a] = (float)f[a];
  y[sidx] = (float)(g.ywall ? cs[(int64_t)(k - 1) * g.ny + j] : cs[k - 1]);
}

// ============================================================================ launcher
template <typename T>
void launch_eddy_viscosity(Ctx& c) {
  const GridP& g = c.g;
  const int model = c.cfg.sgs;
  if (model == LES_SGS_NONE) return;
  const double pts = (double)g.nx * g.ny * g.nz;
  if (model == LES_SGS_SMAG || model == LES_SGS_SMAG_VD) {
    const bool duct_vd = g.ywall && model == LES_SGS_SMAG_VD;
    if (duct_vd) {
      static_assert(VD_BLOCKS * 8 <= 4096, "partials fit the reduction area");
      LES_LAUNCH(c, "vd_duct", 0, k_vd_duct_partial<T>, dim3(VD_BLOCKS), dim3(256), 0, g, (const T*)c.u,
                 (const T*)c.v, (const T*)c.w, c.t.tau, c.t.tauy, c.cfg.zbc == LES_ZBC_WALLMODEL ? 1 : 0, c.t.red);
      LES_LAUNCH(c, "vd_duct_final", 0, k_vd_duct_final, dim3(1), dim3(64), 0, g, c.t.red, c.t.vd4,
                 (int*)nullptr);
    }
    // planes a thread marches: as many as leave the chip 2048 waves
    const int64_t tiles = (int64_t)((g.nx + 31) / 32) * ((g.ny + 7) / 8);
    const int kz = (int)std::min<int64_t>(STRAIN_KZ, std::max<int64_t>(1, tiles * 4 * g.nz / 2048));
    LES_LAUNCH(c, "strain_mag", 4 * pts * sizeof(T), k_strain_mag<T>,
               dim3((g.nx + 31) / 32, (g.ny + 7) / 8, (g.nz + kz - 1) / kz), dim3(32, 8), 0, g, (const T*)c.u,
               (const T*)c.v, (const T*)c.w, (T*)c.nut, duct_vd ? (const double*)c.t.vd4 : nullptr, c.cfg.ly, kz);
    if (model == LES_SGS_SMAG_VD && c.cfg.zbc != LES_ZBC_PERIODIC && !g.ywall) {
      LES_LAUNCH(c, "vd_coef", 0, k_vd_coef_partial<T>, dim3(VD_BLOCKS), dim3(256), 0, g, (const T*)c.u,
                 (const T*)c.v, c.t.tau, c.cfg.zbc == LES_ZBC_WALLMODEL ? 1 : 0, c.t.red);
      LES_LAUNCH(c, "vd_coef_final", 0, k_vd_coef_final, dim3(1), dim3(256), 0, g, c.t.red, c.cfg.cs, c.t.coef);
    }
    return;
  }
  if (model == LES_SGS_DSM || model == LES_SGS_MLP) {
    const bool learned = model == LES_SGS_MLP && c.mlp_params != nullptr;
    // learned closure: the network runs first; the dynamic model of the same velocity runs
    // only if that evaluation flagged a cell (gate = its fallback counter), without storing
    // |S|, and k_mlp_fallback then fills the flagged cells from its coefficients
    const int* gate = learned ? c.mlp_cnt + 1 : nullptr;
    T* dsm_nut = learned ? nullptr : (T*)c.nut;
    const int kc = c.dsm_kc;
    using TL = fused::Tile<T>;
    const dim3 grid((g.nx + fused::TX - 1) / fused::TX, (g.ny + TL::TY - 1) / TL::TY, (g.nz + kc - 1) / kc);
    // FP32 keeps its rounding but in periodic boxes with explicit viscous terms (k_dsm_fused32, 32 x 8 threads)
    const bool rows32 = sizeof(T) == 4 && (g.zbc != LES_ZBC_PERIODIC || c.cfg.implicit_z != LES_VISC_EXPLICIT);
    const dim3 block = rows32 ? dim3(fused32::TX, TL::NT / fused32::TX) : dim3(TL::NT);
    if (learned) {
      MlpNorm nm;
      for (int a = 0; a < 7; ++a) {
        nm.lo[a] = c.mlp_lo[a];
        nm.inv[a] = 1.0 / (c.mlp_hi[a] - c.mlp_lo[a]);
      }
      const int mkc = c.mlp_kc;
      const dim3 tgrid((g.nx + tiled::TX - 1) / tiled::TX, (g.ny + tiled::TY - 1) / tiled::TY, (g.nz + mkc - 1) / mkc);
      if (g.ywall) {
        // ducts: the four walls' friction velocities of the van Driest reduction
        LES_LAUNCH(c, "vd_duct", 0, k_vd_duct_partial<T>, dim3(VD_BLOCKS), dim3(256), 0, g, (const T*)c.u,
                   (const T*)c.v, (const T*)c.w, c.t.tau, c.t.tauy, c.cfg.zbc == LES_ZBC_WALLMODEL ? 1 : 0, c.t.red);
        LES_LAUNCH(c, "vd_duct_final", 0, k_vd_duct_final, dim3(1), dim3(64), 0, g, c.t.red, c.t.vd4, c.mlp_cnt);
        LES_LAUNCH(c, "mlp_nut", 4 * pts * sizeof(T), (k_mlp_nut<T, true>), tgrid, dim3(tiled::TX, tiled::TY), 0, g,
                   (const T*)c.u, (const T*)c.v, (const T*)c.w, (T*)c.nut, c.mlp_params, nm,
                   (const double*)c.t.vd4, c.cfg.ly, c.mlp_cnt, mkc);
      } else {
        LES_LAUNCH(c, "wall_mean", 0, k_wall_mean<T>, dim3(WM_BLOCKS), dim3(256), 0, g, (const T*)c.u,
                   (const T*)c.v, c.t.tau, c.cfg.zbc == LES_ZBC_WALLMODEL ? 1 : 0, c.t.red, c.t.dt, c.mlp_cnt,
                   (unsigned*)(c.mlp_cnt + 2));
        // FP64 with the wall model: the z boundary fixed at compile time (690 -> 677 us on
        // 512x256x128)
        auto km = k_mlp_nut<T, false>;
        if constexpr (sizeof(T) == 8)
          if (g.zbc == LES_ZBC_WALLMODEL) km = k_mlp_nut<T, false, LES_ZBC_WALLMODEL>;
        LES_LAUNCH(c, "mlp_nut", 4 * pts * sizeof(T), km, tgrid, dim3(tiled::TX, tiled::TY), 0, g,
                   (const T*)c.u, (const T*)c.v, (const T*)c.w, (T*)c.nut, c.mlp_params, nm,
                   (const double*)(c.t.dt + 2), c.cfg.ly, c.mlp_cnt, mkc);
      }
    }
    if (g.ywall) {
      // ducts: coefficients along x lines
      auto kfy = [&] {
        if constexpr (sizeof(T) == 4)
          return k_dsm_fused32<T, true>;
        else
          return g.zbc == LES_ZBC_WALLMODEL ? k_dsm_fused<T, true, LES_ZBC_WALLMODEL>
                                            : k_dsm_fused<T, true, LES_ZBC_NOSLIP>;
      }();
      LES_LAUNCH(c, "dsm_fused", 4 * pts * sizeof(T), kfy, grid, block, 0, g,
                 (const T*)c.u, (const T*)c.v, (const T*)c.w, dsm_nut, c.t.dsm_part, kc, gate);
      const int nl = g.nz * g.ny;
      LES_LAUNCH(c, "dsm_reduce", 0, k_dsm_reduce_lines, dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, g,
                 c.t.dsm_part, (int)grid.x, c.t.cs, gate);
      if (!learned) {
        const int64_t ns = (int64_t)(g.nz + 2) * g.nx * g.ny;
        LES_LAUNCH(c, "nut_lines", 2.0 * ns * sizeof(T), k_nut_lines<T>, dim3((unsigned)((ns + 255) / 256)), dim3(256),
                   0, g, (T*)c.nut, (const double*)c.t.cs);
      }
    } else {
      auto kf = k_dsm_fused<T, false, LES_ZBC_PERIODIC>;
      if constexpr (sizeof(T) == 4) {
        if (rows32) kf = k_dsm_fused32<T, false>;
      } else {
        if (g.zbc == LES_ZBC_NOSLIP) kf = k_dsm_fused<T, false, LES_ZBC_NOSLIP>;
        if (g.zbc == LES_ZBC_WALLMODEL) kf = k_dsm_fused<T, false, LES_ZBC_WALLMODEL>;
      }
      LES_LAUNCH(c, "dsm_fused", 4 * pts * sizeof(T), kf, grid, block, 0, g,
                 (const T*)c.u, (const T*)c.v, (const T*)c.w, dsm_nut, c.t.dsm_part, kc, gate);
      const int ntile = (int)(grid.x * grid.y) * TL::WV;
      LES_LAUNCH(c, "dsm_reduce", 0, k_dsm_reduce<T>, dim3(g.nz), dim3(256), 0, g, c.t.dsm_part, ntile, c.t.cs,
                 learned ? nullptr : c.t.coef, gate, learned ? (T*)c.nut : (T*)nullptr);
    }
    if (learned && g.ywall) {   // channels: the fallback ran with the plane coefficients
      const int64_t ni = (int64_t)g.nz * g.nx * g.ny;
      LES_LAUNCH(c, "mlp_fallback", 0, k_mlp_fallback<T>, dim3((unsigned)std::min<int64_t>(1024, (ni + 255) / 256)),
                 dim3(256), 0, g,
                 (T*)c.nut, (const double*)c.t.cs, (const int*)gate);
    }
  }
}

template <typename T>
void batch_eddy_viscosity(hipStream_t st, const BatchMap& m, const int* totals, int any_dsm, int any_smag) {
  if (any_smag) hipLaunchKernelGGL(kb_strain_mag<T>, dim3(totals[BK_POINT]), dim3(32, 8), 0, st, m);
  if (any_dsm) {
    hipLaunchKernelGGL(kb_dsm_fused<T>, dim3(totals[BK_DSM]), dim3(fused::Tile<T>::NT), 0, st, m);
    hipLaunchKernelGGL(kb_dsm_reduce<T>, dim3(totals[BK_DSMRED]), dim3(256), 0, st, m);
  }
}
template void batch_eddy_viscosity<float>(hipStream_t, const BatchMap&, const int*, int, int);
template void batch_eddy_viscosity<double>(hipStream_t, const BatchMap&, const int*, int, int);

template <typename T>
void launch_mlp_sample(Ctx& c, uint64_t seed, int64_t n, float* x, float* y) {
  const GridP& g = c.g;
  const int wm = c.cfg.zbc == LES_ZBC_WALLMODEL ? 1 : 0;
  const double* ut = c.t.dt + 2;
  if (g.ywall) {
    LES_LAUNCH(c, "vd_duct", 0, k_vd_duct_partial<T>, dim3(VD_BLOCKS), dim3(256), 0, g, (const T*)c.u, (const T*)c.v,
               (const T*)c.w, c.t.tau, c.t.tauy, wm, c.t.red);
    LES_LAUNCH(c, "vd_duct_final", 0, k_vd_duct_final, dim3(1), dim3(64), 0, g, c.t.red, c.t.vd4,
                 (int*)nullptr);
    ut = c.t.vd4;
  } else {
    LES_LAUNCH(c, "wall_mean", 0, k_wall_mean<T>, dim3(WM_BLOCKS), dim3(256), 0, g, (const T*)c.u,
               (const T*)c.v, c.t.tau, wm, c.t.red, c.t.dt, (int*)nullptr, (unsigned*)(c.mlp_cnt + 2));
  }
  LES_LAUNCH(c, "mlp_sample", 0, k_mlp_sample<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, g, (const T*)c.u,
             (const T*)c.v, (const T*)c.w, c.t.cs, ut, c.cfg.ly, seed, n, x, y);
}
template void launch_mlp_sample<double>(Ctx&, uint64_t, int64_t, float*, float*);
template void launch_mlp_sample<float>(Ctx&, uint64_t, int64_t, float*, float*);

template <typename T>
__global__ void k_read_nut(GridP g, const T* nut, const double* coef, T* dst, int64_t n) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int k = (int)(e / g.sxy);
  dst[e] = (T)coef[k] * nut[e];
}

template <typename T>
void launch_read_nut(Ctx& c, T* dst) {
  const int64_t n = (int64_t)c.field_elems;
  LES_LAUNCH(c, "read_nut", 2.0 * n * sizeof(T), k_read_nut<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c.g,
                     (const T*)c.nut, c.t.coef, dst, n);
}

template void launch_eddy_viscosity<double>(Ctx&);
template void launch_eddy_viscosity<float>(Ctx&);
template void launch_read_nut<double>(Ctx&, double*);
template void launch_read_nut<float>(Ctx&, float*);

}  // namespace les
