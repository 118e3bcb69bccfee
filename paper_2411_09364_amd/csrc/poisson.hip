// Eigenfunction-expansion Poisson solver (Sec. 2.2: Fourier transforms in the periodic
// directions and the Thomas algorithm along the non-uniform one; Eq. poi).
//
//   k_rfftx      f = D u* / (gamma dt) (or a given field) on two neighbouring x-rows,
//                packed as one complex row, Stockham FFT in LDS, split into the two
//                half spectra l = 0..nx/2; also the flow-rate partial sums of u*.
//   k_fft_lines  complex FFT along y for tiles of consecutive l, from global memory into
//                registers, through LDS once (twice) and back; or along a periodic z the
//                forward FFT, the division by the eigenvalue sum and the inverse.
//   k_thomas_scan  FP64 solve along z for every (l, m) column; the singular (0, 0) column is
//                pinned and mean-corrected.
//   k_irfftx     Hermitian reconstruction of two rows, inverse FFT, real and imaginary
//                parts back to the two rows of phi.
//
// Spectrum layout: complex [nz][ny][nxp] (l fastest, nxp >= nx/2+1), interior planes only.
// Normalisation: forward transforms unscaled; the solve multiplies by 1/(nx ny [nz]) so
// the inverse transforms are plain sums.
#include "les_internal.h"

#include <algorithm>

namespace les {

template <typename R>
struct alignas(2 * sizeof(R)) cpx {
  R x, y;
};

// Passes of an LDS Stockham FFT.  The stages (radix 5, then 3, then 4s, then a 2; a sub-transform
// of Ns points grows by the radix each stage) run two at a time: a thread takes the R1 R2 points
// that both stages of a pair connect, so that a transform of up to 320 points goes through LDS
// once, between its two passes, and one of up to 1024 points twice; the first pass of the strided
// lines loads from global memory and the last one stores there.  Every stage's arithmetic is that
// of the stage alone.  Bound by memory: with a stage per LDS pass (and the index divisions of
// each butterfly) the y transforms of 512 x 256 x 128 in FP64 took 81 and 76 us, now 52 and 48
// (271 MB moved, 5.1 and 5.6 TB/s), those of 1024 x 512 x 256 in FP32 553 and 467, now 255 (4.2
// TB/s, what a large copy reaches).
FftPlan make_plan(int n) {
  FftPlan p{};
  p.n = n;
  int rad[16], s = 0, m = n;
  if (m % 5 == 0) {
    rad[s++] = 5;
    m /= 5;
  }
  if (m % 3 == 0) {
    rad[s++] = 3;
    m /= 3;
  }
  while (m % 4 == 0) {
    rad[s++] = 4;
    m /= 4;
  }
  while (m % 2 == 0) {
    rad[s++] = 2;
    m /= 2;
  }
  // pairs from the front, but of three stages, or of two that make 16 points or fewer, the first
  // stands alone when the groups are smaller and more for it (32 = 4 x (4 2), not (4 4) x 2)
  int i = 0;
  if ((s == 3 && rad[1] * rad[2] < rad[0] * rad[1]) || (s == 2 && n <= 20)) p.pass[p.np++] = 10 * rad[i++] + 1;
  for (; i < s; i += 2) p.pass[p.np++] = 10 * rad[i] + (i + 1 < s ? rad[i + 1] : 1);
  // a last pass of one point per thread where the first already holds the whole transform
  if (p.np == 1) p.pass[p.np++] = 11;
  return p;
}

// Threads of one transform (a team): the power of two that leaves every thread 16 points at
// most, or one group of the first pass; the later passes (16 points or fewer a group) then have
// at most ceil(16 / (R1 R2)) groups a thread.
static int fft_team(int n) {
  const FftPlan p = make_plan(n);
  const int need = std::max((n + 15) / 16, n / (p.pass[0] / 10 * (p.pass[0] % 10)));
  int t = 1;
  while (t < need) t *= 2;
  return t;
}

// Sums of two products are written with their fused multiply-adds, one product rounded and
// the other not: which one the compiler would fuse changes with the code around them, and with
// it the last bits of every transform.
__device__ inline float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// a (c + i s)
template <typename R>
__device__ inline cpx<R> turn(cpx<R> a, R c, R s) {
  return {fmadd(a.x, c, -(a.y * s)), fmadd(a.y, c, a.x * s)};
}

// DIR = -1 forward (exp(-2 pi i q/N)), +1 inverse.  tw holds (cos, sin)(2 pi q/N), q = 0..N-1.
template <typename R, int DIR>
__device__ inline cpx<R> twiddle(cpx<R> a, const R* __restrict__ tw, int qq) {
  return turn(a, tw[2 * qq], (R)DIR * tw[2 * qq + 1]);
}

// butterfly of radix RAD on v[0], v[S], .., in place
template <typename R, int DIR, int RAD, int S>
__device__ __forceinline__ void butterfly(cpx<R>* v) {
  if constexpr (RAD == 2) {
    const cpx<R> v0 = v[0], v1 = v[S];
    v[0] = {v0.x + v1.x, v0.y + v1.y};
    v[S] = {v0.x - v1.x, v0.y - v1.y};
  } else if constexpr (RAD == 4) {
    const cpx<R> v0 = v[0], v1 = v[S], v2 = v[2 * S], v3 = v[3 * S];
    const cpx<R> s02 = {v0.x + v2.x, v0.y + v2.y}, d02 = {v0.x - v2.x, v0.y - v2.y};
    const cpx<R> s13 = {v1.x + v3.x, v1.y + v3.y}, d13 = {v1.x - v3.x, v1.y - v3.y};
    const cpx<R> jd = {-(R)DIR * d13.y, (R)DIR * d13.x};   // DIR * i * d13
    v[0] = {s02.x + s13.x, s02.y + s13.y};
    v[S] = {d02.x + jd.x, d02.y + jd.y};
    v[2 * S] = {s02.x - s13.x, s02.y - s13.y};
    v[3 * S] = {d02.x - jd.x, d02.y - jd.y};
  } else if constexpr (RAD == 3) {
    const R h3 = (R)0.86602540378443864676;
    const cpx<R> v0 = v[0], v1 = v[S], v2 = v[2 * S];
    const cpx<R> s12 = {v1.x + v2.x, v1.y + v2.y}, d12 = {v1.x - v2.x, v1.y - v2.y};
    const cpx<R> m = {v0.x - (R)0.5 * s12.x, v0.y - (R)0.5 * s12.y};
    const R h = (R)DIR * h3;   // m + DIR i h3 d12, m - DIR i h3 d12
    v[0] = {v0.x + s12.x, v0.y + s12.y};
    v[S] = {fmadd(-h, d12.y, m.x), fmadd(h, d12.x, m.y)};
    v[2 * S] = {fmadd(h, d12.y, m.x), fmadd(-h, d12.x, m.y)};
  } else if constexpr (RAD == 5) {
    // with t1 = v1 + v4, t2 = v2 + v3, t3 = v1 - v4, t4 = v2 - v3 (c_q, s_q the cosine and
    // sine of 2 pi q / 5): X1,4 = v0 + c1 t1 + c2 t2 +- DIR i (s1 t3 + s2 t4),
    // X2,3 = v0 + c2 t1 + c1 t2 +- DIR i (s2 t3 - s1 t4), X0 = v0 + t1 + t2
    const R c1 = (R)0.30901699437494742410, c2 = (R)-0.80901699437494742410;
    const R s1 = (R)0.95105651629515357212, s2 = (R)0.58778525229247312917;
    const cpx<R> v0 = v[0], v1 = v[S], v2 = v[2 * S], v3 = v[3 * S], v4 = v[4 * S];
    const cpx<R> t1 = {v1.x + v4.x, v1.y + v4.y}, t2 = {v2.x + v3.x, v2.y + v3.y};
    const cpx<R> t3 = {v1.x - v4.x, v1.y - v4.y}, t4 = {v2.x - v3.x, v2.y - v3.y};
    const cpx<R> a1 = {fmadd(c2, t2.x, fmadd(c1, t1.x, v0.x)), fmadd(c2, t2.y, fmadd(c1, t1.y, v0.y))};
    const cpx<R> a2 = {fmadd(c1, t2.x, fmadd(c2, t1.x, v0.x)), fmadd(c1, t2.y, fmadd(c2, t1.y, v0.y))};
    const cpx<R> b1 = {fmadd(s2, t4.x, s1 * t3.x), fmadd(s2, t4.y, s1 * t3.y)};
    const cpx<R> b2 = {fmadd(s2, t3.x, -(s1 * t4.x)), fmadd(s2, t3.y, -(s1 * t4.y))};
    const cpx<R> j1 = {-(R)DIR * b1.y, (R)DIR * b1.x}, j2 = {-(R)DIR * b2.y, (R)DIR * b2.x};   // DIR i b
    v[0] = {v0.x + t1.x + t2.x, v0.y + t1.y + t2.y};
    v[S] = {a1.x + j1.x, a1.y + j1.y};
    v[4 * S] = {a1.x - j1.x, a1.y - j1.y};
    v[2 * S] = {a2.x + j2.x, a2.y + j2.y};
    v[3 * S] = {a2.x - j2.x, a2.y - j2.y};
  }
}

// Both stages of a pair on the points v[e] = x[b + e N / (R1 R2)] of group b = j Ns + k, k < Ns:
// the stage of radix R1 (sub-transforms of Ns points) joins v[q2], v[q2 + R2], .., the stage of
// radix R2 (of Ns R1) joins v[q R2], v[q R2 + 1], ..  Output q + p R1 of the pair, at v[p + q R2],
// belongs at j Ns R1 R2 + k + (q + p R1) Ns.  ts = N / (Ns R1 R2).  FIRST: Ns = 1, k = 0, where the
// first stage's twiddle factors are 1.
template <typename R, int DIR, int R1, int R2, bool FIRST>
__device__ __forceinline__ void stage_pair(cpx<R>* v, int k, int Ns, int ts, const R* __restrict__ tw) {
  if constexpr (!FIRST) {
    const int i1 = k * ts * R2;
#pragma unroll
    for (int q = 1; q < R1; ++q)
#pragma unroll
      for (int q2 = 0; q2 < R2; ++q2) v[q2 + q * R2] = twiddle<R, DIR>(v[q2 + q * R2], tw, q * i1);
  }
#pragma unroll
  for (int q2 = 0; q2 < R2; ++q2) butterfly<R, DIR, R1, R2>(v + q2);
  if constexpr (R2 > 1) {
#pragma unroll
    for (int q = 0; q < R1; ++q) {
      const int i2 = FIRST ? q * ts : k * ts + q * (Ns * ts);
      if (!FIRST || q > 0) {
#pragma unroll
        for (int q2 = 1; q2 < R2; ++q2) v[q2 + q * R2] = twiddle<R, DIR>(v[q2 + q * R2], tw, q2 * i2);
      }
      butterfly<R, DIR, R2, 1>(v + q * R2);
    }
  }
}

// First pass: in(i) is input point i, out(o, z) takes point o of the pass's result.  SYNC: the
// input lies where the output goes; at most one group per thread then (fft_team), read before
// the barrier and written after it.
template <typename R, int DIR, int R1, int R2, bool SYNC, typename In, typename Out>
__device__ __forceinline__ void pass_first(int N, const R* __restrict__ tw, int lane, int team, In in, Out out) {
  constexpr int RR = R1 * R2;
  const int M = N / RR;
  auto group = [&](int b) {
    cpx<R> v[RR];
    if (b < M) {
#pragma unroll
      for (int e = 0; e < RR; ++e) v[e] = in(b + e * M);
    }
    if (SYNC) __syncthreads();
    if (b < M) {
      stage_pair<R, DIR, R1, R2, true>(v, 0, 1, M, tw);
#pragma unroll
      for (int q = 0; q < R1; ++q)
#pragma unroll
        for (int p = 0; p < R2; ++p) out(b * RR + q + p * R1, v[p + q * R2]);
    }
  };
  if constexpr (SYNC) group(lane);
  else
    for (int b = lane; b < M; b += team) group(b);
}

// Later pass (MID: of radix 4 x 4, before the last), its input in LDS; SYNC as above, with
// all groups of a thread held in registers over the barrier.
template <typename R, int DIR, int R1, int R2, bool MID, bool SYNC, typename In, typename Out>
__device__ __forceinline__ void pass_next(int N, int Ns, const R* __restrict__ tw, int lane, int team, In in, Out out) {
  constexpr int RR = R1 * R2, BPT = SYNC ? (15 + RR) / RR : 1;
  const int M = N / RR;
  cpx<R> v[BPT][RR];
  auto read = [&](cpx<R>* x, int b) {
#pragma unroll
    for (int e = 0; e < RR; ++e) x[e] = in(b + e * M);
  };
  auto finish = [&](cpx<R>* x, int b) {
    const int j = MID ? b / Ns : 0, k = MID ? b - j * Ns : b, o = MID ? j * Ns * RR + k : b;
    const int st = MID ? Ns : M;
    stage_pair<R, DIR, R1, R2, false>(x, k, st, MID ? M / Ns : 1, tw);
#pragma unroll
    for (int q = 0; q < R1; ++q)
#pragma unroll
      for (int p = 0; p < R2; ++p) out(o + (q + p * R1) * st, x[p + q * R2]);
  };
  if constexpr (SYNC) {
#pragma unroll
    for (int t = 0; t < BPT; ++t)
      if (lane + t * team < M) read(v[t], lane + t * team);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < BPT; ++t)
      if (lane + t * team < M) finish(v[t], lane + t * team);
  } else {
    for (int b = lane; b < M; b += team) {
      read(v[0], b);
      finish(v[0], b);
    }
  }
}

// A whole transform of the team's N points: in(i) and out(o, z) as above, ld(i) and st(i, z) its
// N points of LDS.  SYNC_IN: `in` reads those points themselves; SYNC_OUT: `out` writes them.
// Every thread of the block comes through here (barriers); no barrier follows the last write.
template <typename R, int DIR, bool SYNC_IN, bool SYNC_OUT, typename In, typename Out, typename Ld, typename St>
__device__ __forceinline__ void transform(const FftPlan& P, const R* __restrict__ tw, int lane, int team, In in,
                                          Out out, Ld ld, St st) {
  const int N = P.n;
  int Ns = P.pass[0] / 10 * (P.pass[0] % 10);
  switch (P.pass[0]) {
    case 44: pass_first<R, DIR, 4, 4, SYNC_IN>(N, tw, lane, team, in, st); break;
    case 53: pass_first<R, DIR, 5, 3, SYNC_IN>(N, tw, lane, team, in, st); break;
    case 54: pass_first<R, DIR, 5, 4, SYNC_IN>(N, tw, lane, team, in, st); break;
    case 34: pass_first<R, DIR, 3, 4, SYNC_IN>(N, tw, lane, team, in, st); break;
    case 51: pass_first<R, DIR, 5, 1, SYNC_IN>(N, tw, lane, team, in, st); break;
    case 31: pass_first<R, DIR, 3, 1, SYNC_IN>(N, tw, lane, team, in, st); break;
    default: pass_first<R, DIR, 4, 1, SYNC_IN>(N, tw, lane, team, in, st); break;   // 41
  }
  __syncthreads();
  for (int s = 1; s + 1 < P.np; ++s) {
    pass_next<R, DIR, 4, 4, true, true>(N, Ns, tw, lane, team, ld, st);
    __syncthreads();
    Ns *= 16;
  }
  switch (P.pass[P.np - 1]) {
    case 44: pass_next<R, DIR, 4, 4, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    case 42: pass_next<R, DIR, 4, 2, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    case 34: pass_next<R, DIR, 3, 4, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    case 41: pass_next<R, DIR, 4, 1, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    case 32: pass_next<R, DIR, 3, 2, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    case 31: pass_next<R, DIR, 3, 1, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    case 21: pass_next<R, DIR, 2, 1, false, SYNC_OUT>(N, Ns, tw, lane, team, ld, out); break;
    default:   // 11: the points as they are
      for (int i = lane; i < N; i += team) out(i, ld(i));
  }
}

// two neighbouring values, the first of any alignment
template <typename T>
struct pair2 {
  T x, y;
};
template <typename T>
__device__ inline pair2<T> load2(const T* p) {
  typedef T vec __attribute__((ext_vector_type(2), aligned(alignof(T))));
  const vec v = *reinterpret_cast<const vec*>(p);
  return {v.x, v.y};
}

// LDS position of point i of a transform: one point of padding after every 16, so that the
// strided writes of the first pass spread over the banks
__host__ __device__ inline int fft_pos(int i) { return i + (i >> 4); }

template <typename T>
__device__ inline const T* twsel(const double* d, const float* f);
template <>
__device__ inline const double* twsel<double>(const double* d, const float*) { return d; }
template <>
__device__ inline const float* twsel<float>(const double*, const float* f) { return f; }

// ============================================================================ forward x
// MODE 0: f = D u* scaled; MODE 1: f given (les_poisson).  The rows go through LDS before the
// first pass: the divergence reads eleven values a point, too many to hold for the 16 or 20
// points of a group (that spilled).  Bound by those loads: the divergence of 1024 x 512 x 256 in
// FP32 641 us with a load an instruction, 476 with two points a load (2.1 GB, 4.5 TB/s); 512 x
// 256 x 128 in FP64 144 -> 141.  npair_blk teams of blockDim /
// npair_blk threads (a power of two), one row pair each.
template <typename T, int MODE>
__device__ __forceinline__ void rfftx_body(dim3 bid, GridP g, const FftPlan& P, const T* __restrict__ us, const T* __restrict__ vs,
                                               const T* __restrict__ ws, const T* __restrict__ fin,
                                               cpx<T>* __restrict__ spec, const double* __restrict__ twd,
                                               const float* __restrict__ twf, const double* __restrict__ dtp,
                                               double gamma, int npair_blk, double* __restrict__ bulk_part) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nx = g.nx, nxh = nx / 2 + 1, nyh = g.ny / 2;
  const int npairs = g.nz * nyh;   // pair indices fit 32 bits
  // gamma = 0: the plain divergence (initial projection), no time factor
  const T scale = (MODE == 0 && gamma > 0.0) ? (T)(1.0 / (gamma * dtp[0])) : (T)1;
  const int team = blockDim.x / npair_blk, tsh = __builtin_ctz(team);
  const int p = threadIdx.x >> tsh, lane = threadIdx.x & (team - 1);
  cpx<T>* A = reinterpret_cast<cpx<T>*>(smem_raw) + p * fft_pos(nx);
  const int gp = (int)bid.x * npair_blk + p;
  const bool ok = gp < npairs;
  // teams past the last pair repeat pair 0 and store nothing
  const int kk = ok ? gp / nyh : 0, j0 = ok ? 2 * (gp - kk * nyh) : 0, k = kk + 1;
  const int64_t c0 = idx3(g, k, j0, 0);
  double bsum = 0.0;
  auto ld = [&](int i) { return A[fft_pos(i)]; };
  auto st = [&](int i, cpx<T> z) { A[fft_pos(i)] = z; };
  if (MODE == 0) {
    const T *u0 = us + c0, *v0 = vs + c0, *w0 = ws + c0;
    const bool ylow = g.ywall && j0 == 0;   // no face below the first row of a duct
    const T* vm = ylow ? v0 : vs + idx3(g, k, wrap_m(j0, g.ny), 0);
    const T* wm = (k == 1 && g.zbc == LES_ZBC_PERIODIC) ? ws + idx3(g, g.nz, j0, 0) : w0 - g.sxy;
    const T rdx = (T)g.rdx, rdy = (T)g.rdy, rdz = (T)g.rdzf[k];
    const double dz = g.dzf[k];
    // two points at a time (nx is even): nine 2-wide loads and two single ones
#pragma unroll 2
    for (int i = 2 * lane; i < nx; i += 2 * team) {
      const int im = wrap_m(i, nx);
      const pair2<T> ua = load2(u0 + i), ub = load2(u0 + nx + i), va = load2(v0 + i), vb = load2(v0 + nx + i);
      const pair2<T> wa = load2(w0 + i), wb = load2(w0 + nx + i), wc = load2(wm + i), wd = load2(wm + nx + i);
      const T uc = u0[im], ud = u0[nx + im];
      pair2<T> vc = load2(vm + i);
      if (ylow) vc = {(T)0, (T)0};
      auto div = [&](T du, T dv, T dw) { return fmadd(dw, rdz, fmadd(du, rdx, dv * rdy)) * scale; };
      A[fft_pos(i)] = {div(ua.x - uc, va.x - vc.x, wa.x - wc.x), div(ub.x - ud, vb.x - va.x, wb.x - wd.x)};
      A[fft_pos(i + 1)] = {div(ua.y - ua.x, va.y - vc.y, wa.y - wc.y), div(ub.y - ub.x, vb.y - va.y, wb.y - wd.y)};
      if (bulk_part) {
        bsum += (double)ua.x * dz;
        bsum += (double)ub.x * dz;
        bsum += (double)ua.y * dz;
        bsum += (double)ub.y * dz;
      }
    }
  } else {
    const T* f0 = fin + c0;
#pragma unroll 4
    for (int i = lane; i < nx; i += team) A[fft_pos(i)] = {f0[i], f0[nx + i]};
  }
  __syncthreads();
  transform<T, -1, true, true>(P, twsel<T>(twd, twf), lane, team, ld, st, ld, st);
  if (MODE == 0 && bulk_part) {
    __shared__ double red[256];
    red[threadIdx.x] = ok ? bsum : 0.0;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
      if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) bulk_part[bid.x] = red[0];
  }
  __syncthreads();
  if (!ok) return;
  cpx<T>* s0 = spec + ((int64_t)kk * g.ny + j0) * g.nxp;
  cpx<T>* s1 = s0 + g.nxp;
  for (int l = lane; l < nxh; l += team) {
    const cpx<T> a = A[fft_pos(l)];
    const cpx<T> b = A[fft_pos(l == 0 ? 0 : nx - l)];
    // A_l = (Z_l + conj Z_{N-l})/2, B_l = (Z_l - conj Z_{N-l})/(2i)
    s0[l] = {(T)0.5 * (a.x + b.x), (T)0.5 * (a.y - b.y)};
    s1[l] = {(T)0.5 * (a.y + b.y), (T)0.5 * (b.x - a.x)};
  }
}

template <typename T, int MODE>
__global__ void __launch_bounds__(256) k_rfftx(GridP g, FftPlan P, const T* us, const T* vs, const T* ws, const T* fin,
                                               cpx<T>* spec, const double* twd, const float* twf, const double* dtp,
                                               double gamma, int npair_blk, double* bulk_part) {
  rfftx_body<T, MODE>(blockIdx, g, P, us, vs, ws, fin, spec, twd, twf, dtp, gamma, npair_blk, bulk_part);
}

template <typename T>
__global__ void __launch_bounds__(256) kb_rfftx(BatchMap m, double gamma) {
  int box;
  const dim3 bid = batch_bid(m, BK_RFFTX, blockIdx.x, box);
  const BoxDesc& d = m.desc[box];
  rfftx_body<T, 0>(bid, d.g, d.px, (const T*)d.us, (const T*)d.vs, (const T*)d.wsf, nullptr, (cpx<T>*)d.spec, d.twx,
                   d.twx_f, d.dt, gamma, d.pbx, nullptr);
}

// ============================================================================ inverse x
template <typename T>
__device__ __forceinline__ void irfftx_body(dim3 bid, GridP g, const FftPlan& P, const cpx<T>* __restrict__ spec,
                                                T* __restrict__ out, const double* __restrict__ twd,
                                                const float* __restrict__ twf, int npair_blk) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nx = g.nx, nxh = nx / 2 + 1, nyh = g.ny / 2;
  const int npairs = g.nz * nyh;   // pair indices fit 32 bits
  const int team = blockDim.x / npair_blk, tsh = __builtin_ctz(team);
  const int p = threadIdx.x >> tsh, lane = threadIdx.x & (team - 1);
  cpx<T>* A = reinterpret_cast<cpx<T>*>(smem_raw) + p * fft_pos(nx);
  const int gp = (int)bid.x * npair_blk + p;
  const bool ok = gp < npairs;
  // teams past the last pair repeat pair 0 and store nothing
  const int kk = ok ? gp / nyh : 0, j0 = ok ? 2 * (gp - kk * nyh) : 0;
  const cpx<T>* s0 = spec + ((int64_t)kk * g.ny + j0) * g.nxp;
  const cpx<T>* s1 = s0 + g.nxp;
  T* o0 = out + idx3(g, kk + 1, j0, 0);
  T* o1 = o0 + nx;
  // Hermitian reconstruction of two rows' spectra
  auto in = [&](int l) -> cpx<T> {
    const int ls = l < nxh ? l : nx - l;
    const cpx<T> a = s0[ls], b = s1[ls];
    return l < nxh ? cpx<T>{a.x - b.y, a.y + b.x} : cpx<T>{a.x + b.y, -a.y + b.x};
  };
  auto put = [&](int i, cpx<T> z) {
    if (ok) {
      o0[i] = z.x;
      o1[i] = z.y;
    }
  };
  auto ld = [&](int i) { return A[fft_pos(i)]; };
  auto st = [&](int i, cpx<T> z) { A[fft_pos(i)] = z; };
  transform<T, 1, false, false>(P, twsel<T>(twd, twf), lane, team, in, put, ld, st);
}

template <typename T>
__global__ void __launch_bounds__(256) k_irfftx(GridP g, FftPlan P, const cpx<T>* spec, T* out, const double* twd,
                                                const float* twf, int npair_blk) {
  irfftx_body<T>(blockIdx, g, P, spec, out, twd, twf, npair_blk);
}

template <typename T>
__global__ void __launch_bounds__(256) kb_irfftx(BatchMap m) {
  int box;
  const dim3 bid = batch_bid(m, BK_RFFTX, blockIdx.x, box);
  const BoxDesc& d = m.desc[box];
  irfftx_body<T>(bid, d.g, d.px, (const cpx<T>*)d.spec, (T*)d.phi, d.twx, d.twx_f, d.pbx);
}

// ============================================================================ strided lines
// Complex FFT of length P.n along a strided dimension for L consecutive l values:
// element t of line (l, o) is at base + o*ostride + t*lstride + l.  grid.x covers l tiles,
// grid.y covers o.  SOLVE (periodic z only): forward FFT, multiply by the normalisation
// over the eigenvalue lam = lamx + lamy + lamz of the operator, inverse FFT.  The operator
// is the Laplacian when hg = 0 (Poisson; the zero mode is set to 0), else the Helmholtz
// operator 1 - hg dt lam of Crank-Nicolson in all directions (hg = gamma nu / 2, dt from
// the device slot).
//
// DCT = 1 (ducts, walls in y): the lines are transformed by the cosine expansion of the
// zero-flux second difference instead, X_m = sum_t x_t cos(pi m (t + 1/2) / N) (DIR = -1)
// and its unnormalised inverse y_t = X_0 + 2 sum_{m >= 1} X_m cos(pi m (t + 1/2) / N) (DIR =
// +1, so that a forward-inverse pair multiplies by N, like the FFT pair), each through one
// complex FFT of length N of the same line (the lines are complex, and the transforms are
// linear, so real and imaginary parts go through together): forward, the line is loaded
// in the order x_0, x_2, .., x_{N-2}, x_{N-1}, .., x_3, x_1 and X_m = (W_m V_m + conj(W_m)
// V_{N-m}) / 2 with W_m = exp(-i pi m / (2N)) and V its FFT; inverse, V_m = conj(W_m) (X_m -
// i X_{N-m}) (X_N = 0) before the inverse FFT, whose output is stored back in the permuted
// order.  twc holds (cos, sin)(pi m / (2N)).
template <typename T, int DIR, bool SOLVE, int DCT = 0>
__device__ __forceinline__ void fft_lines_body(dim3 bid, const FftPlan& P, cpx<T>* __restrict__ data, int nl, int64_t lstride,
                                                   int64_t ostride, int L, const double* __restrict__ twd,
                                                   const float* __restrict__ twf, const double* __restrict__ lamx,
                                                   const double* __restrict__ lamy, const double* __restrict__ lamz,
                                                   double norm, const double* __restrict__ dtp = nullptr,
                                                   double hg = 0.0, const double* __restrict__ twcd = nullptr,
                                                   const float* __restrict__ twcf = nullptr) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // neighbouring threads take neighbouring lines, in global memory and in LDS
  const int N = P.n, lsh = __builtin_ctz(L), team = blockDim.x >> lsh;
  const int ll = threadIdx.x & (L - 1), lane = threadIdx.x >> lsh;
  cpx<T>* A = reinterpret_cast<cpx<T>*>(smem_raw) + ll;
  const int l = (int)bid.x * L + ll;
  const bool ok = l < nl;
  // lines past the last repeat line 0 and store nothing
  cpx<T>* base = data + (int64_t)bid.y * ostride + (ok ? l : 0);
  const T* tw = twsel<T>(twd, twf);
  const T* twc = DCT ? twsel<T>(twcd, twcf) : nullptr;
  auto ld = [&](int i) { return A[fft_pos(i) << lsh]; };
  auto st = [&](int i, cpx<T> z) { A[fft_pos(i) << lsh] = z; };
  auto get = [&](int t) { return base[(int64_t)t * lstride]; };
  auto put = [&](int t, cpx<T> z) {
    if (ok) base[(int64_t)t * lstride] = z;
  };
  if constexpr (SOLVE) {
    // the transforms are along z here, bid.y indexes the y modes
    const double hc = hg != 0.0 ? hg * dtp[0] : 0.0;
    const double lxy = (ok ? lamx[l] : 0.0) + lamy[bid.y];
    auto scaled = [&](int t, cpx<T> z) {
      const double lam = lxy + lamz[t];
      const double f = hg != 0.0 ? norm / (1.0 - hc * lam) : ((lam != 0.0) ? norm / lam : 0.0);
      st(t, cpx<T>{(T)((double)z.x * f), (T)((double)z.y * f)});
    };
    transform<T, DIR, false, true>(P, tw, lane, team, get, scaled, ld, st);
    __syncthreads();
    transform<T, 1, true, false>(P, tw, lane, team, ld, put, ld, st);
  } else if constexpr (DCT && DIR < 0) {
    // forward cosine transform: even points first, then odd points in reverse
    auto perm = [&](int i) { return get(2 * i < N ? 2 * i : 2 * (N - 1 - i) + 1); };
    transform<T, DIR, false, true>(P, tw, lane, team, perm, st, ld, st);
    __syncthreads();
    for (int t = lane; t < N; t += team) {
      // X_t = (W_t V_t + conj(W_t) V_{N-t}) / 2
      const cpx<T> a = ld(t), b = ld(t == 0 ? 0 : N - t);
      const T c = twc[2 * t], sn = twc[2 * t + 1];
      const cpx<T> wa = turn(a, c, -sn), wb = turn(b, c, sn);
      put(t, cpx<T>{(T)0.5 * (wa.x + wb.x), (T)0.5 * (wa.y + wb.y)});
    }
  } else if constexpr (DCT) {
    // inverse cosine transform: V_m = conj(W_m) (X_m - i X_{N-m})
#pragma unroll 8
    for (int t = lane; t < N; t += team) st(t, get(t));
    __syncthreads();
    auto pre = [&](int m) -> cpx<T> {
      const cpx<T> a = ld(m);
      const cpx<T> b = m == 0 ? cpx<T>{(T)0, (T)0} : ld(N - m);
      return turn(cpx<T>{a.x + b.y, a.y - b.x}, twc[2 * m], twc[2 * m + 1]);
    };
    auto perm = [&](int i, cpx<T> z) { put(2 * i < N ? 2 * i : 2 * (N - 1 - i) + 1, z); };
    transform<T, DIR, true, false>(P, tw, lane, team, pre, perm, ld, st);
  } else {
    transform<T, DIR, false, false>(P, tw, lane, team, get, put, ld, st);
  }
}

template <typename T, int DIR, bool SOLVE, int DCT = 0>
__global__ void __launch_bounds__(256) k_fft_lines(FftPlan P, cpx<T>* data, int nl, int64_t lstride, int64_t ostride,
                                                   int L, const double* twd, const float* twf, const double* lamx,
                                                   const double* lamy, const double* lamz, double norm,
                                                   const double* dtp, double hg, const double* twcd,
                                                   const float* twcf) {
  fft_lines_body<T, DIR, SOLVE, DCT>(blockIdx, P, data, nl, lstride, ostride, L, twd, twf, lamx, lamy, lamz, norm,
                                     dtp, hg, twcd, twcf);
}

// Batched y transforms (SOLVE = false) or periodic-z spectral solve (SOLVE = true).
template <typename T, int DIR, bool SOLVE>
__global__ void __launch_bounds__(256) kb_fft_lines(BatchMap m) {
  int box;
  const dim3 bid = batch_bid(m, SOLVE ? BK_FFTZ : BK_FFTY, blockIdx.x, box);
  const BoxDesc& d = m.desc[box];
  const int nxh = d.g.nx / 2 + 1;
  if (SOLVE)
    fft_lines_body<T, DIR, true>(bid, d.pz, (cpx<T>*)d.spec, nxh, (int64_t)d.g.nxp * d.g.ny, (int64_t)d.g.nxp, d.lz, d.twz,
                                 d.twz_f, d.lamx, d.lamy, d.lamz, 1.0 / ((double)d.g.nx * d.g.ny * d.g.nz));
  else
    fft_lines_body<T, DIR, false>(bid, d.py, (cpx<T>*)d.spec, nxh, (int64_t)d.g.nxp, (int64_t)d.g.nxp * d.g.ny, d.ly,
                                  d.twy, d.twy_f, d.lamx, d.lamy, d.lamz, 1.0);
}

// Factorisation of the z systems of every (l, m) column (Sec. 2.2: one tridiagonal system
// per wavenumber pair), once per grid: the Poisson matrix depends on the geometry only, so
// 1/p_k, p_k = b_k + lambda_x(l) + lambda_y(m) - a_k c'_{k-1}, c'_k = c_k / p_k, are kept in the
// workspace ([k][m][l], FP64) for m <= ny/2; mode ny - m has the same eigenvalue and reads those
// of m.  The solves form c'_k = c_k (1/p_k) again, with the rounding it has here: they are bound
// by memory, and a stored c' would be as many bytes again.
__global__ void __launch_bounds__(256) k_thomas_factor(GridP g, const double* __restrict__ pa,
                                                       const double* __restrict__ pb, const double* __restrict__ pc,
                                                       const double* __restrict__ lamx,
                                                       const double* __restrict__ lamy, double* __restrict__ pfac) {
  const int nxh = g.nx / 2 + 1;
  const int64_t ncol = (int64_t)g.nxp * factor_modes(g);   // l >= nx/2+1 are padding
  const int64_t col = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (col >= ncol) return;
  const int l = (int)(col % g.nxp), m = (int)(col / g.nxp);
  if (l >= nxh) return;
  const double lam = lamx[l] + lamy[m];
  // the singular (0, 0) column pins its last unknown: rows 0..nz-2 factorised, the last row
  // stored as 0 so that the solve returns x = 0 there
  const int nr = col == 0 ? g.nz - 1 : g.nz;
  double cprev = 0.0;
  for (int k = 0; k < nr; ++k) {
    const double a = pa[k];
    const double rr = 1.0 / ((pb[k] + lam) - a * cprev);
    const double cc = pc[k] * rr;
    pfac[(int64_t)k * ncol + col] = rr;
    cprev = cc;
  }
  if (nr < g.nz) pfac[(int64_t)nr * ncol + col] = 0.0;
}

void launch_thomas_factor(Ctx& c) {
  const int64_t ncol = (int64_t)c.g.nxp * factor_modes(c.g);
  hipLaunchKernelGGL(k_thomas_factor, dim3((unsigned)((ncol + 255) / 256)), dim3(256), 0, c.stream, c.g, c.t.pa,
                     c.t.pb, c.t.pc, c.t.lamx, c.t.lamy, c.t.pfac);
}

// Launch shape of the solves of n rows: segments of S rows (8 up to s8 rows, else 16; the segments
// are part of the rounding, and FP32 fields keep those they have), P segments per block, CG columns
// per segment: 64, a wave per segment with scalar loads of its rows' coefficients, up to 12
// segments (256 x 128 x 96 in FP64 17.7 us, 20.8 with 32 columns), beyond that 32, whose blocks of
// half the size overlap better (512 x 256 x 128 in FP64 62 us, 72 with 64 columns; 1024 x 512 x
// 256 in FP32 368 and 375).
struct ThomasShape {
  int S, CG, P;
};
inline ThomasShape thomas_shape(int n, int s8) {
  const int S = n <= s8 ? 8 : 16, P = (n + S - 1) / S;
  return {S, P <= 12 ? 64 : 32, P};
}

// FP64 z solves of every (l, m) column with the stored factors, by segmented scans
// (seg_scan_solve): there are only some ten thousand columns of nz rows, and a plain Thomas sweep
// per column leaves most of the chip idle behind its dependent chain.  Threads: CG consecutive
// columns (adjacent in memory, so each row load of a segment group is contiguous) times the
// segments of S rows, real and imaginary parts together (they share the products of the
// coefficients).  Rows are held in registers, loaded once and stored once.  Bound by memory: with
// one thread per part, pairs (c', 1/pivot) and loads under a condition, each waited for in turn,
// 512 x 256 x 128 in FP64 took 85 us, now 62 (305 MB, 4.9 TB/s); 1024 x 512 x 256 in FP32 676,
// now 368 (1.35 GB, 3.7 TB/s).  ZERO (Poisson): the pinned (0, 0) column has its own factors (last row zero);
// its dzf-weighted mean is removed here and its imaginary part set to zero.  Rows nrow..nz-1 are
// left as they are (the wall face of w in the Helmholtz solves).
template <typename T, int S, int CG, bool ZERO>
__device__ __forceinline__ void thomas_scan_body(unsigned bx, GridP g, cpx<T>* __restrict__ spec,
                                                 const double* __restrict__ pa, const double* __restrict__ pc,
                                                 const double* __restrict__ pfac, double norm, int nrow) {
  __shared__ double2 E[1024 / CG][CG];
  __shared__ double G[1024 / CG][CG];
  // with CG a multiple of the wave size a wave holds one segment, whose a_k and c_k are then
  // wave-uniform (scalar loads)
  const int cl = (int)threadIdx.x % CG, P = (int)blockDim.x / CG;
  const int p = CG % 64 == 0 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / CG) : (int)threadIdx.x / CG;
  const int n = nrow, nxh = g.nx / 2 + 1;
  const int64_t ncol = (int64_t)g.nxp * g.ny;
  const int64_t col = (int64_t)bx * CG + cl;
  const int l = (int)(col % g.nxp), m = (int)(col / g.nxp);
  const bool ok = col < ncol && l < nxh;
  // periodic y: mode ny - m uses the factors of m; ducts: every m has its own
  const int mm = (g.ywall || m <= g.ny / 2) ? m : g.ny - m;
  const int64_t nfac = (int64_t)g.nxp * factor_modes(g);
  const double* fp = pfac + (ok ? (int64_t)mm * g.nxp + l : 0);
  cpx<T>* x = spec + (ok ? col : 0);
  const int k0 = p * S;
  // every load without a condition (rows past the last read it again, columns past the last read
  // column 0), so that all are in flight together; what they read there is replaced by zeros
  double2 v[S];
  double r[S];
  cpx<T> z[S];
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const int k = k0 + j < n ? k0 + j : n - 1;
    z[j] = x[(int64_t)k * ncol];
    r[j] = fp[(int64_t)k * nfac];
  }
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const bool in = ok && k0 + j < n;
    v[j] = in ? make_double2((double)z[j].x * norm, (double)z[j].y * norm) : make_double2(0.0, 0.0);
    if (!in) r[j] = 0.0;
  }
  // a_k, c_k: scalar loads when a wave holds one segment; else (two segments per wave) from a
  // copy in LDS, read where used rather than held in registers (the 16-row variant spilled)
  __shared__ double sa[CG % 64 == 0 ? 1 : 512], sc[CG % 64 == 0 ? 1 : 512];
  if constexpr (CG % 64 != 0) {
    for (int k = (int)threadIdx.x; k < n; k += (int)blockDim.x) {
      sa[k] = pa[k];
      sc[k] = pc[k];
    }
    __syncthreads();
  }
  auto AF = [&](int j) -> double {
    if constexpr (CG % 64 == 0) return pa[k0 + j];
    else return sa[k0 + j];
  };
  // c'_k = c_k / p_k
  auto CF = [&](int j) -> double {
    if constexpr (CG % 64 == 0) return pc[k0 + j] * r[j];
    else return sc[k0 + j] * r[j];
  };
  seg_scan_solve<S, CG>(v, k0, n, p, P, cl, E, G, [&](int j) { return r[j]; }, AF, CF);
  if (ZERO && bx == 0) {
    // zero mode: column 0 of this block
    double sw = 0.0, sd = 0.0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int k = k0 + j;
      if (k < n) {
        sw += v[j].x * g.dzf[k + 1];
        sd += g.dzf[k + 1];
      }
    }
    __syncthreads();
    if (cl == 0) E[p][0] = make_double2(sw, sd);
    __syncthreads();
    if (cl == 0) {
      double tw = 0.0, td = 0.0;
      for (int q = 0; q < P; ++q) {
        tw += E[q][0].x;
        td += E[q][0].y;
      }
      const double mean = tw / td;
#pragma unroll
      for (int j = 0; j < S; ++j) v[j] = make_double2(v[j].x - mean, 0.0);
    }
  }
  if (ok) {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int k = k0 + j;
      if (k < n) x[(int64_t)k * ncol] = {(T)v[j].x, (T)v[j].y};
    }
  }
}

template <typename T, int S, int CG, bool ZERO>
__global__ void __launch_bounds__(1024) k_thomas_scan(GridP g, cpx<T>* __restrict__ spec, const double* __restrict__ pa,
                                                      const double* __restrict__ pc, const double* __restrict__ pfac,
                                                      double norm, int nrow) {
  thomas_scan_body<T, S, CG, ZERO>(blockIdx.x, g, spec, pa, pc, pfac, norm, nrow);
}

// ---------------------------------------------------------------- three components at once
// The Helmholtz solves of CN in all directions transform u*, v* and w* through three spectrum
// buffers (cstride apart), so each stage is one launch over all components (blockIdx.y or z).
// Crank-Nicolson in all directions, wall-bounded z (Eq. onestar_imp3d): after FFTs in x and
// y, every (l, m) column holds the tridiagonal system with rows a_k, b_k - c (lamx(l) +
// lamy(m)), c_k (c = gamma nu dt / 2; a, b, c the CN-z rows of the component, wall folds
// included), solved in FP64.  The pivots depend on dt, so their inverses for this substep are
// formed here, once for the u/v rows and once for the w rows (nb blocks each), for m <= ny/2
// (mode ny - m has the same eigenvalue); the solves are k_thomas_scan.  One thread per column,
// with HFB rows' coefficients (scalar loads) ahead of the chain of divisions that bounds it: 24 us
// for 256 x 128 x 96 when each row's were loaded in turn, 21 so, nearly all of it on an idle chip:
// hence beside the forward x transforms (k_rfftx3), the first blocks of their launch.
constexpr int HFB = 8;
struct Helm3dArgs {
  const double *hfac, *lamx, *lamy, *dtp;
  double hg;
  double* fac;   // null: periodic z, no factors
  int nb;        // blocks per row set
};
__device__ __forceinline__ void helm3d_factor_body(int bx, const GridP& g, const Helm3dArgs& h) {
  const double *__restrict__ hfac = h.hfac, *__restrict__ lamx = h.lamx, *__restrict__ lamy = h.lamy;
  const int nxh = g.nx / 2 + 1, n = g.nz;
  const int64_t nfac = (int64_t)g.nxp * (g.ny / 2 + 1);
  const int w = bx >= h.nb;
  const int64_t col = (bx - w * h.nb) * (int64_t)blockDim.x + threadIdx.x;
  if (col >= nfac) return;
  const int l = (int)(col % g.nxp), m = (int)(col / g.nxp);
  if (l >= nxh) return;
  const double shift = h.hg * h.dtp[0] * (lamx[l] + lamy[m]);
  const double* ra = hfac + (w ? 7 : 6) * n;
  const double* rb = hfac + (w ? 10 : 8) * n;
  const double* rc = hfac + (w ? 11 : 9) * n;
  double* __restrict__ f = h.fac + (w ? (int64_t)n * nfac : 0) + col;
  const int nr = w ? n - 1 : n;
  double na[HFB], nb[HFB], nc[HFB];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int j = 0; j < HFB; ++j) {
      const int k = min(k0 + j, nr - 1);
      na[j] = ro_load(ra, k), nb[j] = ro_load(rb, k), nc[j] = ro_load(rc, k);
    }
  };
  double cprev = 0.0;
  fetch(0);
  for (int k0 = 0; k0 < nr; k0 += HFB) {
    double a[HFB], b[HFB], c[HFB];
#pragma unroll
    for (int j = 0; j < HFB; ++j) a[j] = na[j], b[j] = nb[j], c[j] = nc[j];
    fetch(k0 + HFB);
#pragma unroll
    for (int j = 0; j < HFB; ++j) {
      const double r = 1.0 / ((b[j] - shift) - a[j] * cprev);
      cprev = c[j] * r;
      if (k0 + j < nr) f[(int64_t)(k0 + j) * nfac] = r;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_rfftx3(GridP g, FftPlan P, const T* us, const T* vs, const T* ws,
                                                cpx<T>* spec, int64_t cstride, const double* twd, const float* twf,
                                                int npair_blk, int nblk, Helm3dArgs h) {
  // walls: the first row of blocks forms the z factors
  if (h.fac != nullptr && blockIdx.y == 0) {
    if ((int)blockIdx.x < 2 * h.nb) helm3d_factor_body(blockIdx.x, g, h);
    return;
  }
  if ((int)blockIdx.x >= nblk) return;
  const int comp = (int)blockIdx.y - (h.fac != nullptr ? 1 : 0);
  const T* f = comp == 0 ? us : (comp == 1 ? vs : ws);
  rfftx_body<T, 1>(dim3(blockIdx.x), g, P, nullptr, nullptr, nullptr, f, spec + comp * cstride, twd, twf, nullptr,
                   1.0, npair_blk, nullptr);
}

template <typename T>
__global__ void __launch_bounds__(256) k_irfftx3(GridP g, FftPlan P, const cpx<T>* spec, int64_t cstride, T* us,
                                                 T* vs, T* ws, const double* twd, const float* twf, int npair_blk) {
  const int comp = blockIdx.y;
  T* f = comp == 0 ? us : (comp == 1 ? vs : ws);
  irfftx_body<T>(dim3(blockIdx.x), g, P, spec + comp * cstride, f, twd, twf, npair_blk);
}

template <typename T, int DIR, bool SOLVE>
__global__ void __launch_bounds__(256) k_fft_lines3(FftPlan P, cpx<T>* data, int64_t cstride, int nl, int64_t lstride,
                                                    int64_t ostride, int L, const double* twd, const float* twf,
                                                    const double* lamx, const double* lamy, const double* lamz,
                                                    double norm, const double* dtp, double hg) {
  fft_lines_body<T, DIR, SOLVE>(dim3(blockIdx.x, blockIdx.y), P, data + blockIdx.z * cstride, nl, lstride, ostride,
                                     L, twd, twf, lamx, lamy, lamz, norm, dtp, hg);
}

// component blockIdx.y: u and v take the u/v rows and factors, w the w rows (nz - 1 unknowns);
// hfac: the CN-z rows (a_uv at 6 nz, a_w at 7 nz, c_uv at 9 nz, c_w at 11 nz)
template <typename T, int S, int CG>
__global__ void __launch_bounds__(1024) k_thomas_scan3(GridP g, cpx<T>* __restrict__ spec, int64_t cstride,
                                                       const double* __restrict__ hfac,
                                                       const double* __restrict__ fac_uv,
                                                       const double* __restrict__ fac_w, double norm) {
  const int comp = blockIdx.y, n = g.nz;
  thomas_scan_body<T, S, CG, false>(blockIdx.x, g, spec + comp * cstride, hfac + (comp < 2 ? 6 : 7) * n,
                                    hfac + (comp < 2 ? 9 : 11) * n, comp < 2 ? fac_uv : fac_w, norm,
                                    comp < 2 ? n : n - 1);
}

// ============================================================================ bulk
// s = (U_b - <u*>) / <q>, <.> the dzf-weighted volume mean; stored in dt[1].  One block:
// 256 strided partial sums, then a fixed-order tree (deterministic).
struct BulkArgs {
  const double* part;
  int nblk;
  double* dtp;
  const double* q;
  const double* dzf;
  int nz;
  double ubulk, cells_xy, lz;
};

// sm: 3 x 256 doubles of LDS (the dynamic buffer of the transform it runs beside)
__device__ __forceinline__ void bulk_final_body(const BulkArgs& a_, double (*sm)[256]) {
  const double* part = a_.part;
  const int nblk = a_.nblk, nz = a_.nz;
  const double* q = a_.q;
  const double* dzf = a_.dzf;
  for (int t = threadIdx.x; t < 256; t += blockDim.x) {
    double a = 0.0, b = 0.0, d = 0.0;
    for (int i = t; i < nblk; i += 256) a += part[i];
    for (int k = t; k < nz; k += 256) {
      b += q[k] * dzf[k + 1];
      d += dzf[k + 1];
    }
    sm[0][t] = a;
    sm[1][t] = b;
    sm[2][t] = d;
  }
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    for (int t = threadIdx.x; t < st; t += blockDim.x)
      for (int r = 0; r < 3; ++r) sm[r][t] += sm[r][t + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double mean = sm[0][0] / (a_.cells_xy * a_.lz);
    a_.dtp[1] = (a_.ubulk - mean) / (sm[1][0] / sm[2][0]);
  }
}

// Forward y transform with the flow-rate shift folded in: block (0, 0), dispatched first,
// forms s from the forward-x partials while the others transform (plane = blockIdx.y - 1).
template <typename T, int DCT = 0>
__global__ void __launch_bounds__(256) k_ffty_bulk(FftPlan P, cpx<T>* data, int nl, int64_t lstride, int64_t ostride,
                                                   int L, const double* twd, const float* twf, const double* lamx,
                                                   const double* lamy, const double* lamz, BulkArgs ba,
                                                   const double* twcd, const float* twcf) {
  if (blockIdx.y == 0) {
    extern __shared__ unsigned char smem_raw[];
    if (blockIdx.x == 0) bulk_final_body(ba, reinterpret_cast<double(*)[256]>(smem_raw));
    return;
  }
  fft_lines_body<T, -1, false, DCT>(dim3(blockIdx.x, blockIdx.y - 1), P, data, nl, lstride, ostride, L, twd, twf,
                                         lamx, lamy, lamz, 1.0, nullptr, 0.0, twcd, twcf);
}

// ghost planes of a cell-centred scalar (Neumann walls or periodic copies)
template <typename T>
__global__ void k_scalar_ghosts(GridP g, T* f) {
  const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (c >= g.sxy) return;
  const int64_t s = g.sxy, n = g.nz;
  if (g.zbc == LES_ZBC_PERIODIC) {
    f[c] = f[n * s + c];
    f[(n + 1) * s + c] = f[s + c];
  } else {
    f[c] = f[s + c];
    f[(n + 1) * s + c] = f[n * s + c];
  }
}

// ============================================================================ launchers
// Row pairs per block of the x transforms: blocks of 128 threads (eight pairs of 256 points).
// 64 and 256 threads, or 256 of which half only load, took 525-750 us where 128 take 475 (forward
// x of 1024 x 512 x 256 in FP32) and within 2 us of it on 25 MB of 256 x 128 x 96.  Fewer pairs, with
// more threads to load each, while there would be no block per CU (npairs row pairs in all: a 64^3
// box has 64 blocks of 32 pairs, forward x 13.1 us in FP64 and 11.7 in FP32; 256 of 8 take 9.7 and 9.0).
struct RowShape {
  int pairs, nt;
  size_t sh;       // dynamic LDS bytes
};
static RowShape row_shape(int n, size_t esz, int64_t npairs) {
  int pairs = std::max(1, 128 / fft_team(n));
  const int nt = pairs * fft_team(n);
  while (pairs > 1 && npairs / pairs < 256) pairs /= 2;
  return {pairs, nt, (size_t)pairs * fft_pos(n) * esz};
}

// Lines per block of the strided transforms: neighbouring values of 128 bytes, one cache line
// (256 bytes were no faster), more while a block has fewer than 64 threads, fewer where it would
// have more than 256 (`want`: at most that many, whatever the cache line); down to 64 bytes where
// `groups` groups of nl lines would leave CUs without a block and a thread has 16 points to take
// through (z solve of the 64^3 box in FP64 14.5 -> 13.0 us, 32 bytes no faster; of the 32^3 box, 4
// and 8 points a thread, 8.5 -> 8.7).
struct LineShape {
  int L, nt;
  size_t sh;
};
static LineShape line_shape(int n, size_t esz, int want = 0, int nl = 1, int64_t groups = 256) {
  const int team = fft_team(n);
  int L = want ? want : (int)(128 / esz);
  while (!want && L * team < 64) L *= 2;
  while (L * team > 256) L /= 2;
  while (n >= 64 && L * esz > 64 && groups * ((nl + L - 1) / L) < 256) L /= 2;
  return {L, std::max(64, L * team), (size_t)L * fft_pos(n) * esz};
}

template <typename T>
static void fwd_x(Ctx& c, int mode, const T* us, const T* vs, const T* ws, const T* fin, double gamma, bool bulk) {
  const FftPlan P = make_plan(c.g.nx);
  const int64_t npairs = (int64_t)c.g.nz * (c.g.ny / 2);
  const RowShape rs = row_shape(c.g.nx, sizeof(cpx<T>), npairs);
  const unsigned nblk = (unsigned)((npairs + rs.pairs - 1) / rs.pairs);
  double* bp = bulk ? c.t.bulk : nullptr;
  const double spec_bytes = (double)(c.g.nx / 2 + 1) * c.g.ny * c.g.nz * 2 * sizeof(T);
  const double in_bytes = (mode == 0 ? 3.0 : 1.0) * c.g.sxy * c.g.nz * sizeof(T);
  if (mode == 0)
    LES_LAUNCH(c, "rfftx_div", in_bytes + spec_bytes, (k_rfftx<T, 0>), dim3(nblk), dim3(rs.nt), rs.sh, c.g, P, us, vs, ws, fin,
                       (cpx<T>*)c.spec, c.t.twx, c.t.twx_f, c.t.dt, gamma, rs.pairs, bp);
  else
    LES_LAUNCH(c, "rfftx", in_bytes + spec_bytes, (k_rfftx<T, 1>), dim3(nblk), dim3(rs.nt), rs.sh, c.g, P, us, vs, ws, fin,
                       (cpx<T>*)c.spec, c.t.twx, c.t.twx_f, c.t.dt, gamma, rs.pairs, bp);
  // the flow-rate shift is formed by an extra block of the forward y transform that follows
  c.bulk_nblk = bulk ? (int)nblk : 0;
}

// y transforms of the spectrum buffer (DIR -1 forward, +1 inverse)
template <typename T, int DIR>
static void ffty(Ctx& c, const char* name) {
  const int nxh = c.g.nx / 2 + 1;
  const int ny = c.g.ny, nz = c.g.nz;
  const double spec_bytes = (double)nxh * ny * nz * 2 * sizeof(T);
  const FftPlan P = make_plan(ny);
  const LineShape ls = line_shape(ny, sizeof(cpx<T>), 0, nxh, nz);
  const int L = ls.L;
  dim3 grid((nxh + L - 1) / L, nz);
  // ducts: the cosine transform of the wall-bounded y direction
  auto kern = c.g.ywall ? k_fft_lines<T, DIR, false, 1> : k_fft_lines<T, DIR, false, 0>;
  LES_LAUNCH(c, name, 2 * spec_bytes, kern, grid, dim3(ls.nt), ls.sh, P, (cpx<T>*)c.spec, nxh, (int64_t)c.g.nxp,
             (int64_t)c.g.nxp * ny, L, c.t.twy, c.t.twy_f, c.t.lamx, c.t.lamy, c.t.lamz, 1.0, nullptr, 0.0, c.t.twc,
             c.t.twc_f);
}

// periodic z: FFT, divide by the operator's eigenvalue, inverse FFT (hg = 0: Poisson)
template <typename T>
static void fftz_solve(Ctx& c, const char* name, double hg) {
  const int nxh = c.g.nx / 2 + 1;
  const int ny = c.g.ny, nz = c.g.nz;
  const double spec_bytes = (double)nxh * ny * nz * 2 * sizeof(T);
  const FftPlan P = make_plan(nz);
  const LineShape ls = line_shape(nz, sizeof(cpx<T>), 0, nxh, ny);
  const int L = ls.L;
  dim3 grid((nxh + L - 1) / L, ny);
  const double norm = 1.0 / ((double)c.g.nx * ny * nz);
  LES_LAUNCH(c, name, 2 * spec_bytes, (k_fft_lines<T, -1, true>), grid, dim3(ls.nt), ls.sh, P,
             (cpx<T>*)c.spec, nxh, (int64_t)c.g.nxp * ny, (int64_t)c.g.nxp, L, c.t.twz, c.t.twz_f, c.t.lamx, c.t.lamy,
             c.t.lamz, norm, c.t.dt, hg, (const double*)nullptr, (const float*)nullptr);
}

template <typename T>
static void spectral_solve(Ctx& c) {
  const int nxh = c.g.nx / 2 + 1;
  const int ny = c.g.ny, nz = c.g.nz;
  cpx<T>* sp = (cpx<T>*)c.spec;
  const double spec_bytes = (double)nxh * ny * nz * 2 * sizeof(T);
  if (c.bulk_nblk > 0) {
    const FftPlan P = make_plan(ny);
    const LineShape ls = line_shape(ny, sizeof(cpx<T>), 0, nxh, nz);
    const int L = ls.L;
    dim3 grid((nxh + L - 1) / L, nz + 1);
    const size_t sh = std::max(ls.sh, 3 * 256 * sizeof(double));
    const BulkArgs ba{c.t.bulk, c.bulk_nblk, c.t.dt, c.t.hfac + 4 * nz, c.t.dzf, nz, c.cfg.ubulk,
                      (double)c.g.nx * c.g.ny, c.cfg.lz};
    auto kern = c.g.ywall ? k_ffty_bulk<T, 1> : k_ffty_bulk<T, 0>;
    LES_LAUNCH(c, "ffty_fwd", 2 * spec_bytes, kern, grid, dim3(ls.nt), sh, P, sp, nxh, (int64_t)c.g.nxp,
               (int64_t)c.g.nxp * ny, L, c.t.twy, c.t.twy_f, c.t.lamx, c.t.lamy, c.t.lamz, ba, c.t.twc, c.t.twc_f);
    c.bulk_nblk = 0;
  } else {
    ffty<T, -1>(c, "ffty_fwd");
  }
  if (c.cfg.zbc == LES_ZBC_PERIODIC) {
    fftz_solve<T>(c, "fftz_solve", 0.0);
  } else {
    const int64_t ncol = (int64_t)c.g.nxp * ny;
    const ThomasShape sh = thomas_shape(nz, sizeof(T) == 8 ? 128 : 32);
    const dim3 block(sh.CG * sh.P);
    const double norm = 1.0 / ((double)c.g.nx * ny);
    const double bytes = 2 * spec_bytes + (double)nxh * factor_modes(c.g) * nz * 8;
    auto go = [&](auto kern, int64_t nb) {
      LES_LAUNCH(c, "thomas_z", bytes, kern, dim3((unsigned)nb), block, 0, c.g, sp, c.t.pa, c.t.pc, c.t.pfac,
                 norm, nz);
    };
    if (sh.CG == 64)
      sh.S == 8 ? go(k_thomas_scan<T, 8, 64, true>, (ncol + 64 - 1) / 64)
                : go(k_thomas_scan<T, 16, 64, true>, (ncol + 64 - 1) / 64);
    else
      sh.S == 8 ? go(k_thomas_scan<T, 8, 32, true>, (ncol + 32 - 1) / 32)
                : go(k_thomas_scan<T, 16, 32, true>, (ncol + 32 - 1) / 32);
  }
  ffty<T, 1>(c, "ffty_inv");
}

template <typename T>
static void inv_x(Ctx& c, T* out) {
  const FftPlan P = make_plan(c.g.nx);
  const int64_t npairs = (int64_t)c.g.nz * (c.g.ny / 2);
  const RowShape rs = row_shape(c.g.nx, sizeof(cpx<T>), npairs);
  const unsigned nblk = (unsigned)((npairs + rs.pairs - 1) / rs.pairs);
  const double spec_bytes = (double)(c.g.nx / 2 + 1) * c.g.ny * c.g.nz * 2 * sizeof(T);
  LES_LAUNCH(c, "irfftx", spec_bytes + (double)c.g.sxy * c.g.nz * sizeof(T), (k_irfftx<T>), dim3(nblk),
             dim3(rs.nt), rs.sh, c.g, P, (const cpx<T>*)c.spec, out, c.t.twx, c.t.twx_f, rs.pairs);
}

// Crank-Nicolson in all directions (Eq. onestar_imp3d): the predicted components u*, v*, w*
// (right-hand sides of the Helmholtz systems, wall-model flux included) are transformed in x
// and y into three spectrum buffers, solved per wavenumber pair in z (Thomas in FP64 at
// walls, FFT when z is periodic) and transformed back in place; one launch per stage.
template <typename T>
void launch_helmholtz_3d(Ctx& c, int stage) {
  static const double G[3] = {8.0 / 15.0, 2.0 / 15.0, 1.0 / 3.0};
  const double hg = G[stage] * c.cfg.nu / 2.0;
  const int n = c.g.nz, nx = c.g.nx, ny = c.g.ny, nxh = nx / 2 + 1;
  const double spec_bytes = (double)nxh * ny * n * 2 * sizeof(T);
  const int64_t cstride = (int64_t)c.g.nxp * ny * n;   // complex values per component
  cpx<T>* sp = (cpx<T>*)c.spec;
  const int64_t nfac = (int64_t)c.g.nxp * (ny / 2 + 1);
  const double norm_xy = 1.0 / ((double)nx * ny);
  // forward x of the three components; walls: the z factors of this substep beside them
  {
    const FftPlan P = make_plan(nx);
    const int64_t npairs = (int64_t)n * (ny / 2);
    const RowShape rs = row_shape(nx, sizeof(cpx<T>), 3 * npairs);
    const int nblk = (int)((npairs + rs.pairs - 1) / rs.pairs);
    const bool walls = c.cfg.zbc != LES_ZBC_PERIODIC;
    const Helm3dArgs h{c.t.hfac, c.t.lamx, c.t.lamy, c.t.dt, hg, walls ? c.t.hfac3 : nullptr,
                       (int)((nfac + rs.nt - 1) / rs.nt)};
    LES_LAUNCH(c, "h3d_rfftx", 3 * (spec_bytes + (double)c.g.sxy * n * sizeof(T)) + (walls ? 2.0 * nfac * n * 8 : 0.0),
               (k_rfftx3<T>), dim3((unsigned)(walls ? std::max(nblk, 2 * h.nb) : nblk), walls ? 4 : 3), dim3(rs.nt), rs.sh,
               c.g, P, (const T*)c.us, (const T*)c.vs, (const T*)c.wsf, sp, cstride, c.t.twx, c.t.twx_f, rs.pairs, nblk, h);
  }
  const FftPlan Py = make_plan(ny);
  const LineShape lsy = line_shape(ny, sizeof(cpx<T>));
  const int Ly = lsy.L;
  const dim3 gy((nxh + Ly - 1) / Ly, n, 3);
  LES_LAUNCH(c, "h3d_ffty_fwd", 6 * spec_bytes, (k_fft_lines3<T, -1, false>), gy, dim3(lsy.nt), lsy.sh, Py, sp,
             cstride, nxh, (int64_t)c.g.nxp, (int64_t)c.g.nxp * ny, Ly, c.t.twy, c.t.twy_f, c.t.lamx, c.t.lamy,
             c.t.lamz, 1.0, nullptr, 0.0);
  if (c.cfg.zbc == LES_ZBC_PERIODIC) {
    const FftPlan Pz = make_plan(n);
    const LineShape lsz = line_shape(n, sizeof(cpx<T>));
    const int Lz = lsz.L;
    LES_LAUNCH(c, "h3d_fftz_solve", 6 * spec_bytes, (k_fft_lines3<T, -1, true>),
               dim3((nxh + Lz - 1) / Lz, ny, 3), dim3(lsz.nt), lsz.sh, Pz, sp, cstride, nxh, (int64_t)c.g.nxp * ny,
               (int64_t)c.g.nxp, Lz, c.t.twz, c.t.twz_f, c.t.lamx, c.t.lamy, c.t.lamz, 1.0 / ((double)nx * ny * n),
               c.t.dt, hg);
  } else {
    const int64_t ncol = (int64_t)c.g.nxp * ny;
    const ThomasShape sh = thomas_shape(n, 128);
    const dim3 block(sh.CG * sh.P);
    const double* f_uv = c.t.hfac3;
    const double* f_w = f_uv + (int64_t)n * nfac;
    const double bytes = 6 * spec_bytes + 3.0 * nfac * n * 8;
    auto go = [&](auto kern, int64_t nb) {
      LES_LAUNCH(c, "h3d_thomas_z", bytes, kern, dim3((unsigned)nb, 3), block, 0, c.g, sp, cstride, c.t.hfac, f_uv, f_w,
                 norm_xy);
    };
    if (sh.CG == 64)
      sh.S == 8 ? go(k_thomas_scan3<T, 8, 64>, (ncol + 64 - 1) / 64)
                : go(k_thomas_scan3<T, 16, 64>, (ncol + 64 - 1) / 64);
    else
      sh.S == 8 ? go(k_thomas_scan3<T, 8, 32>, (ncol + 32 - 1) / 32)
                : go(k_thomas_scan3<T, 16, 32>, (ncol + 32 - 1) / 32);
  }
  LES_LAUNCH(c, "h3d_ffty_inv", 6 * spec_bytes, (k_fft_lines3<T, 1, false>), gy, dim3(lsy.nt), lsy.sh, Py, sp,
             cstride, nxh, (int64_t)c.g.nxp, (int64_t)c.g.nxp * ny, Ly, c.t.twy, c.t.twy_f, c.t.lamx, c.t.lamy,
             c.t.lamz, 1.0, nullptr, 0.0);
  {
    const FftPlan P = make_plan(nx);
    const int64_t npairs = (int64_t)n * (ny / 2);
    const RowShape rs = row_shape(nx, sizeof(cpx<T>), 3 * npairs);
    LES_LAUNCH(c, "h3d_irfftx", 3 * (spec_bytes + (double)c.g.sxy * n * sizeof(T)), (k_irfftx3<T>),
               dim3((unsigned)((npairs + rs.pairs - 1) / rs.pairs), 3), dim3(rs.nt), rs.sh, c.g, P, (const cpx<T>*)sp, cstride,
               (T*)c.us, (T*)c.vs, (T*)c.wsf, c.t.twx, c.t.twx_f, rs.pairs);
  }
}

template <typename T>
void launch_poisson_rhs_fwd(Ctx& c, const T* us, const T* vs, const T* ws, double gamma, int stage) {
  (void)stage;
  fwd_x<T>(c, 0, us, vs, ws, nullptr, gamma, c.cfg.ubulk > 0.0);
}

template <typename T>
void launch_poisson_solve_spectral(Ctx& c) {
  spectral_solve<T>(c);
}

template <typename T>
void launch_poisson_inverse(Ctx& c, T* phi_out) {
  inv_x<T>(c, phi_out);
}

template <typename T>
void launch_poisson_field(Ctx& c, T* f) {
  fwd_x<T>(c, 1, nullptr, nullptr, nullptr, f, 1.0, false);
  spectral_solve<T>(c);
  inv_x<T>(c, f);
  LES_LAUNCH(c, "scalar_ghosts", 4.0 * c.g.sxy * sizeof(T), k_scalar_ghosts<T>, dim3((unsigned)((c.g.sxy + 255) / 256)),
             dim3(256), 0, c.g, f);
  if (c.g.ywall) launch_fill_y_scalar<T>(c, f, 1.0);
}

// ============================================================================ initial projection
// One projection of the bound velocity with the substep's operators (Eqs. poi, correc without
// the time factor): phi solves D G phi = D u, u -= G phi; with a constant flow rate the
// streamwise velocity is then shifted uniformly so that its volume mean is U_b.  The interior
// cells are cut into PROJ_BLOCKS contiguous chunks, one block each, so that the flow-rate sum
// runs in a fixed order.
constexpr int PROJ_BLOCKS = 64;

template <typename T>
__global__ void __launch_bounds__(256) k_project_correct(GridP g, T* __restrict__ u, T* __restrict__ v,
                                                         T* __restrict__ w, const T* __restrict__ phi,
                                                         double* __restrict__ part) {
  __shared__ double red[256];
  const int64_t nxy = (int64_t)g.nx * g.ny;
  const int64_t total = (int64_t)g.nz * nxy;
  const int64_t chunk = (total + PROJ_BLOCKS - 1) / PROJ_BLOCKS;
  const int64_t e0 = blockIdx.x * chunk, e1 = e0 + chunk < total ? e0 + chunk : total;
  const bool walls = g.zbc != LES_ZBC_PERIODIC;
  double su = 0.0;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int k = (int)(e / nxy) + 1;
    const int64_t r = e % nxy;
    const int i = (int)(r % g.nx), j = (int)(r / g.nx);
    const int64_t c = idx3(g, k, j, i);
    const T ph = phi[c];
    const T un = u[c] - (phi[idx3(g, k, j, wrap_p(i, g.nx))] - ph) * (T)g.rdx;
    u[c] = un;
    // the y wall face y = ly of a duct (row ny - 1) and the z wall face on top stay at rest
    v[c] = (g.ywall && j == g.ny - 1) ? (T)0 : v[c] - (phi[idx3(g, k, wrap_p(j, g.nys), i)] - ph) * (T)g.rdy;
    w[c] = (walls && k == g.nz) ? (T)0 : w[c] - (phi[c + g.sxy] - ph) * (T)g.rdzc[k];
    su += (double)un * g.dzf[k];
  }
  red[threadIdx.x] = su;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// u += U_b - <u> on every interior cell; each block sums the chunk partials in block order.
template <typename T>
__global__ void __launch_bounds__(256) k_project_shift(GridP g, T* __restrict__ u, const double* __restrict__ part,
                                                       double ubulk, double lz) {
  __shared__ double shift;
  if (threadIdx.x == 0) {
    double a = 0.0;
    for (int b = 0; b < PROJ_BLOCKS; ++b) a += part[b];
    shift = ubulk - a / ((double)g.nx * g.ny * lz);
  }
  __syncthreads();
  const T s = (T)shift;
  const int64_t nxy = (int64_t)g.nx * g.ny;
  const int64_t total = (int64_t)g.nz * nxy;
  const int64_t chunk = (total + PROJ_BLOCKS - 1) / PROJ_BLOCKS;
  const int64_t e0 = blockIdx.x * chunk, e1 = e0 + chunk < total ? e0 + chunk : total;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int k = (int)(e / nxy) + 1;
    const int64_t r = e % nxy;
    u[(int64_t)k * g.sxy + r] += s;
  }
}

template <typename T>
void launch_project(Ctx& c) {
  T* u = (T*)c.u;
  T* v = (T*)c.v;
  T* w = (T*)c.w;
  T* phi = (T*)c.phi;
  launch_bc_fill<T>(c, u, v, w, (T*)c.p);   // wall faces of w (and the periodic copies)
  if (c.g.ywall) launch_bc_fill_y<T>(c, u, v, w, (T*)c.p);
  fwd_x<T>(c, 0, u, v, w, nullptr, 0.0, false);
  spectral_solve<T>(c);
  inv_x<T>(c, phi);
  LES_LAUNCH(c, "scalar_ghosts", 4.0 * c.g.sxy * sizeof(T), k_scalar_ghosts<T>, dim3((unsigned)((c.g.sxy + 255) / 256)),
             dim3(256), 0, c.g, phi);
  if (c.g.ywall) launch_fill_y_scalar<T>(c, phi, 1.0);
  const double cells = (double)c.g.nx * c.g.ny * c.g.nz;
  LES_LAUNCH(c, "project_correct", 7.0 * cells * sizeof(T), k_project_correct<T>, dim3(PROJ_BLOCKS), dim3(256), 0,
             c.g, u, v, w, (const T*)phi, c.t.red);
  if (c.cfg.ubulk > 0.0)
    LES_LAUNCH(c, "project_shift", 2.0 * cells * sizeof(T), k_project_shift<T>, dim3(PROJ_BLOCKS), dim3(256), 0, c.g,
               u, (const double*)c.t.red, c.cfg.ubulk, c.cfg.lz);
}

// ============================================================================ batch launchers
template <typename T>
void batch_poisson(hipStream_t st, const BatchMap& m, const int* totals, const FftLaunch* f, int stage) {
  static const double G[3] = {8.0 / 15.0, 2.0 / 15.0, 1.0 / 3.0};
  hipLaunchKernelGGL(kb_rfftx<T>, dim3(totals[BK_RFFTX]), dim3(f[0].nt), f[0].sh, st, m, G[stage]);
  hipLaunchKernelGGL((kb_fft_lines<T, -1, false>), dim3(totals[BK_FFTY]), dim3(f[1].nt), f[1].sh, st, m);
  hipLaunchKernelGGL((kb_fft_lines<T, -1, true>), dim3(totals[BK_FFTZ]), dim3(f[2].nt), f[2].sh, st, m);
  hipLaunchKernelGGL((kb_fft_lines<T, 1, false>), dim3(totals[BK_FFTY]), dim3(f[1].nt), f[1].sh, st, m);
  hipLaunchKernelGGL(kb_irfftx<T>, dim3(totals[BK_RFFTX]), dim3(f[0].nt), f[0].sh, st, m);
}
template void batch_poisson<float>(hipStream_t, const BatchMap&, const int*, const FftLaunch*, int);
template void batch_poisson<double>(hipStream_t, const BatchMap&, const int*, const FftLaunch*, int);

// shapes of a box in a batch, whose launches take the largest block and LDS of their boxes
FftLaunch fft_rows(int n, size_t esz) {
  const RowShape r = row_shape(n, esz, INT64_MAX);
  return {r.pairs, r.nt, r.sh};
}
FftLaunch fft_lines(int n, size_t esz, int want) {
  const LineShape l = line_shape(n, esz, want);
  return {l.L, l.nt, l.sh};
}

#define INST(T)                                                                              \
  template void launch_poisson_rhs_fwd<T>(Ctx&, const T*, const T*, const T*, double, int); \
  template void launch_poisson_solve_spectral<T>(Ctx&);                                      \
  template void launch_poisson_inverse<T>(Ctx&, T*);                                         \
  template void launch_poisson_field<T>(Ctx&, T*);                                          \
  template void launch_project<T>(Ctx&);                                                     \
  template void launch_helmholtz_3d<T>(Ctx&, int);
INST(double)
INST(float)

}  // namespace les
