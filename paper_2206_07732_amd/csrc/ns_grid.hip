// Grid kernels of the time step on gfx950: level-set advection and
// reinitialisation, material properties, the momentum predictor, the
// projection right-hand side, the velocity correction and diagnostics.
//
// Threads are laid out 64 along x (one wavefront per x-row segment, so every
// load of a row is one contiguous 512-byte FP64 segment) by 4 along y (or
// along z for a 2-D tank).  Out-of-grid neighbours are the nearest interior
// value: zero normal gradient for scalars, free slip for tangential
// velocity, zero for wall-normal velocity (whose faces hold 0).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ns_internal.h"

namespace nsk {

namespace {

constexpr double kPi = 3.14159265358979323846;

struct Geo {
  dim3 grid, block;
};

inline Geo geo3(int mx, int my, int mz) {
  dim3 b = (my >= 4) ? dim3(64, 4, 1) : dim3(64, 1, 4);
  return {dim3((mx + 63) / 64, (my + b.y - 1) / b.y, (mz + b.z - 1) / b.z), b};
}

constexpr double kE = 2.718281828459045235360287471352662;   // e

__device__ __forceinline__ int clampi(int a, int lo, int hi) { return a < lo ? lo : (a > hi ? hi : a); }

// cell value with clamped indices
__device__ __forceinline__ double cv(const double* __restrict__ a, const Dims& n, int i, int j, int k) {
  i = clampi(i, 0, n.nx - 1);
  j = clampi(j, 0, n.ny - 1);
  k = clampi(k, 0, n.nz - 1);
  // 32-bit index arithmetic: every array has fewer than 2^31 entries (the
  // context refuses grids with more than 2e9 faces), and the predictor's
  // ~35 clamped loads per face made 64-bit products a large share of its
  // instructions
  return a[i + n.nx * (j + n.ny * k)];
}

// face value of component C with clamped indices
template <int C>
__device__ __forceinline__ double fv(const double* __restrict__ a, const Dims& n, int i, int j, int k) {
  const int mx = n.nx + (C == 0), my = n.ny + (C == 1), mz = n.nz + (C == 2);
  i = clampi(i, 0, mx - 1);
  j = clampi(j, 0, my - 1);
  k = clampi(k, 0, mz - 1);
  return a[i + mx * (j + my * k)];
}

// The values of two columns, i and i + 1, and their arithmetic: a lane that
// takes both loads them with one 16-byte access, at any 8-byte alignment.  A
// wavefront's access costs the address unit the same 16 clocks at 8 and at 16
// bytes per lane, and that unit is what bounds a stencil of FP64 values.
struct V2 {
  double x, y;
};
struct __attribute__((packed, aligned(8))) V2Mem {
  double x, y;
};
struct __attribute__((packed, aligned(4))) F2Mem {
  float x, y;
};
__device__ __forceinline__ V2 operator+(V2 a, V2 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ V2 operator-(V2 a, V2 b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ V2 operator*(V2 a, V2 b) { return {a.x * b.x, a.y * b.y}; }
__device__ __forceinline__ V2 operator*(double a, V2 b) { return {a * b.x, a * b.y}; }
__device__ __forceinline__ V2 operator*(V2 a, double b) { return {a.x * b, a.y * b}; }
__device__ __forceinline__ void operator+=(V2& a, V2 b) { a.x += b.x, a.y += b.y; }
// Columns i + O and i + O + 1, each clamped to [0, mx), of a row that starts at
// `row` (0 <= i < mx, mx >= 2).  Where the row is the same for the wavefront the
// load's base is a scalar and its offset is shared by every row.
template <int O>
__device__ __forceinline__ V2 pair_at(const double* __restrict__ a, int mx, int i, int row) {
  const unsigned off = 8u * (unsigned)(O < 0 ? max(i + O, 0) : min(i + O, mx - 2));
  const V2Mem m = *reinterpret_cast<const V2Mem*>(reinterpret_cast<const char*>(a + row) + off);
  if (O < 0) return {m.x, i + O < 0 ? m.x : m.y};
  return {i + O > mx - 2 ? m.y : m.x, m.y};
}
// What a sum holds so far is formed here: the compiler would sink a
// direction's arithmetic to the end of the kernel, past the branches of the
// limiters, and keep every direction's loads in registers for it.
__device__ __forceinline__ void settle(double&) {}
__device__ __forceinline__ void settle(V2& a) { asm volatile("" : "+v"(a.x), "+v"(a.y)); }
// cv and fv at column i + O, of one column or of two
template <typename T, int O>
__device__ __forceinline__ T cvt(const double* __restrict__ a, const Dims& n, int i, int j, int k) {
  if constexpr (std::is_same_v<T, V2>)
    return pair_at<O>(a, n.nx, i, n.nx * (clampi(j, 0, n.ny - 1) + n.ny * clampi(k, 0, n.nz - 1)));
  else
    return cv(a, n, i + O, j, k);
}
template <int C, typename T, int O>
__device__ __forceinline__ T fvt(const double* __restrict__ a, const Dims& n, int i, int j, int k) {
  if constexpr (std::is_same_v<T, V2>) {
    const int mx = n.nx + (C == 0), my = n.ny + (C == 1), mz = n.nz + (C == 2);
    return pair_at<O>(a, mx, i, mx * (clampi(j, 0, my - 1) + my * clampi(k, 0, mz - 1)));
  } else {
    return fv<C>(a, n, i + O, j, k);
  }
}

// Koren-limited upwind face value; up2 is the cell behind the upwind cell up,
// dn the downwind cell.  Third order (kappa = 1/3) where smooth, first order
// at extrema, total-variation diminishing.
__device__ __forceinline__ double koren(double up2, double up, double dn) {
  const double a = up - up2;
  const double b = dn - up;
  if (a * b <= 0.0) return up;
  const double fa = fabs(a), fb = fabs(b);
  const double lim = fmin(fmin(2.0 * fa, (2.0 * fb + fa) * (1.0 / 3.0)), 2.0 * fb);
  return up + copysign(0.5 * lim, b);
}

// The Koren value at a face between m (its negative side) and p, with mm
// behind m and pp beyond p, upwind of the advecting velocity a.  The upwind
// side's three values are selected first, so one limiter is evaluated
// instead of both sides' and a select of the two.
__device__ __forceinline__ double koren_face(double a, double mm, double m, double p, double pp) {
  const bool pos = a >= 0.0;
  return koren(pos ? mm : pp, pos ? m : p, pos ? p : m);
}

__device__ __forceinline__ V2 koren_face(V2 a, V2 mm, V2 m, V2 p, V2 pp) {
  return {koren_face(a.x, mm.x, m.x, p.x, pp.x), koren_face(a.y, mm.y, m.y, p.y, pp.y)};
}

__device__ __forceinline__ double heaviside(double phi, double eps) {
  if (phi < -eps) return 0.0;
  if (phi > eps) return 1.0;
  return 0.5 * (1.0 + phi / eps + sin(kPi * phi / eps) * (1.0 / kPi));
}

// level set of one body at (x,y,z,t) and its heave velocity: prescribed
// heave A sin(w t + phi), or the free body's own state
__device__ double body_psi_one(const BodyK& B, double x, double y, double z, double t, double* zdot) {
  double zeta, zd;
  if (B.fh) {
    zeta = B.zeta;
    zd = B.zdot;
  } else {
    const double arg = B.om * t + B.ph;
    zeta = B.amp * sin(arg);
    zd = B.amp * B.om * cos(arg);
  }
  *zdot = zd;
  if (B.kind == 0) return fmax(fabs(x - B.c0) - B.h0, fabs(z - (B.c2 + zeta)) - B.h2);
  const double dx = x - B.c0, dy = y - B.c1;
  const double r = sqrt(dx * dx + dy * dy);
  return fmax(r - B.h0, fmax((B.h1 + zeta) - z, z - (B.h2 + zeta)));
}

// union of the analytic bodies at (x,y,z,t); zdot of the nearest one
__device__ double body_psi(const Phys& P, double x, double y, double z, double t, double* zdot) {
  double best = INFINITY;
  double zd_best = 0.0;
  for (int m = 0; m < P.nb; ++m) {
    double zd;
    const double s = body_psi_one(P.body[m], x, y, z, t, &zd);
    if (s < best) {
      best = s;
      zd_best = zd;
    }
  }
  *zdot = zd_best;
  return best;
}

// --------------------------------------------------------------------------
// numerical wave tank (Sec. "Numerical wave tank")
// --------------------------------------------------------------------------
// the generated wave: elevation, and horizontal (c = 0) or vertical (c = 2)
// potential-flow velocity under the surface at (x, z from the bed, t)
__device__ double tank_eta(const Phys& P, double x, double t) {
  double eta = 0.0;
  for (int q = 0; q < P.nwave; ++q) {
    const double* W = P.waves + 4 * q;
    eta += W[0] * cos(W[1] * x - W[2] * t + W[3]);
  }
  return eta;
}

__device__ double tank_vel(const Phys& P, int c, double x, double z, double t) {
  if (c == 1 || z >= P.depth + tank_eta(P, x, t)) return 0.0;
  double s = 0.0;
  for (int q = 0; q < P.nwave; ++q) {
    const double* W = P.waves + 4 * q;
    const double th = W[1] * x - W[2] * t + W[3];
    const double amp = W[0] * W[2] / sinh(W[1] * P.depth);
    s += (c == 0) ? amp * cosh(W[1] * z) * cos(th) : amp * sinh(W[1] * z) * sin(th);
  }
  return s;
}

// relaxation weight (the relaxation-zone method): 1 at the inner edge, 0 at the end
__device__ __forceinline__ double relax_weight(double chi) {
  return 1.0 - (exp(pow(chi, 3.5)) - 1.0) / (kE - 1.0);
}

// vorticity damping coefficient over the top vort_w of the tank
__device__ __forceinline__ double vort_coeff(const Phys& P, double z, double dt) {
  if (P.vort_w <= 0.0) return 0.0;
  const double zt = (z - P.n.nz * P.h) / P.vort_w;
  return zt < -1.0 ? 0.0 : P.rho_a * (cos(kPi * zt) + 1.0) / (4.0 * dt);
}

// --------------------------------------------------------------------------
// level-set advection: sigma* = sigma - dt/h sum_d [a+ (s+ - s) - a- (s- - s)]
// --------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_advect(Phys P, const double* __restrict__ s,
                                                const double* __restrict__ u,
                                                const double* __restrict__ v,
                                                const double* __restrict__ w, double dt,
                                                double* __restrict__ out) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t c = i + (size_t)n.nx * j + sxy * k;
  const double sc = s[c];
  double acc = 0.0;
  // each direction's four neighbours are loaded before the upwind side is
  // chosen, so no load waits on the velocity's sign
  {  // x
    const size_t fm = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
    const double am = u[fm], ap = u[fm + 1];
    auto S = [&](int o) { return s[c + (clampi(i + o, 0, n.nx - 1) - i)]; };
    const double m2 = S(-2), m1 = S(-1), p1 = S(1), p2 = S(2);
    const double sp = koren_face(ap, m1, sc, p1, p2);
    const double sm = koren_face(am, m2, m1, sc, p1);
    acc += ap * (sp - sc) - am * (sm - sc);
  }
  {  // y
    const size_t fm = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
    const double am = v[fm], ap = v[fm + n.nx];
    auto S = [&](int o) { return s[c + (ptrdiff_t)(clampi(j + o, 0, n.ny - 1) - j) * n.nx]; };
    const double m2 = S(-2), m1 = S(-1), p1 = S(1), p2 = S(2);
    const double sp = koren_face(ap, m1, sc, p1, p2);
    const double sm = koren_face(am, m2, m1, sc, p1);
    acc += ap * (sp - sc) - am * (sm - sc);
  }
  {  // z
    const double am = w[c], ap = w[c + sxy];
    auto S = [&](int o) { return s[c + (ptrdiff_t)(clampi(k + o, 0, n.nz - 1) - k) * (ptrdiff_t)sxy]; };
    const double m2 = S(-2), m1 = S(-1), p1 = S(1), p2 = S(2);
    const double sp = koren_face(ap, m1, sc, p1, p2);
    const double sm = koren_face(am, m2, m1, sc, p1);
    acc += ap * (sp - sc) - am * (sm - sc);
  }
  out[c] = sc - (dt / P.h) * acc;
}

// The same for larger grids: a lane holds kRR rows of a column and marches up
// kz planes.  The plane's two neighbours above and below and most along y are
// then in registers, and the face value above a cell is the one below the next,
// that between two of its rows serves both: 4.5 of the six limiters and 11.5
// of the 19 loads, whose issue (16 clocks for a wavefront's 8-byte load) and
// the index arithmetic around them bound the one-cell form.  Four wavefronts
// per SIMD hide the loads as well as loading a plane ahead with half as many.
// 301 x 125 x 131 (39 us at the copy rate): 66 -> 46 us.
constexpr int kRR = 2, kRW = 8;   // rows of a lane, wavefronts of a block
__global__ void __launch_bounds__(64 * kRW, 4) k_advect_march(Phys P, const double* __restrict__ s,
                                                           const double* __restrict__ u, const double* __restrict__ v,
                                                           const double* __restrict__ w, double dt,
                                                           double* __restrict__ out, int kz) {
  constexpr int R = kRR;
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * 64 + threadIdx.x;
  const int j0 = (tl.y * kRW + __builtin_amdgcn_readfirstlane(threadIdx.y)) * R;
  const int kb = tl.z * kz, ke = min(kb + kz, n.nz);
  if (j0 >= n.ny) return;
  const double c0 = dt / P.h;
  const int ic = min(i, n.nx - 1);
  // byte offsets in a plane (32 bits: a load's base is then a scalar)
  auto at = [](const double* plane, unsigned off) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(plane) + off);
  };
  unsigned row[R + 4], vrow[R + 1], urow[R];
#pragma unroll
  for (int r = 0; r < R + 4; ++r) row[r] = 8u * (unsigned)(n.nx * clampi(j0 + r - 2, 0, n.ny - 1) + ic);
#pragma unroll
  for (int r = 0; r < R + 1; ++r) vrow[r] = 8u * (unsigned)(n.nx * min(j0 + r, n.ny) + ic);
#pragma unroll
  for (int r = 0; r < R; ++r) urow[r] = 8u * (unsigned)((n.nx + 1) * min(j0 + r, n.ny - 1) + ic);
  int ox[4];   // the neighbours along x
#pragma unroll
  for (int o = 0; o < 4; ++o) ox[o] = 8 * (clampi(ic + (o < 2 ? o - 2 : o - 1), 0, n.nx - 1) - ic);
  const size_t sxy = (size_t)n.nx * n.ny;
  struct Plane {
    double x[R][4], y[4], u[R][2], v[R + 1], w[R];
  };
  auto load = [&](int k, Plane& p) {
    const int kc = min(k, n.nz - 1);
    const double* q = s + sxy * kc;
    const double* qu = u + (size_t)(n.nx + 1) * n.ny * kc;
    const double* qv = v + (size_t)n.nx * (n.ny + 1) * kc;
    const double* qw = w + sxy * (kc + 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int o = 0; o < 4; ++o) p.x[r][o] = at(q, row[r + 2] + ox[o]);
      p.u[r][0] = at(qu, urow[r]);
      p.u[r][1] = at(qu, urow[r] + 8);
      p.w[r] = at(qw, row[r + 2]);   // the face above
    }
    p.y[0] = at(q, row[0]);
    p.y[1] = at(q, row[1]);
    p.y[2] = at(q, row[R + 2]);
    p.y[3] = at(q, row[R + 3]);
#pragma unroll
    for (int r = 0; r < R + 1; ++r) p.v[r] = at(qv, vrow[r]);
  };
  auto centre = [&](int k, double (&o)[R]) {
    const double* q = s + sxy * clampi(k, 0, n.nz - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] = at(q, row[r + 2]);
  };
  double z[5][R], wm[R], zm[R];   // planes k - 2 .. k + 2; the face below: velocity and value
  Plane p;
#pragma unroll
  for (int o = 0; o < 5; ++o) centre(kb + o - 2, z[o]);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    wm[r] = at(w + sxy * kb, row[r + 2]);
    zm[r] = koren_face(wm[r], z[0][r], z[1][r], z[2][r], z[3][r]);
  }
#pragma unroll 1
  for (int k = kb; k < ke; ++k) {
    double zn[R];
    load(k, p);
    centre(k + 3, zn);
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double sc = z[2][r];
      const double sp = koren_face(p.u[r][1], p.x[r][1], sc, p.x[r][2], p.x[r][3]);
      const double sm = koren_face(p.u[r][0], p.x[r][0], p.x[r][1], sc, p.x[r][2]);
      acc[r] = p.u[r][1] * (sp - sc) - p.u[r][0] * (sm - sc);
    }
    // rows j0 - 2 .. j0 + R + 1
    double y[R + 4];
    y[0] = p.y[0];
    y[1] = p.y[1];
#pragma unroll
    for (int r = 0; r < R; ++r) y[r + 2] = z[2][r];
    y[R + 2] = p.y[2];
    y[R + 3] = p.y[3];
    double fy = koren_face(p.v[0], y[0], y[1], y[2], y[3]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double fp = koren_face(p.v[r + 1], y[r + 1], y[r + 2], y[r + 3], y[r + 4]);
      const double sc = z[2][r];
      acc[r] += p.v[r + 1] * (fp - sc) - p.v[r] * (fy - sc);
      fy = fp;
      const double zp = koren_face(p.w[r], z[1][r], sc, z[3][r], z[4][r]);
      acc[r] += p.w[r] * (zp - sc) - wm[r] * (zm[r] - sc);
      wm[r] = p.w[r];
      zm[r] = zp;
      if (i < n.nx && j0 + r < n.ny)
        *reinterpret_cast<double*>(reinterpret_cast<char*>(out + sxy * k) + row[r + 2]) = sc - c0 * acc[r];
#pragma unroll
      for (int o = 0; o < 4; ++o) z[o][r] = z[o + 1][r];
      z[4][r] = zn[r];
    }
  }
}

// --------------------------------------------------------------------------
// reinitialisation pseudo-step: Godunov upwind |grad sigma|, smoothed sign of
// the pre-reinitialisation field sigma0.
// --------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_reinit(Phys P, const double* __restrict__ s0,
                                                const double* __restrict__ cur,
                                                double* __restrict__ nxt, double dtau) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t c = i + (size_t)n.nx * j + sxy * k;
  // every load is issued before the sign test, so none waits on it
  const double a0 = s0[c];
  const double sc = cur[c];
  const double nb[6] = {cur[i > 0 ? c - 1 : c],
                        cur[i < n.nx - 1 ? c + 1 : c],
                        cur[j > 0 ? c - n.nx : c],
                        cur[j < n.ny - 1 ? c + n.nx : c],
                        cur[k > 0 ? c - sxy : c],
                        cur[k < n.nz - 1 ? c + sxy : c]};
  const double h = P.h;
  const double sg = a0 / sqrt(a0 * a0 + h * h);
  // (a cell on the interface, sg = 0, keeps its value: selected at the end
  // rather than returned early, so the neighbour loads are not sunk behind
  // the wait for a0)
  const double ih = 1.0 / h;
  double g2 = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double a = (sc - nb[2 * d]) * ih;      // backward difference
    const double b = (nb[2 * d + 1] - sc) * ih;  // forward difference
    double t1, t2;
    if (sg > 0.0) {
      t1 = fmax(a, 0.0);
      t2 = fmin(b, 0.0);
    } else {
      t1 = fmin(a, 0.0);
      t2 = fmax(b, 0.0);
    }
    g2 += fmax(t1 * t1, t2 * t2);
  }
  const double upd = sc - dtau * sg * (sqrt(g2) - 1.0);
  nxt[c] = sg == 0.0 ? sc : upd;
}

// sqrt(x) for x >= 0 and a / sqrt(x) for x > 0 without the scaling that the
// library's forms carry for extreme arguments (which go to those).  The textbook
// Newton iterations on the hardware's reciprocal square root (relative error
// below 2^-22): Goldschmidt's coupled step for the root, a third-order step for
// its reciprocal; each result then takes one correction from its residual in a
// fused multiply-add, as Markstein describes, which rounds it correctly: of
// 2^30 random arguments none differed from sqrt(x), or from the division by it.
__device__ __forceinline__ double root(double x) {
  if (!(x > 1e-280 && x < 1e280)) return sqrt(x);
  const double y = __builtin_amdgcn_rsq(x);
  const double s0 = x * y, h0 = 0.5 * y, r = fma(-h0, s0, 0.5);
  const double s1 = fma(s0, r, s0), h1 = fma(h0, r, h0);
  return fma(fma(-s1, s1, x), h1, s1);
}
__device__ __forceinline__ double over_root(double a, double x) {
  if (!(x > 1e-280 && x < 1e280)) return a / sqrt(x);
  const double y0 = __builtin_amdgcn_rsq(x);
  const double e0 = fma(-x * y0, y0, 1.0), y1 = fma(y0 * e0, fma(0.375, e0, 0.5), y0);
  const double r0 = x * y1, r = fma(fma(-r0, r0, x), 0.5 * y1, r0);   // the rounded root
  const double q = a * y1;
  return fma(fma(-q, r, a), y1, q);
}

// A pseudo-step's update of one cell from its six neighbours, f = the sign of
// sg (1 where positive, else -1): along each direction the larger of the two
// upwind differences is max(f s - min(f s_-, f s_+), 0).
__device__ __forceinline__ double reinit_cell(double sc, double sg, double xm, double xp, double ym, double yp,
                                              double zm, double zp, double dtau, double ih) {
  const double f = sg > 0.0 ? 1.0 : -1.0;
  const double fs = f * sc;
  const double dx = fmax(fs - fmin(f * xm, f * xp), 0.0);
  const double dy = fmax(fs - fmin(f * ym, f * yp), 0.0);
  const double dz = fmax(fs - fmin(f * zm, f * zp), 0.0);
  const double g2 = dx * dx + dy * dy + dz * dz;
  const double upd = sc - dtau * sg * (root(g2) * ih - 1.0);
  return sg == 0.0 ? sc : upd;
}

// STEPS pseudo-steps of the reinitialisation in one launch.  A lane holds
// kRR rows of a column and marches up kz planes, so a plane's neighbours
// along z and most along y are in registers, and the next plane's values are
// loaded a plane ahead.  With two steps the first one's result of the last
// two planes is in LDS for the second (the block's outer ring of cells only
// feeds it); the sign of sigma0 is taken once for both.  The one-cell form is
// bound by its 270 instructions per cell (a root and a division for the sign,
// a root for the gradient) and at 512 x 256 x 256 by its 24 bytes; 301 x 125 x
// 131 (23 us a step at the copy rate): five steps 194 -> 121 us, 512 x 256 x
// 256: 1130 -> 790 us.
template <int STEPS, bool FIRST>
__global__ void __launch_bounds__(64 * kRW) k_reinit_march(Phys P, const double* __restrict__ s0,
                                                         const double* __restrict__ cur, double* __restrict__ nxt,
                                                         double dtau, int kz) {
  constexpr int H = STEPS - 1, R = kRR, kRows = kRW * R;
  __shared__ double lds[STEPS == 2 ? 2 * kRows * 64 : 1];
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int lane = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int i = tl.x * (64 - 2 * H) - H + lane;
  const int j0 = tl.y * (kRows - 2 * H) - H + wv * R;
  const int kb = tl.z * kz, ke = min(kb + kz, n.nz);
  const int sxy = n.nx * n.ny;
  const double h = P.h, h2 = h * h, ih = 1.0 / h;
  const int ic = clampi(i, 0, n.nx - 1), im = max(ic - 1, 0), ip = min(ic + 1, n.nx - 1);
  // byte offsets in a plane (32 bits: a load's base is then a scalar): of the
  // lane's cell in its rows and the rows beside them; of its neighbours along x
  unsigned row[R + 2];
#pragma unroll
  for (int r = 0; r < R + 2; ++r) row[r] = 8u * (unsigned)(n.nx * clampi(j0 + r - 1, 0, n.ny - 1) + ic);
  const int om = 8 * (im - ic), op = 8 * (ip - ic);
  auto at = [](const double* plane, unsigned off) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(plane) + off);
  };
  double cm[R], cc[R], cp[R], a0[R], xm[R], xp[R], ym, yp;
  double sm[R], s1[R], g1[R];   // the first step's result two and one planes down, and its sign
  auto centre = [&](int k, double (&o)[R]) {
    const double* q = cur + (size_t)sxy * clampi(k, 0, n.nz - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] = at(q, row[r + 1]);
  };
  auto beside = [&](int k, double (&m)[R], double (&pl)[R], double& lo, double& hi, double (&a)[R]) {
    const double* q = cur + (size_t)sxy * clampi(k, 0, n.nz - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      m[r] = at(q, row[r + 1] + om);
      pl[r] = at(q, row[r + 1] + op);
    }
    lo = at(q, row[0]);
    hi = at(q, row[R + 1]);
    if (!FIRST) {
      const double* z = s0 + (size_t)sxy * clampi(k, 0, n.nz - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = at(z, row[r + 1]);
    }
  };
  const int p0 = max(kb - H, 0), p1 = ke - 1 + H;   // the first step's planes (the last may lie above the top)
  centre(p0 - 1, cm);
  centre(p0, cc);
  centre(p0 + 1, cp);
  beside(p0, xm, xp, ym, yp, a0);
  auto put = [&](int k, int r, double v) {
    *reinterpret_cast<double*>(reinterpret_cast<char*>(nxt + (size_t)sxy * k) + row[r + 1]) = v;
  };
  const bool outx = i < n.nx && (H == 0 || (lane > 0 && lane < 63));
  const int lm = lane - (i > 0 ? 1 : 0), lp = lane + (i < n.nx - 1 ? 1 : 0);
  const int lrow = wv * R;
#pragma unroll 2
  for (int p = p0; p <= p1; ++p) {
    double cn[R], an[R], xmn[R], xpn[R], ymn, ypn;
    double u[R], sg[R];
    if (STEPS == 1 || p < n.nz) {
      centre(p + 2, cn);
      beside(p + 1, xmn, xpn, ymn, ypn, an);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double a = FIRST ? cc[r] : a0[r];
        sg[r] = over_root(a, a * a + h2);
        u[r] = reinit_cell(cc[r], sg[r], xm[r], xp[r], r > 0 ? cc[r - 1] : ym, r < R - 1 ? cc[r + 1] : yp, cm[r], cp[r],
                           dtau, ih);
      }
    }
    if constexpr (STEPS == 1) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (outx && j0 + r < n.ny) put(p, r, u[r]);
    } else {
      if (p == n.nz) {   // above the top: the top plane's values
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = s1[r];
      } else if (p == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) s1[r] = u[r];   // (below the bed: the bottom plane's)
      }
      double* w = lds + (p & 1) * kRows * 64;
      const double* b = lds + ((p - 1) & 1) * kRows * 64;
      if (p < ke) {
#pragma unroll
        for (int r = 0; r < R; ++r) w[(lrow + r) * 64 + lane] = u[r];
      }
      if (p > kb) {   // the second step, on plane p - 1
        const int jm = j0 > 0 ? max(lrow - 1, 0) : lrow;
        const double lo = b[jm * 64 + lane], hi = b[min(lrow + R, kRows - 1) * 64 + lane];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int y = j0 + r, lr = lrow + r;
          const double vm = b[lr * 64 + max(lm, 0)], vp = b[lr * 64 + min(lp, 63)];
          const double wm = y > 0 ? (r > 0 ? s1[r - 1] : lo) : s1[r];
          const double wp = y < n.ny - 1 ? (r < R - 1 ? s1[r + 1] : hi) : s1[r];
          const double o = reinit_cell(s1[r], g1[r], vm, vp, wm, wp, sm[r], u[r], dtau, ih);
          if (outx && y >= 0 && y < n.ny && lr > 0 && lr < kRows - 1) put(p - 1, r, o);
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < R; ++r) {
        sm[r] = s1[r];
        s1[r] = u[r];
        g1[r] = sg[r];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      cm[r] = cc[r];
      cc[r] = cp[r];
      cp[r] = cn[r];
      a0[r] = an[r];
      xm[r] = xmn[r];
      xp[r] = xpn[r];
    }
    ym = ymn;
    yp = ypn;
  }
}

// All of a 2-D tank's pseudo-steps (up to kR2 of them) in one launch: a block
// takes a tile of 64 x 16 cells with a ring of as many cells as there are steps,
// which each step leaves one cell less of, in two LDS planes; the sign of
// sigma0 is taken once.  A step by itself is a 3 us launch (256 x 64 to 640 x
// 96): five of them 14.7 -> 8.9 us; with the advection 174 -> 116 us on 4096 x
// 1024 cells and 378 -> 283 on 8192 x 1024, the largest timed.
constexpr int kR2 = 5, kR2X = 64, kR2Z = 16, kR2Row = kR2X + 2 * kR2, kR2N = kR2Row * (kR2Z + 2 * kR2);
constexpr int kR2T = 512, kR2C = (kR2N + kR2T - 1) / kR2T;
__global__ void __launch_bounds__(kR2T) k_reinit2d(Phys P, const double* __restrict__ s0, const double* __restrict__ cur,
                                                   double* __restrict__ nxt, double dtau, int steps) {
  __shared__ double lds[2][kR2N];
  const int nx = P.n.nx, nz = P.n.nz;
  const int x0 = blockIdx.x * kR2X - kR2, z0 = blockIdx.y * kR2Z - kR2;
  const double h = P.h, ih = 1.0 / h;
  double sg[kR2C], sc[kR2C];
  int gi[kR2C], gk[kR2C];
#pragma unroll
  for (int q = 0; q < kR2C; ++q) {
    const int e = min((int)threadIdx.x + q * kR2T, kR2N - 1);
    gi[q] = x0 + e % kR2Row;
    gk[q] = z0 + e / kR2Row;
    const int c = clampi(gi[q], 0, nx - 1) + nx * clampi(gk[q], 0, nz - 1);
    const double a = s0[c];
    sc[q] = cur[c];
    sg[q] = a / sqrt(a * a + h * h);
  }
#pragma unroll
  for (int q = 0; q < kR2C; ++q)
    if ((int)threadIdx.x + q * kR2T < kR2N) lds[0][threadIdx.x + q * kR2T] = sc[q];
  __syncthreads();
#pragma unroll 1
  for (int t = 0; t < steps; ++t) {
    const double* b = lds[t & 1];
#pragma unroll
    for (int q = 0; q < kR2C; ++q) {
      // (the ring's own edge reads itself: what it holds is not used)
      const int e = min((int)threadIdx.x + q * kR2T, kR2N - 1);
      const int w = gi[q] > 0 && e > 0 ? e - 1 : e, ea = gi[q] < nx - 1 && e < kR2N - 1 ? e + 1 : e;
      const int d = gk[q] > 0 && e >= kR2Row ? e - kR2Row : e, up = gk[q] < nz - 1 && e < kR2N - kR2Row ? e + kR2Row : e;
      sc[q] = reinit_cell(sc[q], sg[q], b[w], b[ea], sc[q], sc[q], b[d], b[up], dtau, ih);
    }
#pragma unroll
    for (int q = 0; q < kR2C; ++q)
      if ((int)threadIdx.x + q * kR2T < kR2N) lds[1 - (t & 1)][threadIdx.x + q * kR2T] = sc[q];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < kR2C; ++q) {
    const int i = gi[q] - x0 - kR2, k = gk[q] - z0 - kR2;
    if ((int)threadIdx.x + q * kR2T < kR2N && i >= 0 && i < kR2X && k >= 0 && k < kR2Z && gi[q] < nx && gk[q] < nz)
      nxt[gi[q] + nx * gk[q]] = sc[q];
  }
}

__global__ void k_copy(const double* __restrict__ a, double* __restrict__ b, size_t n) {
  size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) b[q] = a[q];
}

// --------------------------------------------------------------------------
// properties at cell centres: two-stage Heaviside blend (flowing phases by
// sigma, then the solid by psi); chi = 1 - H_body.
// --------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_props(Phys P, const double* __restrict__ sigma, double t,
                                               double* __restrict__ rho, double* __restrict__ rfl,
                                               double* __restrict__ mu, double* __restrict__ chi) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const size_t c = i + (size_t)n.nx * (j + (size_t)n.ny * k);
  double zd;
  const double psi = body_psi(P, (i + 0.5) * P.h, (j + 0.5) * P.h, (k + 0.5) * P.h, t, &zd);
  const double hf = heaviside(sigma[c], P.eps);
  const double hb = heaviside(psi, P.eps);
  const double rf = P.rho_w + (P.rho_a - P.rho_w) * hf;
  const double mf = P.mu_w + (P.mu_a - P.mu_w) * hf;
  rfl[c] = rf;
  rho[c] = P.rho_s + (rf - P.rho_s) * hb;
  mu[c] = P.mu_s + (mf - P.mu_s) * hb;
  chi[c] = 1.0 - hb;
}

// --------------------------------------------------------------------------
// momentum predictor for velocity component C (faces normal to C)
// --------------------------------------------------------------------------
// Viscous stress of component C along direction D at a face,
// ((tau_+) - (tau_-))/h: tau = 2 mu du_C/dx_C at the cell centres either side
// (D = C), else mu (du_C/dx_D + du_D/dx_C) on the edges either side with the
// mean of their four cell viscosities.  m1, p1: the face's neighbours along D;
// dvp, dvm: du_D/dx_C on the two edges.  *a (if not null) receives the
// magnitude of the coefficient of the face's own value.
template <int C, int D, typename T = double>
__device__ __forceinline__ T visc_stress(const double* __restrict__ mu, const Dims& n, int i, int j, int k,
                                              T uf, T m1, T p1, T dvp, T dvm, double ih,
                                              T* a) {
  constexpr int ci = (C == 0), cj = (C == 1), ck = (C == 2);
  constexpr int di = (D == 0), dj = (D == 1), dk = (D == 2);
  T tp, tm;
  if constexpr (C == D) {
    const T mup = cvt<T, 0>(mu, n, i, j, k), mum = cvt<T, -ci>(mu, n, i, j - cj, k - ck);
    tp = 2.0 * mup * (p1 - uf) * ih;
    tm = 2.0 * mum * (uf - m1) * ih;
    if (a) *a = 2.0 * (mup + mum) * ih * ih;
  } else {
    const T mep = 0.25 * (cvt<T, -ci>(mu, n, i, j - cj, k - ck) + cvt<T, 0>(mu, n, i, j, k) +
                               cvt<T, -ci + di>(mu, n, i, j - cj + dj, k - ck + dk) +
                               cvt<T, di>(mu, n, i, j + dj, k + dk));
    const T mem = 0.25 * (cvt<T, -ci - di>(mu, n, i, j - cj - dj, k - ck - dk) +
                               cvt<T, -di>(mu, n, i, j - dj, k - dk) + cvt<T, -ci>(mu, n, i, j - cj, k - ck) +
                               cvt<T, 0>(mu, n, i, j, k));
    tp = mep * ((p1 - uf) * ih + dvp);
    tm = mem * ((uf - m1) * ih + dvm);
    if (a) *a = (mep + mem) * ih * ih;
  }
  return (tp - tm) * ih;
}

// One direction D of the predictor of component C: advection (advective
// form), viscous stress, and with CONS the consistent transport's mass flux
// (Koren-limited upwind face density at t^n times the advecting velocity)
// and the momentum it carries (times the same upwind velocity).
template <int C, int D, bool CONS, typename T>
__device__ __forceinline__ void mom_dir(const double* __restrict__ uc, const double* __restrict__ ud,
                                        const double* __restrict__ mu, const double* __restrict__ rho_n,
                                        const Dims& n, int i, int j, int k, T uf, double ih, T& adv,
                                        T& visc, T& conv, T& mflux) {
  constexpr int ci = (C == 0), cj = (C == 1), ck = (C == 2);
  constexpr int di = (D == 0), dj = (D == 1), dk = (D == 2);
  const T m2 = fvt<C, T, -2 * di>(uc, n, i, j - 2 * dj, k - 2 * dk);
  const T m1 = fvt<C, T, -di>(uc, n, i, j - dj, k - dk);
  const T p1 = fvt<C, T, di>(uc, n, i, j + dj, k + dk);
  const T p2 = fvt<C, T, 2 * di>(uc, n, i, j + 2 * dj, k + 2 * dk);
  T ap, am, dvp{}, dvm{};
  if constexpr (C == D) {
    ap = 0.5 * (uf + p1);
    am = 0.5 * (m1 + uf);
  } else {
    // transverse velocity on the two faces meeting the edge above / below
    const T vpp = fvt<D, T, di>(ud, n, i, j + dj, k + dk);
    const T vpm = fvt<D, T, di - ci>(ud, n, i, j + dj - cj, k + dk - ck);
    const T vmp = fvt<D, T, 0>(ud, n, i, j, k);
    const T vmm = fvt<D, T, -ci>(ud, n, i, j - cj, k - ck);
    ap = 0.5 * (vpm + vpp);
    am = 0.5 * (vmm + vmp);
    dvp = (vpp - vpm) * ih;
    dvm = (vmp - vmm) * ih;
  }
  const T vp = koren_face(ap, m1, uf, p1, p2);
  const T vm = koren_face(am, m2, m1, uf, p1);
  if constexpr (!CONS) adv += ap * (vp - uf) - am * (vm - uf);
  if constexpr (CONS) {
    // face density at t^n of the face o steps along D: mean of its two cells
    auto rf = [&](auto oc) {
      constexpr int o = decltype(oc)::value;
      return 0.5 * (cvt<T, -ci + o * di>(rho_n, n, i, j - cj + o * dj, k - ck + o * dk) +
                    cvt<T, o * di>(rho_n, n, i, j + o * dj, k + o * dk));
    };
    const T rm2 = rf(std::integral_constant<int, -2>{}), rm1 = rf(std::integral_constant<int, -1>{});
    const T r0 = rf(std::integral_constant<int, 0>{}), rp1 = rf(std::integral_constant<int, 1>{});
    const T rp2 = rf(std::integral_constant<int, 2>{});
    const T mp = ap * koren_face(ap, rm1, r0, rp1, rp2);
    const T mm = am * koren_face(am, rm2, rm1, r0, rp1);
    conv += mp * vp - mm * vm;
    mflux += mp - mm;
    settle(conv);
    settle(mflux);
  } else {
    settle(adv);
  }
  visc += visc_stress<C, D, T>(mu, n, i, j, k, uf, m1, p1, dvp, dvm, ih, (T*)nullptr);
  settle(visc);
}

// The predictor of component C.  CONS: the conservative form with
// consistent mass/momentum transport, from the cell density rho_n at t^n:
// (rb u* - rho^n_f u^n)/dt + conv/h = forces, rb = rho^n_f - dt mflux/h, and
// beta from rb; otherwise the advective form with rho_f at t^{n+1}.
// A wall's face f of it:
template <int C>
__device__ __forceinline__ void mom_wall(const Phys& P, int i, int k, unsigned f, double t1, double* __restrict__ out,
                                         double* __restrict__ beta, float* __restrict__ betaf,
                                         double* __restrict__ cn_rhs, double* __restrict__ cn_diag) {
  // the inlet of a wave tank carries the generated wave's velocity
  out[f] = (C == 0 && i == 0 && P.gen_len > 0.0) ? tank_vel(P, 0, 0.0, (k + 0.5) * P.h, t1) : 0.0;
  beta[f] = 0.0;
  betaf[f] = 0.0f;
  if (cn_rhs) {
    cn_rhs[f] = 0.0;
    cn_diag[f] = 0.0;   // marks a face the Crank-Nicolson sweeps keep
  }
}
// and any other, from its sums over the directions: advection and mass flux
// (times h), viscous stress, momentum flux (times h); r0, rff, xf: the face's
// density (CONS: at t^n), flowing density (C = 2) and solid fraction; damp: the
// row's damping coefficient
struct MomFace {
  double u, beta, num, den;
};
template <int C, bool CONS>
__device__ __forceinline__ MomFace mom_face(const Phys& P, double uf, double r0, double rff,
                                            double xf, double adv, double visc, double conv, double mflux, double damp,
                                            double ub, double dt, bool cn, double* __restrict__ flag) {
  const double ih = 1.0 / P.h;
  const double grav = (C == 2) ? -P.g * rff : 0.0;
  const double pen = xf * P.inv_kp;
  // Crank-Nicolson keeps half the viscous term at t^n on the right-hand side
  // and writes the first iterate of its sweeps (the explicit value)
  const double wv = cn ? 0.5 : 1.0;
  MomFace m;
  if constexpr (CONS) {
    const double rb = r0 - dt * mflux * ih;
    // a carried density at or below zero makes the projection operator
    // indefinite: the step is past the transport's Courant bound
    if (!(rb > 0.0)) *flag = 1.0;
    m.num = r0 * uf / dt - conv * ih + wv * visc + grav + pen * ub;
    m.den = rb / dt + pen + damp;
    m.beta = 1.0 / (rb + P.pen_w * dt * pen);
  } else {
    m.num = r0 * (uf / dt - adv * ih) + wv * visc + grav + pen * ub;
    m.den = r0 / dt + pen + damp;
    m.beta = 1.0 / (r0 + P.pen_w * dt * pen);
  }
  m.u = cn ? (m.num + 0.5 * visc) / m.den : m.num / m.den;
  return m;
}
// (the nearest body's heave velocity, at a z-face)
template <int C>
__device__ __forceinline__ double mom_heave(const Phys& P, int i, int j, int k, double t1) {
  double ub = 0.0;
  if (C == 2 && P.nb > 0) body_psi(P, (i + 0.5) * P.h, (j + 0.5) * P.h, k * P.h, t1, &ub);
  return ub;
}
template <int C>
__device__ __forceinline__ double mom_damp(const Phys& P, int k, double dt) {
  return vort_coeff(P, (C == 2) ? k * P.h : (k + 0.5) * P.h, dt);   // -g u, implicit
}

template <int C, bool CONS>
__device__ __forceinline__ void mom_point(const Phys& P, int i, int j, int k, const double* __restrict__ u,
                                                  const double* __restrict__ v,
                                                  const double* __restrict__ w,
                                                  const double* __restrict__ rho,
                                                  const double* __restrict__ rfl,
                                                  const double* __restrict__ mu,
                                                  const double* __restrict__ chi,
                                                  const double* __restrict__ rho_n, double dt, double t1,
                                                  double* __restrict__ out, double* __restrict__ beta,
                                                  float* __restrict__ betaf, double* __restrict__ cn_rhs,
                                                  double* __restrict__ cn_diag, double* __restrict__ flag) {
  const Dims n = P.n;
  constexpr int ci = (C == 0), cj = (C == 1), ck = (C == 2);
  const int mx = n.nx + ci, my = n.ny + cj, mz = n.nz + ck;
  if (i >= mx || j >= my || k >= mz) return;
  const size_t f = i + (size_t)mx * (j + (size_t)my * k);
  const bool wall = (C == 0) ? (i == 0 || i == n.nx) : (C == 1) ? (j == 0 || j == n.ny) : (k == 0);
  if (wall) {
    mom_wall<C>(P, i, k, (unsigned)f, t1, out, beta, betaf, cn_rhs, cn_diag);
    return;
  }
  const double* uc = (C == 0) ? u : (C == 1) ? v : w;
  const double uf = uc[f];
  const double ih = 1.0 / P.h;
  double adv = 0.0, visc = 0.0, conv = 0.0, mflux = 0.0;
  mom_dir<C, 0, CONS>(uc, u, mu, rho_n, n, i, j, k, uf, ih, adv, visc, conv, mflux);
  mom_dir<C, 1, CONS>(uc, v, mu, rho_n, n, i, j, k, uf, ih, adv, visc, conv, mflux);
  mom_dir<C, 2, CONS>(uc, w, mu, rho_n, n, i, j, k, uf, ih, adv, visc, conv, mflux);
  const double r0 = CONS ? 0.5 * (cv(rho_n, n, i - ci, j - cj, k - ck) + cv(rho_n, n, i, j, k))
                         : 0.5 * (cv(rho, n, i - ci, j - cj, k - ck) + cv(rho, n, i, j, k));
  const double rff = C == 2 ? 0.5 * (cv(rfl, n, i - ci, j - cj, k - ck) + cv(rfl, n, i, j, k)) : 0.0;
  const double xf = 0.5 * (cv(chi, n, i - ci, j - cj, k - ck) + cv(chi, n, i, j, k));
  const MomFace m = mom_face<C, CONS>(P, uf, r0, rff, xf, adv, visc, conv, mflux, mom_damp<C>(P, k, dt),
                                      mom_heave<C>(P, i, j, k, t1), dt, cn_rhs != nullptr, flag);
  out[f] = m.u;
  beta[f] = m.beta;
  betaf[f] = (float)m.beta;
  if (cn_rhs) {
    cn_rhs[f] = m.num;
    cn_diag[f] = m.den;
  }
}
// The three components in one launch: the first third of the blocks along x
// takes the x-faces, then the y- and the z-faces (along x, where a launch may
// have 2^31 blocks: three times a tall tank's planes would pass the 65536 of z)
struct MomOut {
  double* u[3];
  double* beta[3];
  float* betaf[3];
  double* rhs[3];
  double* diag[3];
};
template <bool CONS>
__global__ void __launch_bounds__(256) k_momentum(Phys P, const double* __restrict__ u, const double* __restrict__ v,
                                                  const double* __restrict__ w, const double* __restrict__ rho,
                                                  const double* __restrict__ rfl, const double* __restrict__ mu,
                                                  const double* __restrict__ chi, const double* __restrict__ rho_n,
                                                  double dt, double t1, MomOut O, double* __restrict__ flag) {
  const int nb = gridDim.x / 3, C = blockIdx.x / nb;
  const int i = (blockIdx.x - C * nb) * 64 + threadIdx.x;
  const int j = blockIdx.y * blockDim.y + __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int k = blockIdx.z * blockDim.z + __builtin_amdgcn_readfirstlane(threadIdx.z);
  if (C == 0)
    mom_point<0, CONS>(P, i, j, k, u, v, w, rho, rfl, mu, chi, rho_n, dt, t1, O.u[0], O.beta[0], O.betaf[0], O.rhs[0],
                       O.diag[0], flag);
  else if (C == 1)
    mom_point<1, CONS>(P, i, j, k, u, v, w, rho, rfl, mu, chi, rho_n, dt, t1, O.u[1], O.beta[1], O.betaf[1], O.rhs[1],
                       O.diag[1], flag);
  else
    mom_point<2, CONS>(P, i, j, k, u, v, w, rho, rfl, mu, chi, rho_n, dt, t1, O.u[2], O.beta[2], O.betaf[2], O.rhs[2],
                       O.diag[2], flag);
}

// One component, its tiles in the XCD order: larger grids of short rows
template <int C, bool CONS>
__global__ void __launch_bounds__(256) k_momentum_face(Phys P, const double* __restrict__ u,
                                                       const double* __restrict__ v, const double* __restrict__ w,
                                                       const double* __restrict__ rho, const double* __restrict__ rfl,
                                                       const double* __restrict__ mu, const double* __restrict__ chi,
                                                       const double* __restrict__ rho_n, double dt, double t1,
                                                       double* __restrict__ out, double* __restrict__ beta,
                                                       float* __restrict__ betaf, double* __restrict__ cn_rhs,
                                                       double* __restrict__ cn_diag, double* __restrict__ flag) {
  const Tile tl = xcd_tile();
  mom_point<C, CONS>(P, tl.x * blockDim.x + threadIdx.x, tl.y * blockDim.y + threadIdx.y,
                     tl.z * blockDim.z + threadIdx.z, u, v, w, rho, rfl, mu, chi, rho_n, dt, t1, out, beta, betaf,
                     cn_rhs, cn_diag, flag);
}

// The same for larger grids, two faces along x per lane (V2): half the accesses,
// which bound the one-face form (55 to 59 of them per face, the address unit busy
// 85% of the time), and the rows' arithmetic on scalars.  256 x 128 x 128, the
// three components with consistent transport (3 x 56 us for the bytes at the
// copy rate): 481 -> 352 us, advective 345 -> 272; 512 x 256 x 256 3.72 -> 2.55 ms.
// (The last x-face of a row, a wall, is written with the one before it, so that
// every component's row is nx wide.)
template <int C, bool CONS>
__global__ void __launch_bounds__(256, 4) k_momentum_pair(
    Phys P, const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    const double* __restrict__ rho, const double* __restrict__ rfl, const double* __restrict__ mu,
    const double* __restrict__ chi, const double* __restrict__ rho_n, double dt, double t1, double* __restrict__ out,
    double* __restrict__ beta, float* __restrict__ betaf, double* __restrict__ cn_rhs, double* __restrict__ cn_diag,
    double* __restrict__ flag) {
  const Dims n = P.n;
  constexpr int ci = (C == 0), cj = (C == 1), ck = (C == 2);
  const int mx = n.nx + ci, my = n.ny + cj, mz = n.nz + ck;
  const Tile tl = xcd_tile();
  // (a wavefront lies in one row)
  const int i = 2 * (tl.x * 64 + threadIdx.x);
  const int j = tl.y * blockDim.y + __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int k = tl.z * blockDim.z + __builtin_amdgcn_readfirstlane(threadIdx.z);
  if (i >= n.nx || j >= my || k >= mz) return;
  const unsigned f = (unsigned)(i + mx * (j + my * k));
  const bool wall = (C == 1) ? (j == 0 || j == n.ny) : (C == 2) ? k == 0 : false;   // (the row is)
  // (before the stencil, whose registers their library functions would add to)
  const double damp = mom_damp<C>(P, k, dt);
  const double ub0 = mom_heave<C>(P, i, j, k, t1), ub1 = mom_heave<C>(P, i + 1, j, k, t1);
  __builtin_amdgcn_sched_barrier(0);
  MomFace m[2];
  if (wall) {
    m[0] = m[1] = MomFace{0.0, 0.0, 0.0, 0.0};
  } else {
    const double* uc = (C == 0) ? u : (C == 1) ? v : w;
    const V2 uf = fvt<C, V2, 0>(uc, n, i, j, k);
    const double ih = 1.0 / P.h;
    V2 adv{}, visc{}, conv{}, mflux{};
    mom_dir<C, 0, CONS>(uc, u, mu, rho_n, n, i, j, k, uf, ih, adv, visc, conv, mflux);
    mom_dir<C, 1, CONS>(uc, v, mu, rho_n, n, i, j, k, uf, ih, adv, visc, conv, mflux);
    mom_dir<C, 2, CONS>(uc, w, mu, rho_n, n, i, j, k, uf, ih, adv, visc, conv, mflux);
    auto mean = [&](const double* a) {
      return 0.5 * (cvt<V2, -ci>(a, n, i, j - cj, k - ck) + cvt<V2, 0>(a, n, i, j, k));
    };
    const V2 r0 = mean(CONS ? rho_n : rho), xf = mean(chi);
    const V2 rff = C == 2 ? mean(rfl) : V2{};
    const bool cn = cn_rhs != nullptr;
    // (a face that is a wall or past the row raises no flag)
    const bool ok0 = C != 0 || i > 0, ok1 = i + 1 < n.nx;
    m[0] = mom_face<C, CONS>(P, uf.x, ok0 ? r0.x : 1.0, rff.x, xf.x, adv.x, visc.x, conv.x, ok0 ? mflux.x : 0.0,
                             damp, ub0, dt, cn, flag);
    m[1] = mom_face<C, CONS>(P, uf.y, ok1 ? r0.y : 1.0, rff.y, xf.y, adv.y, visc.y, conv.y,
                             ok1 ? mflux.y : 0.0, damp, ub1, dt, cn, flag);
    if (C == 0 && i == 0)   // the inlet of a wave tank carries the generated wave's velocity
      m[0] = MomFace{P.gen_len > 0.0 ? tank_vel(P, 0, 0.0, (k + 0.5) * P.h, t1) : 0.0, 0.0, 0.0, 0.0};
  }
  const bool two = i + 1 < n.nx;
  if (two) {
    *reinterpret_cast<V2Mem*>(out + f) = V2Mem{m[0].u, m[1].u};
    *reinterpret_cast<V2Mem*>(beta + f) = V2Mem{m[0].beta, m[1].beta};
    *reinterpret_cast<F2Mem*>(betaf + f) = F2Mem{(float)m[0].beta, (float)m[1].beta};
    if (cn_rhs) {
      *reinterpret_cast<V2Mem*>(cn_rhs + f) = V2Mem{m[0].num, m[1].num};
      *reinterpret_cast<V2Mem*>(cn_diag + f) = V2Mem{m[0].den, m[1].den};
    }
  } else {
    out[f] = m[0].u;
    beta[f] = m[0].beta;
    betaf[f] = (float)m[0].beta;
    if (cn_rhs) {
      cn_rhs[f] = m[0].num;
      cn_diag[f] = m[0].den;
    }
  }
  if (C == 0 && i + 2 >= n.nx) mom_wall<0>(P, n.nx, k, f + (two ? 2u : 1u), t1, out, beta, betaf, cn_rhs, cn_diag);
}

// Viscous stress of component C along D from the iterate, with its diagonal.
template <int C, int D, typename T>
__device__ __forceinline__ void sweep_dir(const double* __restrict__ uc, const double* __restrict__ ud,
                                          const double* __restrict__ mu, const Dims& n, int i, int j, int k,
                                          T uf, double ih, T& L, T& a) {
  constexpr int ci = (C == 0), cj = (C == 1), ck = (C == 2);
  constexpr int di = (D == 0), dj = (D == 1), dk = (D == 2);
  const T m1 = fvt<C, T, -di>(uc, n, i, j - dj, k - dk);
  const T p1 = fvt<C, T, di>(uc, n, i, j + dj, k + dk);
  T dvp{}, dvm{};
  if constexpr (C != D) {
    dvp = (fvt<D, T, di>(ud, n, i, j + dj, k + dk) - fvt<D, T, di - ci>(ud, n, i, j + dj - cj, k + dk - ck)) * ih;
    dvm = (fvt<D, T, 0>(ud, n, i, j, k) - fvt<D, T, -ci>(ud, n, i, j - cj, k - ck)) * ih;
  }
  T ad;
  L += visc_stress<C, D, T>(mu, n, i, j, k, uf, m1, p1, dvp, dvm, ih, &ad);
  a += ad;
  settle(L);
  settle(a);
}

// Largest value over a 256-thread block (64 x 4 or 64 x 1 x 4), two
// quantities at once; thread 0 returns them.
__device__ __forceinline__ void block_max2(double& a, double& b) {
  for (int off = 32; off > 0; off >>= 1) {
    a = fmax(a, __shfl_down(a, off, 64));
    b = fmax(b, __shfl_down(b, off, 64));
  }
  __shared__ double sm[4][2];
  const int tid = threadIdx.x + 64 * (threadIdx.y + blockDim.y * threadIdx.z);
  if ((tid & 63) == 0) {
    sm[tid >> 6][0] = a;
    sm[tid >> 6][1] = b;
  }
  __syncthreads();
  if (tid == 0) {
    a = fmax(fmax(sm[0][0], sm[1][0]), fmax(sm[2][0], sm[3][0]));
    b = fmax(fmax(sm[0][1], sm[1][1]), fmax(sm[2][1], sm[3][1]));
  }
}

// One point-Jacobi sweep of the Crank-Nicolson viscous system of component C,
//   D_f u_f - 1/2 L(u)_f = rhs_f,
// from the iterate (u, v, w): u_f <- (rhs_f + 1/2 (L(u)_f + a_f u_f)) / (D_f + 1/2 a_f),
// a_f the magnitude of L's diagonal; a face with D_f = 0 (a wall or the
// inlet) keeps its value.  With part, the block's largest |u_new - u| and
// largest |u_new| over the faces it updates go to part[2 lin], part[2 lin + 1].
// Larger grids take two faces along x per lane (T = V2), a row then nx wide: the
// last x-face of a row, a wall, goes with the one before it.
template <int C, typename T>
__global__ void __launch_bounds__(256) k_cn_sweep(Phys P, const double* __restrict__ u,
                                                  const double* __restrict__ v,
                                                  const double* __restrict__ w,
                                                  const double* __restrict__ mu,
                                                  const double* __restrict__ rhs,
                                                  const double* __restrict__ diag, double* __restrict__ out,
                                                  double* __restrict__ part) {
  const Dims n = P.n;
  constexpr int ci = (C == 0), cj = (C == 1), ck = (C == 2);
  const int mx = n.nx + ci, my = n.ny + cj, mz = n.nz + ck;
  const double* uc = (C == 0) ? u : (C == 1) ? v : w;
  const Tile tl = xcd_tile();
  double du = 0.0, um = 0.0;
  if constexpr (std::is_same_v<T, double>) {
    const int i = tl.x * blockDim.x + threadIdx.x;
    const int j = tl.y * blockDim.y + threadIdx.y;
    const int k = tl.z * blockDim.z + threadIdx.z;
    if (i < mx && j < my && k < mz) {
      const size_t f = i + (size_t)mx * (j + (size_t)my * k);
      const double uf = uc[f], dg = diag[f];
      double nv = uf;
      if (dg != 0.0) {
        const double ih = 1.0 / P.h;
        double L = 0.0, a = 0.0;
        sweep_dir<C, 0, T>(uc, u, mu, n, i, j, k, uf, ih, L, a);
        sweep_dir<C, 1, T>(uc, v, mu, n, i, j, k, uf, ih, L, a);
        sweep_dir<C, 2, T>(uc, w, mu, n, i, j, k, uf, ih, L, a);
        nv = (rhs[f] + 0.5 * (L + a * uf)) / (dg + 0.5 * a);
        du = fabs(nv - uf);
        um = fabs(nv);
      }
      out[f] = nv;
    }
  } else {
    const int i = 2 * (tl.x * 64 + threadIdx.x);
    const int j = tl.y * blockDim.y + __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int k = tl.z * blockDim.z + __builtin_amdgcn_readfirstlane(threadIdx.z);
    if (i < n.nx && j < my && k < mz) {
      const unsigned f = (unsigned)(i + mx * (j + my * k));
      const bool two = i + 1 < n.nx;
      const T uf = fvt<C, T, 0>(uc, n, i, j, k);
      const double dg[2] = {diag[f], two ? diag[f + 1] : 0.0};
      auto update = [&](double u0, double d0, double r0, double L, double a) {
        const double nv = (r0 + 0.5 * (L + a * u0)) / (d0 + 0.5 * a);
        if (d0 == 0.0) return u0;
        du = fmax(du, fabs(nv - u0));
        um = fmax(um, fabs(nv));
        return nv;
      };
      if (dg[0] != 0.0 || dg[1] != 0.0) {
        const double ih = 1.0 / P.h;
        T L{}, a{};
        sweep_dir<C, 0, T>(uc, u, mu, n, i, j, k, uf, ih, L, a);
        sweep_dir<C, 1, T>(uc, v, mu, n, i, j, k, uf, ih, L, a);
        sweep_dir<C, 2, T>(uc, w, mu, n, i, j, k, uf, ih, L, a);
        const double nx = update(uf.x, dg[0], rhs[f], L.x, a.x);
        if (two)
          *reinterpret_cast<V2Mem*>(out + f) = V2Mem{nx, update(uf.y, dg[1], rhs[f + 1], L.y, a.y)};
        else
          out[f] = nx;
      } else {
        out[f] = uf.x;
        if (two) out[f + 1] = uf.y;
      }
      if (C == 0 && i + 2 >= n.nx) {
        const unsigned fw = f + (two ? 2u : 1u);
        out[fw] = uc[fw];
      }
    }
  }
  if (!part) return;
  block_max2(du, um);
  if (threadIdx.x == 0 && threadIdx.y == 0 && threadIdx.z == 0) {
    part[2 * (size_t)tl.lin] = du;
    part[2 * (size_t)tl.lin + 1] = um;
  }
}

// The CFL rule's per-block maximum of |u_c| + |v_c| + |w_c|, each cell
// velocity the mean of its two faces; a value that is not finite counts as
// infinite (a maximum would otherwise drop a NaN).
__global__ void __launch_bounds__(256) k_cfl(Phys P, const double* __restrict__ u, const double* __restrict__ v,
                                             const double* __restrict__ w, double* __restrict__ partials) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  double m = 0.0, unused = 0.0;
  if (i < n.nx && j < n.ny && k < n.nz) {
    const size_t sxy = (size_t)n.nx * n.ny;
    const size_t c = i + (size_t)n.nx * j + sxy * k;
    const size_t fu = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
    const size_t fvv = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
    const double uc = 0.5 * fabs(u[fu] + u[fu + 1]);
    const double vc = 0.5 * fabs(v[fvv] + v[fvv + n.nx]);
    const double wc = 0.5 * fabs(w[c] + w[c + sxy]);
    const double sum = (uc + vc) + wc;
    m = isfinite(sum) ? sum : INFINITY;
  }
  block_max2(m, unused);
  if (threadIdx.x + threadIdx.y + threadIdx.z == 0) partials[tl.lin] = m;
}

// out[q] = max over p of partials[K p + q], q < K (one 1024-thread block)
template <int K>
__global__ void __launch_bounds__(1024) k_max_finalize(const double* __restrict__ partials, int nparts,
                                                       double* __restrict__ out) {
  double m[2] = {0.0, 0.0};
  for (int p = threadIdx.x; p < nparts; p += 1024)
#pragma unroll
    for (int q = 0; q < K; ++q) m[q] = fmax(m[q], partials[(size_t)K * p + q]);
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < K; ++q) m[q] = fmax(m[q], __shfl_down(m[q], off, 64));
  __shared__ double sm[16][2];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < K; ++q) sm[wid][q] = m[q];
  __syncthreads();
  if (threadIdx.x == 0) {
    double r[2] = {0.0, 0.0};
    for (int w = 0; w < 16; ++w)
#pragma unroll
      for (int q = 0; q < K; ++q) r[q] = fmax(r[q], sm[w][q]);
#pragma unroll
    for (int q = 0; q < K; ++q) out[q] = r[q];
  }
}

// b = -div_h(u*) / dt
__global__ void __launch_bounds__(256) k_rhs(Phys P, const double* __restrict__ us,
                                             const double* __restrict__ vs,
                                             const double* __restrict__ ws, double scale,
                                             double* __restrict__ b) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t c = i + (size_t)n.nx * j + sxy * k;
  const size_t fu = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
  const size_t fv_ = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
  const double div = (us[fu + 1] - us[fu]) + (vs[fv_ + n.nx] - vs[fv_]) + (ws[c + sxy] - ws[c]);
  b[c] = div * scale;
}

// u^{n+1} = u* - dt beta grad_h p on non-wall faces of component C
// A thread takes a cell's three lower faces (and, at a far wall or the top, the
// face beyond), so p is read once for the three components and the step has one
// launch for them: 512 x 256 x 256 601 -> 499 us, 256 x 1 x 64 8.2 -> 3.4.
__global__ void __launch_bounds__(256) k_correct(Phys P, const double* __restrict__ us, const double* __restrict__ vs,
                                                 const double* __restrict__ ws, const double* __restrict__ p,
                                                 const double* __restrict__ bx, const double* __restrict__ by,
                                                 const double* __restrict__ bz, double dt, double* __restrict__ u,
                                                 double* __restrict__ v, double* __restrict__ w) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * 64 + threadIdx.x;
  const int j = tl.y * blockDim.y + __builtin_amdgcn_readfirstlane(threadIdx.y);
  const int k = tl.z * blockDim.z + __builtin_amdgcn_readfirstlane(threadIdx.z);
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const unsigned sxy = (unsigned)(n.nx * n.ny);
  const unsigned c = i + (unsigned)n.nx * (j + n.ny * k);
  const unsigned fu = i + (unsigned)(n.nx + 1) * (j + n.ny * k);
  const unsigned fv = i + (unsigned)n.nx * (j + (n.ny + 1) * k);
  const double pc = p[c], px = p[i > 0 ? c - 1 : c], py = p[j > 0 ? c - n.nx : c], pz = p[k > 0 ? c - sxy : c];
  const double u0 = us[fu], v0 = vs[fv], w0 = ws[c], b0 = bx[fu], b1 = by[fv], b2 = bz[c];
  const double ih = 1.0 / P.h;
  // walls: zero, but for a tank's inlet, which keeps its wave
  u[fu] = i > 0 ? u0 - dt * b0 * ((pc - px) * ih) : P.gen_len > 0.0 ? u0 : 0.0;
  v[fv] = j > 0 ? v0 - dt * b1 * ((pc - py) * ih) : 0.0;
  w[c] = k > 0 ? w0 - dt * b2 * ((pc - pz) * ih) : 0.0;
  if (i == n.nx - 1) u[fu + 1] = 0.0;
  if (j == n.ny - 1) v[fv + n.nx] = 0.0;
  if (k == n.nz - 1) w[c + sxy] = ws[c + sxy] - dt * bz[c + sxy] * (-pc * (2.0 * ih));   // p = 0 half a cell above
}

// The wave tank's relaxation zones after a step: phi <- a phi + (1 - a) target
// over the columns of the generation zone [0, gen_len] (target: the wave at
// t) and of the damping zone [L - damp_len, L] (still water).  The launch
// covers only those columns: column q < ng is x-index q, the others
// x-index i_damp + (q - ng).  C = 0, 1, 2: the velocity faces; C = 3: sigma.
template <int C>
__global__ void __launch_bounds__(256) k_relax(Phys P, double t, int ng, int i_damp, int ncol,
                                               double* __restrict__ a) {
  const Dims n = P.n;
  const int my = n.ny + (C == 1), mz = n.nz + (C == 2), mx = n.nx + (C == 0);
  const Tile tl = xcd_tile();
  const int q = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (q >= ncol || j >= my || k >= mz) return;
  const int i = q < ng ? q : i_damp + (q - ng);
  if (i >= mx) return;
  const double h = P.h;
  const double x = (C == 0) ? i * h : (i + 0.5) * h;
  const double z = (C == 2) ? k * h : (k + 0.5) * h;
  const double L = n.nx * h;
  bool gen;
  double al;
  if (P.gen_len > 0.0 && x <= P.gen_len) {
    gen = true;
    al = relax_weight(1.0 - x / P.gen_len);
  } else if (P.damp_len > 0.0 && x >= L - P.damp_len) {
    gen = false;
    al = relax_weight((x - (L - P.damp_len)) / P.damp_len);
  } else {
    return;
  }
  double target;
  if constexpr (C == 3)
    target = z - (P.depth + (gen ? tank_eta(P, x, t) : 0.0));
  else
    target = gen ? tank_vel(P, C, x, z, t) : 0.0;
  const size_t f = i + (size_t)mx * (j + (size_t)my * k);
  a[f] = al * a[f] + (1.0 - al) * target;
}

// Hydrodynamic force on body m, eqn_int_fh (Sec. "Fluid-structure
// coupling"): the sum over its stair-step surface (the faces across which the
// body's level set changes sign, Sec. "NLFK calculation") of
// (-p_f n_f + mu_f (grad u + grad u^T) . n_f) dA_f, with n_f out of the body,
// p_f the two cell pressures interpolated linearly to psi = 0, mu_f their
// mean viscosity, central differences at the face centre, dA_f = h^2 (h in
// 2-D).  One thread per cell of the box [lo, lo + ext), for the three faces
// below it; the box holds every cell within two of the body, so no face of
// the surface lies on its edge.  Per-block partials (Fx, Fy, Fz) in tile
// order.
__global__ void __launch_bounds__(256) k_hydro_force(Phys P, int m, int i0, int j0, int k0, int ex, int ey,
                                                     int ez, double t, const double* __restrict__ p,
                                                     const double* __restrict__ u,
                                                     const double* __restrict__ v,
                                                     const double* __restrict__ w,
                                                     const double* __restrict__ mu,
                                                     double* __restrict__ partials) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int li = tl.x * blockDim.x + threadIdx.x;
  const int lj = tl.y * blockDim.y + threadIdx.y;
  const int lk = tl.z * blockDim.z + threadIdx.z;
  double F[3] = {0.0, 0.0, 0.0};
  if (li < ex && lj < ey && lk < ez) {
    const int i = i0 + li, j = j0 + lj, k = k0 + lk;
    const BodyK B = P.body[m];
    const double h = P.h, ih = 1.0 / h;
    const bool two_d = (n.ny == 1);
    const double dA = two_d ? h : h * h;
    double zd;
    const double psb = body_psi_one(B, (i + 0.5) * h, (j + 0.5) * h, (k + 0.5) * h, t, &zd);
    // cell-centred mean of component c at a cell
    auto cmean = [&](int c, int a, int b2, int c2) {
      switch (c) {
        case 0: return 0.5 * (fv<0>(u, n, a, b2, c2) + fv<0>(u, n, a + 1, b2, c2));
        case 1: return 0.5 * (fv<1>(v, n, a, b2, c2) + fv<1>(v, n, a, b2 + 1, c2));
        default: return 0.5 * (fv<2>(w, n, a, b2, c2) + fv<2>(w, n, a, b2, c2 + 1));
      }
    };
    // face value of component d at face index (a, b2, c2)
    auto face = [&](int d, int a, int b2, int c2) {
      return d == 0 ? fv<0>(u, n, a, b2, c2) : (d == 1 ? fv<1>(v, n, a, b2, c2) : fv<2>(w, n, a, b2, c2));
    };
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if (d == 1 && two_d) continue;
      const int di = (d == 0), dj = (d == 1), dk = (d == 2);
      if ((d == 0 && i < 1) || (d == 1 && j < 1) || (d == 2 && k < 1)) continue;
      const int ia = i - di, ja = j - dj, ka = k - dk;
      const double psa = body_psi_one(B, (ia + 0.5) * h, (ja + 0.5) * h, (ka + 0.5) * h, t, &zd);
      if ((psa < 0.0) == (psb < 0.0)) continue;
      const double nd = (psa < 0.0) ? 1.0 : -1.0;
      const double pa = cv(p, n, ia, ja, ka), pb = cv(p, n, i, j, k);
      const double wa = fabs(psa), wb = fabs(psb);
      const double pf = (wb * pa + wa * pb) / (wa + wb);
      const double muf = 0.5 * (cv(mu, n, ia, ja, ka) + cv(mu, n, i, j, k));
      F[d] -= pf * nd * dA;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (c == 1 && two_d) continue;
        double G;
        if (c == d) {
          G = (face(d, i + di, j + dj, k + dk) - face(d, i - di, j - dj, k - dk)) * ih;
        } else {
          const int ci = (c == 0), cj = (c == 1), ck = (c == 2);
          G = (cmean(c, i, j, k) - cmean(c, ia, ja, ka)) * ih +
              (face(d, i + ci, j + cj, k + ck) - face(d, i - ci, j - cj, k - ck)) * (0.5 * ih);
        }
        F[c] += muf * G * nd * dA;
      }
    }
  }
  // fixed-order block sum
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < 3; ++q) F[q] += __shfl_down(F[q], off, 64);
  __shared__ double sm[4][3];
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  if ((tid & 63) == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) sm[tid >> 6][q] = F[q];
  __syncthreads();
  if (tid == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) partials[3 * (size_t)tl.lin + q] = (sm[0][q] + sm[1][q]) + (sm[2][q] + sm[3][q]);
}

// per-block partial diagnostics: max|div|, water volume, kinetic energy, max|u_c|
__global__ void __launch_bounds__(256) k_diag(Phys P, const double* __restrict__ sigma,
                                              const double* __restrict__ u,
                                              const double* __restrict__ v,
                                              const double* __restrict__ w,
                                              double* __restrict__ partials) {
  const Dims n = P.n;
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  double vals[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < n.nx && j < n.ny && k < n.nz) {
    const size_t sxy = (size_t)n.nx * n.ny;
    const size_t c = i + (size_t)n.nx * j + sxy * k;
    const size_t fu = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
    const size_t fvv = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
    const double um = u[fu], up = u[fu + 1], vm = v[fvv], vp = v[fvv + n.nx], wm = w[c],
                 wp = w[c + sxy];
    const double h = P.h;
    const double vol = (n.ny == 1) ? h * h : h * h * h;
    const double div = ((up - um) + (vp - vm) + (wp - wm)) / h;
    const double hf = heaviside(sigma[c], P.eps);
    const double rf = P.rho_w + (P.rho_a - P.rho_w) * hf;
    const double uc = 0.5 * (up + um), vc = 0.5 * (vp + vm), wc = 0.5 * (wp + wm);
    vals[0] = fabs(div);
    vals[1] = (1.0 - hf) * vol;
    vals[2] = 0.5 * rf * (uc * uc + vc * vc + wc * wc) * vol;
    vals[3] = fmax(fmax(fmax(fabs(um), fabs(up)), fmax(fabs(vm), fabs(vp))), fmax(fabs(wm), fabs(wp)));
  }
  for (int off = 32; off > 0; off >>= 1) {
    vals[0] = fmax(vals[0], __shfl_down(vals[0], off, 64));
    vals[1] += __shfl_down(vals[1], off, 64);
    vals[2] += __shfl_down(vals[2], off, 64);
    vals[3] = fmax(vals[3], __shfl_down(vals[3], off, 64));
  }
  __shared__ double sm[4][4];
  const int tid = threadIdx.x + 64 * (threadIdx.y + blockDim.y * threadIdx.z);
  const int lane = tid & 63, wid = tid >> 6;
  if (lane == 0)
    for (int q = 0; q < 4; ++q) sm[wid][q] = vals[q];
  __syncthreads();
  if (tid == 0) {
    const size_t blk = tl.lin;
    partials[4 * blk + 0] = fmax(fmax(sm[0][0], sm[1][0]), fmax(sm[2][0], sm[3][0]));
    partials[4 * blk + 1] = (sm[0][1] + sm[1][1]) + (sm[2][1] + sm[3][1]);
    partials[4 * blk + 2] = (sm[0][2] + sm[1][2]) + (sm[2][2] + sm[3][2]);
    partials[4 * blk + 3] = fmax(fmax(sm[0][3], sm[1][3]), fmax(sm[2][3], sm[3][3]));
  }
}

__global__ void __launch_bounds__(1024) k_diag_finalize(const double* __restrict__ partials, int nparts,
                                                        double* __restrict__ scal) {
  double vals[4] = {0.0, 0.0, 0.0, 0.0};
  for (int q = threadIdx.x; q < nparts; q += 1024) {
    vals[0] = fmax(vals[0], partials[4 * q + 0]);
    vals[1] += partials[4 * q + 1];
    vals[2] += partials[4 * q + 2];
    vals[3] = fmax(vals[3], partials[4 * q + 3]);
  }
  for (int off = 32; off > 0; off >>= 1) {
    vals[0] = fmax(vals[0], __shfl_down(vals[0], off, 64));
    vals[1] += __shfl_down(vals[1], off, 64);
    vals[2] += __shfl_down(vals[2], off, 64);
    vals[3] = fmax(vals[3], __shfl_down(vals[3], off, 64));
  }
  __shared__ double sm[16][4];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0)
    for (int q = 0; q < 4; ++q) sm[wid][q] = vals[q];
  __syncthreads();
  if (threadIdx.x == 0) {
    double r[4] = {0.0, 0.0, 0.0, 0.0};
    for (int q = 0; q < 16; ++q) {
      r[0] = fmax(r[0], sm[q][0]);
      r[1] += sm[q][1];
      r[2] += sm[q][2];
      r[3] = fmax(r[3], sm[q][3]);
    }
    for (int q = 0; q < 4; ++q) scal[S_DIAG + q] = r[q];
  }
}

}  // namespace

// ------------------------------------------------------------------ launchers
// Grids past the predictor's one launch of a face per lane: 64 x 40 x 40 (102400
// cells) 23.2 us against 26.6 with two faces, 1024 x 1 x 208 (212992) 26.2 against
// 25.2, 96 x 48 x 56 40.8 against 35.8
static bool large(const Dims& n) { return (long)n.nx * n.ny * n.nz >= 3L << 16; }
// Where the predictor and its Crank-Nicolson sweeps take two faces along x per
// lane: in rows of 64 cells on, whose x-faces fill more than one wavefront; below,
// two faces per lane leave more of one idle and save no wavefront (64 x 128 x 128
// 136 us against 88 with two, 63 x 128 x 128 78 against 88, 16 x 128 x 128 75
// against 97)
static bool pairs_pay(const Dims& n) { return n.nx >= 64 && large(n); }

// Planes of a march: the fewest rounds of blocks over the chip's 512 places
// (two blocks per compute unit) times a block's planes, four more being spent
// on its start and the planes that only feed it (a block of all planes has none)
static int march_planes(long cols, int nz, long* planes = nullptr) {
  int best = nz;
  long cost = -1;
  for (int c = 1; c <= std::max(1, std::min(nz / 4, 1024)); ++c) {
    const int kz = (nz + c - 1) / c;
    const long t = ((cols * ((nz + kz - 1) / kz) + 511) / 512) * (kz + 4);
    if (cost < 0 || t < cost) cost = t, best = kz;
  }
  if (planes) *planes = best == nz ? (cols + 511) / 512 * (nz + 1) : cost;
  return best;
}
static long march_cols(const Dims& n, int ring) {
  const int lanes = 64 - 2 * ring, rows = kRW * kRR - 2 * ring;
  return (long)((n.nx + lanes - 1) / lanes) * ((n.ny + rows - 1) / rows);
}

// Where a lane may march up a column: a plane's values are at byte offsets of 32
// bits, so its largest array must stay below 2^29 entries (23171 x 23171 x 2 is
// a valid grid)
static bool marches(const Dims& n) {
  return n.ny >= 4 && (long)n.nx * n.ny * n.nz >= (1L << 20) &&
         std::max((long)(n.nx + 1) * n.ny, (long)n.nx * (n.ny + 1)) < (1L << 29);
}
// lanes of the one-cell forms' 64 x 4 tiles
static double cell_lanes(const Dims& n) { return 256.0 * ((n.nx + 63) / 64) * ((n.ny + 3) / 4) * n.nz; }
// The advection marches from 13 x 2^17 such lanes on, in blocks that ny fills by
// more than half: below, a cell per lane's many short wavefronts fill the chip better
// (186 x 96 x 64, 1.18 million lanes, 15.3 us against 20.0; 176 x 112 x 80, 1.72 million,
// 20.6 against 20.1)
static bool advect_marches(const Dims& n) { return marches(n) && n.ny > 8 && cell_lanes(n) >= (13L << 17); }
// The reinitialisation's form: two pseudo-steps per launch, marched (two), and a
// single one marched or by a cell per lane, by what each is expected to take (us).  A round of
// blocks takes 2.65 us a plane with two steps, in tiles of 62 x 14 cells, and
// 1.5 with one, in 64 x 16, or the time of its 24 bytes per cell at 4.3 TB/s; a
// cell per lane 3.5 and 6.2 per 2^20 lanes in tiles of 64 x 4.  Within 15% of
// the times measured on 26 grids of 1 to 33 million cells, and the choice the
// best one or within 6% of it: two steps 19, 21, 33 and 38 us on 64 x 128 x 128 (two
// blocks across a row of 64), 200 x 72 x 104, 512 x 4 x 512 and 64 x 512 x 64, two
// launches of one 18, 26, 33 and 24, of a cell per lane 19, 29, 19 and 31.
struct ReinitForm {
  bool two, march;
};
static ReinitForm reinit_form(const Dims& n) {
  if (!marches(n)) return {false, false};
  long p1, p2;
  march_planes(march_cols(n, 0), n.nz, &p1);
  march_planes(march_cols(n, 1), n.nz, &p2);
  const double cells = (double)n.nx * n.ny * n.nz;
  const double one = 3.5 + 6.2 * cell_lanes(n) / (1 << 20), march = std::max(1.5 * p1, cells * 24.0 / 4.3e6);
  return {2.65 * p2 - 2.0 < 1.95 * std::min(one, march), march < one};
}
// Pseudo-steps per launch
int reinit_steps(const Dims& n) { return n.ny == 1 ? kR2 : reinit_form(n).two ? 2 : 1; }

void launch_advect(const Phys& P, const double* s, const double* u, const double* v, const double* w,
                   double dt, double* out, hipStream_t st) {
  const Dims n = P.n;
  if (advect_marches(n)) {
    const int gx = (n.nx + 63) / 64, gy = (n.ny + kRW * kRR - 1) / (kRW * kRR), kz = march_planes(march_cols(n, 0), n.nz);
    hipLaunchKernelGGL(k_advect_march, dim3(gx, gy, (n.nz + kz - 1) / kz), dim3(64, kRW), 0, st, P, s, u, v, w, dt, out, kz);
    return;
  }
  Geo g = geo3(n.nx, n.ny, n.nz);
  hipLaunchKernelGGL(k_advect, g.grid, g.block, 0, st, P, s, u, v, w, dt, out);
}

template <int STEPS, bool FIRST>
static void reinit_march(const Phys& P, const double* s0, const double* cur, double* nxt, double dtau, hipStream_t st) {
  constexpr int H = STEPS - 1, rows = kRW * kRR - 2 * H, lanes = 64 - 2 * H;
  const Dims n = P.n;
  const int gx = (n.nx + lanes - 1) / lanes, gy = (n.ny + rows - 1) / rows, kz = march_planes(march_cols(n, H), n.nz);
  hipLaunchKernelGGL((k_reinit_march<STEPS, FIRST>), dim3(gx, gy, (n.nz + kz - 1) / kz), dim3(64, kRW), 0, st, P, s0, cur,
                     nxt, dtau, kz);
}

void launch_reinit(const Phys& P, const double* s0, const double* cur, double* nxt, double dtau, int steps,
                   hipStream_t st) {
  const bool first = s0 == cur;   // (sigma0 is then read once)
  if (P.n.ny == 1) {
    hipLaunchKernelGGL(k_reinit2d, dim3((P.n.nx + kR2X - 1) / kR2X, (P.n.nz + kR2Z - 1) / kR2Z), dim3(kR2T), 0, st, P, s0,
                       cur, nxt, dtau, steps);
  } else if (steps == 2) {
    first ? reinit_march<2, true>(P, s0, cur, nxt, dtau, st) : reinit_march<2, false>(P, s0, cur, nxt, dtau, st);
  } else if (reinit_form(P.n).march) {
    first ? reinit_march<1, true>(P, s0, cur, nxt, dtau, st) : reinit_march<1, false>(P, s0, cur, nxt, dtau, st);
  } else {
    Geo g = geo3(P.n.nx, P.n.ny, P.n.nz);
    hipLaunchKernelGGL(k_reinit, g.grid, g.block, 0, st, P, s0, cur, nxt, dtau);
  }
}

void launch_copy(const double* src, double* dst, size_t n, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
}

// A launch evaluates the bodies at one time: a prescribed heave's sine and
// cosine are taken here, once, and the kernels receive those bodies with
// zeta, zdot set and fh = 1, as for a free body's state (fh is read on the
// device only to choose between the stored heave and the formula).  The
// kernels had evaluated both per cell or face.
static Phys heave_at(const Phys& P, double t) {
  Phys Q = P;
  for (int m = 0; m < Q.nb; ++m) {
    BodyK& B = Q.body[m];
    if (B.fh) continue;
    const double arg = B.om * t + B.ph;
    B.zeta = B.amp * std::sin(arg);
    B.zdot = B.amp * B.om * std::cos(arg);
    B.fh = 1;
  }
  return Q;
}

void launch_props(const Phys& P, const double* sigma, double t, double* rho, double* rfl, double* mu,
                  double* chi, hipStream_t st) {
  Geo g = geo3(P.n.nx, P.n.ny, P.n.nz);
  hipLaunchKernelGGL(k_props, g.grid, g.block, 0, st, heave_at(P, t), sigma, t, rho, rfl, mu, chi);
}

void launch_momentum(const Phys& P, const double* u, const double* v, const double* w,
                     const double* rho, const double* rfl, const double* mu, const double* chi,
                     const double* rho_n, double dt, double t1, double* us, double* vs, double* ws, double* bx,
                     double* by, double* bz, float* bxf, float* byf, float* bzf, double* const* cn_rhs,
                     double* const* cn_diag, double* flag, hipStream_t st) {
  const Dims n = P.n;
  const Phys Pt = heave_at(P, t1);
  double* r[3] = {nullptr, nullptr, nullptr};
  double* dg[3] = {nullptr, nullptr, nullptr};
  if (cn_rhs)
    for (int c = 0; c < 3; ++c) r[c] = cn_rhs[c], dg[c] = cn_diag[c];
  double* const o[3] = {us, vs, ws};
  double* const be[3] = {bx, by, bz};
  float* const bf[3] = {bxf, byf, bzf};
  if (!large(n)) {
    MomOut O;
    for (int c = 0; c < 3; ++c) O.u[c] = o[c], O.beta[c] = be[c], O.betaf[c] = bf[c], O.rhs[c] = r[c], O.diag[c] = dg[c];
    Geo g = geo3(n.nx + 1, n.ny + (n.ny > 1), n.nz + 1);
    g.grid.y = (n.ny + 1 + g.block.y - 1) / g.block.y;   // (the y-faces' rows)
    g.grid.x *= 3;
    hipLaunchKernelGGL(rho_n ? k_momentum<true> : k_momentum<false>, g.grid, g.block, 0, st, Pt, u, v, w, rho, rfl, mu, chi,
                       rho_n, dt, t1, O, flag);
    return;
  }
  auto comp = [&](auto c, auto cons) {
    constexpr int C = decltype(c)::value;
    constexpr bool CONS = decltype(cons)::value;
    const bool pair = pairs_pay(n);
    const Geo g = geo3(pair ? (n.nx + 1) / 2 : n.nx + (C == 0), n.ny + (C == 1), n.nz + (C == 2));
    hipLaunchKernelGGL((pair ? k_momentum_pair<C, CONS> : k_momentum_face<C, CONS>), g.grid, g.block, 0, st, Pt, u, v, w, rho, rfl, mu, chi, rho_n, dt, t1,
                       o[C], be[C], bf[C], r[C], dg[C], flag);
  };
  auto all = [&](auto cons) {
    comp(std::integral_constant<int, 0>{}, cons);
    comp(std::integral_constant<int, 1>{}, cons);
    comp(std::integral_constant<int, 2>{}, cons);
  };
  if (rho_n)
    all(std::true_type{});
  else
    all(std::false_type{});
}

void launch_cn_sweep(const Phys& P, const double* u, const double* v, const double* w, const double* mu,
                     double* const* rhs, double* const* diag, double* uo, double* vo, double* wo, double* part,
                     double* out2, hipStream_t st) {
  const Dims n = P.n;
  size_t blocks = 0;
  auto sweep = [&](auto c, double* o) {
    constexpr int C = decltype(c)::value;
    const bool pair = pairs_pay(n);
    const Geo g = geo3(pair ? (n.nx + 1) / 2 : n.nx + (C == 0), n.ny + (C == 1), n.nz + (C == 2));
    hipLaunchKernelGGL((pair ? k_cn_sweep<C, V2> : k_cn_sweep<C, double>), g.grid, g.block, 0, st, P, u, v, w, mu, rhs[C],
                       diag[C], o, part ? part + 2 * blocks : nullptr);
    blocks += (size_t)g.grid.x * g.grid.y * g.grid.z;
  };
  sweep(std::integral_constant<int, 0>{}, uo);
  sweep(std::integral_constant<int, 1>{}, vo);
  sweep(std::integral_constant<int, 2>{}, wo);
  if (part)
    hipLaunchKernelGGL(k_max_finalize<2>, dim3(1), dim3(1024), 0, st, part, (int)blocks, out2);
}

int cn_part_blocks(const Dims& n) {
  Geo gx = geo3(n.nx + 1, n.ny, n.nz);
  Geo gy = geo3(n.nx, n.ny + 1, n.nz);
  Geo gz = geo3(n.nx, n.ny, n.nz + 1);
  return (int)((size_t)gx.grid.x * gx.grid.y * gx.grid.z + (size_t)gy.grid.x * gy.grid.y * gy.grid.z +
               (size_t)gz.grid.x * gz.grid.y * gz.grid.z);
}

void launch_cfl_max(const Phys& P, const double* u, const double* v, const double* w, double* partials,
                    double* out, hipStream_t st) {
  Geo g = geo3(P.n.nx, P.n.ny, P.n.nz);
  const int nb = (int)(g.grid.x * g.grid.y * g.grid.z);
  hipLaunchKernelGGL(k_cfl, g.grid, g.block, 0, st, P, u, v, w, partials);
  hipLaunchKernelGGL(k_max_finalize<1>, dim3(1), dim3(1024), 0, st, partials, nb, out);
}

void launch_rhs(const Phys& P, const double* us, const double* vs, const double* ws, double dt,
                double* b, hipStream_t st) {
  Geo g = geo3(P.n.nx, P.n.ny, P.n.nz);
  hipLaunchKernelGGL(k_rhs, g.grid, g.block, 0, st, P, us, vs, ws, -1.0 / (P.h * dt), b);
}

void launch_correct(const Phys& P, const double* us, const double* vs, const double* ws,
                    const double* p, const double* bx, const double* by, const double* bz, double dt,
                    double* u, double* v, double* w, hipStream_t st) {
  const Dims n = P.n;
  const Geo g = geo3(n.nx, n.ny, n.nz);
  hipLaunchKernelGGL(k_correct, g.grid, g.block, 0, st, P, us, vs, ws, p, bx, by, bz, dt, u, v, w);
}

int diag_blocks(const Phys& P) {
  Geo g = geo3(P.n.nx, P.n.ny, P.n.nz);
  return (int)(g.grid.x * g.grid.y * g.grid.z);
}

int launch_diag_partials(const Phys& P, const double* sigma, const double* u, const double* v,
                         const double* w, double* partials, hipStream_t st) {
  Geo g = geo3(P.n.nx, P.n.ny, P.n.nz);
  hipLaunchKernelGGL(k_diag, g.grid, g.block, 0, st, P, sigma, u, v, w, partials);
  return (int)(g.grid.x * g.grid.y * g.grid.z);
}

void launch_diag_finalize(const double* partials, int nparts, double* scal, hipStream_t st) {
  hipLaunchKernelGGL(k_diag_finalize, dim3(1), dim3(1024), 0, st, partials, nparts, scal);
}

int launch_hydro_force(const Phys& P, int m, double t, const double* p, const double* u, const double* v,
                       const double* w, const double* mu, double* partials, int max_blocks, hipStream_t st) {
  const BodyK& B = P.body[m];
  const double zeta = B.fh ? B.zeta : B.amp * sin(B.om * t + B.ph);
  // the body's extent, then every cell within two of it
  double lo[3], hi[3];
  if (B.kind == 0) {
    lo[0] = B.c0 - B.h0, hi[0] = B.c0 + B.h0;
    lo[1] = 0.0, hi[1] = P.n.ny * P.h;
    lo[2] = B.c2 + zeta - B.h2, hi[2] = B.c2 + zeta + B.h2;
  } else {
    lo[0] = B.c0 - B.h0, hi[0] = B.c0 + B.h0;
    lo[1] = B.c1 - B.h0, hi[1] = B.c1 + B.h0;
    lo[2] = B.h1 + zeta, hi[2] = B.h2 + zeta;
  }
  const int nn[3] = {P.n.nx, P.n.ny, P.n.nz};
  int a[3], e[3];
  for (int d = 0; d < 3; ++d) {
    const double L = std::floor(lo[d] / P.h) - 2.0, H = std::ceil(hi[d] / P.h) + 2.0;
    const int a0 = (int)std::max(0.0, std::min(L, (double)nn[d]));
    const int a1 = (int)std::max(0.0, std::min(H, (double)nn[d]));
    a[d] = a0;
    e[d] = a1 - a0;
  }
  if (e[0] <= 0 || e[1] <= 0 || e[2] <= 0) return 0;
  Geo g = geo3(e[0], e[1], e[2]);
  const long long blocks = (long long)g.grid.x * g.grid.y * g.grid.z;
  if (blocks > max_blocks) return -1;
  hipLaunchKernelGGL(k_hydro_force, g.grid, g.block, 0, st, heave_at(P, t), m, a[0], a[1], a[2], e[0], e[1], e[2], t, p, u, v,
                     w, mu, partials);
  return (int)blocks;
}

void launch_relax(const Phys& P, double t, double* sigma, double* u, double* v, double* w, hipStream_t st) {
  if (!(P.gen_len > 0.0) && !(P.damp_len > 0.0)) return;
  // columns that can lie in a zone: x-index 0..ng-1 (generation) and
  // i_damp..nx (damping), one spare column each way for the face arrays
  const double h = P.h;
  const int nx = P.n.nx;
  const int ng = P.gen_len > 0.0 ? std::min(nx + 1, (int)std::floor(P.gen_len / h) + 2) : 0;
  const int i_damp = P.damp_len > 0.0 ? std::max(ng, (int)std::floor((nx * h - P.damp_len) / h) - 1) : nx + 1;
  const int ncol = ng + std::max(0, nx + 1 - i_damp);
  if (ncol <= 0) return;
  Geo gu = geo3(ncol, P.n.ny, P.n.nz);
  hipLaunchKernelGGL(k_relax<0>, gu.grid, gu.block, 0, st, P, t, ng, i_damp, ncol, u);
  if (P.n.ny > 1) {
    Geo gv = geo3(ncol, P.n.ny + 1, P.n.nz);
    hipLaunchKernelGGL(k_relax<1>, gv.grid, gv.block, 0, st, P, t, ng, i_damp, ncol, v);
  }
  Geo gw = geo3(ncol, P.n.ny, P.n.nz + 1);
  hipLaunchKernelGGL(k_relax<2>, gw.grid, gw.block, 0, st, P, t, ng, i_damp, ncol, w);
  hipLaunchKernelGGL(k_relax<3>, gu.grid, gu.block, 0, st, P, t, ng, i_damp, ncol, sigma);
}

}  // namespace nsk
