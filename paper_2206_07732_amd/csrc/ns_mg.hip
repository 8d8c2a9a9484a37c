// Multigrid (red-black Gauss-Seidel V-cycle) and conjugate-gradient kernels
// for the pressure projection on gfx950.
//
// Operator on a level with spacing h (walls carry beta = 0, so every cell
// sums all six faces; the open top face couples to the ghost -x_c):
//   (A x)_c = (1/h^2) [ sum_f beta_f (x_c - x_nb) + 2 beta_top x_c (top row) ]
// V-cycle kernels are templated on the arithmetic type (double or float);
// the CG vectors and their reductions are always FP64.
//
// Launch count, not bandwidth, limits the small levels, so the schedule fuses
// what the algorithm allows:
//   * the first pre-smoothing pass (red from a zero guess) and the black pass
//     after it are one kernel: the red values h^2 b / D are recomputed by
//     the black cells from b and 1/D;
//   * prolongation and the first post-smoothing (black) pass are one kernel:
//     the black cells read their red neighbours plus the parent correction,
//     and the red cells are left for the red pass that follows, which
//     overwrites them without reading them;
//   * the levels from 4096 cells (FP32 6144) down run in one workgroup, the
//     first out of registers, those below out of LDS, and the cycle from 256
//     cells down is a product with its matrix;
//   * a 2-D level's visit is one launch down and one up;
//   * the direction update d = z + beta d is folded into the operator
//     application, which carries q = A d by its recurrence A z + beta q;
//     every CG reduction ends in one fixed-order pass over the per-block
//     partials, so results are bitwise reproducible.
#include <hip/hip_ext.h>

#include <type_traits>

#include "ns_internal.h"

namespace nsk {

namespace {

struct Geo {
  dim3 grid, block;
};

inline Geo geo3(int mx, int my, int mz) {
  dim3 b = (my >= 4) ? dim3(64, 4, 1) : dim3(64, 1, 4);
  return {dim3((mx + 63) / 64, (my + b.y - 1) / b.y, (mz + b.z - 1) / b.z), b};
}

// sum_f beta_f (x_c - x_nb) + top term, without the 1/h^2 factor
template <typename T>
__device__ __forceinline__ T stencil(const Dims& n, const T* __restrict__ bx, const T* __restrict__ by,
                                     const T* __restrict__ bz, const T* __restrict__ x, int i, int j,
                                     int k, size_t c) {
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t fx = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
  const size_t fy = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
  const T xc = x[c];
  const T xw = x[i > 0 ? c - 1 : c];
  const T xe = x[i < n.nx - 1 ? c + 1 : c];
  const T xs = x[j > 0 ? c - n.nx : c];
  const T xn = x[j < n.ny - 1 ? c + n.nx : c];
  const T xd = x[k > 0 ? c - sxy : c];
  const T xu = x[k < n.nz - 1 ? c + sxy : c];
  const T bu = bz[c + sxy];
  T acc = bx[fx] * (xc - xw) + bx[fx + 1] * (xc - xe) + by[fy] * (xc - xs) +
          by[fy + n.nx] * (xc - xn) + bz[c] * (xc - xd);
  acc += (k < n.nz - 1) ? bu * (xc - xu) : (T)2 * bu * xc;
  return acc;
}

// ------------------------------------------------------------ line tables
template <typename T>
struct TabBits;
template <>
struct TabBits<double> {
  using U = unsigned long long;
};
template <>
struct TabBits<float> {
  using U = unsigned;
};

// true with v the value every face of the line holds, where the table says
// so; else false (v = 0), also without a table.  With a line that is the
// same on every lane the entry is a scalar load, and a branch on the result
// a scalar branch.
template <typename T>
__device__ __forceinline__ bool line_val(const T* __restrict__ tab, int line, T& v) {
  using U = typename TabBits<T>::U;
  v = (T)0;
  if (tab == nullptr) return false;
  const T t = tab[line];
  if (__builtin_bit_cast(U, t) == ~U(0)) return false;
  v = t;
  return true;
}

// The six faces of one cell per lane, for a wavefront whose lanes share the
// cell's j and k (ju, ku: those values, the same on every lane; blockDim.x is
// 64): the x-line (j, k), the y-lines j and j + 1 and the z-lines k and k + 1
// of plane k, each taken from its table where the line is one value, else
// loaded.  load() issues the loads, under scalar branches, so that a
// wavefront on lines of one value issues none; get(), called after the
// caller's loads are all in flight (past its sched_barrier), picks the
// values, so no wait is placed between the loads.  TAB false: plain loads,
// no table code (the coarse levels' first-pass instance; their colour and
// prolongation passes keep the table code with null tables, see k_gs).
template <typename T, bool TAB = true>
struct FaceLd {
  T t[5];
  bool u[5];
  T l[6];
  // fx, fy: the x- and y-face index of the cell's west and south faces; fz:
  // its down face (the cell's natural index)
  __device__ __forceinline__ void load(const Dims& n, const FaceTab<T>& ft, const T* __restrict__ bx,
                                       const T* __restrict__ by, const T* __restrict__ bz, int ju, int ku,
                                       size_t fx, size_t fy, size_t fz) {
    if constexpr (!TAB) {
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        u[q] = false;
        t[q] = (T)0;
      }
      l[0] = bx[fx];
      l[1] = bx[fx + 1];
      l[2] = by[fy];
      l[3] = by[fy + n.nx];
      l[4] = bz[fz];
      l[5] = bz[fz + (size_t)n.nx * n.ny];
      return;
    }
    u[0] = line_val(ft.x, ju + n.ny * ku, t[0]);
    u[1] = line_val(ft.y, ju + (n.ny + 1) * ku, t[1]);
    u[2] = line_val(ft.y, ju + 1 + (n.ny + 1) * ku, t[2]);
    u[3] = line_val(ft.z, ju + n.ny * ku, t[3]);
    u[4] = line_val(ft.z, ju + n.ny * (ku + 1), t[4]);
    // a face of a one-value line is left unset (get() never reads it):
    // zeroing it on that side of the branch made the compiler wait there,
    // in some instances, for every load in flight
    if (!u[0]) {
      l[0] = bx[fx];
      l[1] = bx[fx + 1];
    }
    if (!u[1]) l[2] = by[fy];
    if (!u[2]) l[3] = by[fy + n.nx];
    if (!u[3]) l[4] = bz[fz];
    if (!u[4]) l[5] = bz[fz + (size_t)n.nx * n.ny];
  }
  // the faces of the lane's cell, in column i (a line of one value has zero
  // wall faces)
  __device__ __forceinline__ void get(const Dims& n, int i, T& bw, T& be, T& bs, T& bn, T& bd, T& bu) const {
    bw = u[0] ? (i > 0 ? t[0] : (T)0) : l[0];
    be = u[0] ? (i < n.nx - 1 ? t[0] : (T)0) : l[1];
    bs = u[1] ? t[1] : l[2];
    bn = u[2] ? t[2] : l[3];
    bd = u[3] ? t[3] : l[4];
    bu = u[4] ? t[4] : l[5];
  }
};

// the line tables of a level's three face arrays in one launch, a
// wavefront per line: lines [0, lx) of bx ((nx + 1) faces each, walls first
// and last, which must be zero), then [lx, lx + ly) of by and the rest of bz
// (nx faces each); the comparison is of bit patterns, so a line of equal
// values is exactly one value
template <typename T>
__global__ void __launch_bounds__(256) k_face_table(Dims n, const T* __restrict__ bx, const T* __restrict__ by,
                                                    const T* __restrict__ bz, T* __restrict__ tx,
                                                    T* __restrict__ ty, T* __restrict__ tz) {
  using U = typename TabBits<T>::U;
  const int lx = n.ny * n.nz, ly = (n.ny + 1) * n.nz, lz = n.ny * (n.nz + 1);
  int line = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (line >= lx + ly + lz) return;
  const bool xw = line < lx;
  const T* a = bx;
  T* tab = tx;
  if (!xw) {
    line -= lx;
    a = by;
    tab = ty;
    if (line >= ly) {
      line -= ly;
      a = bz;
      tab = tz;
    }
  }
  const int len = xw ? n.nx + 1 : n.nx;
  const T* p = a + (size_t)line * len;
  const int lo = xw ? 1 : 0, hi = xw ? len - 1 : len;
  const U v = lo < hi ? __builtin_bit_cast(U, p[lo]) : U(0);
  bool same = true;
  for (int i = lo + lane; i < hi; i += 64) same &= __builtin_bit_cast(U, p[i]) == v;
  if (xw && lane == 0) same &= __builtin_bit_cast(U, p[0]) == U(0) && __builtin_bit_cast(U, p[len - 1]) == U(0);
  const bool all = __all(same);
  if (lane == 0) tab[line] = __builtin_bit_cast(T, all ? v : ~U(0));
}

// --------------------------------------------------------------- reductions
__device__ __forceinline__ int block_tid() {
  return threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
}

// sum NV values over the block; the totals end in thread 0 (fixed tree)
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV]) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] += __shfl_down(v[q], off, 64);
  __shared__ double sm[16][NV];
  const int tid = block_tid();
  const int nw = (blockDim.x * blockDim.y * blockDim.z + 63) >> 6;
  if ((tid & 63) == 0)
#pragma unroll
    for (int q = 0; q < NV; ++q) sm[tid >> 6][q] = v[q];
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += sm[w][q];
      v[q] = s;
    }
  }
  __syncthreads();
}

// the totals of np partials of NV values, in every lane: each wavefront sums
// them all, lane l partials l, l + 64, ..
template <int NV>
__device__ __forceinline__ void wave_totals(const double* __restrict__ p, int np, double (&t)[NV]) {
  const int lane = block_tid() & 63;
#pragma unroll
  for (int q = 0; q < NV; ++q) t[q] = 0.0;
#pragma unroll 1
  for (int base = lane; base < np; base += 4 * 64) {
    double a[4][NV];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < NV; ++q) a[u][q] = p[NV * min(base + 64 * u, np - 1) + q];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < NV; ++q) t[q] += base + 64 * u < np ? a[u][q] : 0.0;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < NV; ++q) t[q] += __shfl_xor(t[q], off, 64);
}

// write the block's NV sums to partials[NV * slot + q] (thread 0); slot is
// the block's tile index, so the partials lie in tile order
template <int NV>
__device__ __forceinline__ void block_partials(double (&v)[NV], double* __restrict__ partials, int slot) {
  block_sum<NV>(v);
  if (block_tid() == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) partials[NV * (size_t)slot + q] = v[q];
  }
}

// --------------------------------------------------------------- smoothers
// Levels above the coarse-level tail keep b, e and 1/D colour-split: cell
// (i, j, k) of colour c = (i + j + k) & 1 lives at c P + p with the pair index
// p = (i >> 1) + hx (j + ny k), hx = ceil(nx / 2), P = hx ny nz.  A colour pass
// then reads and writes only its own colour's entries (and the other
// colour's as neighbours), instead of whole lines of both.  The face
// coefficients stay in their natural layout.
struct SplitGeo {
  int hx;
  size_t P;
};
__host__ __device__ inline SplitGeo split_geo(const Dims& n) {
  const int hx = (n.nx + 1) >> 1;
  return SplitGeo{hx, (size_t)hx * n.ny * n.nz};
}
__device__ __forceinline__ size_t sidx(const Dims& n, const SplitGeo& g, int i, int j, int k) {
  return (size_t)((i + j + k) & 1) * g.P + (size_t)(i >> 1) + (size_t)g.hx * (j + (size_t)n.ny * k);
}
// index of cell (i, j, k) of a level's correction, split or natural
__device__ __forceinline__ size_t lidx(const Dims& n, const SplitGeo& g, bool split, int i, int j, int k) {
  return split ? sidx(n, g, i, j, k) : (size_t)i + (size_t)n.nx * (j + (size_t)n.ny * k);
}

// Threads own cell pairs (2ti, 2ti+1) of a row; the red cell of the pair is
// 2ti + ((j+k) & 1), the black one the other; pos is the pair index.
// (a 64 x bdy x bdz = 256-thread block of geo3; bdz is derived, since
// reading blockDim.y and .z together made the compiler fetch both in one
// misaligned vector load, waited on before any other load)
#define PAIR_INDEX                                                        \
  const Tile tl = xcd_tile();                                             \
  const int bdy = blockDim.y, bdz = 4 / bdy;                              \
  const int ti = tl.x * 64 + threadIdx.x;                                 \
  const int j = tl.y * bdy + threadIdx.y;                                 \
  const int k = tl.z * bdz + threadIdx.z;                                 \
  if (j >= n.ny || k >= n.nz) return;                                     \
  const SplitGeo sg = split_geo(n);                                       \
  if (ti >= sg.hx) return;                                                \
  const size_t sxy = (size_t)n.nx * n.ny;                                 \
  const size_t row = (size_t)n.nx * j + sxy * k;                          \
  const size_t pos = (size_t)ti + (size_t)sg.hx * (j + (size_t)n.ny * k)

// Gauss-Seidel value of cell (i, j, k) with pair index pos: (h^2 b + sum over
// non-wall faces of beta_f x_nb) / D, the neighbour values o(q) taken from the
// other colour at the neighbours' pair indices.  Wall terms are dropped by
// selects and every load goes through an in-range index (a wall neighbour
// through the cell's own pair index), so all of a thread's loads are in
// flight together and a 0 * garbage product never enters a sum.
// The loads of that value (faces; y and z neighbours), gathered apart from
// its arithmetic so that a kernel can issue them with its other loads,
// before anything waits on one.
template <typename T>
struct GsIn {
  T bw, be, bs, bn, bd, bu;   // faces: west, east, south, north, down, up
  T vs, vn, vd, vu;           // neighbour values: south, north, down, up
};
template <typename T, typename O>
__device__ __forceinline__ GsIn<T> gs_gather(const Dims& n, const SplitGeo& sg, const T* __restrict__ bx,
                                             const T* __restrict__ by, const T* __restrict__ bz, int i, int j,
                                             int k, size_t pos, O o) {
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t c = i + (size_t)n.nx * j + sxy * k;
  const size_t fx = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
  const size_t fy = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
  const bool top = (k == n.nz - 1);
  const bool S = j > 0, N = j < n.ny - 1, D = k > 0;
  const size_t sz = (size_t)sg.hx * n.ny;
  const size_t ps = S ? pos - sg.hx : pos, pn = N ? pos + sg.hx : pos;
  const size_t pd = D ? pos - sz : pos, pu = top ? pos : pos + sz;
  return GsIn<T>{bx[fx], bx[fx + 1], by[fy], by[fy + n.nx], bz[c], bz[c + sxy], o(ps), o(pn), o(pd), o(pu)};
}
// the neighbour values of gs_gather alone (the faces left zero, for a
// FaceLd to fill)
template <typename T, typename O>
__device__ __forceinline__ GsIn<T> gs_gather_nb(const Dims& n, const SplitGeo& sg, int j, int k, size_t pos, O o) {
  const bool top = (k == n.nz - 1);
  const bool S = j > 0, N = j < n.ny - 1, D = k > 0;
  const size_t sz = (size_t)sg.hx * n.ny;
  const size_t ps = S ? pos - sg.hx : pos, pn = N ? pos + sg.hx : pos;
  const size_t pd = D ? pos - sz : pos, pu = top ? pos : pos + sz;
  return GsIn<T>{(T)0, (T)0, (T)0, (T)0, (T)0, (T)0, o(ps), o(pn), o(pd), o(pu)};
}
template <typename T>
__device__ __forceinline__ T gs_combine(const Dims& n, const GsIn<T>& g, T h2, T bc, int i, int j, int k, T vw,
                                        T ve) {
  const bool top = (k == n.nz - 1);
  const bool W = i > 0, E = i < n.nx - 1, S = j > 0, N = j < n.ny - 1, D = k > 0;
  const T diag = g.bw + g.be + g.bs + g.bn + g.bd + (top ? (T)2 * g.bu : g.bu);
  const T num = h2 * bc + (W ? g.bw * vw : (T)0) + (E ? g.be * ve : (T)0) + (S ? g.bs * g.vs : (T)0) +
                (N ? g.bn * g.vn : (T)0) + (D ? g.bd * g.vd : (T)0) + (top ? (T)0 : g.bu * g.vu);
  return num / diag;
}
template <typename T, typename O>
__device__ __forceinline__ T gs_split_value_x(const Dims& n, const SplitGeo& sg, T h2, const T* __restrict__ bx,
                                             const T* __restrict__ by, const T* __restrict__ bz, T bc, int i,
                                             int j, int k, size_t pos, T vw, T ve, O o) {
  return gs_combine<T>(n, gs_gather<T>(n, sg, bx, by, bz, i, j, k, pos, o), h2, bc, i, j, k, vw, ve);
}

// the same with the x neighbours loaded: cell i - 1 is in pair (i - 1) >> 1,
// cell i + 1 in pair (i + 1) >> 1
template <typename T, typename O>
__device__ __forceinline__ T gs_split_value(const Dims& n, const SplitGeo& sg, T h2, const T* __restrict__ bx,
                                           const T* __restrict__ by, const T* __restrict__ bz, T bc, int i, int j,
                                           int k, size_t pos, O o) {
  const bool W = i > 0, E = i < n.nx - 1;
  const size_t pw = W ? pos - (size_t)((i & 1) ? 0 : 1) : pos;
  const size_t pe = E ? pos + (size_t)((i & 1) ? 1 : 0) : pos;
  return gs_split_value_x<T>(n, sg, h2, bx, by, bz, bc, i, j, k, pos, o(pw), o(pe), o);
}

// one colour of Gauss-Seidel on colour-split b, e (FINE: finest-level
// instance, own symbol).  With nat set (the last pass of the finest level's
// V-cycle) the pair is written, both colours, to nat in natural order
// instead of back into e.
// NZ (gs_planes: two on the finest level in FP32, else one): planes per
// thread.  A pass over a level whose line tables spare most face loads is
// bound by its loads' latency, a block living about one memory round trip: a
// thread taking two planes k, k + 1 (its loads all issued before it waits on
// one) halves the rounds of blocks.  On 512x256x256 that took the FP32
// colour pass from 108 to 84 us and the prolongation pass from 128 to 123;
// the FP64 ones, which move twice the bytes, stayed at 154 us and went from
// 198 to 206, and keep one plane.
template <typename T>
constexpr int gs_planes(bool fine) { return fine && sizeof(T) == 4 ? 2 : 1; }
// The pass's body: TAB, the instance with line-table code (the finest
// level's, and the first coarse level's where it has tables); NZ planes per
// thread.
template <typename T, bool TAB, int NZ>
__device__ __forceinline__ void gs_body(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                        const T* __restrict__ bz, const T* __restrict__ b, T* __restrict__ e,
                                        int colour, T* __restrict__ nat, FaceTab<T> ft) {
  // the block is 64 x by x bz = 256 threads (geo3); blockDim.z is derived,
  // since reading blockDim.y and .z together made the compiler fetch both in
  // one misaligned vector load, waited on before any other load
  const Tile tl = xcd_tile();
  const int bdy = blockDim.y, bdz = 4 / bdy;
  const int tix = tl.x * 64 + threadIdx.x;
  const int j = tl.y * bdy + threadIdx.y;
  const int k0 = (tl.z * bdz + threadIdx.z) * NZ;
  if (j >= n.ny || k0 >= n.nz) return;
  const SplitGeo sg = split_geo(n);
  // a lane past the row's end works on its last pair and stores nothing:
  // returning it early made the compiler put the other lanes' loads under
  // that branch, past the barrier
  const bool tlive = tix < sg.hx;
  const int ti = tlive ? tix : sg.hx - 1;
  const T* eo = e + (size_t)(1 - colour) * sg.P;
  const auto o = [&](size_t q) { return eo[q]; };
  if constexpr (NZ == 1) {
    // One plane: written out.  In the per-plane form below the compiler
    // moved this case's loads past the barrier, a second memory round trip
    // per wavefront (the FP64 pass 153 -> 158 us on 512x256x256).
    if (!tlive) return;
    const int k = k0;
    const int par = (j + k + colour) & 1;
    const int i = 2 * ti + par, io = 2 * ti + 1 - par;
    const size_t pos = (size_t)ti + (size_t)sg.hx * (j + (size_t)n.ny * k);
    const size_t row = (size_t)n.nx * j + (size_t)n.nx * n.ny * k;
    // a cell past the row's end gathers through the row's last cell and stores nothing
    const int ic = i < n.nx ? i : n.nx - 1;
    const bool W = ic > 0, E = ic < n.nx - 1;
    const size_t pw = W ? pos - (size_t)((ic & 1) ? 0 : 1) : pos;
    const size_t pe = E ? pos + (size_t)((ic & 1) ? 1 : 0) : pos;
    GsIn<T> g = gs_gather_nb<T>(n, sg, j, k, pos, o);
    const T vw = o(pw), ve = o(pe), bc = b[(size_t)colour * sg.P + pos];
    FaceLd<T, TAB> F;
    F.load(n, ft, bx, by, bz, __builtin_amdgcn_readfirstlane(j), __builtin_amdgcn_readfirstlane(k),
           ic + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k), ic + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k),
           row + ic);
    __builtin_amdgcn_sched_barrier(0);
    F.get(n, ic, g.bw, g.be, g.bs, g.bn, g.bd, g.bu);
    if (i < n.nx) {
      const T v = gs_combine<T>(n, g, h2, bc, i, j, k, vw, ve);
      if (nat)
        nat[row + i] = v;
      else
        e[(size_t)colour * sg.P + pos] = v;
    }
    if (nat && io < n.nx) nat[row + io] = eo[pos];
    return;
  }
  // per plane: a plane past the grid's top repeats the last one and stores
  // nothing; a cell past the row's end gathers through the row's last cell
  // and stores nothing
  int kq[NZ], iq[NZ], icq[NZ];
  size_t posq[NZ], rowq[NZ];
  GsIn<T> g[NZ];
  T vw[NZ], ve[NZ], bc[NZ];
  FaceLd<T, TAB> F[NZ];
#pragma unroll
  for (int q = 0; q < NZ; ++q) {
    const int k = min(k0 + q, n.nz - 1);
    const int par = (j + k + colour) & 1;
    const int i = 2 * ti + par, ic = i < n.nx ? i : n.nx - 1;
    const size_t pos = (size_t)ti + (size_t)sg.hx * (j + (size_t)n.ny * k);
    const size_t row = (size_t)n.nx * j + (size_t)n.nx * n.ny * k;
    const bool W = ic > 0, E = ic < n.nx - 1;
    const size_t pw = W ? pos - (size_t)((ic & 1) ? 0 : 1) : pos;
    const size_t pe = E ? pos + (size_t)((ic & 1) ? 1 : 0) : pos;
    // the faces' branches first, then the plain loads: issued before the
    // branches, these were moved past the barrier (to their uses) by the
    // compiler, a second memory round trip per wavefront
    F[q].load(n, ft, bx, by, bz, __builtin_amdgcn_readfirstlane(j), __builtin_amdgcn_readfirstlane(k),
              ic + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k), ic + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k),
              row + ic);
    g[q] = gs_gather_nb<T>(n, sg, j, k, pos, o);
    vw[q] = o(pw);
    ve[q] = o(pe);
    bc[q] = b[(size_t)colour * sg.P + pos];
    kq[q] = k;
    iq[q] = i;
    icq[q] = ic;
    posq[q] = pos;
    rowq[q] = row;
  }
  __builtin_amdgcn_sched_barrier(0);
  // every value is formed (a repeated plane's or a clamped cell's too) and
  // only the stores are guarded: a value formed under the guard let the
  // compiler sink its loads past the barrier, into the guarded block
#pragma unroll
  for (int q = 0; q < NZ; ++q) {
    F[q].get(n, icq[q], g[q].bw, g[q].be, g[q].bs, g[q].bn, g[q].bd, g[q].bu);
    const int i = iq[q], io = 2 * ti + 1 - (i & 1);
    const T v = gs_combine<T>(n, g[q], h2, bc[q], icq[q], j, kq[q], vw[q], ve[q]);
    const bool live = tlive && k0 + q < n.nz;
    if (live && i < n.nx) {
      if (nat)
        nat[rowq[q] + i] = v;
      else
        e[(size_t)colour * sg.P + posq[q]] = v;
    }
    if (live && nat && io < n.nx) nat[rowq[q] + io] = eo[posq[q]];
  }
}

// one colour pass (FINE: the finest level's instance, its own symbol).  The
// coarse instance keeps the table code's shape with no tables: with plain
// face loads the compiler moved all its loads past the barrier.
template <typename T, bool FINE>
__global__ void __launch_bounds__(256) k_gs(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                            const T* __restrict__ bz, const T* __restrict__ b, T* __restrict__ e,
                                            int colour, T* __restrict__ nat, FaceTab<T> ft) {
  gs_body<T, true, gs_planes<T>(FINE)>(n, h2, bx, by, bz, b, e, colour, nat, ft);
}

// the same on the first coarse level where it has line tables (own symbol)
template <typename T>
__global__ void __launch_bounds__(256) k_gs_c1(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                               const T* __restrict__ bz, const T* __restrict__ b, T* __restrict__ e,
                                               int colour, T* __restrict__ nat, FaceTab<T> ft) {
  gs_body<T, true, gs_planes<T>(true)>(n, h2, bx, by, bz, b, e, colour, nat, ft);
}

// The last red pass of the finest level, writing the V-cycle's result z in
// natural order and in FP64 (as k_gs with nat; an FP32 cycle's values are
// widened exactly), fused with the product r z the flexible CG needs next:
// its per-block sums, red cell then black cell of each pair, in tile order.  Every thread reaches the block reduction (no
// early return).
template <typename T>
__global__ void __launch_bounds__(256) k_gs_last_dots(Dims n, T h2, const T* __restrict__ bx,
                                                      const T* __restrict__ by, const T* __restrict__ bz,
                                                      const T* __restrict__ b, const T* __restrict__ e,
                                                      double* __restrict__ nat, const double* __restrict__ r,
                                                      double* __restrict__ partials, FaceTab<T> ft) {
  const Tile tl = xcd_tile();
  const int ti = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  const SplitGeo sg = split_geo(n);
  double v[1] = {0.0};
  const bool live = j < n.ny && k < n.nz && ti < sg.hx;
  const size_t pos = live ? (size_t)ti + (size_t)sg.hx * (j + (size_t)n.ny * k) : 0;
  const T* eo = e + sg.P;   // the black plane
  // This pair's black value.  The red cell's x neighbours are this pair's
  // black cell and the adjacent pair's, which the adjacent lane holds (a
  // wavefront is 64 consecutive pairs of one row); every lane takes part in
  // the shuffles, and only a row's end lanes load their neighbour.  Every
  // load is issued before the shuffles wait for eb, through in-range indices
  // (a lane outside the grid, or a red cell past the row's end, reads cells
  // of the grid and stores nothing).
  const int par = (j + k) & 1;
  const int i = 2 * ti + par, io = 2 * ti + 1 - par;
  const int jj = live ? j : 0, kk = live ? k : 0;
  const int ir = live ? min(i, n.nx - 1) : 0, iq = live ? min(io, n.nx - 1) : 0;
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t row = (size_t)n.nx * jj + sxy * kk;
  const int lane = threadIdx.x;
  const T eb = eo[pos];
  GsIn<T> g = gs_gather_nb<T>(n, sg, jj, kk, pos, [&](size_t q) { return eo[q]; });
  FaceLd<T> F;   // the wavefront's lines (j, k), clamped into the grid for a wavefront outside it
  F.load(n, ft, bx, by, bz, __builtin_amdgcn_readfirstlane(min(j, n.ny - 1)),
         __builtin_amdgcn_readfirstlane(min(k, n.nz - 1)), ir + (size_t)(n.nx + 1) * (jj + (size_t)n.ny * kk),
         ir + (size_t)n.nx * (jj + (size_t)(n.ny + 1) * kk), row + ir);
  const T bc = b[pos];
  T ex = 0;   // the row-end lanes' x neighbour from outside the wavefront
  if (live && lane == 0 && par == 0 && ir > 0) ex = eo[pos - 1];
  if (live && lane == 63 && par == 1 && ir < n.nx - 1) ex = eo[pos + 1];
  const double rr = r[row + ir], rq = r[row + iq];
  __builtin_amdgcn_sched_barrier(0);
  F.get(n, ir, g.bw, g.be, g.bs, g.bn, g.bd, g.bu);
  const T ebl = __shfl_up(eb, 1, 64), ebr = __shfl_down(eb, 1, 64);
  // formed on every lane from in-grid values, then kept by selects: a use
  // under a branch would let the compiler sink r's loads past the shuffles
  T vw = eb, ve = eb;   // par 1: west is this pair's black; par 0: east is
  if (par == 0 && ir > 0) vw = lane > 0 ? ebl : ex;
  if (par == 1 && ir < n.nx - 1) ve = lane < 63 ? ebr : ex;
  const double z = (double)gs_combine<T>(n, g, h2, bc, ir, jj, kk, vw, ve), zb = (double)eb;
  const bool red_ok = live && i < n.nx, black_ok = live && io < n.nx;
  if (red_ok) nat[row + i] = z;
  if (black_ok) nat[row + io] = zb;
  v[0] = (red_ok ? rr * z : 0.0) + (black_ok ? rq * zb : 0.0);
  block_partials<1>(v, partials, tl.lin);
}

// red pass from a zero guess followed by the black pass, in one launch: the
// red values the black cells need are recomputed from b and 1/D.  NAT: b is
// read in natural order (the finest level, whose b is a CG vector) and its
// colour-split copy is written to bs for the later passes; a natural b may
// be FP64 under an FP32 cycle (TB = double), rounded to T as it is read.
template <typename T, bool TAB, bool NAT, typename TB>
__device__ __forceinline__ void gs_first_body(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                              const T* __restrict__ bz, const TB* __restrict__ b,
                                              const T* __restrict__ invd, T* __restrict__ e, T* __restrict__ bs,
                                              T* __restrict__ bcopy, FaceTab<T> ft, int red_out) {
  static_assert(NAT || sizeof(TB) == sizeof(T), "a colour-split b has the cycle's type");
  PAIR_INDEX;
  const int par = (j + k) & 1;
  const int ir = 2 * ti + par, ib = 2 * ti + 1 - par;
  const size_t sz = (size_t)sg.hx * n.ny;
  // b of the cell (ii, jj, kk) of colour c with pair index q, as stored (an
  // FP64 b is rounded to T after the loads: rounded as it arrived, each
  // conversion waited for its load)
  auto bval = [&](int c, size_t q, int ii, int jj, int kk) -> TB {
    if constexpr (NAT)
      return b[(size_t)ii + (size_t)n.nx * jj + sxy * kk];
    else
      return b[(size_t)c * sg.P + q];
  };
  // This pair's red value h2 b / D, formed also where the red cell lies past
  // the row's end (b clamped into the row, an unused 1/D entry), since the
  // adjacent lane reads it: the black cell's x neighbours are this pair's red
  // cell and the adjacent pair's (a wavefront is 64 consecutive pairs of one
  // row), and only a row's end lanes load theirs.  Every load is issued
  // before the shuffles wait for that value; a black cell past the row's end
  // gathers through the row's last cell and stores nothing.
  const int lane = threadIdx.x;
  const int irc = ir < n.nx ? ir : n.nx - 1, ibc = ib < n.nx ? ib : n.nx - 1;
  const TB br0 = bval(0, pos, irc, j, k);
  const T idr = invd[pos];
  const TB bb0 = bval(1, pos, ibc, j, k);
  // the red neighbours' b and 1/D through in-range indices (walls: own pair)
  const bool W = ibc > 0, E = ibc < n.nx - 1, S = j > 0, N = j < n.ny - 1, D = k > 0, U = k < n.nz - 1;
  const size_t ps = S ? pos - sg.hx : pos, pn = N ? pos + sg.hx : pos, pd = D ? pos - sz : pos, pu = U ? pos + sz : pos;
  const int js = S ? j - 1 : j, jn = N ? j + 1 : j;
  const int kd = D ? k - 1 : k, ku = U ? k + 1 : k;
  const TB bS0 = bval(0, ps, ibc, js, k), bN0 = bval(0, pn, ibc, jn, k);
  const T iS = invd[ps], iN = invd[pn];
  const TB bD0 = bval(0, pd, ibc, j, kd), bU0 = bval(0, pu, ibc, j, ku);
  const T iD = invd[pd], iU = invd[pu];
  TB bX0 = 0;   // lane 63's east or lane 0's west red neighbour, outside the wavefront
  T iX = 0;
  const bool xe = lane == 63 && par == 0 && E, xw = lane == 0 && par == 1 && W;
  if (xe || xw) {   // one block of loads: two made the second wait for the first's
    const int dx = xe ? 1 : -1;
    bX0 = bval(0, pos + dx, ibc + dx, j, k);
    iX = invd[pos + dx];
  }
  const size_t c = row + ibc;
  const size_t fx = ibc + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
  const size_t fy = ibc + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
  FaceLd<T, TAB> F;
  F.load(n, ft, bx, by, bz, __builtin_amdgcn_readfirstlane(j), __builtin_amdgcn_readfirstlane(k), fx, fy, c);
  __builtin_amdgcn_sched_barrier(0);
  T bw, be, bsy, bn, bd, bu;
  F.get(n, ibc, bw, be, bsy, bn, bd, bu);
  const T br = (T)br0, bb = (T)bb0, bS = (T)bS0, bN = (T)bN0, bD = (T)bD0, bU = (T)bU0, bX = (T)bX0;
  const T rv = h2 * br * idr;
  if (ir < n.nx) {
    // the red values are not stored where the next pass is a red one, which
    // overwrites them without reading them
    if (red_out) e[pos] = rv;
    if constexpr (NAT) bs[pos] = br;
  }
  const T rl = __shfl_up(rv, 1, 64), rr = __shfl_down(rv, 1, 64);
  if (ib >= n.nx) return;
  if constexpr (NAT) bs[sg.P + pos] = bb;
  T vw = rv, ve = rv;   // par 0: west is this pair's red cell; par 1: east is
  if (par == 0 && E) ve = lane < 63 ? rr : h2 * bX * iX;
  if (par == 1 && W) vw = lane > 0 ? rl : h2 * bX * iX;
  const T vs = h2 * bS * iS, vn = h2 * bN * iN, vd = h2 * bD * iD, vu = h2 * bU * iU;
  const bool top = !U;
  const T diag = bw + be + bsy + bn + bd + (top ? (T)2 * bu : bu);
  const T num = h2 * bb + (W ? bw * vw : (T)0) + (E ? be * ve : (T)0) + (S ? bsy * vs : (T)0) +
                (N ? bn * vn : (T)0) + (D ? bd * vd : (T)0) + (top ? (T)0 : bu * vu);
  const T vb = num / diag;
  e[sg.P + pos] = vb;
  if (bcopy) bcopy[pos] = vb;   // the black plane as a fused red-black pass will read it
}

// (FINE: the finest level's instance, its own symbol)
template <typename T, bool FINE, bool NAT, typename TB = T>
__global__ void __launch_bounds__(256) k_gs_first(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                                  const T* __restrict__ bz, const TB* __restrict__ b,
                                                  const T* __restrict__ invd, T* __restrict__ e, T* __restrict__ bs,
                                                  T* __restrict__ bcopy, FaceTab<T> ft, int red_out) {
  gs_first_body<T, FINE, NAT, TB>(n, h2, bx, by, bz, b, invd, e, bs, bcopy, ft, red_out);
}

// the same on the first coarse level where it has line tables (own symbol)
template <typename T>
__global__ void __launch_bounds__(256) k_gs_first_c1(Dims n, T h2, const T* __restrict__ bx,
                                                     const T* __restrict__ by, const T* __restrict__ bz,
                                                     const T* __restrict__ b, const T* __restrict__ invd,
                                                     T* __restrict__ e, T* __restrict__ bs, T* __restrict__ bcopy,
                                                     FaceTab<T> ft, int red_out) {
  gs_first_body<T, true, false, T>(n, h2, bx, by, bz, b, invd, e, bs, bcopy, ft, red_out);
}

// prolongation e += P ec followed by the black pass, in one launch; only the
// black cells are written (the red pass that follows overwrites the red ones
// without reading them).  ec is the next level's correction, colour-split
// (csplit) or natural (a tail level).
template <typename T, bool TAB, int NZ>
__device__ __forceinline__ void gs_prolong_body(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                                const T* __restrict__ bz, const T* __restrict__ b,
                                                T* __restrict__ e, Dims nc, int sxc, int syc, int szc, int csplit,
                                                const T* __restrict__ ec, T* __restrict__ bcopy, FaceTab<T> ft) {
  // NZ planes per thread, as in k_gs
  // the block is 64 x by x bz = 256 threads (geo3); blockDim.z is derived,
  // since reading blockDim.y and .z together made the compiler fetch both in
  // one misaligned vector load, waited on before any other load
  const Tile tl = xcd_tile();
  const int bdy = blockDim.y, bdz = 4 / bdy;
  const int tix = tl.x * 64 + threadIdx.x;
  const int j = tl.y * bdy + threadIdx.y;
  const int k0 = (tl.z * bdz + threadIdx.z) * NZ;
  if (j >= n.ny || k0 >= n.nz) return;
  const SplitGeo sg = split_geo(n);
  // a lane past the row's end works on its last pair and stores nothing:
  // returning it early made the compiler put the other lanes' loads under
  // that branch, past the barrier
  const bool tlive = tix < sg.hx;
  const int ti = tlive ? tix : sg.hx - 1;
  // the parent's entry in 32-bit arithmetic (a level's arrays have fewer
  // than 2^31 entries; six of these per thread dominated its instruction count)
  const int chx = (nc.nx + 1) >> 1, cP = chx * nc.ny * nc.nz;
  auto cidx = [&](int ii, int jj, int kk) {
    const int I = ii >> sxc, J = jj >> syc, K = kk >> szc;
    return csplit ? ((I + J + K) & 1) * cP + (I >> 1) + chx * (J + nc.ny * K) : I + nc.nx * (J + nc.ny * K);
  };
  const size_t sz = (size_t)sg.hx * n.ny, sxy = (size_t)n.nx * n.ny;
  // per plane (a plane past the grid's top repeats the last one, and a black
  // cell past the row's end its row's last cell; neither is stored): the red
  // neighbours' values and their parents' corrections, the faces and b,
  // every load before the first wait.  The indices are all formed first:
  // interleaved with the loads, the compiler's 32-bit multiply-adds read a
  // register pair whose upper half was a load's destination, and waited.
  T ev[NZ][6], qv[NZ][6], bcell[NZ];
  int iq[NZ], kq[NZ], qi[NZ][6];
  size_t posq[NZ], en[NZ][6], fxq[NZ], fyq[NZ], cq[NZ];
  FaceLd<T, TAB> F[NZ];
#pragma unroll
  for (int q = 0; q < NZ; ++q) {
    const int k = min(k0 + q, n.nz - 1);
    const int ib = 2 * ti + 1 - ((j + k) & 1);   // the black cell
    const int i = ib < n.nx ? ib : n.nx - 1;
    const size_t pos = (size_t)ti + (size_t)sg.hx * (j + (size_t)n.ny * k);
    const bool W = i > 0, E = i < n.nx - 1, S = j > 0, N = j < n.ny - 1, D = k > 0, U = k < n.nz - 1;
    en[q][0] = W ? pos - (size_t)((i & 1) ? 0 : 1) : pos;
    en[q][1] = E ? pos + (size_t)((i & 1) ? 1 : 0) : pos;
    en[q][2] = S ? pos - sg.hx : pos;
    en[q][3] = N ? pos + sg.hx : pos;
    en[q][4] = D ? pos - sz : pos;
    en[q][5] = U ? pos + sz : pos;
    qi[q][0] = cidx(W ? i - 1 : i, j, k);
    qi[q][1] = cidx(E ? i + 1 : i, j, k);
    qi[q][2] = cidx(i, S ? j - 1 : j, k);
    qi[q][3] = cidx(i, N ? j + 1 : j, k);
    qi[q][4] = cidx(i, j, D ? k - 1 : k);
    qi[q][5] = cidx(i, j, U ? k + 1 : k);
    cq[q] = (size_t)n.nx * j + sxy * k + i;
    fxq[q] = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
    fyq[q] = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
    iq[q] = ib;
    kq[q] = k;
    posq[q] = pos;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < NZ; ++q) {
#pragma unroll
    for (int d = 0; d < 6; ++d) ev[q][d] = e[en[q][d]];
#pragma unroll
    for (int d = 0; d < 6; ++d) qv[q][d] = ec[qi[q][d]];
    F[q].load(n, ft, bx, by, bz, __builtin_amdgcn_readfirstlane(j), __builtin_amdgcn_readfirstlane(kq[q]), fxq[q],
              fyq[q], cq[q]);
    bcell[q] = b[sg.P + posq[q]];
  }
  __builtin_amdgcn_sched_barrier(0);
  // every value formed, only the stores guarded (as in gs_body)
#pragma unroll
  for (int q = 0; q < NZ; ++q) {
    const int k = kq[q], i = min(iq[q], n.nx - 1);
    const bool W = i > 0, E = i < n.nx - 1, S = j > 0, N = j < n.ny - 1, D = k > 0, U = k < n.nz - 1;
    T bw, be, bs, bn, bd, bu;
    F[q].get(n, i, bw, be, bs, bn, bd, bu);
    const T vw = ev[q][0] + qv[q][0], ve = ev[q][1] + qv[q][1], vs = ev[q][2] + qv[q][2];
    const T vn = ev[q][3] + qv[q][3], vd = ev[q][4] + qv[q][4], vu = ev[q][5] + qv[q][5];
    const bool top = !U;
    const T diag = bw + be + bs + bn + bd + (top ? (T)2 * bu : bu);
    const T num = h2 * bcell[q] + (W ? bw * vw : (T)0) + (E ? be * ve : (T)0) + (S ? bs * vs : (T)0) +
                  (N ? bn * vn : (T)0) + (D ? bd * vd : (T)0) + (top ? (T)0 : bu * vu);
    const T vb = num / diag;
    if (tlive && k0 + q < n.nz && iq[q] < n.nx) {
      e[sg.P + posq[q]] = vb;
      if (bcopy) bcopy[posq[q]] = vb;   // the black plane as a fused red-black pass will read it
    }
  }
}

// (FINE: the finest level's instance, its own symbol; the coarse one keeps
// the table code's shape, as k_gs)
template <typename T, bool FINE>
__global__ void __launch_bounds__(256) k_gs_prolong(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                                    const T* __restrict__ bz, const T* __restrict__ b,
                                                    T* __restrict__ e, Dims nc, int sxc, int syc, int szc, int csplit,
                                                    const T* __restrict__ ec, T* __restrict__ bcopy, FaceTab<T> ft) {
  gs_prolong_body<T, true, gs_planes<T>(FINE)>(n, h2, bx, by, bz, b, e, nc, sxc, syc, szc, csplit, ec, bcopy, ft);
}

// the same on the first coarse level where it has line tables (own symbol)
template <typename T>
__global__ void __launch_bounds__(256) k_gs_prolong_c1(Dims n, T h2, const T* __restrict__ bx,
                                                       const T* __restrict__ by, const T* __restrict__ bz,
                                                       const T* __restrict__ b, T* __restrict__ e, Dims nc, int sxc,
                                                       int syc, int szc, int csplit, const T* __restrict__ ec,
                                                       T* __restrict__ bcopy, FaceTab<T> ft) {
  gs_prolong_body<T, true, gs_planes<T>(true)>(n, h2, bx, by, bz, b, e, nc, sxc, syc, szc, csplit, ec, bcopy, ft);
}

// ---------------------------------------------------------- wide passes
// The smoothing passes of a level with long rows (wide_pairs), V adjacent
// pairs of a row per lane.  What bounds the one-pair passes on a large level
// is the vector L1's address rate, not HBM: measured with loads that hit it,
// a wavefront's 8-byte-per-lane load takes 16 clocks (32 B/clk per compute
// unit), and so does a 16-byte one (64 B/clk; a 4-byte load takes 5, a
// strided 4-byte one 16).  A one-pair FP64 pass issues eight 8-byte
// instructions per 64 pairs, up to twenty where a line is not one value, and
// kept the address unit busy most of the time at 3.5 TB/s of traffic.  With
// V = 2 in FP64 and 4 in FP32 every access of a row is one 16-byte load or
// store per lane.  (512 x 256 x 256, one finest colour pass: FP64 150 ->
// 126 us, with faces all one value 132 -> 83; 256 x 128 x 128: 18.3 -> 13.3.)

// V consecutive values, by loads and stores of up to 16 bytes per lane
template <typename T, int V>
__device__ __forceinline__ void vload(T (&d)[V], const T* __restrict__ p) {
  typedef T VT __attribute__((ext_vector_type(V)));
  typedef VT VU __attribute__((aligned(sizeof(T))));   // a caller's field array is only 8-byte aligned
  const VU v = *reinterpret_cast<const VU*>(p);
#pragma unroll
  for (int q = 0; q < V; ++q) d[q] = v[q];
}
template <typename T, int V>
__device__ __forceinline__ void vstore(T* __restrict__ p, const T (&d)[V]) {
  typedef T VT __attribute__((ext_vector_type(V)));
  typedef VT VU __attribute__((aligned(sizeof(T))));
  VU v;
#pragma unroll
  for (int q = 0; q < V; ++q) v[q] = d[q];
  *reinterpret_cast<VU*>(p) = v;
}
// the same for values no other wavefront touches: not kept in the L2, which
// the values that neighbouring rows and planes share then have to themselves
template <typename T, int V>
__device__ __forceinline__ void vload_once(T (&d)[V], const T* __restrict__ p) {
  typedef T VT __attribute__((ext_vector_type(V)));
  typedef VT VU __attribute__((aligned(sizeof(T))));
  const VU v = __builtin_nontemporal_load(reinterpret_cast<const VU*>(p));
#pragma unroll
  for (int q = 0; q < V; ++q) d[q] = v[q];
}
template <typename T, int V>
__device__ __forceinline__ void vstore_once(T* __restrict__ p, const T (&d)[V]) {
  typedef T VT __attribute__((ext_vector_type(V)));
  typedef VT VU __attribute__((aligned(sizeof(T))));
  VU v;
#pragma unroll
  for (int q = 0; q < V; ++q) v[q] = d[q];
  __builtin_nontemporal_store(v, reinterpret_cast<VU*>(p));
}

// The faces of the V cells i0, i0 + 2, .. of one row, the cells of one colour
// of V adjacent pairs; i0 = 2 tp + par, tp the first pair.  As FaceLd: load()
// under scalar branches, get() once every load is in flight.  In FP32 the y
// and z faces are read as whole rows of 2 V faces from the even column 2 tp
// (two or four times fewer instructions than strided 4-byte loads) and the
// cells' own picked by par; in FP64 the whole row would cost as much as the
// cells' own.
template <typename T, int V>
struct FaceLdV {
  static constexpr bool ROW = sizeof(T) == 4;
  static constexpr int NF = ROW ? 2 * V : V;
  T t[5];
  bool u[5];
  T lx[2 * V], ls[NF], ln[NF], ld[NF], lu[NF];
  int par;
  __device__ __forceinline__ void row(T (&d)[NF], const T* __restrict__ p) const {   // p: the face at column i0
    if constexpr (ROW) {
      vload<T, NF>(d, p - par);
    } else {
#pragma unroll
      for (int q = 0; q < V; ++q) d[q] = p[2 * q];
    }
  }
  __device__ __forceinline__ T pick(const T (&d)[NF], int q) const {
    if constexpr (ROW)
      return par ? d[2 * q + 1] : d[2 * q];
    else
      return d[q];
  }
  __device__ __forceinline__ void load(const Dims& n, const FaceTab<T>& ft, const T* __restrict__ bx,
                                       const T* __restrict__ by, const T* __restrict__ bz, int ju, int ku, int p,
                                       int i0, int j, int k) {
    par = p;
    u[0] = line_val(ft.x, ju + n.ny * ku, t[0]);
    u[1] = line_val(ft.y, ju + (n.ny + 1) * ku, t[1]);
    u[2] = line_val(ft.y, ju + 1 + (n.ny + 1) * ku, t[2]);
    u[3] = line_val(ft.z, ju + n.ny * ku, t[3]);
    u[4] = line_val(ft.z, ju + n.ny * (ku + 1), t[4]);
    const size_t fy = i0 + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
    const size_t fz = i0 + (size_t)n.nx * (j + (size_t)n.ny * k);
    if (!u[0]) vload<T, 2 * V>(lx, bx + i0 + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k));
    if (!u[1]) row(ls, by + fy);
    if (!u[2]) row(ln, by + fy + n.nx);
    if (!u[3]) row(ld, bz + fz);
    if (!u[4]) row(lu, bz + fz + (size_t)n.nx * n.ny);
  }
  // the faces of the q-th cell, in column i
  __device__ __forceinline__ void get(const Dims& n, int i, int q, T& bw, T& be, T& bs, T& bn, T& bd, T& bu) const {
    bw = u[0] ? (i > 0 ? t[0] : (T)0) : lx[2 * q];
    be = u[0] ? (i < n.nx - 1 ? t[0] : (T)0) : lx[2 * q + 1];
    bs = u[1] ? t[1] : pick(ls, q);
    bn = u[2] ? t[2] : pick(ln, q);
    bd = u[3] ? t[3] : pick(ld, q);
    bu = u[4] ? t[4] : pick(lu, q);
  }
};

// The lane's place: pairs tp .. tp + V - 1 of row j of plane k (a 64 x 4
// block), pos the first one's pair index.  A level of the wide passes has an
// even nx and a multiple of V pairs per row, so a lane's pairs are all in the
// row or all past its end; such a lane, or one in a row past the last,
// works on pairs inside the grid (tp, j clamped) and stores nothing.  A tile
// holds more of a row here, so the band of tile rows is wider where the grid
// has enough of them: at 512 x 256 x 256 sixteen (64 rows) took a projection
// from 38.6 to 36.6 ms (FP32 cycle 29.6 to 28.3), thirty-two 37.2; at 256 x
// 128 x 128 eight 5.12 ms, sixteen 5.17.
#define WIDE_INDEX                                                                     \
  const Tile tl = xcd_tile(max(kTileBand, min(2 * kTileBand, (int)gridDim.y >> 2)));   \
  const int lane = threadIdx.x, hx = n.nx >> 1;                                        \
  const int tpr = V * (tl.x * 64 + lane), jr = tl.y * 4 + (int)threadIdx.y, k = tl.z;  \
  const bool live = tpr < hx && jr < n.ny;                                             \
  const int tp = min(tpr, hx - V), j = min(jr, n.ny - 1);                              \
  [[maybe_unused]] const int ju = __builtin_amdgcn_readfirstlane(j);                   \
  const size_t P = (size_t)hx * n.ny * n.nz, sz = (size_t)hx * n.ny;                   \
  const size_t pos = (size_t)tp + (size_t)hx * (j + (size_t)n.ny * k);                 \
  const bool S = j > 0, N = j < n.ny - 1, D = k > 0, U = k < n.nz - 1;                 \
  [[maybe_unused]] const size_t ps = S ? pos - hx : pos, pn = N ? pos + hx : pos;      \
  [[maybe_unused]] const size_t pd = D ? pos - sz : pos, pu = U ? pos + sz : pos

// The other colour's values around V cells of one colour: own pairs, rows
// beside, planes below and above, and the pair beyond the lane's own that the
// first (par = 0) or last (par = 1) cell has as its x neighbour.
template <typename T, int V>
struct WideNb {
  T o[V], s[V], n[V], d[V], u[V], x;
  __device__ __forceinline__ void load(const T* __restrict__ eo, size_t pos, size_t ps, size_t pn, size_t pd,
                                       size_t pu, int tp, int hx, int par) {
    vload<T, V>(o, eo + pos);
    vload<T, V>(s, eo + ps);
    vload<T, V>(n, eo + pn);
    vload<T, V>(d, eo + pd);
    vload<T, V>(u, eo + pu);
    x = eo[par ? (tp + V < hx ? pos + V : pos) : (tp > 0 ? pos - 1 : pos)];
  }
  __device__ __forceinline__ T west(int q, int par) const { return par ? o[q] : q > 0 ? o[q > 0 ? q - 1 : 0] : x; }
  __device__ __forceinline__ T east(int q, int par) const { return par ? (q < V - 1 ? o[q < V - 1 ? q + 1 : q] : x) : o[q]; }
};

// the Gauss-Seidel values of the lane's V cells, as gs_combine
template <typename T, int V>
__device__ __forceinline__ void wide_values(const Dims& n, const FaceLdV<T, V>& F, const WideNb<T, V>& w, T h2,
                                            const T (&bc)[V], int i0, int j, int k, int par, T (&v)[V]) {
#pragma unroll
  for (int q = 0; q < V; ++q) {
    GsIn<T> g;
    const int i = i0 + 2 * q;
    F.get(n, i, q, g.bw, g.be, g.bs, g.bn, g.bd, g.bu);
    g.vs = w.s[q];
    g.vn = w.n[q];
    g.vd = w.d[q];
    g.vu = w.u[q];
    v[q] = gs_combine<T>(n, g, h2, bc[q], i, j, k, w.west(q, par), w.east(q, par));
  }
}

// one colour pass (as k_gs)
template <typename T, int V>
__global__ void __launch_bounds__(256) k_gs_wide(Dims n, T h2, const T* __restrict__ bx, const T* __restrict__ by,
                                                 const T* __restrict__ bz, const T* __restrict__ b,
                                                 T* __restrict__ e, int colour, FaceTab<T> ft) {
  WIDE_INDEX;
  const int par = (j + k + colour) & 1, i0 = 2 * tp + par;
  WideNb<T, V> w;
  w.load(e + (size_t)(1 - colour) * P, pos, ps, pn, pd, pu, tp, hx, par);
  T bc[V], v[V];
  vload<T, V>(bc, b + (size_t)colour * P + pos);
  FaceLdV<T, V> F;
  F.load(n, ft, bx, by, bz, ju, k, par, i0, j, k);
  __builtin_amdgcn_sched_barrier(0);
  wide_values<T, V>(n, F, w, h2, bc, i0, j, k, par, v);
  if (live) vstore<T, V>(e + (size_t)colour * P + pos, v);
}

// The V-cycle's first kernel on such a level (as k_gs_first), b colour-split:
// the level's own b, or on the finest level the CG residual, which split CG
// vectors keep colour-split.  An FP32 cycle reads it in FP64 and leaves its
// FP32 copy in bs for the passes that follow; an FP64 cycle reads the
// residual itself in all of them.
template <typename T, int V, typename TB>
__global__ void __launch_bounds__(256) k_gs_first_wide(Dims n, T h2, const T* __restrict__ bx,
                                                       const T* __restrict__ by, const T* __restrict__ bz,
                                                       const TB* __restrict__ b, const T* __restrict__ invd,
                                                       T* __restrict__ e, T* __restrict__ bs, T* __restrict__ bcopy,
                                                       FaceTab<T> ft, int red_out) {
  constexpr bool COPY = sizeof(TB) != sizeof(T);
  WIDE_INDEX;
  const int par = (j + k) & 1, i0 = 2 * tp + 1 - par;   // the first black cell
  // b and 1/D of the lane's red cells and of the red neighbours of its black
  // ones, whose values from zero are h^2 b / D
  WideNb<TB, V> rb;
  WideNb<T, V> w;
  rb.load(b, pos, ps, pn, pd, pu, tp, hx, 1 - par);
  w.load(invd, pos, ps, pn, pd, pu, tp, hx, 1 - par);
  TB bb[V];
  vload<TB, V>(bb, b + P + pos);
  FaceLdV<T, V> F;
  F.load(n, ft, bx, by, bz, ju, k, 1 - par, i0, j, k);
  __builtin_amdgcn_sched_barrier(0);
  T red[V], black[V], v[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    red[q] = (T)rb.o[q];
    black[q] = (T)bb[q];
    w.o[q] = h2 * red[q] * w.o[q];
    w.s[q] = h2 * (T)rb.s[q] * w.s[q];
    w.n[q] = h2 * (T)rb.n[q] * w.n[q];
    w.d[q] = h2 * (T)rb.d[q] * w.d[q];
    w.u[q] = h2 * (T)rb.u[q] * w.u[q];
  }
  w.x = h2 * (T)rb.x * w.x;
  wide_values<T, V>(n, F, w, h2, black, i0, j, k, 1 - par, v);
  if (!live) return;
  if (red_out) vstore<T, V>(e + pos, w.o);
  if constexpr (COPY) {
    vstore<T, V>(bs + pos, red);
    vstore<T, V>(bs + P + pos, black);
  }
  vstore<T, V>(e + P + pos, v);
  if (bcopy) vstore<T, V>(bcopy + pos, v);
}

// The last red pass of the finest level with the product r z the flexible CG
// needs next (as k_gs_last_dots), z and r colour-split.  An FP64 cycle works
// in z itself (e == z: its black values are final, so only the red ones are
// stored) and has r for its b; an FP32 cycle writes both colours, widened.
template <typename T, int V>
__global__ void __launch_bounds__(256) k_gs_last_dots_wide(Dims n, T h2, const T* __restrict__ bx,
                                                           const T* __restrict__ by, const T* __restrict__ bz,
                                                           const T* __restrict__ b, const T* e, double* z,
                                                           const double* __restrict__ r,
                                                           double* __restrict__ partials, FaceTab<T> ft) {
  constexpr bool WIDEN = sizeof(T) != sizeof(double);
  WIDE_INDEX;
  const int par = (j + k) & 1, i0 = 2 * tp + par;
  WideNb<T, V> w;
  w.load(e + P, pos, ps, pn, pd, pu, tp, hx, par);
  T bc[V], v[V];
  vload<T, V>(bc, b + pos);
  double rr[V], rk[V];
  if constexpr (WIDEN) vload<double, V>(rr, r + pos);
  vload<double, V>(rk, r + P + pos);
  FaceLdV<T, V> F;
  F.load(n, ft, bx, by, bz, ju, k, par, i0, j, k);
  __builtin_amdgcn_sched_barrier(0);
  wide_values<T, V>(n, F, w, h2, bc, i0, j, k, par, v);
  double s[1] = {0.0}, zr[V], zk[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    zr[q] = (double)v[q];
    zk[q] = (double)w.o[q];
    if constexpr (!WIDEN) rr[q] = bc[q];
  }
  if (live) {
    vstore<double, V>(z + pos, zr);
    if constexpr (WIDEN) vstore<double, V>(z + P + pos, zk);
#pragma unroll
    for (int q = 0; q < V; ++q) s[0] += rr[q] * zr[q] + rk[q] * zk[q];
  }
  block_partials<1>(s, partials, tl.lin);
}

// prolongation + black (as k_gs_prolong).  A red neighbour's parent is the
// cell's own, or, for one neighbour each along x, y and z, the next one's, so
// four parents are read per cell instead of six.
template <typename T, int V>
__global__ void __launch_bounds__(256) k_gs_prolong_wide(Dims n, T h2, const T* __restrict__ bx,
                                                         const T* __restrict__ by, const T* __restrict__ bz,
                                                         const T* __restrict__ b, T* __restrict__ e, Dims nc, int syc,
                                                         int szc, int csplit, const T* __restrict__ ec,
                                                         T* __restrict__ bcopy, FaceTab<T> ft) {
  WIDE_INDEX;
  const int par = (j + k + 1) & 1, i0 = 2 * tp + par;
  const int chx = (nc.nx + 1) >> 1, cP = chx * nc.ny * nc.nz;
  auto cidx = [&](int I, int J, int K) {
    return csplit ? ((I + J + K) & 1) * cP + (I >> 1) + chx * (J + nc.ny * K) : I + nc.nx * (J + nc.ny * K);
  };
  // the parents' rows: the cell's own, and the one that holds its neighbour
  // across the coarse cell's y or z face
  const int J = j >> syc, K = k >> szc;
  const int js = (S ? j - 1 : j) >> syc, jn = (N ? j + 1 : j) >> syc;
  const int kd = (D ? k - 1 : k) >> szc, ku = (U ? k + 1 : k) >> szc;
  const int xI = par ? min(tp + V, hx - 1) : max(tp - 1, 0);
  WideNb<T, V> w;
  w.load(e, pos, ps, pn, pd, pu, tp, hx, par);
  T bc[V], v[V], co[V], cy[V], cz[V];
  const int jy = js != J ? js : jn, kz = kd != K ? kd : ku;
#pragma unroll
  for (int q = 0; q < V; ++q) {
    co[q] = ec[cidx(tp + q, J, K)];
    cy[q] = ec[cidx(tp + q, jy, K)];
    cz[q] = ec[cidx(tp + q, J, kz)];
  }
  const T cx = ec[cidx(xI, J, K)];
  vload<T, V>(bc, b + P + pos);
  FaceLdV<T, V> F;
  F.load(n, ft, bx, by, bz, ju, k, par, i0, j, k);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < V; ++q) {
    w.o[q] += co[q];
    w.s[q] += js != J ? cy[q] : co[q];
    w.n[q] += jn != J ? cy[q] : co[q];
    w.d[q] += kd != K ? cz[q] : co[q];
    w.u[q] += ku != K ? cz[q] : co[q];
  }
  w.x += cx;
  wide_values<T, V>(n, F, w, h2, bc, i0, j, k, par, v);
  if (!live) return;
  vstore<T, V>(e + P + pos, v);
  if (bcopy) vstore<T, V>(bcopy + pos, v);
}

// A red pass then a black pass of Gauss-Seidel in one launch, on a level
// whose rows are at most 32 pairs (ceil(nx/2) <= 32), where launch latency,
// not bytes, bounds a pass.  A block takes whole rows: TY rows by TZ planes
// of pairs (TX >= ceil(nx/2) lanes per row).  It forms the red values of its
// tile and of a ring one row wide in y and z around it (the red cells its
// black cells read) from the black plane as it stood before the launch,
// which the previous kernel copied to bold (this launch overwrites the
// black plane while other blocks still read it).  It then forms its black
// values from those red values, held in LDS.  Each value comes from the same
// arithmetic, on the same inputs, as in the two separate passes, so the
// results are theirs bit for bit.  Every global load of a thread is issued
// before it waits on any.
constexpr int kRbThreads = 256;
constexpr int kRbMaxIter = 3;   // ring-extended tile entries per thread
constexpr int kRbMaxExt = kRbThreads * kRbMaxIter;

template <typename T>
__global__ void __launch_bounds__(kRbThreads) k_gs_rb(Dims n, T h2, const T* __restrict__ bx,
                                                      const T* __restrict__ by, const T* __restrict__ bz,
                                                      const T* __restrict__ b, T* __restrict__ e,
                                                      const T* __restrict__ bold, int TX, int TY, int TZ) {
  __shared__ T R[kRbMaxExt];
  const SplitGeo sg = split_geo(n);
  const Tile tl = xcd_tile_flat();
  const int ty0 = tl.y * TY, tz0 = tl.z * TZ;
  const int ry = n.ny > 1 ? 1 : 0;   // ring width in y (none in a 2-D tank)
  const int EY = TY + 2 * ry, NE = TX * EY * (TZ + 2);
  const int t = threadIdx.x;
  const size_t sxy = (size_t)n.nx * n.ny;
  auto ob = [&](size_t q) { return bold[q]; };
  // red entries of the ring-extended tile: entry q is pair q % TX of row
  // (ty0 + ey - ry, tz0 + ez - 1); an entry outside the grid gathers through
  // red cell (parity, 0, 0) and is stored as 0
  GsIn<T> gr[kRbMaxIter];
  T br[kRbMaxIter], rw[kRbMaxIter], re[kRbMaxIter];
  int ri[kRbMaxIter], rj[kRbMaxIter], rk[kRbMaxIter];
  size_t rp[kRbMaxIter];
  bool rok[kRbMaxIter];
#pragma unroll
  for (int u = 0; u < kRbMaxIter; ++u) {
    const int q = t + u * kRbThreads;
    const int ex = q % TX, ey = (q / TX) % EY, ez = q / (TX * EY);
    const int j = ty0 + ey - ry, k = tz0 + ez - 1;
    const int i = 2 * ex + ((j + k) & 1);
    rok[u] = q < NE && j >= 0 && j < n.ny && k >= 0 && k < n.nz && i < n.nx;
    rj[u] = rok[u] ? j : 0;
    rk[u] = rok[u] ? k : 0;
    ri[u] = rok[u] ? i : 0;
    rp[u] = (size_t)(ri[u] >> 1) + (size_t)sg.hx * (rj[u] + (size_t)n.ny * rk[u]);
    gr[u] = gs_gather<T>(n, sg, bx, by, bz, ri[u], rj[u], rk[u], rp[u], ob);
    br[u] = b[rp[u]];
    const bool W = ri[u] > 0, E = ri[u] < n.nx - 1;
    rw[u] = bold[W ? rp[u] - (size_t)((ri[u] & 1) ? 0 : 1) : rp[u]];
    re[u] = bold[E ? rp[u] + (size_t)((ri[u] & 1) ? 1 : 0) : rp[u]];
  }
  // this thread's black cell: pair px of row (ty0 + py, tz0 + pz); the tile
  // has exactly kRbThreads cells (TX TY TZ = kRbThreads), so pz < TZ
  const int px = t % TX, py = (t / TX) % TY, pz = t / (TX * TY);
  const int jb = ty0 + py, kb = tz0 + pz;
  const int ib = 2 * px + 1 - ((jb + kb) & 1);
  const bool bok = jb < n.ny && kb < n.nz && ib < n.nx;
  const int jc = bok ? jb : 0, kc = bok ? kb : 0, ic = bok ? ib : 1;
  const size_t pb = (size_t)(ic >> 1) + (size_t)sg.hx * (jc + (size_t)n.ny * kc);
  const size_t cb = ic + (size_t)n.nx * jc + sxy * kc;
  const size_t fxb = ic + (size_t)(n.nx + 1) * (jc + (size_t)n.ny * kc);
  const size_t fyb = ic + (size_t)n.nx * (jc + (size_t)(n.ny + 1) * kc);
  const T bw = bx[fxb], be = bx[fxb + 1], bs = by[fyb], bn = by[fyb + n.nx], bd = bz[cb], bu = bz[cb + sxy];
  const T bb = b[sg.P + pb];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < kRbMaxIter; ++u) {
    const int q = t + u * kRbThreads;
    if (q < NE) {
      T v = (T)0;
      if (rok[u]) {
        v = gs_combine<T>(n, gr[u], h2, br[u], ri[u], rj[u], rk[u], rw[u], re[u]);
        const int ey = (q / TX) % EY, ez = q / (TX * EY);
        if (ey >= ry && ey < ry + TY && ez >= 1 && ez <= TZ) e[rp[u]] = v;
      }
      R[q] = v;
    }
  }
  __syncthreads();
  if (bok) {
    const int ey = py + ry, ez = pz + 1;
    const int row = TX * (ey + EY * ez);
    const int L = px + row;
    const bool W = ib > 0, E = ib < n.nx - 1, S = jb > 0, N = jb < n.ny - 1, D = kb > 0, U = kb < n.nz - 1;
    const T vw = R[W ? ((ib - 1) >> 1) + row : L], ve = R[E ? ((ib + 1) >> 1) + row : L];
    const GsIn<T> g{bw, be, bs, bn, bd, bu, R[S ? L - TX : L], R[N ? L + TX : L], R[D ? L - TX * EY : L],
                    R[U ? L + TX * EY : L]};
    e[sg.P + pb] = gs_combine<T>(n, g, h2, bb, ib, jb, kb, vw, ve);
  }
}

// A red pass then a black pass of Gauss-Seidel in one launch on the finest
// level, reading each face coefficient once.  Every face borders one red and
// one black cell, so the black update takes its six coefficients from the
// red updates beside it instead of loading them again:
//   * its z-faces are the down face of the red cell above it and the up face
//     of the red cell below it, both in the same pair column, which the same
//     thread computes on the planes above and below;
//   * its x-faces are the faces of the red cell of its own pair and of the
//     adjacent pair (the adjacent lane: a row of the block is one wave of 64
//     consecutive pairs; the end lanes load their outer face);
//   * its y-faces are those of the red cells of the rows beside it (LDS).
// A block marches up a chunk of KZ planes: at plane m it forms the red
// values of plane m, then the black values of plane m - 1, whose red
// neighbours are then all known.  Its 64 lanes by TY + 2 rows of pairs store
// every lane of the TY inner rows; the first and last rows form a ring whose
// red values the block's own black cells read.  One more wave, the halo,
// forms for each inner row the red values of the two pairs just beyond the
// row's ends (lanes 0 .. TY - 1 the west pair, 32 .. 31 + TY the east one),
// which the end lanes' black cells read from LDS.  Ring and halo values are
// recomputed (the neighbouring block forms and stores them too).  Red values
// are formed from the black plane as it stood before the launch, which the
// previous kernel copied to bold (this launch overwrites the black plane
// while other blocks still read it).  Each value comes from the same
// arithmetic on the same inputs as in the two separate passes, so the
// results are theirs bit for bit.
//
// The march is bound by memory latency, not bandwidth: a plane's work is a
// few dozen instructions per thread against one trip to HBM.  So every load
// of a plane is issued, unconditionally from clamped addresses, before the
// planes below it are computed, and waits only at its first use: one plane
// ahead in FP64, two in FP32, whose planes carry half the bytes each (with
// one plane in flight the FP32 march moved 3.2 TB/s, the FP64 one 4.3; a
// second FP64 plane would not fit the 128 registers a 1024-thread block
// allows).  The loop is unrolled by the depth so that the planes' registers
// rotate without copies.
constexpr int kRbfLanes = 64;
template <typename T>
constexpr int rbf_depth() { return sizeof(T) == 4 ? 3 : 2; }

template <typename T>
struct RbfLoads {
  T fw, fe, fs, fn, fd, fu;  // the faces of the red cell of plane m
  T bc;                      // its right-hand side
  T bo_u;                    // this pair's black value (before the launch) on plane m + 1
  T xo, yo;                  // black values beside the row ends and the ring rows on plane m
  T bb;                      // the right-hand side of this pair's black cell on plane m - 1
  T xf;                      // that cell's outer x-face, for a row's end lanes
};

// what a halo lane loads for the red cell of its pair on plane m
template <typename T>
struct RbfHaloLoads {
  T fw, fe, fs, fn, fd, fu, bc;
  T own, xo;   // black values (before the launch) of its pair and of the x-adjacent pair
  T ys, yn;    // of the rows beside it
  T zd, zu;    // of the planes below and above
};

template <typename T, int TY>
__global__ void __launch_bounds__(kRbfLanes * (TY + 3)) k_gs_rb_fine(Dims n, T h2, const T* __restrict__ bx,
                                                                     const T* __restrict__ by,
                                                                     const T* __restrict__ bz,
                                                                     const T* __restrict__ b, T* __restrict__ e,
                                                                     const T* __restrict__ bold, int KZ) {
  constexpr int R = TY + 2;
  static_assert(TY <= 32, "a halo lane per inner row and side");
  // One barrier per plane, between its red and black phases.  A wave may
  // then form the red values of plane m + 1 while another still reads those
  // of plane m - 1 in its black phase, so the red values, their y-faces and
  // the halo's values take three slots (plane mod 3); the black values
  // before the launch need two, since their readers (the red phase) all
  // finish before the barrier.
  __shared__ T BO[2][R][kRbfLanes];    // black values (as before the launch) of a plane
  __shared__ T RN[3][R][kRbfLanes];    // red values of a plane
  __shared__ T RYS[3][R][kRbfLanes];   // their south and north faces
  __shared__ T RYN[3][R][kRbfLanes];
  __shared__ T HH[3][2][R];            // the halo's red values: [plane mod 3][west, east][row]
  const SplitGeo sg = split_geo(n);
  const Tile tl = xcd_tile_flat();
  const int lane = threadIdx.x, r = threadIdx.y;
  const bool halo = r == R;            // the halo wave (wave-uniform)
  const int tx0 = tl.x * kRbfLanes;    // this block's first pair of a row
  const int k0 = tl.z * KZ, kz1 = min(k0 + KZ, n.nz);
  const size_t sz = (size_t)sg.hx * n.ny;   // pairs per plane
  const size_t fxs = (size_t)(n.nx + 1) * n.ny, fys = (size_t)n.nx * (n.ny + 1), fzs = (size_t)n.nx * n.ny;
  const auto clampz = [&](int m) { return (size_t)min(max(m, 0), n.nz - 1); };
  // ---- a main lane: pair ti of row j
  const int ti = tx0 + lane, j = tl.y * TY - 1 + r;
  const bool ok = !halo && ti < sg.hx && j >= 0 && j < n.ny;
  const bool inner = ok && r >= 1 && r <= TY;
  const int tic = min(ti, sg.hx - 1), jc = min(max(j, 0), n.ny - 1);
  const size_t prow = (size_t)tic + (size_t)sg.hx * jc;   // this pair in plane 0
  // the pairs whose black values the row ends and the ring rows read
  const size_t xrow = (size_t)(lane == 0 ? max(tic - 1, 0) : lane == kRbfLanes - 1 ? min(tic + 1, sg.hx - 1) : tic) +
                      (size_t)sg.hx * jc;
  const size_t yrow = (size_t)tic + (size_t)sg.hx * (r == 0 ? max(jc - 1, 0) : r == R - 1 ? min(jc + 1, n.ny - 1) : jc);
  // the outer x-face of a black cell on a row's end lane: the west face of
  // an even column on lane 0, the east face of an odd one on lane 63 (a
  // shuffle there would return the lane's own face)
  const int xfi = lane == 0 ? 2 * ti : 2 * ti + 2;
  // ---- a halo lane: the pair beyond the west (side 0) or east (side 1) row end, inner row hr
  const int side = lane >> 5, hr = (lane & 31) + 1;
  const int hp = side ? tx0 + kRbfLanes : tx0 - 1, hj = tl.y * TY - 1 + hr;
  const bool hok = halo && hr <= TY && hp >= 0 && hp < sg.hx && hj < n.ny;
  const int hpc = min(max(hp, 0), sg.hx - 1), hjc = min(hj, n.ny - 1);
  // face indices from the unclamped cell, kept in the face range: a ring
  // cell outside the grid holds the wall face it shares with the grid; at
  // m = -1 the up face is the bed, at m = nz the down face is the open top
  const auto load = [&](int m, RbfLoads<T>& L) {
    const size_t mc = clampz(m);
    const int iru = 2 * ti + ((j + m) & 1);
    const int irc = min(max(iru, 0), n.nx - 1);
    const size_t xf = (size_t)(n.nx + 1) * jc + fxs * mc;
    L.fw = bx[(size_t)min(max(iru, 0), n.nx) + xf];
    L.fe = bx[(size_t)min(max(iru + 1, 0), n.nx) + xf];
    L.fs = by[(size_t)irc + (size_t)n.nx * min(max(j, 0), n.ny) + fys * mc];
    L.fn = by[(size_t)irc + (size_t)n.nx * min(max(j + 1, 0), n.ny) + fys * mc];
    L.fd = bz[(size_t)irc + (size_t)n.nx * jc + fzs * (size_t)min(max(m, 0), n.nz)];
    L.fu = bz[(size_t)irc + (size_t)n.nx * jc + fzs * (size_t)min(max(m + 1, 0), n.nz)];
    L.bc = b[prow + sz * mc];
    L.bo_u = bold[prow + sz * clampz(m + 1)];
    L.xo = bold[xrow + sz * mc];
    L.yo = bold[yrow + sz * mc];
    L.bb = b[sg.P + prow + sz * clampz(m - 1)];
    L.xf = bx[(size_t)min(max(xfi, 0), n.nx) + (size_t)(n.nx + 1) * jc + fxs * clampz(m - 1)];
  };
  const auto load_h = [&](int m, RbfHaloLoads<T>& H) {
    const size_t mc = clampz(m);
    const int par = (hj + m) & 1;
    const int iru = 2 * hp + par;
    const int irc = min(max(iru, 0), n.nx - 1);
    const size_t xf = (size_t)(n.nx + 1) * hjc + fxs * mc;
    const size_t pr = (size_t)hpc + (size_t)sg.hx * hjc;
    H.fw = bx[(size_t)min(max(iru, 0), n.nx) + xf];
    H.fe = bx[(size_t)min(max(iru + 1, 0), n.nx) + xf];
    H.fs = by[(size_t)irc + (size_t)n.nx * hjc + fys * mc];
    H.fn = by[(size_t)irc + (size_t)n.nx * (hjc + 1) + fys * mc];
    H.fd = bz[(size_t)irc + (size_t)n.nx * hjc + fzs * mc];
    H.fu = bz[(size_t)irc + (size_t)n.nx * hjc + fzs * (mc + 1)];
    H.bc = b[pr + sz * mc];
    H.own = bold[pr + sz * mc];
    H.xo = bold[(size_t)min(max(par ? hpc + 1 : hpc - 1, 0), sg.hx - 1) + (size_t)sg.hx * hjc + sz * mc];
    H.ys = bold[(size_t)hpc + (size_t)sg.hx * max(hjc - 1, 0) + sz * mc];
    H.yn = bold[(size_t)hpc + (size_t)sg.hx * min(hjc + 1, n.ny - 1) + sz * mc];
    H.zd = bold[pr + sz * clampz(m - 1)];
    H.zu = bold[pr + sz * clampz(m + 1)];
  };
  T bo_d = bold[prow + sz * clampz(k0 - 2)], bo_c = bold[prow + sz * clampz(k0 - 1)];
  if (!(ok && k0 - 2 >= 0)) bo_d = (T)0;
  if (!(ok && k0 - 1 >= 0)) bo_c = (T)0;
  T rv1 = 0, rv2 = 0, fu1 = 0, fu2 = 0, fw1 = 0, fe1 = 0;
  // the halo wave's plane: the red value of its pair on plane m, to LDS
  const auto plane_h = [&](int m, const RbfHaloLoads<T>& H) {
    const int par = (hj + m) & 1;
    const int iru = 2 * hp + par;
    T rv = (T)0;
    if (hok && m >= 0 && m < n.nz && iru < n.nx) {
      const int mc = m;
      const T vw = par == 0 ? H.xo : H.own, ve = par == 0 ? H.own : H.xo;
      const T vd = m > 0 ? H.zd : (T)0, vu = m + 1 < n.nz ? H.zu : (T)0;
      const GsIn<T> g{H.fw, H.fe, H.fs, H.fn, H.fd, H.fu, H.ys, H.yn, vd, vu};
      rv = gs_combine<T>(n, g, h2, H.bc, iru, hj, mc, vw, ve);
    }
    if (hr <= TY) HH[(m + 3) % 3][side][hr] = rv;
    __syncthreads();
  };
  const auto plane = [&](int m, const RbfLoads<T>& L) {
    // ---- the red cell of this pair on plane m (ring rows included)
    const int mc = (int)clampz(m);
    const int par = (j + m) & 1;
    const int iru = 2 * ti + par;                     // possibly outside the grid
    const int irc = min(max(iru, 0), n.nx - 1);
    const bool live = ok && m >= 0 && m < n.nz;
    const T bo_u = (ok && m + 1 >= 0 && m + 1 < n.nz) ? L.bo_u : (T)0;
    // x neighbours: this pair's black cell and the adjacent pair's (the
    // adjacent lane; the row's end lanes loaded theirs)
    const T bl = __shfl_up(bo_c, 1, kRbfLanes), br = __shfl_down(bo_c, 1, kRbfLanes);
    const T xo = live ? L.xo : (T)0, yo = live ? L.yo : (T)0;
    const T vw = par == 0 ? (lane > 0 ? bl : xo) : bo_c;
    const T ve = par == 1 ? (lane < kRbfLanes - 1 ? br : xo) : bo_c;
    const T vs = r > 0 ? BO[m & 1][r - 1][lane] : yo;
    const T vn = r < R - 1 ? BO[m & 1][r + 1][lane] : yo;
    T rv = (T)0;
    if (live && iru < n.nx) {
      const GsIn<T> g{L.fw, L.fe, L.fs, L.fn, L.fd, L.fu, vs, vn, bo_d, bo_u};
      rv = gs_combine<T>(n, g, h2, L.bc, irc, jc, mc, vw, ve);
      if (inner && m >= k0 && m < kz1) e[prow + sz * mc] = rv;
    }
    const int sm = (m + 3) % 3, sb = (m + 2) % 3;   // the slots of planes m and m - 1
    RN[sm][r][lane] = rv;
    RYS[sm][r][lane] = L.fs;
    RYN[sm][r][lane] = L.fn;
    BO[(m + 1) & 1][r][lane] = bo_u;
    // the adjacent lanes' red values and x-faces of plane m - 1 (every lane
    // takes part in the shuffles)
    const T xfe = __shfl_up(fe1, 1, kRbfLanes), xrl = __shfl_up(rv1, 1, kRbfLanes);
    const T xfw = __shfl_down(fw1, 1, kRbfLanes), xrr = __shfl_down(rv1, 1, kRbfLanes);
    __syncthreads();
    // ---- the black cell of this pair on plane m - 1 (inner threads)
    const int mb = m - 1;
    if (inner && mb >= k0 && mb < kz1) {
      const int ib = iru;      // the black cell of plane m - 1 shares the column of plane m's red cell
      if (ib < n.nx) {
        const bool even = (ib & 1) == 0;
        const T bw = lane > 0 ? xfe : L.xf, be = lane < kRbfLanes - 1 ? xfw : L.xf;
        const T vwb = lane > 0 ? xrl : HH[sb][0][r], veb = lane < kRbfLanes - 1 ? xrr : HH[sb][1][r];
        const GsIn<T> g{even ? bw : fe1, even ? fw1 : be, RYN[sb][r - 1][lane], RYS[sb][r + 1][lane],
                        fu2, L.fd, RN[sb][r - 1][lane], RN[sb][r + 1][lane], rv2, rv};
        const T bb = L.bb;
        e[sg.P + prow + sz * (size_t)mb] = gs_combine<T>(n, g, h2, bb, ib, j, mb, even ? vwb : rv1, even ? rv1 : veb);
      }
    }
    rv2 = rv1;
    rv1 = rv;
    fu2 = fu1;
    fu1 = L.fu;
    fw1 = L.fw;
    fe1 = L.fe;
    bo_d = bo_c;
    bo_c = bo_u;
  };
  // plane p's loads sit in buffer (p - k0 + 1) % D; the halo wave and the
  // main waves pass the same planes, so they meet the same barriers (the
  // two-deep form is written out: as the general loop it spilled in FP64)
  constexpr int D = rbf_depth<T>();
  if (halo) {
    if constexpr (D == 2) {
      RbfHaloLoads<T> A, B;
      load_h(k0 - 1, A);
      __syncthreads();
      for (int m = k0 - 1; m <= kz1; m += 2) {
        load_h(m + 1, B);
        __builtin_amdgcn_sched_barrier(0);
        plane_h(m, A);
        if (m + 1 > kz1) break;
        load_h(m + 2, A);
        __builtin_amdgcn_sched_barrier(0);
        plane_h(m + 1, B);
      }
    } else {
      RbfHaloLoads<T> H[D];
#pragma unroll
      for (int q = 0; q < D - 1; ++q) load_h(k0 - 1 + q, H[q]);
      __syncthreads();
      for (int m = k0 - 1; m <= kz1; m += D) {
#pragma unroll
        for (int q = 0; q < D; ++q) {
          if (q > 0 && m + q > kz1) return;
          load_h(m + q + D - 1, H[(q + D - 1) % D]);
          __builtin_amdgcn_sched_barrier(0);
          plane_h(m + q, H[q]);
        }
      }
    }
    return;
  }
  if constexpr (D == 2) {
    RbfLoads<T> A, B;
    load(k0 - 1, A);
    BO[(k0 - 1) & 1][r][lane] = bo_c;
    __syncthreads();
    for (int m = k0 - 1; m <= kz1; m += 2) {
      load(m + 1, B);
      __builtin_amdgcn_sched_barrier(0);
      plane(m, A);
      if (m + 1 > kz1) break;
      load(m + 2, A);
      __builtin_amdgcn_sched_barrier(0);
      plane(m + 1, B);
    }
  } else {
    RbfLoads<T> A[D];
#pragma unroll
    for (int q = 0; q < D - 1; ++q) load(k0 - 1 + q, A[q]);
    BO[(k0 - 1) & 1][r][lane] = bo_c;
    __syncthreads();
    for (int m = k0 - 1; m <= kz1; m += D) {
#pragma unroll
      for (int q = 0; q < D; ++q) {
        if (q > 0 && m + q > kz1) return;
        load(m + q + D - 1, A[(q + D - 1) % D]);
        __builtin_amdgcn_sched_barrier(0);
        plane(m + q, A[q]);
      }
    }
  }
}

// A x (without 1/h^2) and the residual b - A x of one cell from its value,
// its neighbours' (a wall neighbour given as the cell's own value) and its six
// faces; up: the cell is below the top row (else the open top's ghost term
// 2 beta_top x_c)
template <typename T>
__device__ __forceinline__ T cell_A(T xc, T xw, T xe, T xs, T xn, T xd, T xu, T cw, T ce, T cs, T cn, T cd, T bu,
                                    bool up) {
  T acc = cw * (xc - xw) + ce * (xc - xe) + cs * (xc - xs) + cn * (xc - xn) + cd * (xc - xd);
  acc += up ? bu * (xc - xu) : (T)2 * bu * xc;
  return acc;
}
template <typename T>
__device__ __forceinline__ T cell_resid(T bcell, T ih2, T xc, T xw, T xe, T xs, T xn, T xd, T xu, T cw, T ce, T cs,
                                        T cn, T cd, T bu, bool up) {
  return bcell - ih2 * cell_A<T>(xc, xw, xe, xs, xn, xd, xu, cw, ce, cs, cn, cd, bu, up);
}

// coarse rhs = mean over the children of the fine residual b - A e (fine b,
// e colour-split; the coarse b colour-split when csplit, else natural).  A
// block takes a tile of fine cells (32 x 4 x 2; 64 x 1 x 4 in 2-D), one
// thread per cell: each computes its cell's residual into LDS, then one
// thread per coarse cell of the tile sums its children from LDS in the
// order (dk, dj, di).  Tile extents are even, so a coarse cell's children
// never straddle two tiles.
template <typename T>
__global__ void __launch_bounds__(256) k_resid_restrict(Dims nf, int fx, int fy, int fz, T ih2,
                                                        const T* __restrict__ bx, const T* __restrict__ by,
                                                        const T* __restrict__ bz, const T* __restrict__ b,
                                                        const T* __restrict__ e, Dims nc, int csplit, T inv,
                                                        T* __restrict__ bc) {
  __shared__ T sr[256];
  const int TX = blockDim.x, TY = blockDim.y;
  const int tx = threadIdx.x, ty = threadIdx.y, tz = threadIdx.z;
  const Tile tl = xcd_tile();
  const int i = tl.x * TX + tx, j = tl.y * TY + ty, k = tl.z * blockDim.z + tz;
  // Index arithmetic in 32 bits (every array of a level has fewer than 2^31
  // entries): the kernel issues more integer instructions than loads, and
  // 64-bit products cost several each.
  const int hx = (nf.nx + 1) >> 1, P = hx * nf.ny * nf.nz;
  const int sxy = nf.nx * nf.ny, sz = hx * nf.ny;
  T r = 0;
  if (i < nf.nx && j < nf.ny && k < nf.nz) {
    const int c = i + nf.nx * j + sxy * k;
    const int fxi = i + (nf.nx + 1) * (j + nf.ny * k);
    const int fyi = i + nf.nx * (j + (nf.ny + 1) * k);
    const int par = (i + j + k) & 1;
    const int rowp = hx * (j + nf.ny * k);          // first pair of the cell's row
    const int own = par * P + (i >> 1) + rowp;      // the cell's own entry
    const int oth = (1 - par) * P + rowp;           // the other colour's row (all six neighbours)
    const int pc = oth + (i >> 1);
    // walls read the cell's own entry, so their (x_c - x_nb) is zero
    const T xc = e[own];
    const T xw = e[i > 0 ? oth + ((i - 1) >> 1) : own];
    const T xe = e[i < nf.nx - 1 ? oth + ((i + 1) >> 1) : own];
    const T xs = e[j > 0 ? pc - hx : own];
    const T xn = e[j < nf.ny - 1 ? pc + hx : own];
    const T xd = e[k > 0 ? pc - sz : own];
    const T xu = e[k < nf.nz - 1 ? pc + sz : own];
    const T cw = bx[fxi], ce = bx[fxi + 1], cs = by[fyi], cn = by[fyi + nf.nx], cd = bz[c], bu = bz[c + sxy];
    const T bcell = b[own];
    // all loads above are in flight together: the compiler may not sink the
    // up neighbour's load into the branch that uses it
    __builtin_amdgcn_sched_barrier(0);
    r = cell_resid<T>(bcell, ih2, xc, xw, xe, xs, xn, xd, xu, cw, ce, cs, cn, cd, bu, k < nf.nz - 1);
  }
  const int t = (tz * TY + ty) * TX + tx;
  sr[t] = r;
  __syncthreads();
  // each coarse cell of the tile is summed by the thread of its corner child
  // (the factors are 1 or 2 and the tile's extents even, so shifts replace
  // divisions)
  const int sx = fx - 1, sy = fy - 1, sz2 = fz - 1;
  if ((tx & sx) | (ty & sy) | (tz & sz2)) return;
  const int CX = TX >> sx, CY = TY >> sy, CZ = (int)blockDim.z >> sz2;
  const int I = tl.x * CX + (tx >> sx), J = tl.y * CY + (ty >> sy), K = tl.z * CZ + (tz >> sz2);
  if (I >= nc.nx || J >= nc.ny || K >= nc.nz) return;
  T sum = 0;
  for (int dk = 0; dk < fz; ++dk)
    for (int dj = 0; dj < fy; ++dj)
      for (int di = 0; di < fx; ++di) sum += sr[((tz + dk) * TY + ty + dj) * TX + tx + di];
  const int chx = (nc.nx + 1) >> 1, cP = chx * nc.ny * nc.nz;
  const int ci = csplit ? ((I + J + K) & 1) * cP + (I >> 1) + chx * (J + nc.ny * K) : I + nc.nx * (J + nc.ny * K);
  bc[ci] = sum * inv;
}

// The same on a level whose extents are all even and which is halved in
// every direction, so that coarse cell (I, J, K) holds fine pair I of rows
// 2J, 2J + 1 and planes 2K, 2K + 1.  One thread per pair of cells: every
// load of a wave is 64 consecutive pairs of one colour, or the faces of one
// row (y and z faces as two-element vector loads), and a pair's x
// neighbours come from the adjacent lanes; a cell-per-thread tile issues
// half as many loads again, at stride two.  A block takes 64 pairs x 2 rows
// x 2 planes, the children of 64 coarse cells, and its first wave sums each
// coarse cell's eight residuals in k_resid_restrict's order (dk, dj, di), so
// the result is the same.
template <typename T>
__global__ void __launch_bounds__(256) k_resid_restrict_pairs(Dims nf, T ih2, const T* __restrict__ bx,
                                                              const T* __restrict__ by, const T* __restrict__ bz,
                                                              const T* __restrict__ b, const T* __restrict__ e,
                                                              Dims nc, int csplit, T inv, T* __restrict__ bc,
                                                              FaceTab<T> ft) {
  using T2 = T __attribute__((ext_vector_type(2)));
  __shared__ T sr[2][2][2][64];   // [dk][dj][di][lane]
  const Tile tl = xcd_tile();
  const int lane = threadIdx.x, dj = threadIdx.y, dk = threadIdx.z;
  const int hx = nf.nx >> 1;
  const int ti = tl.x * 64 + lane, j = 2 * tl.y + dj, k = 2 * tl.z + dk;
  const bool live = ti < hx;
  const int tc = live ? ti : hx - 1;   // lanes past the row's end work on its last pair and store nothing
  // 32-bit index arithmetic: every array of a level has fewer than 2^31 entries
  const int P = hx * nf.ny * nf.nz, sz = hx * nf.ny, sxy = nf.nx * nf.ny;
  const int pos = tc + hx * (j + nf.ny * k);
  const int par = (j + k) & 1;   // colour of the pair's first cell A (i = 2 tc); B is i = 2 tc + 1
  const int pa = par * P + pos, pb = (1 - par) * P + pos;
  const bool W = tc > 0, E = tc < hx - 1, S = j > 0, N = j < nf.ny - 1, D = k > 0, U = k < nf.nz - 1;
  // A's y and z neighbours have B's colour, and B's have A's; a wall
  // neighbour reads the cell's own entry
  const T xa = e[pa], xb = e[pb];
  const T xas = e[S ? pb - hx : pa], xan = e[N ? pb + hx : pa], xad = e[D ? pb - sz : pa], xau = e[U ? pb + sz : pa];
  const T xbs = e[S ? pa - hx : pb], xbn = e[N ? pa + hx : pb], xbd = e[D ? pa - sz : pb], xbu = e[U ? pa + sz : pb];
  // outside the wavefront: lane 0 loads A's west neighbour (B of the pair
  // before), lane 63 B's east one (A of the pair after)
  const T xo = e[lane == 0 ? (W ? pb - 1 : pa) : lane == 63 ? (E ? pa + 1 : pb) : pa];
  const int fx = 2 * tc + (nf.nx + 1) * (j + nf.ny * k);
  const int fy = 2 * tc + nf.nx * (j + (nf.ny + 1) * k);
  const int c = 2 * tc + nf.nx * j + sxy * k;
  // the faces: each line (the x-line j, k; y-lines j, j + 1; z-lines k, k + 1)
  // through its table where it is one value (the wavefront is one row), else
  // loaded under a scalar branch; picked after every load is in flight
  const int ju = __builtin_amdgcn_readfirstlane(j), ku = __builtin_amdgcn_readfirstlane(k);
  T tx, ts, tn, td, tu;
  const bool ux = line_val(ft.x, ju + nf.ny * ku, tx), us = line_val(ft.y, ju + (nf.ny + 1) * ku, ts);
  const bool un = line_val(ft.y, ju + 1 + (nf.ny + 1) * ku, tn), ud = line_val(ft.z, ju + nf.ny * ku, td);
  const bool uu = line_val(ft.z, ju + nf.ny * (ku + 1), tu);
  // A's west face; the face between A and B; B's east face, for lane 63.  A
  // face of a one-value line is left unset until it is taken from the
  // table below: zeroing it on that side of the branch made the FP32
  // instance wait there for every load in flight.
  T fwa, fab, feo;
  T2 fs, fn, fd, fu;
  if (!ux) {
    fwa = bx[fx];
    fab = bx[fx + 1];
    feo = bx[lane == 63 ? fx + 2 : fx];
  }
  if (!us) fs = *reinterpret_cast<const T2*>(by + fy);
  if (!un) fn = *reinterpret_cast<const T2*>(by + fy + nf.nx);
  if (!ud) fd = *reinterpret_cast<const T2*>(bz + c);
  if (!uu) fu = *reinterpret_cast<const T2*>(bz + c + sxy);
  const T ba = b[pa], bb = b[pb];
  __builtin_amdgcn_sched_barrier(0);
  if (ux) {   // walls: face 0 and face nx (nx is even, so 2 tc + 1 is inside)
    fwa = tc > 0 ? tx : (T)0;
    fab = tx;
    feo = 2 * tc + 2 < nf.nx ? tx : (T)0;
  }
  if (us) fs = T2{ts, ts};
  if (un) fn = T2{tn, tn};
  if (ud) fd = T2{td, td};
  if (uu) fu = T2{tu, tu};
  const T xbl = __shfl_up(xb, 1, 64), xar = __shfl_down(xa, 1, 64), fwr = __shfl_down(fwa, 1, 64);
  const T xaw = W ? (lane > 0 ? xbl : xo) : xa;
  const T xbe = E ? (lane < 63 ? xar : xo) : xb;
  const T feb = lane < 63 ? fwr : feo;
  sr[dk][dj][0][lane] = cell_resid<T>(ba, ih2, xa, xaw, xb, xas, xan, xad, xau, fwa, fab, fs.x, fn.x, fd.x, fu.x, U);
  sr[dk][dj][1][lane] = cell_resid<T>(bb, ih2, xb, xa, xbe, xbs, xbn, xbd, xbu, fab, feb, fs.y, fn.y, fd.y, fu.y, U);
  __syncthreads();
  if (dj | dk) return;
  T sum = 0;
#pragma unroll
  for (int qk = 0; qk < 2; ++qk)
#pragma unroll
    for (int qj = 0; qj < 2; ++qj)
#pragma unroll
      for (int qi = 0; qi < 2; ++qi) sum += sr[qk][qj][qi][lane];
  if (!live) return;
  const int I = ti, J = tl.y, K = tl.z;
  const int chx = (nc.nx + 1) >> 1, cP = chx * nc.ny * nc.nz;
  const int ci = csplit ? ((I + J + K) & 1) * cP + (I >> 1) + chx * (J + nc.ny * K) : I + nc.nx * (J + nc.ny * K);
  bc[ci] = sum * inv;
}

// Both cells of V adjacent pairs of a row and what the operator reads around
// them, for the wide kernels.  A is a pair's first cell (even column, colour
// par = (j + k) & 1), B its second; pa, pb: their entries in v's two planes.
// A's y and z neighbours have B's colour, and B's have A's; a wall neighbour
// reads the cell's own entry.
template <typename T, int V>
struct PairNb {
  T a[V], b[V], as[V], an[V], ad[V], au[V], bs[V], bn[V], bd[V], bu[V], w, e;
  __device__ __forceinline__ void load(const T* __restrict__ v, size_t pa, size_t pb, int hx, size_t sz, int tp, bool S,
                                       bool N, bool D, bool U) {
    vload<T, V>(a, v + pa);
    vload<T, V>(b, v + pb);
    vload<T, V>(as, v + (S ? pb - hx : pa));
    vload<T, V>(an, v + (N ? pb + hx : pa));
    vload<T, V>(ad, v + (D ? pb - sz : pa));
    vload<T, V>(au, v + (U ? pb + sz : pa));
    vload<T, V>(bs, v + (S ? pa - hx : pb));
    vload<T, V>(bn, v + (N ? pa + hx : pb));
    vload<T, V>(bd, v + (D ? pa - sz : pb));
    vload<T, V>(bu, v + (U ? pa + sz : pb));
    w = v[tp > 0 ? pb - 1 : pa];               // west of the first A
    e = v[tp + V < hx ? pa + V : pb + V - 1];  // east of the last B
  }
};
// Their faces: each line through its table where it is one value, else loaded
// under a scalar branch (as FaceLd), in loads of up to 16 bytes per lane.
template <typename T, int V>
struct PairFaces {
  static constexpr int W = 16 / sizeof(T) < 2 * V ? 16 / sizeof(T) : 2 * V;
  T t[5];
  bool u[5];
  T x[2 * V + 1], s[2 * V], n[2 * V], d[2 * V], up[2 * V];
  __device__ __forceinline__ static void row(T* d, const T* __restrict__ p) {
#pragma unroll
    for (int q = 0; q < 2 * V; q += W) vload<T, W>(*reinterpret_cast<T(*)[W]>(d + q), p + q);
  }
  __device__ __forceinline__ void load(const Dims& nn, const FaceTab<T>& ft, const T* __restrict__ bx,
                                       const T* __restrict__ by, const T* __restrict__ bz, int ju, int ku, int tp,
                                       int j, int k) {
    u[0] = line_val(ft.x, ju + nn.ny * ku, t[0]);
    u[1] = line_val(ft.y, ju + (nn.ny + 1) * ku, t[1]);
    u[2] = line_val(ft.y, ju + 1 + (nn.ny + 1) * ku, t[2]);
    u[3] = line_val(ft.z, ju + nn.ny * ku, t[3]);
    u[4] = line_val(ft.z, ju + nn.ny * (ku + 1), t[4]);
    const size_t fx = 2 * tp + (size_t)(nn.nx + 1) * (j + (size_t)nn.ny * k);
    const size_t fy = 2 * tp + (size_t)nn.nx * (j + (size_t)(nn.ny + 1) * k);
    const size_t fz = 2 * tp + (size_t)nn.nx * (j + (size_t)nn.ny * k);
    if (!u[0]) {
      row(x, bx + fx);
      x[2 * V] = bx[fx + 2 * V];
    }
    if (!u[1]) row(s, by + fy);
    if (!u[2]) row(n, by + fy + nn.nx);
    if (!u[3]) row(d, bz + fz);
    if (!u[4]) row(up, bz + fz + (size_t)nn.nx * nn.ny);
  }
  // A v at the p-th cell of the lane's 2 V (p = 2 q: A of pair q), without
  // 1/h^2; i: its column (nx is even, so a pair's middle face is inside);
  // inner: the cell is below the top row
  __device__ __forceinline__ T apply(const Dims& nn, int p, int i, T c, T w, T e, T vs, T vn, T vd, T vu,
                                     bool inner) const {
    const T cw = u[0] ? (i > 0 ? t[0] : (T)0) : x[p], ce = u[0] ? (i < nn.nx - 1 ? t[0] : (T)0) : x[p + 1];
    return cell_A<T>(c, w, e, vs, vn, vd, vu, cw, ce, u[1] ? t[1] : s[p], u[2] ? t[2] : n[p], u[3] ? t[3] : d[p],
                     u[4] ? t[4] : up[p], inner);
  }
  // both cells of pair q
  __device__ __forceinline__ void apply2(const Dims& nn, const PairNb<T, V>& v, int q, int tp, bool inner, T& a,
                                         T& b) const {
    const int i = 2 * (tp + q);
    const T w = q > 0 ? v.b[q > 0 ? q - 1 : 0] : v.w, e = q < V - 1 ? v.a[q < V - 1 ? q + 1 : q] : v.e;
    a = apply(nn, 2 * q, i, v.a[q], w, v.b[q], v.as[q], v.an[q], v.ad[q], v.au[q], inner);
    b = apply(nn, 2 * q + 1, i + 1, v.b[q], v.a[q], e, v.bs[q], v.bn[q], v.bd[q], v.bu[q], inner);
  }
};

// k_resid_restrict_pairs with V adjacent pairs per lane (the wide passes' levels)
template <typename T, int V>
__global__ void __launch_bounds__(256) k_resid_restrict_wide(Dims nf, T ih2, const T* __restrict__ bx,
                                                             const T* __restrict__ by, const T* __restrict__ bz,
                                                             const T* __restrict__ b, const T* __restrict__ e,
                                                             Dims nc, int csplit, T inv, T* __restrict__ bc,
                                                             FaceTab<T> ft) {
  __shared__ T sr[2][2][2][V][64];   // [dk][dj][di][pair of the lane][lane]
  const Tile tl = xcd_tile();
  const int lane = threadIdx.x, dj = threadIdx.y, dk = threadIdx.z;
  const int hx = nf.nx >> 1;
  const int tpr = V * (tl.x * 64 + lane), j = 2 * tl.y + dj, k = 2 * tl.z + dk;
  const bool live = tpr < hx;
  const int tp = min(tpr, hx - V);   // a lane past the row's end stores nothing
  const size_t P = (size_t)hx * nf.ny * nf.nz, sz = (size_t)hx * nf.ny;
  const size_t pos = tp + (size_t)hx * (j + (size_t)nf.ny * k);
  const int par = (j + k) & 1;
  const size_t pa = par * P + pos, pb = (1 - par) * P + pos;
  PairNb<T, V> v;
  v.load(e, pa, pb, hx, sz, tp, j > 0, j < nf.ny - 1, k > 0, k < nf.nz - 1);
  T ba[V], bb[V];
  vload<T, V>(ba, b + pa);
  vload<T, V>(bb, b + pb);
  PairFaces<T, V> F;
  F.load(nf, ft, bx, by, bz, __builtin_amdgcn_readfirstlane(j), __builtin_amdgcn_readfirstlane(k), tp, j, k);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < V; ++q) {
    T a, c;
    F.apply2(nf, v, q, tp, k < nf.nz - 1, a, c);
    sr[dk][dj][0][q][lane] = ba[q] - ih2 * a;
    sr[dk][dj][1][q][lane] = bb[q] - ih2 * c;
  }
  __syncthreads();
  if ((dj | dk) || !live) return;
  const int J = tl.y, K = tl.z;
  const int chx = (nc.nx + 1) >> 1, cP = chx * nc.ny * nc.nz;
#pragma unroll
  for (int q = 0; q < V; ++q) {
    T sum = 0;
#pragma unroll
    for (int qk = 0; qk < 2; ++qk)
#pragma unroll
      for (int qj = 0; qj < 2; ++qj)
#pragma unroll
        for (int qi = 0; qi < 2; ++qi) sum += sr[qk][qj][qi][q][lane];
    const int I = tp + q;
    const int ci = csplit ? ((I + J + K) & 1) * cP + (I >> 1) + chx * (J + nc.ny * K) : I + nc.nx * (J + nc.ny * K);
    bc[ci] = sum * inv;
  }
}

// colour-split fine correction += parent's coarse correction (nu_post == 0)
template <typename T>
__global__ void __launch_bounds__(256) k_prolong(Dims nf, int sx, int sy, int sz, T* __restrict__ e, Dims nc,
                                                 int csplit, const T* __restrict__ ec) {
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= nf.nx || j >= nf.ny || k >= nf.nz) return;
  const SplitGeo sg = split_geo(nf), cg = split_geo(nc);
  e[sidx(nf, sg, i, j, k)] += ec[lidx(nc, cg, csplit != 0, i >> sx, j >> sy, k >> sz)];
}

// natural <-> colour-split copies (the finest level's edge cases)
template <typename T>
__global__ void __launch_bounds__(256) k_split_copy(Dims n, const T* __restrict__ src, T* __restrict__ dst,
                                                    int to_split) {
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const SplitGeo sg = split_geo(n);
  const size_t c = i + (size_t)n.nx * (j + (size_t)n.ny * k), s = sidx(n, sg, i, j, k);
  if (to_split)
    dst[s] = src[c];
  else
    dst[c] = src[s];
}

// 1 / (sum of the cell's face coefficients, top face counted twice), stored
// colour-split (levels above the tail) or natural (tail levels)
template <typename T>
__global__ void __launch_bounds__(256) k_invdiag(Dims n, const T* __restrict__ bx, const T* __restrict__ by,
                                                 const T* __restrict__ bz, int split, T* __restrict__ invd) {
  const Tile tl = xcd_tile();
  const int i = tl.x * blockDim.x + threadIdx.x;
  const int j = tl.y * blockDim.y + threadIdx.y;
  const int k = tl.z * blockDim.z + threadIdx.z;
  if (i >= n.nx || j >= n.ny || k >= n.nz) return;
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t c = i + (size_t)n.nx * j + sxy * k;
  const size_t fx = i + (size_t)(n.nx + 1) * (j + (size_t)n.ny * k);
  const size_t fy = i + (size_t)n.nx * (j + (size_t)(n.ny + 1) * k);
  const T bu = bz[c + sxy];
  const T diag = bx[fx] + bx[fx + 1] + by[fy] + by[fy + n.nx] + bz[c] + (k == n.nz - 1 ? (T)2 * bu : bu);
  invd[lidx(n, split_geo(n), split != 0, i, j, k)] = (T)1 / diag;
}

// Coarse face coefficient of component C at coarse face (I, J, K): the mean
// of the fine faces covering it, summed in the order (dk, dj, di).
// (the coarsening factors fx, fy, fz are 1 or 2).  The candidate fine faces
// are loaded through indices clamped into the array (coarse_face_load), and
// those within the factors summed in the order (dk, dj, di)
// (coarse_face_sum); a kernel loads all six faces before it sums any, so
// that every load is in flight before the first wait.
template <typename T>
struct FaceIn {
  T v[2][2][2];   // [dk][dj][di]
};
template <typename T, int C>
__device__ __forceinline__ FaceIn<T> coarse_face_load(const Dims& nf, int fx, int fy, int fz,
                                                      const T* __restrict__ fb, int I, int J, int K) {
  const int fmx = nf.nx + (C == 0), fmy = nf.ny + (C == 1), fmz = nf.nz + (C == 2);
  FaceIn<T> f;
#pragma unroll
  for (int dk = 0; dk < 2; ++dk)
#pragma unroll
    for (int dj = 0; dj < 2; ++dj)
#pragma unroll
      for (int di = 0; di < 2; ++di) {
        const int i = min(I * fx + di, fmx - 1), j = min(J * fy + dj, fmy - 1), k = min(K * fz + dk, fmz - 1);
        f.v[dk][dj][di] = fb[i + (size_t)fmx * (j + (size_t)fmy * k)];
      }
  return f;
}
template <typename T, int C>
__device__ __forceinline__ T coarse_face_sum(int fx, int fy, int fz, const FaceIn<T>& f) {
  const int ni = (C == 0) ? 1 : fx, nj = (C == 1) ? 1 : fy, nk = (C == 2) ? 1 : fz;
  T sum = 0;
#pragma unroll
  for (int dk = 0; dk < 2; ++dk)
#pragma unroll
    for (int dj = 0; dj < 2; ++dj)
#pragma unroll
      for (int di = 0; di < 2; ++di)
        if (dk < nk && dj < nj && di < ni) sum += f.v[dk][dj][di];
  return sum / (T)(ni * nj * nk);
}

// One coarse level of the hierarchy in one launch: each coarse cell forms its
// six face coefficients from the fine level, writes the faces it owns (its
// lower faces, and its upper ones on the grid's upper edges) and its 1/D
// (the sum of its faces, the top face twice, as in k_invdiag), colour-split
// (split) or natural.  A face shared by two cells is formed by both with the
// same arithmetic, and written once.
template <typename T>
__device__ __forceinline__ void coarsen_cell(const Dims& nf, int fx, int fy, int fz, const T* __restrict__ fbx,
                                             const T* __restrict__ fby, const T* __restrict__ fbz, const Dims& nc,
                                             T* __restrict__ cbx, T* __restrict__ cby, T* __restrict__ cbz, bool split,
                                             T* __restrict__ invd, int I, int J, int K) {
  const FaceIn<T> fw = coarse_face_load<T, 0>(nf, fx, fy, fz, fbx, I, J, K);
  const FaceIn<T> fe = coarse_face_load<T, 0>(nf, fx, fy, fz, fbx, I + 1, J, K);
  const FaceIn<T> fs = coarse_face_load<T, 1>(nf, fx, fy, fz, fby, I, J, K);
  const FaceIn<T> fn = coarse_face_load<T, 1>(nf, fx, fy, fz, fby, I, J + 1, K);
  const FaceIn<T> fd = coarse_face_load<T, 2>(nf, fx, fy, fz, fbz, I, J, K);
  const FaceIn<T> fu = coarse_face_load<T, 2>(nf, fx, fy, fz, fbz, I, J, K + 1);
  // (the barrier keeps the compiler from sinking a load into the branch of
  // the sum that uses it)
  __builtin_amdgcn_sched_barrier(0);
  const T bw = coarse_face_sum<T, 0>(fx, fy, fz, fw), be = coarse_face_sum<T, 0>(fx, fy, fz, fe);
  const T bs = coarse_face_sum<T, 1>(fx, fy, fz, fs), bn = coarse_face_sum<T, 1>(fx, fy, fz, fn);
  const T bd = coarse_face_sum<T, 2>(fx, fy, fz, fd), bu = coarse_face_sum<T, 2>(fx, fy, fz, fu);
  const size_t fxi = I + (size_t)(nc.nx + 1) * (J + (size_t)nc.ny * K);
  const size_t fyi = I + (size_t)nc.nx * (J + (size_t)(nc.ny + 1) * K);
  const size_t c = I + (size_t)nc.nx * (J + (size_t)nc.ny * K);
  const size_t sxy = (size_t)nc.nx * nc.ny;
  cbx[fxi] = bw;
  if (I == nc.nx - 1) cbx[fxi + 1] = be;
  cby[fyi] = bs;
  if (J == nc.ny - 1) cby[fyi + nc.nx] = bn;
  cbz[c] = bd;
  if (K == nc.nz - 1) cbz[c + sxy] = bu;
  const T diag = bw + be + bs + bn + bd + (K == nc.nz - 1 ? (T)2 * bu : bu);
  invd[lidx(nc, split_geo(nc), split, I, J, K)] = (T)1 / diag;
}
template <typename T>
__global__ void __launch_bounds__(256) k_coarsen_level(Dims nf, int fx, int fy, int fz, const T* __restrict__ fbx,
                                                       const T* __restrict__ fby, const T* __restrict__ fbz,
                                                       Dims nc, T* __restrict__ cbx, T* __restrict__ cby,
                                                       T* __restrict__ cbz, int split, T* __restrict__ invd) {
  const Tile tl = xcd_tile();
  const int I = tl.x * blockDim.x + threadIdx.x;
  const int J = tl.y * blockDim.y + threadIdx.y;
  const int K = tl.z * blockDim.z + threadIdx.z;
  if (I >= nc.nx || J >= nc.ny || K >= nc.nz) return;
  coarsen_cell<T>(nf, fx, fy, fz, fbx, fby, fbz, nc, cbx, cby, cbz, split != 0, invd, I, J, K);
}
// The small coarse levels (kCoarsenChain cells at most, all in the tail) one
// after the other in one workgroup, each from the one before: a launch of 3.4 us
// per level otherwise
template <typename T>
__global__ void __launch_bounds__(1024) k_coarsen_chain(CoarsenChain<T> D) {
#pragma unroll 1
  for (int l = 1; l < D.nl; ++l) {
    const Dims nc = D.n[l];
    const float inx = 1.0f / (float)nc.nx, iny = 1.0f / (float)nc.ny;
#pragma unroll 1
    for (int c = threadIdx.x; c < nc.nx * nc.ny * nc.nz; c += 1024) {
      const int r = (int)(((float)c + 0.5f) * inx), K = (int)(((float)r + 0.5f) * iny);
      coarsen_cell<T>(D.n[l - 1], D.f[l - 1][0], D.f[l - 1][1], D.f[l - 1][2], D.bx[l - 1], D.by[l - 1], D.bz[l - 1], nc,
                      D.bx[l], D.by[l], D.bz[l], false, D.invd[l], c - r * nc.nx, r - K * nc.ny, K);
    }
    __threadfence_block();
    __syncthreads();
  }
}

// ------------------------------------------------------- coarse-level tail
// Every level from the first tail level down to the coarsest runs in one
// workgroup, so a smoothing pass costs a barrier instead of a launch: the first
// level (and without a matrix the coarsest) in registers (RegLevel), the ones
// between with coefficients, 1/D, right-hand sides and corrections in LDS, and
// from the first level of at most kTailMatrixCells down a product with the
// cycle's matrix.  Each thread decodes its cell pairs once per level visit, and a
// pass is its loads and its arithmetic.
//
// A launch runs every instruction of this kernel a few times at most, on a
// compute unit whose instruction cache holds none of them: with each level's
// passes written out for both colours and directions it was 54 KB of code, and
// fetching it took more of the 20 us of a 128 x 64 x 64 cycle's tail than the
// passes.  So there is one body: a loop over the level visits, one loop over
// a visit's passes, and the colour a number.
//
// Walls carry beta = 0 and every correction in LDS is finite (the tail zeroes
// them all before its first level), so a wall term beta_f e_nb is an exact
// zero and the passes add it unconditionally; only the open top face, whose
// coefficient is not zero, is dropped by a select.
// t / n for 0 <= t < 8192 with inv = 1.0f / n, exact ((t + 1/2) / n is at least
// 1/(2n) from a whole number, and the product's error below 2^-10 / n): an
// integer division by a number that is not a constant takes some thirty
// instructions
__device__ __forceinline__ int tail_div(int t, float inv) { return (int)(((float)t + 0.5f) * inv); }

// num / D from inv = 1 / D, rounded, and what that rounding left out, rest =
// (1 - D inv) inv: the rounded quotient, as the separate passes' division gives
// it, for one more multiplication.  The product with inv alone is a unit
// further off, and always to the same side in a cell: after the coarsest
// level's 40 passes the cycle's error against extended precision was 2.6
// times the dividing passes' (25 x 9 x 13: FP64 1.5e-16 against 3.8e-16, FP32 0.7e-7
// against 2.0e-7).
template <typename T>
__device__ __forceinline__ T fused(T a, T b, T c) {
  if constexpr (sizeof(T) == 8)
    return __builtin_fma(a, b, c);
  else
    return __builtin_fmaf(a, b, c);
}
template <typename T>
__device__ __forceinline__ float inv_rest(T diag, T inv) { return (float)(fused<T>(-diag, inv, (T)1) * inv); }
template <typename T>
__device__ __forceinline__ T quotient(T num, T inv, float rest) { return fused<T>(num, inv, num * (T)rest); }

struct TailCell {
  int c;                  // cell index (b, e, 1/D, bz of the lower face)
  int fx, fy;             // west x-face and south y-face
  int w, e, s, n, d, u;   // neighbour cells; the cell itself through a wall or the top
  bool ok, top;           // the cell exists (i < nx; else the pair's other cell); it lies in the top row
};
// a thread's pairs: t and t + nthr
struct TailPairs {
  int np;
  int i[2], j[2], k[2];                          // first column, row, plane
  int c[2], fx[2], fy[2];                        // cell, west x-face and south y-face of the first column
  int ds[2], dn[2], dd[2], du[2];                // distances of the neighbours, zero through a wall or the top
};
__device__ __forceinline__ void tail_decode(const Dims& n, int tid, int nthr, TailPairs& tp) {
  const int hx = (n.nx + 1) >> 1, sxy = n.nx * n.ny;
  const int NP = hx * n.ny * n.nz;
  const float ihx = 1.0f / (float)hx, iny = 1.0f / (float)n.ny;
  tp.np = tid < NP ? (tid + nthr < NP ? 2 : 1) : 0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int t = min(tid + q * nthr, NP - 1), r = tail_div(t, ihx);
    const int k = tail_div(r, iny), j = r - k * n.ny, i = 2 * (t - r * hx);
    tp.i[q] = i;
    tp.j[q] = j;
    tp.k[q] = k;
    tp.c[q] = i + n.nx * j + sxy * k;
    tp.fx[q] = i + (n.nx + 1) * (j + n.ny * k);
    tp.fy[q] = i + n.nx * (j + (n.ny + 1) * k);
    tp.ds[q] = j > 0 ? -n.nx : 0;
    tp.dn[q] = j < n.ny - 1 ? n.nx : 0;
    tp.dd[q] = k > 0 ? -sxy : 0;
    tp.du[q] = k < n.nz - 1 ? sxy : 0;
  }
}
// pair q's cell of a colour
__device__ __forceinline__ TailCell tail_cell(const Dims& n, const TailPairs& tp, int q, int colour) {
  const int o = (tp.j[q] + tp.k[q] + colour) & 1;
  TailCell x;
  x.ok = q < tp.np && tp.i[q] + o < n.nx;
  const int oc = tp.i[q] + o < n.nx ? o : 0, i = tp.i[q] + oc;
  x.top = tp.du[q] == 0;
  x.c = tp.c[q] + oc;
  x.fx = tp.fx[q] + oc;
  x.fy = tp.fy[q] + oc;
  x.w = x.c - (i > 0 ? 1 : 0);
  x.e = x.c + (i < n.nx - 1 ? 1 : 0);
  x.s = x.c + tp.ds[q];
  x.n = x.c + tp.dn[q];
  x.d = x.c + tp.dd[q];
  x.u = x.c + tp.du[q];
  return x;
}

// a level's arrays in LDS
template <typename T>
struct TailArrays {
  const T *bx, *by, *bz, *id, *b;
  T* e;
};
// what a cell's update reads: six faces, six neighbours, its own b and 1/D
template <typename T>
struct TailLoads {
  T f[6], v[6], b, id;
  __device__ __forceinline__ TailLoads(const TailArrays<T>& A, const TailCell& x, int nx, int sxy) {
    f[0] = A.bx[x.fx];
    f[1] = A.bx[x.fx + 1];
    f[2] = A.by[x.fy];
    f[3] = A.by[x.fy + nx];
    f[4] = A.bz[x.c];
    f[5] = A.bz[x.c + sxy];
    v[0] = A.e[x.w];
    v[1] = A.e[x.e];
    v[2] = A.e[x.s];
    v[3] = A.e[x.n];
    v[4] = A.e[x.d];
    v[5] = A.e[x.u];
    b = A.b[x.c];
    id = A.id[x.c];
  }
};

// one colour pass.  Every load of the thread's cells is issued before the
// arithmetic starts (the scheduling barrier keeps the compiler from
// interleaving them with the sums, which would wait on each pair in turn).
// DIVIDE: the quotient by the diagonal, rounded, for one correction of the product
// with 1/D (which an FP32 cycle's matrix has in FP32 only).
template <typename T, bool DIVIDE>
__device__ __forceinline__ void tail_pass(const Dims& n, const TailPairs& tp, const TailArrays<T>& A, T h2, int colour,
                                          bool from_zero) {
  const int sxy = n.nx * n.ny;
  const TailCell x0 = tail_cell(n, tp, 0, colour);
  auto value = [&](const TailCell& x, const TailLoads<T>& l) {
    T num = h2 * l.b;
    if (!from_zero) {
#pragma unroll
      for (int q = 0; q < 5; ++q) num += l.f[q] * l.v[q];   // west, east, south, north, down, up
      const T with_up = num + l.f[5] * l.v[5];
      num = x.top ? num : with_up;
    }
    T v = num * l.id;
    if constexpr (DIVIDE) {
      const T diag = l.f[0] + l.f[1] + l.f[2] + l.f[3] + l.f[4] + (x.top ? (T)2 * l.f[5] : l.f[5]);
      v = fused<T>(fused<T>(-v, diag, num), l.id, v);
    }
    return v;
  };
  if (tp.np == 2) {
    const TailCell x1 = tail_cell(n, tp, 1, colour);
    const TailLoads<T> l0(A, x0, n.nx, sxy), l1(A, x1, n.nx, sxy);
    __builtin_amdgcn_sched_barrier(0);
    const T v0 = value(x0, l0), v1 = value(x1, l1);
    if (x0.ok) A.e[x0.c] = v0;
    if (x1.ok) A.e[x1.c] = v1;
  } else if (x0.ok) {
    const TailLoads<T> l0(A, x0, n.nx, sxy);
    __builtin_amdgcn_sched_barrier(0);
    A.e[x0.c] = value(x0, l0);
  }
  __syncthreads();
}

// A coarsest level of one or two cells in a row: the same sweeps, with the
// same arithmetic, done by one thread in registers.  Cell 0 is red, cell 1
// black; the face between them is bx[1]; there is no other neighbour.
template <typename T, bool DIVIDE>
__device__ __forceinline__ void tail_coarsest_row(const TailArrays<T>& A, bool two, T h2, int S, int tid) {
  if (tid == 0) {
    const int nx = two ? 2 : 1;
    const T r0 = h2 * A.b[0], i0 = A.id[0];
    const T r1 = two ? h2 * A.b[1] : (T)0, i1 = two ? A.id[1] : (T)0, w = two ? A.bx[1] : (T)0;
    T d0 = 0, d1 = 0;
    if constexpr (DIVIDE) {
      d0 = A.bx[0] + A.bx[1] + A.by[0] + A.by[nx] + A.bz[0] + (T)2 * A.bz[nx];
      if (two) d1 = A.bx[1] + A.bx[2] + A.by[1] + A.by[3] + A.bz[1] + (T)2 * A.bz[3];
    }
    auto over = [&](T num, T id, T d) {
      const T v = num * id;
      return DIVIDE ? fused<T>(fused<T>(-v, d, num), id, v) : v;
    };
    T e0 = 0, e1 = 0;
#pragma unroll 1
    for (int s = 0; s < 2 * S; ++s) {   // forward: red, black; backward: black, red
      if (s < S) {
        T num = r0;
        if (s > 0) num += w * e1;
        e0 = over(num, i0, d0);
      }
      T num = r1;
      num += w * e0;
      e1 = over(num, i1, d1);
      if (s >= S) {
        T n0 = r0;
        n0 += w * e1;
        e0 = over(n0, i0, d0);
      }
    }
    A.e[0] = e0;
    if (two) A.e[1] = e1;
  }
  __syncthreads();
}

// The cycle from the last level of D down, e = M b.  A level of up to 128 pairs
// keeps a wavefront or two busy, and its passes (40 of them on the coarsest
// level) are a chain of LDS round trips, 0.3 us each; the cycle is a
// linear map, so its matrix, formed once per solve, gives the same values in one
// product: 256 x 1 x 64's levels of 64, 16 and 4 cells took 20 of the tail's
// 40 us.  R: the level's cells, rounded up; thread (g, i) sums columns g, g + G,
// .. of row i (32 loads in flight at a time), in FP64 and in up to eight sums that
// are added pairwise (one sum of 128 terms was 5e-16 from the exact product, these
// 3e-16), then the G sums are added in order.  SUM2: each sum's rounding is summed
// beside it, for a matrix that is the whole tail (of a grid of up to 256 cells,
// whose correction is the product itself).
// Past 256 cells the matrix outgrows what one compute unit loads in the time
// of the passes (512 cells: 2 MB at 64 B per clock, 14 us).
template <typename T, int R, bool SUM2>
__device__ __forceinline__ void matrix_product(const TailDesc<T>& D, T* sm, int tid, int N) {
  constexpr int G = kTailThreads / R, K = R / G, U = K < 32 ? K : 32, S = U < 8 ? U : 8;
  const int l = D.nl - 1, i = tid % R, g = tid / R;
  const T* b = sm + D.ob[l];
  double* mv = reinterpret_cast<double*>(sm + D.omv);
  T m[U];
  double s[S] = {}, r[S] = {};
#pragma unroll 1
  for (int c0 = g; c0 < N; c0 += G * U) {
#pragma unroll
    for (int q = 0; q < U; ++q) m[q] = D.M[min(c0 + G * q, N - 1) * N + min(i, N - 1)];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const T bq = b[min(c0 + G * q, N - 1)];
      const double bc = c0 + G * q < N ? (double)bq : 0.0, t = __builtin_fma((double)m[q], bc, s[q % S]);
      if constexpr (SUM2) r[q % S] += __builtin_fma((double)m[q], bc, s[q % S] - t);
      s[q % S] = t;
    }
  }
#pragma unroll
  for (int o = S / 2; o > 0; o >>= 1)
#pragma unroll
    for (int q = 0; q < o; ++q) {
      if constexpr (SUM2) {
        const double t = s[q] + s[q + o], a = t - s[q];
        r[q] += r[q + o] + ((s[q] - (t - a)) + (s[q + o] - a));
        s[q] = t;
      } else {
        s[q] += s[q + o];
      }
    }
  mv[tid] = s[0] + r[0];
  __syncthreads();
  if (tid < N) {
    double t = 0;
#pragma unroll 4
    for (int q = 0; q < G; ++q) t += mv[tid + q * R];
    sm[D.oe[l] + tid] = (T)t;
  }
  __syncthreads();
}
template <typename T, bool SUM2>
__device__ __forceinline__ void tail_matrix_product(const TailDesc<T>& D, T* sm, int tid) {
  const Dims n = D.n[D.nl - 1];
  const int N = n.nx * n.ny * n.nz;
  if (N > 128)
    matrix_product<T, 256, SUM2>(D, sm, tid, N);
  else if (N > 64)
    matrix_product<T, 128, SUM2>(D, sm, tid, N);
  else if (N > 32)
    matrix_product<T, 64, SUM2>(D, sm, tid, N);
  else
    matrix_product<T, 32, SUM2>(D, sm, tid, N);
}

// The tail's first level, and a coarsest level that is no matrix: its face
// coefficients, 1/D and right-hand side live in registers, NP pairs per thread
// (pair tid + q kTailThreads), and only its correction is in LDS, by colour and
// pair index (reg_planes), so that a wavefront's reads are consecutive and a
// neighbour is a fixed distance away.  Same passes, in the same order, as the
// separate launches.  A pass is six LDS reads per cell, a dozen FP64 operations
// and a barrier: 0.46 us for 25 x 9 x 13 cells against a launch of 3.4
// (200 x 72 x 104, whose coarsest level that is: 40 passes, 1.42 times the
// step's speed); with the coefficients in LDS, 14 reads per cell, 18 x 8 x 9's
// 40 passes (72 x 32 x 36) made the step 5 to 10% slower.
template <typename T>
struct RegView {
  Dims n, nc;      // the level and the next one
  int fy, fz;      // coarsening factors (fx is 2)
  T h2;
  const T *bx, *by, *bz, *id, *b;
  T *planes, *rs;  // LDS: the correction (reg_planes entries), the residual scratch in natural order
};
// WAVE: a level of at most 64 pairs by the first wavefront alone, ordered by
// wavefront-level fences instead of workgroup barriers.
template <typename T, int NP, bool WAVE = false>
struct RegLevel {
  RegView<T> V;
  T* e;      // the red plane; the black one is P + sz further
  int tid, hx, sz, P;
  // per pair: the face between its cells, each colour's five other faces (x
  // outer, south, north, down, up), 1/D with its rest, and b
  T fm[NP], f[NP][2][5], id[NP][2], b[NP][2];
  float rest[NP][2];
  unsigned ok, odd, top;   // per (pair, colour): exists; odd column; per pair: top row

  __device__ __forceinline__ static void sync() {
    if constexpr (WAVE) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  }
  __device__ __forceinline__ int pair(int q) const {   // (the last pairs of the last thread groups repeat one)
    return q < NP - 1 ? tid + q * kTailThreads : min(tid + q * kTailThreads, P - 1);
  }
  // every load from a clamped index, so that all are in flight together; what
  // lies outside the level is then dropped
  __device__ __forceinline__ RegLevel(const RegView<T>& V_, int t) : V(V_), tid(t) { load(); }
  __device__ __forceinline__ void load() {
    const Dims& g = V.n;
    const int sxy = g.nx * g.ny;
    hx = (g.nx + 1) >> 1;
    sz = hx * g.ny;
    P = sz * g.nz;
    e = V.planes + sz;
    ok = odd = top = 0;
    const float ihx = 1.0f / (float)hx, iny = 1.0f / (float)g.ny;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int p = pair(q);
      const int r = tail_div(p, ihx), ti = p - r * hx, k = tail_div(r, iny), j = r - k * g.ny;
      const bool t = k == g.nz - 1;
      if (t) top |= 1u << q;
      const int row = (g.nx + 1) * (j + g.ny * k);
      const T xm = V.bx[row + 2 * ti + 1];   // (past an odd row's end: the wall face)
      fm[q] = 2 * ti + 1 < g.nx ? xm : (T)0;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int o = (j + k + c) & 1, i = min(2 * ti + o, g.nx - 1);
        if (tid + q * kTailThreads < P && 2 * ti + o < g.nx) ok |= 1u << (2 * q + c);
        if (o) odd |= 1u << (2 * q + c);
        const int fy = i + g.nx * (j + (g.ny + 1) * k), cc = i + g.nx * j + sxy * k;
        // (a wall face is zero here whatever a caller's array holds: the entry
        // beyond it is another row's)
        const T xo = V.bx[row + (o ? i + 1 : i)], ys = V.by[fy], yn = V.by[fy + g.nx], zd = V.bz[cc];
        const T zu = V.bz[cc + sxy];
        f[q][c][0] = (o ? i + 1 < g.nx : i > 0) ? xo : (T)0;
        f[q][c][1] = j > 0 ? ys : (T)0;
        f[q][c][2] = j < g.ny - 1 ? yn : (T)0;
        f[q][c][3] = k > 0 ? zd : (T)0;
        f[q][c][4] = zu;
        id[q][c] = V.id[cc];
        rest[q][c] = inv_rest<T>(xo + xm + ys + yn + zd + (t ? (T)2 * zu : zu), id[q][c]);
        b[q][c] = V.b[cc];
      }
    }
  }
  __device__ __forceinline__ void zero() {
    for (int q = tid; q < 2 * P + 3 * sz; q += WAVE ? 64 : kTailThreads) e[q - sz] = (T)0;
    sync();
  }
  template <int C>
  __device__ __forceinline__ T* plane() const { return C ? e + P + sz : e; }
  // the other colour's values around a pair's cell of colour C: in the pair,
  // beyond it along x, south, north, down, up (the entries above the top row
  // stay zero)
  template <int C>
  __device__ __forceinline__ void around(int q, T (&v)[6]) const {
    const T* o = plane<1 - C>() + pair(q);
    v[0] = o[0];
    v[1] = o[odd >> (2 * q + C) & 1u ? 1 : -1];
    v[2] = o[-hx];
    v[3] = o[hx];
    v[4] = o[-sz];
    v[5] = o[sz];
  }

  template <int C>
  __device__ __forceinline__ void pass(bool from_zero) {
    T v[NP][6];
    if (!from_zero) {
#pragma unroll
      for (int q = 0; q < NP; ++q) around<C>(q, v[q]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      T num = V.h2 * b[q][C];
      if (!from_zero) {
        num += fm[q] * v[q][0];
#pragma unroll
        for (int i = 0; i < 4; ++i) num += f[q][C][i] * v[q][i + 1];
        const T with_up = num + f[q][C][4] * v[q][5];
        num = top >> q & 1u ? num : with_up;
      }
      if (ok >> (2 * q + C) & 1u) plane<C>()[pair(q)] = quotient<T>(num, id[q][C], rest[q][C]);
    }
    sync();
  }

  template <int C>
  __device__ __forceinline__ void residual(T ih2) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      T v[6];
      around<C>(q, v);
      const T xc = plane<C>()[pair(q)];
      T acc = fm[q] * (xc - v[0]);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc += f[q][C][i] * (xc - v[i + 1]);
      acc += top >> q & 1u ? (T)2 * f[q][C][4] * xc : f[q][C][4] * (xc - v[5]);
      if (ok >> (2 * q + C) & 1u) V.rs[2 * pair(q) + (odd >> (2 * q + C) & 1u)] = b[q][C] - ih2 * acc;
    }
  }

  // the red, black, .. passes of a visit: down from zero (up 0), up (1), or the
  // coarsest level's sweeps forward then backward
  __device__ __forceinline__ void smooth(int passes, bool up, bool bottom) {
#pragma unroll 1
    for (int s = 0; s < passes; ++s) {
      const bool zero = !up && s == 0;
      if ((s + (up || (bottom && 2 * s >= passes))) & 1)
        pass<1>(zero);
      else
        pass<0>(zero);
    }
  }
  // the residual and its restriction
  __device__ __forceinline__ void restrict_to(T* bc) {
    const T ih2 = (T)1 / V.h2;
    residual<0>(ih2);
    residual<1>(ih2);
    __syncthreads();
    // each coarse cell's mean of its children (a level that is restricted has
    // an even nx, so entry 2 p + odd of the scratch is the cell's natural
    // index)
    const Dims &g = V.n, nc = V.nc;
    const int sy = V.fy - 1, sk = V.fz - 1, sxy = g.nx * g.ny;
    const T inv = (T)1 / (T)(2 << (sy + sk));
    const float inx = 1.0f / (float)nc.nx, iny = 1.0f / (float)nc.ny;
#pragma unroll 1
    for (int c = tid; c < nc.nx * nc.ny * nc.nz; c += kTailThreads) {
      const int r = tail_div(c, inx), K = tail_div(r, iny), f0 = 2 * (c - r * nc.nx) + g.nx * ((r - K * nc.ny) << sy) + (sxy << sk) * K;
      T sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int dj = q & 1, dk = q >> 1;
        if (dj <= sy && dk <= sk) {
          sum += V.rs[f0 + g.nx * dj + sxy * dk];
          sum += V.rs[f0 + g.nx * dj + sxy * dk + 1];
        }
      }
      bc[c] = sum * inv;
    }
    __syncthreads();
  }
  __device__ __forceinline__ void prolong(const T* ec) {
    const float ihx = 1.0f / (float)hx, iny = 1.0f / (float)V.n.ny;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int p = pair(q), r = tail_div(p, ihx), k = tail_div(r, iny), j = r - k * V.n.ny;
      const T add = ec[p - r * hx + V.nc.nx * ((j >> (V.fy - 1)) + V.nc.ny * (k >> (V.fz - 1)))];
      if (ok >> (2 * q) & 1u) plane<0>()[p] += add;
      if (ok >> (2 * q) & 2u) plane<1>()[p] += add;
    }
    __syncthreads();
  }

  __device__ __forceinline__ void store(T* ge) const {
    const float ihx = 1.0f / (float)hx;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int p = pair(q), r = tail_div(p, ihx), c = 2 * (p - r * hx) + V.n.nx * r;   // the first column's cell
      if (ok >> (2 * q) & 1u) ge[c + (odd >> (2 * q) & 1u)] = plane<0>()[p];
      if (ok >> (2 * q) & 2u) ge[c + (odd >> (2 * q + 1) & 1u)] = plane<1>()[p];
    }
  }
};

// The V-cycle over the levels in LDS by nthr threads: the visits go down the
// levels and up again
template <typename T, bool REG>
__device__ __forceinline__ void tail_levels(const TailDesc<T>& D, T* sm, int tid, int nthr) {
  const int nl = D.nl;
#pragma unroll 1
  for (int it = 0; it < 2 * nl - 1; ++it) {
    const bool up = it >= nl;
    const int l = up ? 2 * nl - 2 - it : it;
    const bool bottom = l == nl - 1;
    if (bottom && D.M) {
      tail_matrix_product<T, false>(D, sm, tid);
      continue;
    }
    const Dims n = D.n[l];
    const int sxy = n.nx * n.ny;
    const T h2 = D.h2[l];
    const TailArrays<T> A{sm + D.obx[l], sm + D.oby[l], sm + D.obz[l], sm + D.oid[l], sm + D.ob[l], sm + D.oe[l]};
    if (bottom && n.nx <= 2 && n.ny == 1 && n.nz == 1) {
      tail_coarsest_row<T, !REG>(A, n.nx == 2, h2, D.coarse_sweeps, tid);
      continue;
    }
    if constexpr (REG) {
      if (bottom) {
        auto sweeps = [&](auto wave) {
          RegLevel<T, 1, decltype(wave)::value> t({n, n, 1, 1, h2, A.bx, A.by, A.bz, A.id, A.b, sm + D.oeb, nullptr}, tid);
          t.zero();
          t.smooth(4 * D.coarse_sweeps, false, true);
          t.store(A.e);
        };
        if ((n.nx + 1) / 2 * n.ny * n.nz > 64)
          sweeps(std::false_type{});
        else if (tid < 64)
          sweeps(std::true_type{});
        __syncthreads();
        continue;
      }
    }
    TailPairs tp;
    tail_decode(n, tid, nthr, tp);
    const Dims nc = bottom ? n : D.n[l + 1];
    const int sy = D.f[l][1] - 1, sz = D.f[l][2] - 1;   // the halved directions' shifts
    if (up) {
      // prolongation: both cells of a pair share one coarse cell (fx = 2)
      const T* ec = sm + D.oe[l + 1];
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (q < tp.np) {
          const T add = ec[(tp.i[q] >> 1) + nc.nx * ((tp.j[q] >> sy) + nc.ny * (tp.k[q] >> sz))];
          A.e[tp.c[q]] += add;
          if (tp.i[q] + 1 < n.nx) A.e[tp.c[q] + 1] += add;
        }
      __syncthreads();
    }
    // red, black, .. down from zero; black, red, .. up; on the coarsest level
    // the sweeps forward, then backward
    const int passes = bottom ? 4 * D.coarse_sweeps : 2 * (up ? D.nu_post : D.nu_pre);
#pragma unroll 1
    for (int s = 0; s < passes; ++s)
      tail_pass<T, !REG>(n, tp, A, h2, (s + (up || (bottom && 2 * s >= passes))) & 1, !up && s == 0);
    if (up || bottom) continue;
    // every fine cell's residual b - A e, each thread for both cells of its
    // pairs (a wall term is an exact zero) ...
    T* rs = sm + D.ors;
    const T ih2 = (T)1 / h2;
#pragma unroll 1
    for (int col = 0; col < 2; ++col)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const TailCell x = tail_cell(n, tp, q, col);
        if (!x.ok) continue;
        const TailLoads<T> a(A, x, n.nx, sxy);
        const T xc = A.e[x.c];
        __builtin_amdgcn_sched_barrier(0);
        T acc = 0;
#pragma unroll
        for (int d = 0; d < 5; ++d) acc += a.f[d] * (xc - a.v[d]);
        acc += x.top ? (T)2 * a.f[5] * xc : a.f[5] * (xc - a.v[5]);
        rs[x.c] = a.b - ih2 * acc;
      }
    __syncthreads();
    // ... then each coarse cell's mean of its children, summed in the order
    // (dk, dj, di) (a level that is restricted has an even nx: fx = 2; fy, fz
    // are 1 along a dimension of one cell, else 2)
    T* bc = sm + D.ob[l + 1];
    const T inv = (T)1 / (T)(2 << (sy + sz));
    const float inx = 1.0f / (float)nc.nx, iny = 1.0f / (float)nc.ny;
#pragma unroll 1
    for (int c = tid; c < nc.nx * nc.ny * nc.nz; c += nthr) {
      const int r = tail_div(c, inx), K = tail_div(r, iny), f = 2 * (c - r * nc.nx) + n.nx * ((r - K * nc.ny) << sy) + (sxy << sz) * K;
      T sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int dj = q & 1, dk = q >> 1;
        if (dj <= sy && dk <= sz) {
          sum += rs[f + n.nx * dj + sxy * dk];
          sum += rs[f + n.nx * dj + sxy * dk + 1];
        }
      }
      bc[c] = sum * inv;
    }
    __syncthreads();
  }
}

// Column blockIdx.x of that matrix: the cycle over D's levels, one wavefront,
// from a unit right-hand side.  An FP32 cycle's is computed in FP64 from
// its FP32 coefficients and rounded once, and its products are summed in FP64:
// nearer the exact cycle than the FP32 passes' own.  An FP64 cycle's is about as
// near as the passes (a whole cycle from the oracle's, 16 x 1 x 16 2.9e-16 and 3.0e-16,
// 8 x 4 x 8 2.8e-16 and 2.0e-16, 256 x 1 x 64 3.0e-16 and 2.8e-16).
template <typename T>
__global__ void __launch_bounds__(64) k_tail_matrix(TailDesc<double> D, const T* __restrict__ pack, T* __restrict__ M) {
  extern __shared__ double tail_smem[];
  double* sm = tail_smem;
  const int tid = threadIdx.x, N = D.n[0].nx * D.n[0].ny * D.n[0].nz;
  for (int q = tid; q < D.npack; q += 64) sm[q] = (double)pack[q];
  for (int q = D.npack + tid; q < D.omv; q += 64) sm[q] = 0.0;
  __syncthreads();
  if (tid == 0) sm[D.ob[0] + blockIdx.x] = 1.0;
  __syncthreads();
  tail_levels<double, false>(D, sm, tid, 64);
  for (int q = tid; q < N; q += 64) M[(size_t)blockIdx.x * N + q] = (T)sm[D.oe[0] + q];
}

// The tail whose first level is held in registers, NP pairs per thread
template <typename T, int NP>
__global__ void __launch_bounds__(kTailThreads) k_vcycle_tail(TailDesc<T> D) {
  extern __shared__ double tail_smem[];
  T* sm = reinterpret_cast<T*>(tail_smem);
  const int nl = D.nl;
  const int tid = threadIdx.x;
  RegLevel<T, NP> t({D.nt, D.n[0], D.ft[1], D.ft[2], D.h2t, D.tbx, D.tby, D.tbz, D.tid, D.b0, sm + D.oet, sm + D.ors}, tid);
  // stage the pack (every coefficient array and 1/D of the levels below) while
  // those loads are in flight: one flat loop, sixteen independent loads per
  // thread at a time
#pragma unroll 1
  for (int base = tid; base < D.npack; base += 16 * kTailThreads) {
    T v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = D.pack[min(base + u * kTailThreads, D.npack - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (base + u * kTailThreads < D.npack) sm[base + u * kTailThreads] = v[u];
  }
  // every level's correction starts at zero: the passes read a cell's own
  // entry through a wall before it is first written
#pragma unroll 1
  for (int l = 0; l < nl; ++l) {
    const int N = D.n[l].nx * D.n[l].ny * D.n[l].nz;
#pragma unroll 1
    for (int c = tid; c < N; c += kTailThreads) sm[D.oe[l] + c] = (T)0;
  }
  t.zero();
#pragma unroll 1
  for (bool up = false;; up = true) {
    t.smooth(nl == 0 ? 4 * D.coarse_sweeps : 2 * (up ? D.nu_post : D.nu_pre), up, nl == 0);
    if (nl == 0 || up) break;
    t.restrict_to(sm + D.ob[0]);
    tail_levels<T, true>(D, sm, tid, kTailThreads);
    if constexpr (NP * sizeof(T) >= 16) {
      // read again rather than kept: the levels between want the registers
      // (also the ones its indices would take: hiding that the thread's number
      // is the same keeps them from being formed once)
      asm volatile("" : "+v"(t.tid));
      t.load();
    }
    t.prolong(sm + D.oe[0]);
  }
  t.store(D.ge);
}

// The tail whose first level's cycle is a matrix
template <typename T>
__global__ void __launch_bounds__(kTailThreads) k_vcycle_matrix(TailDesc<T> D) {
  extern __shared__ double tail_smem[];
  T* sm = reinterpret_cast<T*>(tail_smem);
  const int tid = threadIdx.x, N = D.n[0].nx * D.n[0].ny * D.n[0].nz;
  if (tid < N) sm[D.ob[0] + tid] = D.b0[tid];
  __syncthreads();
  tail_matrix_product<T, sizeof(T) == 8>(D, sm, tid);
  if (tid < N) D.ge[tid] = sm[D.oe[0] + tid];
}

// ------------------------------------------------------------ 2-D levels
// A level of a 2-D tank is small: each of its passes is a launch of 3 to 5 us
// for a fraction of that of work.  So a visit is one launch each way: a block
// takes a tile of 64 x 8 cells and a ring of four around it, holds the ring's
// and the tile's coefficients in registers (three cell pairs per thread) and
// the correction in LDS by colour and pair, and runs all four passes on both;
// each pass's values are right one cell further in from the ring's edge than
// the last one's, so the tile's are right at the end.  A value differs from the
// separate passes' in the order of its sums alone.  With its ring a tile is 2.25
// times its cells, loaded once where the separate passes load them four to
// five times; 256 x 64: 16.5 us of launches for 5.9 down, 18.2 for 7.1 up.
constexpr int kT2X = 64, kT2Z = 8, kT2H = 4;                         // tile, ring
constexpr int kT2Row = (kT2X + 2 * kT2H) / 2, kT2Rows = kT2Z + 2 * kT2H;   // pairs per row, rows
constexpr int kT2P = kT2Row * kT2Rows, kT2Threads = 192, kT2N = kT2P / kT2Threads;
static_assert(kT2P % kT2Threads == 0, "whole threads");

template <typename T>
struct Tile2d {
  T* e;     // LDS: the red plane, kT2P + 2 kT2Row entries before the black one's
  int x0, z0, nx, nz;
  T fm[kT2N], f[kT2N][2][3], id[kT2N][2], b[kT2N][2];   // as RegLevel: x outer, down, up
  float rest[kT2N][2];
  unsigned in = 0, odd = 0, top = 0;

  static constexpr int kLds = 2 * kT2P + 3 * kT2Row;   // planes, and a row before, between and after
  __device__ __forceinline__ int pair(int q) const { return (int)threadIdx.x + q * kT2Threads; }
  // the global cell of pair q's colour c
  __device__ __forceinline__ int col(int q, int c) const {
    return x0 - kT2H + 2 * (pair(q) % kT2Row) + (int)(odd >> (2 * q + c) & 1u);
  }
  __device__ __forceinline__ int row(int q) const { return z0 - kT2H + pair(q) / kT2Row; }
  __device__ __forceinline__ bool has(int q, int c) const { return in >> (2 * q + c) & 1u; }
  // whether the cell lies in the tile (and the grid)
  __device__ __forceinline__ bool tile(int q, int c) const {
    const int i = col(q, c) - x0, k = row(q) - z0;
    return has(q, c) && i >= 0 && i < kT2X && k >= 0 && k < kT2Z;
  }

  // b natural, 1/D colour-split; every load from a clamped index, what lies
  // outside the grid zero
  template <typename TB>
  __device__ __forceinline__ void load(T* lds, int nx_, int nz_, const T* __restrict__ bx, const T* __restrict__ bz,
                                       const T* __restrict__ invd, const TB* __restrict__ bg) {
    e = lds + kT2Row;
    nx = nx_;
    nz = nz_;
    x0 = blockIdx.x * kT2X;
    z0 = blockIdx.y * kT2Z;
    const int hx = nx >> 1, P = hx * nz;   // (a level that is halved has an even nx)
    TB bb[kT2N][2];
#pragma unroll
    for (int q = 0; q < kT2N; ++q) {
      const int k = row(q), kc = min(max(k, 0), nz - 1), i0 = x0 - kT2H + 2 * (pair(q) % kT2Row);
      const int ic = min(max(i0, 0), nx - 2);
      const bool ok = k >= 0 && k < nz && i0 >= 0 && i0 < nx;
      if (k == nz - 1) top |= 1u << q;
      fm[q] = bx[ic + 1 + (nx + 1) * kc];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int o = (k + c) & 1, g = ic + o + nx * kc;
        if (o) odd |= 1u << (2 * q + c);
        if (ok) in |= 1u << (2 * q + c);
        f[q][c][0] = bx[ic + 2 * o + (nx + 1) * kc];
        f[q][c][1] = bz[g];
        f[q][c][2] = bz[g + nx];
        id[q][c] = invd[c * P + (ic >> 1) + hx * kc];
        bb[q][c] = bg[g];
      }
    }
    for (int q = threadIdx.x; q < kLds; q += kT2Threads) lds[q] = (T)0;
#pragma unroll
    for (int q = 0; q < kT2N; ++q) {
      const bool ok = in >> (2 * q) & 1u;
      fm[q] = ok ? fm[q] : (T)0;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        // (without the y-walls' faces, which are not read here: where those are
        // not zero, 1/D is taken as it is)
        const T zu = f[q][c][2], diag = f[q][c][0] + fm[q] + f[q][c][1] + (top >> q & 1u ? (T)2 * zu : zu);
        rest[q][c] = ok && fabs(fused<T>(-diag, id[q][c], (T)1)) < (sizeof(T) == 8 ? (T)0x1p-48 : (T)0x1p-19)
                         ? inv_rest<T>(diag, id[q][c])
                         : 0.0f;
#pragma unroll
        for (int d = 0; d < 3; ++d) f[q][c][d] = ok ? f[q][c][d] : (T)0;
        id[q][c] = ok ? id[q][c] : (T)0;
        b[q][c] = ok ? (T)bb[q][c] : (T)0;
      }
    }
    __syncthreads();
  }
  template <int C>
  __device__ __forceinline__ T* plane() const { return C ? e + kT2P + kT2Row : e; }
  template <int C>
  __device__ __forceinline__ void around(int q, T (&v)[4]) const {
    const T* o = plane<1 - C>() + pair(q);
    v[0] = o[0];
    v[1] = o[odd >> (2 * q + C) & 1u ? 1 : -1];
    v[2] = o[-kT2Row];
    v[3] = o[kT2Row];
  }
  template <int C>
  __device__ __forceinline__ void pass(bool from_zero) {
    T v[kT2N][4];
    if (!from_zero) {
#pragma unroll
      for (int q = 0; q < kT2N; ++q) around<C>(q, v[q]);
    }
#pragma unroll
    for (int q = 0; q < kT2N; ++q) {
      T num = h2 * b[q][C];
      if (!from_zero) {
        num += fm[q] * v[q][0];
        num += f[q][C][0] * v[q][1];
        num += f[q][C][1] * v[q][2];
        const T with_up = num + f[q][C][2] * v[q][3];
        num = top >> q & 1u ? num : with_up;
      }
      plane<C>()[pair(q)] = quotient<T>(num, id[q][C], rest[q][C]);
    }
    __syncthreads();
  }
  template <int C>
  __device__ __forceinline__ void residual(T ih2, T* rs) const {
#pragma unroll
    for (int q = 0; q < kT2N; ++q) {
      T v[4];
      around<C>(q, v);
      const T xc = plane<C>()[pair(q)];
      // a pass may read the zero beyond a wall whatever the wall's coefficient
      // is; the residual drops the term
      const int i = col(q, C);
      const bool wall = odd >> (2 * q + C) & 1u ? i == nx - 1 : i == 0;
      T acc = fm[q] * (xc - v[0]);
      acc += wall ? (T)0 : f[q][C][0] * (xc - v[1]);
      acc += row(q) == 0 ? (T)0 : f[q][C][1] * (xc - v[2]);
      acc += top >> q & 1u ? (T)2 * f[q][C][2] * xc : f[q][C][2] * (xc - v[3]);
      if (tile(q, C)) rs[col(q, C) - x0 + kT2X * (row(q) - z0)] = b[q][C] - ih2 * acc;
    }
  }
  T h2;
};

// Down: V(2,.)'s two pre-smoothing sweeps from zero, the correction (natural),
// and the restricted residual into the next level's b (colour-split when
// csplit, else natural)
template <typename T, typename TB>
__global__ void __launch_bounds__(kT2Threads) k_pre2d(int nx, int nz, T h2, const T* __restrict__ bx,
                                                      const T* __restrict__ bz, const T* __restrict__ invd,
                                                      const TB* __restrict__ b, T* __restrict__ e, int csplit,
                                                      T* __restrict__ bc) {
  __shared__ T lds[Tile2d<T>::kLds];
  __shared__ T rs[kT2X * kT2Z];
  Tile2d<T> t;
  t.h2 = h2;
  t.load(lds, nx, nz, bx, bz, invd, b);
  t.template pass<0>(true);
  t.template pass<1>(false);
  t.template pass<0>(false);
  t.template pass<1>(false);
  const T ih2 = (T)1 / h2;
  t.template residual<0>(ih2, rs);
  t.template residual<1>(ih2, rs);
#pragma unroll
  for (int q = 0; q < kT2N; ++q) {
    const int p = t.pair(q);
    if (t.tile(q, 0)) e[t.col(q, 0) + nx * t.row(q)] = t.template plane<0>()[p];
    if (t.tile(q, 1)) e[t.col(q, 1) + nx * t.row(q)] = t.template plane<1>()[p];
  }
  __syncthreads();
  const int ncx = nx >> 1, chx = (ncx + 1) >> 1, cP = chx * (nz >> 1);
  for (int q = threadIdx.x; q < kT2X * kT2Z / 4; q += kT2Threads) {
    const int li = q % (kT2X / 2), lk = q / (kT2X / 2), I = t.x0 / 2 + li, K = t.z0 / 2 + lk;
    if (I >= ncx || K >= nz >> 1) continue;
    const T* r = rs + 2 * li + 2 * kT2X * lk;
    T sum = 0;
    sum += r[0];
    sum += r[1];
    sum += r[kT2X];
    sum += r[kT2X + 1];
    bc[csplit ? ((I + K) & 1) * cP + (I >> 1) + chx * K : I + ncx * K] = sum * (T)0.25;
  }
}

// Up: prolongation of the next level's correction ec, two post-smoothing
// sweeps, and the result to out (natural: the FP64 z of the CG loop, or the
// second half of a coarse level's vector).  out is another buffer than e, whose
// values the rings of tiles that run later still read.  With r
// (the CG residual) also the per-block sums of r out.
template <typename T, typename TB, typename TO>
__global__ void __launch_bounds__(kT2Threads) k_post2d(int nx, int nz, T h2, const T* __restrict__ bx,
                                                       const T* __restrict__ bz, const T* __restrict__ invd,
                                                       const TB* __restrict__ b, const T* __restrict__ e, int csplit,
                                                       const T* __restrict__ ec, TO* __restrict__ out,
                                                       const double* __restrict__ r, double* __restrict__ partials) {
  __shared__ T lds[Tile2d<T>::kLds];
  Tile2d<T> t;
  t.h2 = h2;
  // the red cells' starting values (the first pass overwrites the black ones)
  T st[kT2N], sc[kT2N];
  {
    const int ncx = nx >> 1, chx = (ncx + 1) >> 1, cP = chx * (nz >> 1);
    const int x0 = blockIdx.x * kT2X, z0 = blockIdx.y * kT2Z;
#pragma unroll
    for (int q = 0; q < kT2N; ++q) {
      const int p = (int)threadIdx.x + q * kT2Threads;
      const int k = min(max(z0 - kT2H + p / kT2Row, 0), nz - 1), i = min(max(x0 - kT2H + 2 * (p % kT2Row), 0), nx - 2);
      const int I = i >> 1, K = k >> 1;
      st[q] = e[i + (k & 1) + nx * k];
      sc[q] = ec[csplit ? ((I + K) & 1) * cP + (I >> 1) + chx * K : I + ncx * K];
    }
  }
  t.load(lds, nx, nz, bx, bz, invd, b);
#pragma unroll
  for (int q = 0; q < kT2N; ++q) t.template plane<0>()[t.pair(q)] = t.has(q, 0) ? st[q] + sc[q] : (T)0;
  __syncthreads();
  t.template pass<1>(false);
  t.template pass<0>(false);
  t.template pass<1>(false);
  t.template pass<0>(false);
  double v[1] = {0.0};
#pragma unroll
  for (int q = 0; q < kT2N; ++q)
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (t.tile(q, c)) {
        const int g = t.col(q, c) + nx * t.row(q);
        const TO z = (TO)(c ? t.template plane<1>()[t.pair(q)] : t.template plane<0>()[t.pair(q)]);
        out[g] = z;
        if (r) v[0] += r[g] * (double)z;
      }
  if (r) block_partials<1>(v, partials, (int)(blockIdx.x + gridDim.x * blockIdx.y));
}

template <typename T>
__global__ void k_fill(T* __restrict__ a, size_t n) {
  size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) a[q] = (T)0;
}

__global__ void k_d2f(const double* __restrict__ a, float* __restrict__ b, size_t n) {
  size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) b[q] = (float)a[q];
}

__global__ void k_f2d(const float* __restrict__ a, double* __restrict__ b, size_t n) {
  size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) b[q] = (double)a[q];
}

// the FP32 V-cycle's result to FP64 z, fused with the per-block sums of r z
// (block order); every thread reaches the reduction
__global__ void __launch_bounds__(256) k_f2d_dots(const float* __restrict__ a, double* __restrict__ z, size_t n,
                                                  const double* __restrict__ r, double* __restrict__ partials) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  double v[1] = {0.0};
  if (q < n) {
    const double zq = (double)a[q];
    z[q] = zq;
    v[0] = r[q] * zq;
  }
  block_partials<1>(v, partials, (int)blockIdx.x);
}

// ------------------------------------------------------------------ CG (FP64)
#define CELL_INDEX                                                         \
  const Tile tl = xcd_tile();                                              \
  const int i = tl.x * blockDim.x + threadIdx.x;                           \
  const int j = tl.y * blockDim.y + threadIdx.y;                           \
  const int k = tl.z * blockDim.z + threadIdx.z;                           \
  const bool inside = (i < n.nx && j < n.ny && k < n.nz);                  \
  const size_t c = inside ? i + (size_t)n.nx * (j + (size_t)n.ny * k) : 0

// r = b - A x; totals (r.r, b.b) -> scal (RESID0: S_RR, S_BB; TRR: S_TRR)
__global__ void __launch_bounds__(256) k_resid_norm(Dims n, double ih2, const double* __restrict__ bx,
                                                    const double* __restrict__ by,
                                                    const double* __restrict__ bz,
                                                    const double* __restrict__ b,
                                                    const double* __restrict__ x,
                                                    double* __restrict__ r,
                                                    double* __restrict__ partials, FaceTab<double> ft) {
  CELL_INDEX;
  double v[2] = {0.0, 0.0};
  // As k_dir_spmv: a wavefront is one x-row of 64 cells (blockDim.x == 64);
  // every load is issued before the first wait, through in-range indices (a
  // lane outside the grid reads around cell 0), the x neighbours come from
  // the adjacent lanes (a row's end lanes load theirs), and the faces of the
  // wavefront's lines through their tables where a line is one value.
  const int lane = threadIdx.x;
  const int ii = inside ? i : 0, jj = inside ? j : 0, kk = inside ? k : 0;
  const size_t sxy = (size_t)n.nx * n.ny;
  const double xc = x[c];
  const double xs = x[jj > 0 ? c - n.nx : c], xn = x[jj < n.ny - 1 ? c + n.nx : c];
  const double xd = x[kk > 0 ? c - sxy : c], xu = x[kk < n.nz - 1 ? c + sxy : c];
  const bool xlo = lane == 0 && ii > 0, xhi = lane == 63 && ii < n.nx - 1;
  double xx = 0.0;
  if (xlo || xhi) xx = x[xhi ? c + 1 : c - 1];
  const double bc = b[c];
  const int ju = __builtin_amdgcn_readfirstlane(min(j, n.ny - 1)), ku = __builtin_amdgcn_readfirstlane(min(k, n.nz - 1));
  FaceLd<double> F;
  F.load(n, ft, bx, by, bz, ju, ku, ii + (size_t)(n.nx + 1) * (jj + (size_t)n.ny * kk),
         ii + (size_t)n.nx * (jj + (size_t)(n.ny + 1) * kk), c);
  __builtin_amdgcn_sched_barrier(0);
  double cw, ce, cs, cn, cd, cu;
  F.get(n, ii, cw, ce, cs, cn, cd, cu);
  const double xl = __shfl_up(xc, 1, 64), xr = __shfl_down(xc, 1, 64);
  if (inside) {
    double xw = xc, xe = xc;
    if (i > 0) xw = lane > 0 ? xl : xx;
    if (i < n.nx - 1) xe = lane < 63 ? xr : xx;
    double acc = cw * (xc - xw) + ce * (xc - xe) + cs * (xc - xs) + cn * (xc - xn) + cd * (xc - xd);
    acc += (k < n.nz - 1) ? cu * (xc - xu) : 2.0 * cu * xc;
    const double rc = bc - ih2 * acc;
    r[c] = rc;
    v[0] = rc * rc;
    v[1] = bc * bc;
  }
  block_partials<2>(v, partials, tl.lin);
}

// <r, z>
__global__ void __launch_bounds__(256) k_dot_rho(Dims n, const double* __restrict__ r,
                                                 const double* __restrict__ z, double* __restrict__ partials) {
  CELL_INDEX;
  double v[1] = {inside ? r[c] * z[c] : 0.0};
  block_partials<1>(v, partials, tl.lin);
}

// d = zn + beta d_old, q = A d = A zn + beta q_old (first: d = zn, q = A zn);
// alpha = rho / <d, q>, and <z, q>, from which the next iteration's
// <r, z_old> follows (see k_finalize).  Carrying q = A d by its recurrence keeps the
// stencil on zn alone, and d_old and q_old are read pointwise: the stencil's
// load count, not its bytes, limits this kernel.  With xupd it also applies
// the previous iteration's x += alpha d_old (alpha still in scal, d_old
// already loaded here), which the vector update then leaves out.  A wavefront is one x-row of
// 64 cells (blockDim.x == 64), so the x neighbours of zn come from the
// adjacent lanes and only a row's end lanes load them; every lane takes part
// in the shuffles (c is 0 outside the grid).  ndot > 0: <r, zn> is still in
// ndot partials (dotp), which every wavefront sums for itself, and beta follows
// here; the first block leaves the sum in S_RHON.
__global__ void __launch_bounds__(256) k_dir_spmv(Dims n, double ih2, const double* __restrict__ bx,
                                                  const double* __restrict__ by,
                                                  const double* __restrict__ bz,
                                                  const double* __restrict__ zn,
                                                  const double* __restrict__ dold,
                                                  double* __restrict__ dnew, double* __restrict__ q,
                                                  int first, double* __restrict__ scal,
                                                  double* __restrict__ partials, double* __restrict__ x,
                                                  int xupd, FaceTab<double> ft, const double* __restrict__ dotp,
                                                  int ndot) {
  CELL_INDEX;
  double v[2] = {0.0, 0.0};
  double beta = 0.0;
  // Every load is issued before the shuffles wait for zc: the faces and the
  // y and z neighbours through in-range indices (a lane outside the grid
  // reads around cell 0), the row-end lanes' x neighbour, and d_old, q_old
  // (also on a first iteration, which does not use them).
  const int lane = threadIdx.x;
  const int ii = inside ? i : 0, jj = inside ? j : 0, kk = inside ? k : 0;
  const size_t sxy = (size_t)n.nx * n.ny;
  const size_t fx = ii + (size_t)(n.nx + 1) * (jj + (size_t)n.ny * kk);
  const size_t fy = ii + (size_t)n.nx * (jj + (size_t)(n.ny + 1) * kk);
  const double zc = zn[c];
  const double zs = zn[jj > 0 ? c - n.nx : c], zno = zn[jj < n.ny - 1 ? c + n.nx : c];
  const double zd = zn[kk > 0 ? c - sxy : c], zu = zn[kk < n.nz - 1 ? c + sxy : c];
  double zx = 0.0;   // lane 0's west and lane 63's east neighbour lie outside the wavefront
  if (lane == 0 && ii > 0) zx = zn[c - 1];
  if (lane == 63 && ii < n.nx - 1) zx = zn[c + 1];
  const double dol = dold[c], qol = q[c];
  const double xo = xupd ? x[c] : 0.0;
  // the faces: of the wavefront's x-line (j, k), the y-lines j, j + 1 and the
  // z-lines k, k + 1, each through its table where the line is one value
  const int ju = __builtin_amdgcn_readfirstlane(min(j, n.ny - 1)), ku = __builtin_amdgcn_readfirstlane(min(k, n.nz - 1));
  FaceLd<double> F;
  F.load(n, ft, bx, by, bz, ju, ku, fx, fy, c);
  __builtin_amdgcn_sched_barrier(0);
  if (ndot > 0) {
    double t[1];
    wave_totals<1>(dotp, ndot, t);
    const double rho = scal[S_RHO];
    beta = (t[0] - (rho - scal[S_ALPHA] * scal[S_ZQ])) / rho;   // (as k_finalize)
    if (tl.lin == 0 && block_tid() == 0) scal[S_RHON] = t[0];
  } else if (!first) {
    beta = scal[S_BETA];
  }
  double cw, ce, cs, cn, cd, cu;
  F.get(n, ii, cw, ce, cs, cn, cd, cu);
  const double zl = __shfl_up(zc, 1, 64), zr = __shfl_down(zc, 1, 64);
  if (inside) {
    if (xupd) x[c] = xo + scal[S_ALPHA] * dol;
    double zw = zc, ze = zc;
    if (i > 0) zw = lane > 0 ? zl : zx;
    if (i < n.nx - 1) ze = lane < 63 ? zr : zx;
    double acc = cw * (zc - zw) + ce * (zc - ze) + cs * (zc - zs) + cn * (zc - zno) + cd * (zc - zd);
    acc += (k < n.nz - 1) ? cu * (zc - zu) : 2.0 * cu * zc;
    const double qz = ih2 * acc;
    double dc = zc, qc = qz;
    if (!first) {
      dc = zc + beta * dol;
      qc = qz + beta * qol;
    }
    dnew[c] = dc;
    q[c] = qc;
    v[0] = dc * qc;
    v[1] = zc * qc;
  }
  block_partials<2>(v, partials, tl.lin);
}

// The split CG vectors' kernels.  On a finest level of the wide passes r, z,
// d and q are colour-split like the V-cycle's vectors, so the cycle reads r
// and leaves z in place: no split copy of r is written (8 B per cell), the
// last pass stores only the red half of z, and every access of these kernels
// is a whole 16-byte load or store per lane.  b and the caller's pressure stay
// in natural order: the residual leaves a split copy of the guess, the
// direction updates advance it, and the last update writes the result back in
// natural order.  A lane takes two pairs.
//
// d, q, alpha and <z, q> as k_dir_spmv
__global__ void __launch_bounds__(256) k_dir_spmv_split(Dims n, double ih2, const double* __restrict__ bx,
                                                        const double* __restrict__ by,
                                                        const double* __restrict__ bz,
                                                        const double* __restrict__ zn,
                                                        const double* __restrict__ dold,
                                                        double* __restrict__ dnew, double* __restrict__ q, int first,
                                                        double* __restrict__ scal,
                                                        double* __restrict__ partials, double* __restrict__ x,
                                                        int xupd, FaceTab<double> ft,
                                                        const double*, int) {
  constexpr int V = 2;
  WIDE_INDEX;
  const int par = (j + k) & 1;
  const size_t pa = par * P + pos, pb = (1 - par) * P + pos;
  PairNb<double, V> z;
  z.load(zn, pa, pb, hx, sz, tp, S, N, D, U);
  double da[V], db[V], qa[V], qb[V], xa[V] = {}, xb[V] = {};
  vload_once<double, V>(da, dold + pa);
  vload_once<double, V>(db, dold + pb);
  vload_once<double, V>(qa, q + pa);
  vload_once<double, V>(qb, q + pb);
  if (xupd) {
    vload_once<double, V>(xa, x + pa);
    vload_once<double, V>(xb, x + pb);
  }
  PairFaces<double, V> F;
  F.load(n, ft, bx, by, bz, ju, k, tp, j, k);
  __builtin_amdgcn_sched_barrier(0);
  double v[2] = {0.0, 0.0};
  const double al = xupd ? scal[S_ALPHA] : 0.0, beta = first ? 0.0 : scal[S_BETA];
  double aa[V], ab[V];
#pragma unroll
  for (int p = 0; p < V; ++p) F.apply2(n, z, p, tp, k < n.nz - 1, aa[p], ab[p]);
  if (live) {
    if (xupd) {
#pragma unroll
      for (int p = 0; p < V; ++p) {
        xa[p] = xa[p] + al * da[p];
        xb[p] = xb[p] + al * db[p];
      }
      vstore_once<double, V>(x + pa, xa);
      vstore_once<double, V>(x + pb, xb);
    }
#pragma unroll
    for (int p = 0; p < V; ++p) {
      da[p] = first ? z.a[p] : z.a[p] + beta * da[p];
      db[p] = first ? z.b[p] : z.b[p] + beta * db[p];
      qa[p] = first ? ih2 * aa[p] : ih2 * aa[p] + beta * qa[p];
      qb[p] = first ? ih2 * ab[p] : ih2 * ab[p] + beta * qb[p];
      v[0] += da[p] * qa[p] + db[p] * qb[p];
      v[1] += z.a[p] * qa[p] + z.b[p] * qb[p];
    }
    vstore_once<double, V>(dnew + pa, da);
    vstore_once<double, V>(dnew + pb, db);
    vstore_once<double, V>(q + pa, qa);
    vstore_once<double, V>(q + pb, qb);
  }
  block_partials<2>(v, partials, tl.lin);
}

// r = b - A x (b, x natural, r split) and the totals, as k_resid_norm; xs, when
// set, receives x split
__global__ void __launch_bounds__(256) k_resid_norm_split(Dims n, double ih2, const double* __restrict__ bx,
                                                          const double* __restrict__ by,
                                                          const double* __restrict__ bz,
                                                          const double* __restrict__ b,
                                                          const double* __restrict__ x, double* __restrict__ r,
                                                          double* __restrict__ partials, FaceTab<double> ft,
                                                          double* __restrict__ xs_) {
  constexpr int V = 2;
  WIDE_INDEX;
  const int par = (j + k) & 1;
  const size_t sxy = (size_t)n.nx * n.ny, c = 2 * (size_t)tp + (size_t)n.nx * (j + (size_t)n.ny * k);
  double xc[4], xs[4], xn[4], xd[4], xu[4], bc[4];
  auto four = [](double (&d)[4], const double* __restrict__ p) {
    vload<double, 2>(*reinterpret_cast<double(*)[2]>(&d[0]), p);
    vload<double, 2>(*reinterpret_cast<double(*)[2]>(&d[2]), p + 2);
  };
  four(xc, x + c);
  four(xs, x + (S ? c - n.nx : c));
  four(xn, x + (N ? c + n.nx : c));
  four(xd, x + (D ? c - sxy : c));
  four(xu, x + (U ? c + sxy : c));
  four(bc, b + c);
  const double xw = x[tp > 0 ? c - 1 : c], xe = x[tp + V < hx ? c + 4 : c + 3];
  PairFaces<double, V> F;
  F.load(n, ft, bx, by, bz, ju, k, tp, j, k);
  __builtin_amdgcn_sched_barrier(0);
  double v[2] = {0.0, 0.0}, rc[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const double a = F.apply(n, p, 2 * tp + p, xc[p], p > 0 ? xc[p > 0 ? p - 1 : 0] : xw, p < 3 ? xc[p < 3 ? p + 1 : p] : xe,
                             xs[p], xn[p], xd[p], xu[p], k < n.nz - 1);
    rc[p] = bc[p] - ih2 * a;
    if (live) {
      v[0] += rc[p] * rc[p];
      v[1] += bc[p] * bc[p];
    }
  }
  if (live) {
    const double ra[2] = {rc[0], rc[2]}, rb[2] = {rc[1], rc[3]};
    vstore<double, 2>(r + par * P + pos, ra);
    vstore<double, 2>(r + (1 - par) * P + pos, rb);
    if (xs_) {
      const double ya[2] = {xc[0], xc[2]}, yb[2] = {xc[1], xc[3]};
      vstore<double, 2>(xs_ + par * P + pos, ya);
      vstore<double, 2>(xs_ + (1 - par) * P + pos, yb);
    }
  }
  block_partials<2>(v, partials, tl.lin);
}

// x = xs + alpha d, xs and d split, x natural
__global__ void __launch_bounds__(256) k_x_update_split(Dims n, const double* __restrict__ d,
                                                        const double* __restrict__ xs, double* __restrict__ x,
                                                        const double* __restrict__ scal) {
  constexpr int V = 2;
  WIDE_INDEX;
  if (!live) return;
  const int par = (j + k) & 1;
  const size_t c = 2 * (size_t)tp + (size_t)n.nx * (j + (size_t)n.ny * k);
  double da[V], db[V], xa[V], xb[V];
  vload<double, V>(da, d + par * P + pos);
  vload<double, V>(db, d + (1 - par) * P + pos);
  vload<double, V>(xa, xs + par * P + pos);
  vload<double, V>(xb, xs + (1 - par) * P + pos);
  const double al = scal[S_ALPHA];
#pragma unroll
  for (int p = 0; p < V; ++p) {
    const double y[2] = {xa[p] + al * da[p], xb[p] + al * db[p]};
    vstore<double, 2>(x + c + 2 * p, y);
  }
}

// r -= alpha q; ||r||^2 (the matching x += alpha d is applied by the next
// direction update, or by k_x_update before x is read).  ndq > 0: <d, q> and
// <z, q> are still in ndq partials, which every wavefront sums for itself; the
// first block then leaves what the finalizing kernels would have in scal.
__global__ void __launch_bounds__(256) k_cg_update(Dims n, const double* __restrict__ q, double* __restrict__ r,
                                                   double* __restrict__ scal, double* __restrict__ partials,
                                                   const double* __restrict__ dqp, int ndq) {
  CELL_INDEX;
  double v[1] = {0.0};
  const double r0 = inside ? r[c] : 0.0, q0 = inside ? q[c] : 0.0;
  double alpha;
  if (ndq > 0) {
    double t[2];
    wave_totals<2>(dqp, ndq, t);
    const double rho = scal[S_RHON];
    alpha = rho / t[0];
    if (tl.lin == 0 && block_tid() == 0) {
      scal[S_RHO] = rho;
      scal[S_DQ] = t[0];
      scal[S_ZQ] = t[1];
      scal[S_ALPHA] = alpha;
    }
  } else {
    alpha = scal[S_ALPHA];
  }
  if (inside) {
    const double rc = r0 - alpha * q0;
    r[c] = rc;
    v[0] = rc * rc;
  }
  block_partials<1>(v, partials, tl.lin);
}

// x += alpha d: the update the CG vector update leaves pending
__global__ void __launch_bounds__(256) k_x_update(Dims n, const double* __restrict__ d, double* __restrict__ x,
                                                  const double* __restrict__ scal) {
  CELL_INDEX;
  if (inside) x[c] = x[c] + scal[S_ALPHA] * d[c];
}

__global__ void __launch_bounds__(256) k_apply_A(Dims n, double ih2, const double* __restrict__ bx,
                                                 const double* __restrict__ by,
                                                 const double* __restrict__ bz,
                                                 const double* __restrict__ x,
                                                 double* __restrict__ y) {
  CELL_INDEX;
  if (inside) y[c] = ih2 * stencil<double>(n, bx, by, bz, x, i, j, k, c);
}


// first stage of a large reduction: block g sums partials [g W, (g + 1) W),
// W = 4 x 1024, thread t the four consecutive ones from g W + 4 t in order,
// then the block's fixed tree; out[nv g + q] gets the block's sums
constexpr int kFinChunk = 4 * 1024;
__global__ void __launch_bounds__(1024) k_finalize_chunks(const double* __restrict__ partials, int nparts, int nv,
                                                          double* __restrict__ out) {
  const int q0 = (int)blockIdx.x * kFinChunk + 4 * (int)threadIdx.x;
  double a[4], c[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int q = min(q0 + u, nparts - 1);
    a[u] = partials[nv * q];
    c[u] = nv > 1 ? partials[nv * q + 1] : 0.0;
  }
  double v[2] = {0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (q0 + u < nparts) {
      v[0] += a[u];
      v[1] += c[u];
    }
  block_sum<2>(v);
  if (threadIdx.x == 0) {
    out[nv * (size_t)blockIdx.x] = v[0];
    if (nv > 1) out[nv * (size_t)blockIdx.x + 1] = v[1];
  }
}

// fixed-order sum of the per-block partials and the CG scalar recurrences;
// the values the host tests are also stored to its pinned mirror
template <int B>
__global__ void __launch_bounds__(1024) k_finalize(const double* __restrict__ partials, int nparts,
                                                   int nv, int mode, double* __restrict__ scal,
                                                   double* __restrict__ hscal) {
  // thread t sums partials t, t + 1024, t + 2048, ... in that order; each
  // batch of B is loaded (clamped, unconditional) before it is added, so the
  // loads are in flight together.  B only sets how many loads one batch
  // issues, never the order of the additions.
  double v[2] = {0.0, 0.0};
  for (int base = threadIdx.x; base < nparts; base += 1024 * B) {
    double a[B], c[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int q = min(base + 1024 * u, nparts - 1);
      a[u] = partials[nv * q];
      c[u] = nv > 1 ? partials[nv * q + 1] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (base + 1024 * u < nparts) {
        v[0] += a[u];
        if (nv > 1) v[1] += c[u];
      }
  }
  block_sum<2>(v);
  if (threadIdx.x == 0) {
    const double a = v[0], b = v[1];
    switch (mode) {
      case FIN_RESID0:
        scal[S_RR] = a;
        scal[S_BB] = b;
        hscal[S_RR] = a;
        hscal[S_BB] = b;
        break;
      case FIN_TRR:
        scal[S_TRR] = a;
        hscal[S_TRR] = a;
        break;
      case FIN_RHO: scal[S_RHO] = a; break;
      case FIN_BETA: {
        // flexible (Polak-Ribiere) beta = (<r, z> - <r, z_old>) / rho, then
        // rho = <r, z>.  r = r_old - alpha q, so <r, z_old> = rho - alpha
        // <q, z_old>, whose product the direction update took where it had
        // z_old and q at hand: summing r z_old here would read z_old again,
        // 8 B per cell.  It differs from that sum by rounding of rho's size,
        // 1e-16 in beta.
        const double rho = scal[S_RHO];
        scal[S_BETA] = (a - (rho - scal[S_ALPHA] * scal[S_ZQ])) / rho;
        scal[S_RHO] = a;
        break;
      }
      case FIN_ALPHA:
        scal[S_DQ] = a;
        scal[S_ZQ] = b;
        scal[S_ALPHA] = scal[S_RHO] / a;
        break;
      case FIN_RR:
        scal[S_RR] = a;
        hscal[S_RR] = a;
        break;
    }
  }
}


}  // namespace

// ------------------------------------------------------------------ launchers
// Pairs per lane of a level's smoothing passes: 0 where the one-pair forms
// run.  The wide forms need whole lanes (hx a multiple of V) and rows that
// fill most of a wavefront, and pay where the level has enough of them to keep
// the chip busy: at 256 x 128 x 128 an FP64 colour pass takes 13.3 us against
// 18.3 (FP32: 11.4 against 13.5), at 128 x 64 x 64, where a row fills half a
// wavefront, 5.2 against 4.3 (FP32: 5.0 against 3.7).  At a million cells, where
// the rule begins, eight FP64 iterations take 1990 us against 1955 on 384 x 52 x
// 54 and less on the other shapes timed (256 x 64 x 64: 1425 against 1468).
// FP32 takes four pairs where such a row still fills a wavefront.
template <typename T>
static int wide_pairs(const Dims& n) {
  const int hx = n.nx / 2;
  if (n.ny < 4 || n.nx % 2 || (long)n.nx * n.ny * n.nz < (1L << 20)) return 0;
  if (sizeof(T) == 4 && hx % 4 == 0 && hx / 4 >= 48) return 4;
  return hx % 2 == 0 && hx / 2 >= 48 ? 2 : 0;
}
static dim3 wide_grid(const Dims& n, int V) {
  return dim3((n.nx / 2 / V + 63) / 64, (n.ny + 3) / 4, n.nz);
}
bool cg_split(const Dims& n) { return wide_pairs<double>(n) == 2; }

template <typename T>
void launch_gs(const Level& L, const T* bx, const T* by, const T* bz, const T* b, T* e, int colour,
               hipStream_t st, KTimer* kt, T* nat) {
  const bool fine = (L.h == L.h0);
  const FaceTab<T> ft = face_tab(L, bx);
  const bool tab1 = !fine && ft.x != nullptr;   // a coarse level with line tables
  if (const int V = nat ? 0 : wide_pairs<T>(L.n)) {
    auto kern = V == 2 ? k_gs_wide<T, 2> : k_gs_wide<T, 16 / sizeof(T)>;
    const dim3 grid = wide_grid(L.n, V), blk(64, 4);
    if (kt && kt->n < kt->cap) {
      hipExtLaunchKernelGGL(kern, grid, blk, 0, st, kt->ev[2 * kt->n], kt->ev[2 * kt->n + 1], 0, L.n,
                            (T)(L.h * L.h), bx, by, bz, b, e, colour, ft);
      ++kt->n;
    } else {
      hipLaunchKernelGGL(kern, grid, blk, 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, colour, ft);
    }
    return;
  }
  const int pl = gs_planes<T>(fine || tab1);   // planes per thread
  Geo g = geo3((L.n.nx + 1) / 2, L.n.ny, (L.n.nz + pl - 1) / pl);
  auto kern = fine ? k_gs<T, true> : tab1 ? k_gs_c1<T> : k_gs<T, false>;
  if (kt && kt->n < kt->cap) {
    hipExtLaunchKernelGGL(kern, g.grid, g.block, 0, st, kt->ev[2 * kt->n], kt->ev[2 * kt->n + 1], 0, L.n,
                          (T)(L.h * L.h), bx, by, bz, b, e, colour, nat, ft);
    ++kt->n;
    return;
  }
  hipLaunchKernelGGL(kern, g.grid, g.block, 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, colour, nat, ft);
}

template <typename T>
void launch_gs_first(const Level& L, const T* bx, const T* by, const T* bz, const T* b, bool b_natural,
                     const T* invd, T* e, T* bs, hipStream_t st, T* bcopy, bool red_out) {
  Geo g = geo3((L.n.nx + 1) / 2, L.n.ny, L.n.nz);
  const bool fine = (L.h == L.h0);
  const FaceTab<T> ft = face_tab(L, bx);
  const bool tab1 = !fine && ft.x != nullptr && !b_natural;   // a coarse level with line tables
  if (const int V = b_natural ? 0 : wide_pairs<T>(L.n)) {
    auto kern = V == 2 ? k_gs_first_wide<T, 2, T> : k_gs_first_wide<T, 16 / sizeof(T), T>;
    hipLaunchKernelGGL(kern, wide_grid(L.n, V), dim3(64, 4), 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, invd, e, bs,
                       bcopy, ft, red_out ? 1 : 0);
    return;
  }
  void (*kern)(Dims, T, const T*, const T*, const T*, const T*, const T*, T*, T*, T*, FaceTab<T>, int);
  if (b_natural)
    kern = fine ? k_gs_first<T, true, true> : k_gs_first<T, false, true>;
  else
    kern = fine ? k_gs_first<T, true, false> : tab1 ? k_gs_first_c1<T> : k_gs_first<T, false, false>;
  hipLaunchKernelGGL(kern, g.grid, g.block, 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, invd, e, bs, bcopy, ft,
                     red_out ? 1 : 0);
}

template <typename T>
void launch_gs_prolong(const Level& L, const T* bx, const T* by, const T* bz, const T* b, T* e,
                       const Level& C, const T* ec, bool ec_split, hipStream_t st, T* bcopy) {
  const bool fine = (L.h == L.h0);
  const FaceTab<T> ft = face_tab(L, bx);
  const bool tab1 = !fine && ft.x != nullptr;   // a coarse level with line tables
  if (const int V = L.f[0] == 2 ? wide_pairs<T>(L.n) : 0) {
    auto kern = V == 2 ? k_gs_prolong_wide<T, 2> : k_gs_prolong_wide<T, 16 / sizeof(T)>;
    hipLaunchKernelGGL(kern, wide_grid(L.n, V), dim3(64, 4), 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, C.n,
                       L.f[1] >> 1, L.f[2] >> 1, ec_split ? 1 : 0, ec, bcopy, ft);
    return;
  }
  const int pl = gs_planes<T>(fine || tab1);   // planes per thread
  Geo g = geo3((L.n.nx + 1) / 2, L.n.ny, (L.n.nz + pl - 1) / pl);
  auto kern = fine ? k_gs_prolong<T, true> : tab1 ? k_gs_prolong_c1<T> : k_gs_prolong<T, false>;
  hipLaunchKernelGGL(kern, g.grid, g.block, 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, C.n, L.f[0] >> 1,
                     L.f[1] >> 1, L.f[2] >> 1, ec_split ? 1 : 0, ec, bcopy, ft);
}

// the fused red-black pass's tile (TX lanes per row, TY rows, TZ planes), or
// false where a row does not fit one tile
static bool gs_rb_tile(const Dims& n, int& TX, int& TY, int& TZ) {
  const int hx = (n.nx + 1) / 2;
  if (hx > 32) return false;
  TX = hx > 16 ? 32 : hx > 8 ? 16 : 8;
  TY = n.ny > 1 ? 4 : 1;
  // TX TY is 8 to 128, a divisor of kRbThreads: the tile has one black cell
  // per thread
  static_assert(kRbThreads % (32 * 4) == 0, "every TX TY divides the block");
  TZ = kRbThreads / (TX * TY);
  // the ring-extended tile within the kernel's LDS and its unrolled loads
  return TX * (TY + (n.ny > 1 ? 2 : 0)) * (TZ + 2) <= kRbMaxExt;
}

bool gs_rb_fits(const Dims& n) {
  int TX, TY, TZ;
  return gs_rb_tile(n, TX, TY, TZ);
}

template <typename T>
void launch_gs_rb(const Level& L, const T* bx, const T* by, const T* bz, const T* b, T* e, const T* bold,
                  hipStream_t st) {
  int TX, TY, TZ;
  if (!gs_rb_tile(L.n, TX, TY, TZ)) return;   // callers check gs_rb_fits first
  const dim3 grid(1, (L.n.ny + TY - 1) / TY, (L.n.nz + TZ - 1) / TZ);
  hipLaunchKernelGGL(k_gs_rb<T>, grid, dim3(kRbThreads), 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, bold, TX,
                     TY, TZ);
}

// the finest level's fused red-black sweep: where it applies (a 3-D level
// whose rows fill at least half a wave), where it pays, and its launch.  A
// block runs 64 lanes by kRbfRows + 2 rows of pairs and the halo wave (1024
// threads) up a chunk of planes.
constexpr int kRbfRows = 13;    // inner rows of a block (TY)

bool gs_rb_fine_fits(const Dims& n) {
  return n.ny >= 4 && n.nz >= 4 && (n.nx + 1) / 2 >= 32;
}

// A block's march is a chain of dependent planes: the launch wins over two
// colour passes on large grids only, in FP64 only, and only where the
// passes load every face (on 512 x 256 x 256 378 us against 2 x 223 in FP64,
// but 249 against 2 x 116 in FP32, whose planes carry half the bytes for the
// same instructions; slower in both on 256 x 128 x 128 and 128 x 64 x 64).
// With the line tables a colour pass loads few faces and takes 153 us there,
// and the two passes win (the march's loads stay as many).
bool gs_rb_fine_pays(const Dims& n, bool fp64, bool tables) {
  return fp64 && !tables && gs_rb_fine_fits(n) && (long)n.nx * n.ny * n.nz >= (1L << 24);
}

// compute units of the current device (one block of the sweep per unit)
static int device_cus() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] > 0) return cache[dev];
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
  cache[dev] = v;
  return v;
}

// The chunk of planes a block marches.  A block holds its compute unit for
// its whole march (KZ + 2 planes), so the sweep takes about (rounds of
// blocks) x (KZ + 2) plane times: the chunk is chosen to minimise that
// product, ties going to fewer chunks.  512 x 256 x 256 gets 3 chunks of 86
// planes, 240 blocks, one round.
static int rbf_planes(int tiles, int nz, int cus) {
  long best = -1;
  int best_kz = nz;
  for (int nzc = 1; nzc <= nz; ++nzc) {
    const int kz = (nz + nzc - 1) / nzc;
    const int chunks = (nz + kz - 1) / kz;
    const long rounds = ((long)tiles * chunks + cus - 1) / cus;
    const long cost = rounds * (kz + 2);
    if (best < 0 || cost < best) {
      best = cost;
      best_kz = kz;
    }
  }
  return best_kz;
}

template <typename T>
void launch_gs_rb_fine(const Level& L, const T* bx, const T* by, const T* bz, const T* b, T* e, const T* bold,
                       hipStream_t st, KTimer* kt) {
  constexpr int TY = kRbfRows;
  static_assert(kRbfLanes * (TY + 3) == 1024, "a block of 1024 threads");
  const int hx = (L.n.nx + 1) / 2;
  const int gx = (hx + kRbfLanes - 1) / kRbfLanes, gy = (L.n.ny + TY - 1) / TY;
  const int KZ = rbf_planes(gx * gy, L.n.nz, device_cus());
  const dim3 grid(gx, gy, (L.n.nz + KZ - 1) / KZ);
  const dim3 blk(kRbfLanes, TY + 3);
  const T h2 = (T)(L.h * L.h);
  if (kt && kt->n < kt->cap) {
    hipExtLaunchKernelGGL((k_gs_rb_fine<T, TY>), grid, blk, 0, st, kt->ev[2 * kt->n], kt->ev[2 * kt->n + 1], 0, L.n,
                          h2, bx, by, bz, b, e, bold, KZ);
    ++kt->n;
    return;
  }
  hipLaunchKernelGGL((k_gs_rb_fine<T, TY>), grid, blk, 0, st, L.n, h2, bx, by, bz, b, e, bold, KZ);
}

// the pair form of the residual-restriction: even extents, halved in every
// direction (the fine level is colour-split wherever it is called)
static bool resid_pairs_fit(const Level& F) {
  return F.f[0] == 2 && F.f[1] == 2 && F.f[2] == 2 && F.n.nx % 2 == 0 && F.n.ny % 2 == 0 && F.n.nz % 2 == 0;
}

template <typename T>
void launch_resid_restrict(const Level& F, const T* bx, const T* by, const T* bz, const T* b,
                           const T* e, const Level& C, T* bc, bool c_split, hipStream_t st) {
  const T ih2 = (T)(1.0 / (F.h * F.h));
  if (resid_pairs_fit(F)) {
    if (const int V = wide_pairs<T>(F.n)) {
      auto kern = V == 2 ? k_resid_restrict_wide<T, 2> : k_resid_restrict_wide<T, 16 / sizeof(T)>;
      hipLaunchKernelGGL(kern, dim3((F.n.nx / 2 / V + 63) / 64, F.n.ny / 2, F.n.nz / 2), dim3(64, 2, 2), 0, st, F.n,
                         ih2, bx, by, bz, b, e, C.n, c_split ? 1 : 0, (T)0.125, bc, face_tab(F, bx));
      return;
    }
    const dim3 grid((F.n.nx / 2 + 63) / 64, F.n.ny / 2, F.n.nz / 2);
    hipLaunchKernelGGL(k_resid_restrict_pairs<T>, grid, dim3(64, 2, 2), 0, st, F.n, ih2, bx, by, bz, b, e, C.n,
                       c_split ? 1 : 0, (T)0.125, bc, face_tab(F, bx));
    return;
  }
  // fine-cell tiles with even extents (a coarse cell's children in one tile)
  const dim3 blk = (F.n.ny > 1) ? dim3(32, 4, 2) : dim3(64, 1, 4);
  const Geo g{dim3((F.n.nx + blk.x - 1) / blk.x, (F.n.ny + blk.y - 1) / blk.y, (F.n.nz + blk.z - 1) / blk.z), blk};
  const T inv = (T)(1.0 / (F.f[0] * F.f[1] * F.f[2]));
  hipLaunchKernelGGL(k_resid_restrict<T>, g.grid, g.block, 0, st, F.n, F.f[0], F.f[1], F.f[2], ih2, bx,
                     by, bz, b, e, C.n, c_split ? 1 : 0, inv, bc);
}

template <typename T>
void launch_prolong(const Level& F, T* e, const Level& C, const T* ec, bool ec_split, hipStream_t st) {
  Geo g = geo3(F.n.nx, F.n.ny, F.n.nz);
  hipLaunchKernelGGL(k_prolong<T>, g.grid, g.block, 0, st, F.n, F.f[0] >> 1, F.f[1] >> 1, F.f[2] >> 1, e, C.n,
                     ec_split ? 1 : 0, ec);
}

template <typename T>
void launch_split_copy(const Level& L, const T* src, T* dst, bool to_split, hipStream_t st) {
  Geo g = geo3(L.n.nx, L.n.ny, L.n.nz);
  hipLaunchKernelGGL(k_split_copy<T>, g.grid, g.block, 0, st, L.n, src, dst, to_split ? 1 : 0);
}

template <typename T>
void launch_invdiag(const Level& L, const T* bx, const T* by, const T* bz, T* invd, bool split, hipStream_t st) {
  Geo g = geo3(L.n.nx, L.n.ny, L.n.nz);
  hipLaunchKernelGGL(k_invdiag<T>, g.grid, g.block, 0, st, L.n, bx, by, bz, split ? 1 : 0, invd);
}

template <typename T>
void launch_coarsen_chain(const CoarsenChain<T>& D, hipStream_t st) {
  hipLaunchKernelGGL(k_coarsen_chain<T>, dim3(1), dim3(1024), 0, st, D);
}
template <typename T>
void launch_coarsen_level(const Level& F, const T* fbx, const T* fby, const T* fbz, const Level& C, T* cbx,
                          T* cby, T* cbz, T* invd, bool split, hipStream_t st) {
  Geo g = geo3(C.n.nx, C.n.ny, C.n.nz);
  hipLaunchKernelGGL(k_coarsen_level<T>, g.grid, g.block, 0, st, F.n, F.f[0], F.f[1], F.f[2], fbx, fby, fbz, C.n,
                     cbx, cby, cbz, split ? 1 : 0, invd);
}

template <typename T>
void launch_vcycle_tail(const TailDesc<T>& D, size_t lds_bytes, hipStream_t st) {
  // dynamic LDS above 64 KB needs the kernel's limit raised (once per process)
  using Kern = void (*)(TailDesc<T>);
  constexpr int M = tail_top_pairs<T>();
  static const Kern kerns[] = {k_vcycle_matrix<T>, k_vcycle_tail<T, 1>, k_vcycle_tail<T, 2>, k_vcycle_tail<T, 3>,
                               k_vcycle_tail<T, 4>, k_vcycle_tail<T, M < 5 ? M : 5>, k_vcycle_tail<T, M < 6 ? M : 6>};
  static bool raised[7] = {};
  // pairs per thread of the level in registers
  const int v = D.top ? ((D.nt.nx + 1) / 2 * D.nt.ny * D.nt.nz + kTailThreads - 1) / kTailThreads : 0;
  if (lds_bytes > 64 * 1024 && !raised[v]) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kerns[v]), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)kTailLdsBytes);
    raised[v] = true;
  }
  hipLaunchKernelGGL(kerns[v], dim3(1), dim3(kTailThreads), lds_bytes, st, D);
}

template <typename T>
void launch_tail_matrix(const TailDesc<T>& D, int elems, T* M, hipStream_t st) {
  TailDesc<double> C{};
  C.nl = D.nl;
  C.nu_pre = D.nu_pre;
  C.nu_post = D.nu_post;
  C.coarse_sweeps = D.coarse_sweeps;
  for (int l = 0; l < D.nl; ++l) {
    C.n[l] = D.n[l];
    for (int d = 0; d < 3; ++d) C.f[l][d] = D.f[l][d];
    C.h2[l] = (double)D.h2[l];
    C.obx[l] = D.obx[l];
    C.oby[l] = D.oby[l];
    C.obz[l] = D.obz[l];
    C.oid[l] = D.oid[l];
    C.ob[l] = D.ob[l];
    C.oe[l] = D.oe[l];
  }
  C.ors = D.ors;
  C.npack = D.npack;
  C.omv = D.omv;
  const int N = D.n[0].nx * D.n[0].ny * D.n[0].nz;
  hipLaunchKernelGGL(k_tail_matrix<T>, dim3(N), dim3(64), (size_t)elems * sizeof(double), st, C, D.pack, M);
}

// 2-D levels that are halved both ways (k_pre2d, k_post2d)
bool tank2d_fits(const Level& L) { return L.n.ny == 1 && L.f[0] == 2 && L.f[2] == 2; }
static dim3 grid2d(const Dims& n) { return dim3((n.nx + kT2X - 1) / kT2X, (n.nz + kT2Z - 1) / kT2Z); }

template <typename T, typename TB>
void launch_pre2d(const Level& L, const T* bx, const T* bz, const T* invd, const TB* b, T* e, bool csplit, T* bc,
                  hipStream_t st) {
  hipLaunchKernelGGL((k_pre2d<T, TB>), grid2d(L.n), dim3(kT2Threads), 0, st, L.n.nx, L.n.nz, (T)(L.h * L.h), bx, bz, invd,
                     b, e, csplit ? 1 : 0, bc);
}
template <typename T, typename TB, typename TO>
int launch_post2d(const Level& L, const T* bx, const T* bz, const T* invd, const TB* b, const T* e, bool csplit,
                  const T* ec, TO* out, const double* r, double* partials, hipStream_t st) {
  const dim3 g = grid2d(L.n);
  hipLaunchKernelGGL((k_post2d<T, TB, TO>), g, dim3(kT2Threads), 0, st, L.n.nx, L.n.nz, (T)(L.h * L.h), bx, bz, invd, b,
                     e, csplit ? 1 : 0, ec, out, r, partials);
  return (int)(g.x * g.y);
}
#define NSK_INST2(T, TB)                                                                                        \
  template void launch_pre2d<T, TB>(const Level&, const T*, const T*, const T*, const TB*, T*, bool, T*, hipStream_t);
#define NSK_INST3(T, TB, TO)                                                                                    \
  template int launch_post2d<T, TB, TO>(const Level&, const T*, const T*, const T*, const TB*, const T*, bool, \
                                        const T*, TO*, const double*, double*, hipStream_t);
NSK_INST2(double, double)
NSK_INST2(float, float)
NSK_INST2(float, double)
NSK_INST3(double, double, double)
NSK_INST3(float, float, float)
NSK_INST3(float, double, double)
NSK_INST3(float, double, float)
#undef NSK_INST2
#undef NSK_INST3

template <typename T>
void launch_fill(T* a, size_t n, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, n);
}

template <typename T>
void launch_face_tables(const Dims& n, const T* bx, const T* by, const T* bz, T* tx, T* ty, T* tz, hipStream_t st) {
  const int lines = n.ny * n.nz + (n.ny + 1) * n.nz + n.ny * (n.nz + 1);
  hipLaunchKernelGGL(k_face_table<T>, dim3((lines + 3) / 4), dim3(256), 0, st, n, bx, by, bz, tx, ty, tz);
}

// Where the line tables pay: each kernel that reads them waits one cache
// round trip for its lines' entries before it issues their faces' loads, which
// a latency-bound level cannot hide (128 x 64 x 64: the FP64 step 2.5% slower
// with them); from 2^21 cells on the bytes they spare win (256 x 128 x 128:
// 7.00 -> 6.27 ms, 512 x 256 x 256: 51.1 -> 41.5 ms).
bool face_tables_pay(const Dims& n) { return (long)n.nx * n.ny * n.nz >= (1L << 21); }


void launch_d2f(const double* a, float* b, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_d2f, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, b, n);
}

template <typename T>
int launch_gs_last_dots(const Level& L, const T* bx, const T* by, const T* bz, const T* b, const T* e,
                        double* nat, const double* r, double* partials, hipStream_t st) {
  Geo g = geo3((L.n.nx + 1) / 2, L.n.ny, L.n.nz);
  hipLaunchKernelGGL(k_gs_last_dots<T>, g.grid, g.block, 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, nat, r,
                     partials, face_tab(L, bx));
  return (int)(g.grid.x * g.grid.y * g.grid.z);
}

// Two pairs per lane in both precisions: FP64 vectors take part, whose 16
// bytes are two values (four pairs read them at a lane stride of 32 bytes).
template <typename T>
void launch_gs_first_split(const Level& L, const T* bx, const T* by, const T* bz, const double* r, const T* invd, T* e,
                           T* bs, hipStream_t st, bool red_out) {
  hipLaunchKernelGGL((k_gs_first_wide<T, 2, double>), wide_grid(L.n, 2), dim3(64, 4), 0, st, L.n, (T)(L.h * L.h), bx,
                     by, bz, r, invd, e, bs, (T*)nullptr, face_tab(L, bx), red_out ? 1 : 0);
}

template <typename T>
int launch_gs_last_dots_split(const Level& L, const T* bx, const T* by, const T* bz, const T* b, const T* e, double* z,
                              const double* r, double* partials, hipStream_t st) {
  const dim3 g = wide_grid(L.n, 2);
  hipLaunchKernelGGL((k_gs_last_dots_wide<T, 2>), g, dim3(64, 4), 0, st, L.n, (T)(L.h * L.h), bx, by, bz, b, e, z, r,
                     partials, face_tab(L, bx));
  return (int)(g.x * g.y * g.z);
}

void launch_gs_first_nat64(const Level& L, const float* bx, const float* by, const float* bz, const double* b,
                           const float* invd, float* e, float* bs, hipStream_t st, float* bcopy, bool red_out) {
  Geo g = geo3((L.n.nx + 1) / 2, L.n.ny, L.n.nz);
  hipLaunchKernelGGL((k_gs_first<float, true, true, double>), g.grid, g.block, 0, st, L.n, (float)(L.h * L.h), bx,
                     by, bz, b, invd, e, bs, bcopy, face_tab(L, bx), red_out ? 1 : 0);
}

int launch_f2d_dots(const float* a, double* z, size_t n, const double* r, double* partials, hipStream_t st) {
  const int nb = (int)((n + 255) / 256);
  hipLaunchKernelGGL(k_f2d_dots, dim3(nb), dim3(256), 0, st, a, z, n, r, partials);
  return nb;
}

void launch_f2d(const float* a, double* b, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_f2d, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, b, n);
}

int cg_blocks(const Dims& n) {
  Geo g = geo3(n.nx, n.ny, n.nz);
  return (int)(g.grid.x * g.grid.y * g.grid.z);
}

static void finalize(const CgScratch& cs, int nparts, int mode, hipStream_t st) {
  const int nv = (mode == FIN_RESID0 || mode == FIN_TRR || mode == FIN_ALPHA) ? 2 : 1;
  const double* src = cs.partials;
  // Beyond one batch of 16 loads per thread, one workgroup walking every
  // partial waits on a chain of batches (27 us for the 131072 blocks of a
  // 512 x 256 x 256 level): the chunks are summed first, one workgroup
  // each, into the partials buffer's free room after the nv * nparts values
  // (the buffer holds 4 per block of the finest level; nv <= 2), and their
  // sums finalized.  Up to one batch a single launch is cheaper.
  if (nparts > 16 * 1024) {
    const int G = (nparts + kFinChunk - 1) / kFinChunk;
    double* mid = cs.partials + (size_t)nv * nparts;
    hipLaunchKernelGGL(k_finalize_chunks, dim3(G), dim3(1024), 0, st, cs.partials, nparts, nv, mid);
    src = mid;
    nparts = G;
  }
  // loads per thread per batch: as many as the partials need, at most 16
  const int per = (nparts + 1023) / 1024;
  const dim3 g(1), b(1024);
  if (per <= 1)
    hipLaunchKernelGGL(k_finalize<1>, g, b, 0, st, src, nparts, nv, mode, cs.scal, cs.hscal);
  else if (per <= 2)
    hipLaunchKernelGGL(k_finalize<2>, g, b, 0, st, src, nparts, nv, mode, cs.scal, cs.hscal);
  else if (per <= 4)
    hipLaunchKernelGGL(k_finalize<4>, g, b, 0, st, src, nparts, nv, mode, cs.scal, cs.hscal);
  else
    hipLaunchKernelGGL(k_finalize<16>, g, b, 0, st, src, nparts, nv, mode, cs.scal, cs.hscal);
}

void launch_finalize_dot(const CgScratch& cs, int nparts, int mode, hipStream_t st) { finalize(cs, nparts, mode, st); }

int launch_resid_norm(const Dims& n, double h, const double* bx, const double* by, const double* bz, const double* b,
                      const double* x, double* r, const CgScratch& cs, int mode, hipStream_t st,
                      const FaceTab<double>& ft, bool split, double* xs) {
  // blockDim.x == 64: a wavefront per x-line
  const Geo g = split ? Geo{wide_grid(n, 2), dim3(64, 4)} : geo3(n.nx, n.ny, n.nz);
  double* part = cs.hpart ? cs.hpart : cs.partials;
  if (split)
    hipLaunchKernelGGL(k_resid_norm_split, g.grid, g.block, 0, st, n, 1.0 / (h * h), bx, by, bz, b, x, r, part, ft, xs);
  else
    hipLaunchKernelGGL(k_resid_norm, g.grid, g.block, 0, st, n, 1.0 / (h * h), bx, by, bz, b, x, r, part, ft);
  const int np = (int)(g.grid.x * g.grid.y * g.grid.z);
  if (!cs.hpart) finalize(cs, np, mode, st);
  return np;
}

// Where the direction update and the vector update sum the partials before
// them for themselves instead of waiting for a finalizing launch each: up to
// 512 partials (131072 cells), which a wavefront sums in a microsecond against
// the launch's 3.3 to 4 us (256 x 1 x 64 steps 2.85 -> 2.65 ms, 640 x 1 x 96 3.55 -> 3.32)
bool cg_folds(const Dims& n) { return cg_blocks(n) <= 512; }

int launch_dot(const Dims& n, const double* r, const double* z, const CgScratch& cs, int mode, hipStream_t st,
               bool fold) {
  Geo g = geo3(n.nx, n.ny, n.nz);
  hipLaunchKernelGGL(k_dot_rho, g.grid, g.block, 0, st, n, r, z, cs.partials);
  const int np = (int)(g.grid.x * g.grid.y * g.grid.z);
  if (!fold) finalize(cs, np, mode, st);
  return np;
}

void launch_dir_spmv(const Dims& n, double h, const double* bx, const double* by, const double* bz,
                     const double* zn, const double* dold, double* dnew, double* q, int first,
                     const CgScratch& cs, hipStream_t st, KTimer* kt, double* x, const FaceTab<double>& ft, bool split,
                     int ndot) {
  // blockDim.x == 64: a wavefront per x-line
  const Geo g = split ? Geo{wide_grid(n, 2), dim3(64, 4)} : geo3(n.nx, n.ny, n.nz);
  const int xupd = x ? 1 : 0, np = (int)(g.grid.x * g.grid.y * g.grid.z);
  // (folded: its partials go behind those of <r, z>, which its blocks read)
  double* part = ndot > 0 ? cs.partials + 2 * (size_t)np : cs.partials;
  auto kern = split ? k_dir_spmv_split : k_dir_spmv;
  if (kt && kt->n < kt->cap) {
    (void)hipStreamSynchronize(st);
    hipExtLaunchKernelGGL(kern, g.grid, g.block, 0, st, kt->ev[2 * kt->n], kt->ev[2 * kt->n + 1], 0, n, 1.0 / (h * h), bx,
                          by, bz, zn, dold, dnew, q, first, cs.scal, part, x, xupd, ft, (const double*)cs.partials, ndot);
    ++kt->n;
  } else {
    hipLaunchKernelGGL(kern, g.grid, g.block, 0, st, n, 1.0 / (h * h), bx, by, bz, zn, dold, dnew, q, first, cs.scal, part,
                       x, xupd, ft, (const double*)cs.partials, ndot);
  }
  if (ndot == 0) finalize(cs, np, FIN_ALPHA, st);
}

void launch_cg_update(const Dims& n, const double* q, double* r, const CgScratch& cs, hipStream_t st, bool fold) {
  Geo g = geo3(n.nx, n.ny, n.nz);
  const int np = (int)(g.grid.x * g.grid.y * g.grid.z);
  hipLaunchKernelGGL(k_cg_update, g.grid, g.block, 0, st, n, q, r, cs.scal, cs.hpart ? cs.hpart : cs.partials,
                     (const double*)(cs.partials + 2 * (size_t)np), fold ? np : 0);
  if (!cs.hpart) finalize(cs, np, FIN_RR, st);
}

void launch_x_update(const Dims& n, const double* d, double* x, const CgScratch& cs, hipStream_t st, const double* xs) {
  if (xs) {
    hipLaunchKernelGGL(k_x_update_split, wide_grid(n, 2), dim3(64, 4), 0, st, n, d, xs, x, (const double*)cs.scal);
    return;
  }
  Geo g = geo3(n.nx, n.ny, n.nz);
  hipLaunchKernelGGL(k_x_update, g.grid, g.block, 0, st, n, d, x, (const double*)cs.scal);
}

void launch_apply_A(const Dims& n, double h, const double* bx, const double* by, const double* bz,
                    const double* x, double* y, hipStream_t st) {
  Geo g = geo3(n.nx, n.ny, n.nz);
  hipLaunchKernelGGL(k_apply_A, g.grid, g.block, 0, st, n, 1.0 / (h * h), bx, by, bz, x, y);
}

#define NSK_INST(T)                                                                                   \
  template void launch_gs<T>(const Level&, const T*, const T*, const T*, const T*, T*, int, hipStream_t,   \
                             KTimer*, T*);                                                                \
  template int launch_gs_last_dots<T>(const Level&, const T*, const T*, const T*, const T*, const T*,     \
                                      double*, const double*, double*, hipStream_t);                      \
  template int launch_gs_last_dots_split<T>(const Level&, const T*, const T*, const T*, const T*, const T*, \
                                            double*, const double*, double*, hipStream_t);                \
  template void launch_gs_first_split<T>(const Level&, const T*, const T*, const T*, const double*, const T*, T*, \
                                         T*, hipStream_t, bool);                                          \
  template void launch_gs_first<T>(const Level&, const T*, const T*, const T*, const T*, bool, const T*,  \
                                   T*, T*, hipStream_t, T*, bool);                                        \
  template void launch_gs_prolong<T>(const Level&, const T*, const T*, const T*, const T*, T*,           \
                                     const Level&, const T*, bool, hipStream_t, T*);                      \
  template void launch_gs_rb<T>(const Level&, const T*, const T*, const T*, const T*, T*, const T*,     \
                                hipStream_t);                                                             \
  template void launch_gs_rb_fine<T>(const Level&, const T*, const T*, const T*, const T*, T*, const T*,  \
                                     hipStream_t, KTimer*);                                               \
  template void launch_resid_restrict<T>(const Level&, const T*, const T*, const T*, const T*, const T*,  \
                                         const Level&, T*, bool, hipStream_t);                            \
  template void launch_prolong<T>(const Level&, T*, const Level&, const T*, bool, hipStream_t);           \
  template void launch_split_copy<T>(const Level&, const T*, T*, bool, hipStream_t);                     \
  template void launch_invdiag<T>(const Level&, const T*, const T*, const T*, T*, bool, hipStream_t);    \
  template void launch_coarsen_level<T>(const Level&, const T*, const T*, const T*, const Level&, T*, \
                                        T*, T*, T*, bool, hipStream_t);                               \
  template void launch_fill<T>(T*, size_t, hipStream_t);                                              \
  template void launch_face_tables<T>(const Dims&, const T*, const T*, const T*, T*, T*, T*, hipStream_t); \
  template void launch_vcycle_tail<T>(const TailDesc<T>&, size_t, hipStream_t);                       \
  template void launch_coarsen_chain<T>(const CoarsenChain<T>&, hipStream_t);                         \
  template void launch_tail_matrix<T>(const TailDesc<T>&, int, T*, hipStream_t);
NSK_INST(double)
NSK_INST(float)
#undef NSK_INST

}  // namespace nsk
