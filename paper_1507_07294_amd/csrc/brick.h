// One-kernel time step of small lattices (part of kernels.hip's translation
// unit): every block owns a three-dimensional brick of BX x BY x BZ nodes, one
// per thread, and does the whole step of it in one pass (the z-marching
// kernels of fused.hip carry a column of planes through LDS rings instead).
//
// A lattice that cannot fill the chip is bound by the length of the chain of
// memory round trips in its step, not by bytes: a march makes one per plane
// and one per warm-up plane.  A brick makes one: all its loads (its nodes' own
// populations and history, and the f of its halo, from which phi is summed)
// go out together, then phi, mu and the collisions follow from LDS behind two
// barriers.  The price is the halo: a node pulls more f than in a march, which
// a lattice that stays in the caches can afford.
//
// Measured, march against bricks, us per step: 32^3 droplet FP64 30.7 / 7.6
// (about 2 us of it the launch), 64^3 FP32 27.3 / 12.7, 48 x 48 x 192 with BF16
// populations 25.1 / 18.1, 70 x 77 x 69 with walls on every axis FP32 32.1 /
// 22.4, D3Q19 64 x 64 x 256 FP32 56.2 / 45.7 (5.3 TB/s), CHE-only 64^3 FP32
// 14.1 / 6.3, 128^3 29.4 / 27.6 (4.9 TB/s).  What is left on the larger of these
// is the traffic of the last-level cache (a copy of their size moves 6-7 TB/s)
// and the vector-memory instructions of the halo pulls: halo nodes per node of
// the brick (16 x 4 x 4, 16 x 8 x 4, 32 x 4 x 4) 4.0, 2.75, 3.5 in the coupled
// step, 1.53, 1.11, 1.39 in the CHE-only one.
#pragma once

#include "common.h"
#include "device.h"
#include "launch.h"

namespace mplb {
namespace {

using namespace dev;

// Buffer accesses at a byte offset per lane plus a scalar one (the start of an
// array): array offsets cost no vector instruction.
template <class S>
__device__ inline S ld_off(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
  if constexpr (sizeof(S) == 2) {
    return __builtin_bit_cast(S, (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, off, soff, 0));
  } else if constexpr (sizeof(S) == 4) {
    return __builtin_bit_cast(S, (unsigned int)__builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
  } else {
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
  }
}
template <class S>
__device__ inline void st_off(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff, S v) {
  if constexpr (sizeof(S) == 2) {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, off, soff, 0);
  } else if constexpr (sizeof(S) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, soff, 0);
  } else {
    using U2 = unsigned int __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, off, soff, 0);
  }
}

// map_axis for a position from two nodes before an axis to two nodes past it
// (two steps of wrapping, for axes of one node; no division).  Positions
// further out belong to no node of the lattice; they take some valid node.
__device__ inline int near_axis(int v, int n, int wall) {
  if (wall) return clamp_axis(v, n);
  v = v < n + 1 ? v : n + 1;
  v += v < 0 ? n : 0;
  v += v < 0 ? n : 0;
  v -= v >= n ? n : 0;
  v -= v >= n ? n : 0;
  return v;
}

// A brick padded by H nodes on every side, and its halo positions.
template <int BX, int BY, int BZ, int H>
struct Pad {
  static constexpr int PX = BX + 2 * H, PY = BY + 2 * H, PZ = BZ + 2 * H;
  static constexpr int PXY = PX * PY, NPHI = PXY * PZ;
  static constexpr int NT = BX * BY * BZ, NHALO = NPHI - NT;
  static constexpr int HPT = (NHALO + NT - 1) / NT;

  // Halo position h: first the whole rows above, below, before and behind the
  // brick, then the 2 H columns at the sides of the brick's own rows (each of
  // those a cache line of its own).
  __device__ static void pos(int h, int& px, int& py, int& pz) {
    constexpr int ZROWS = 2 * H * PY, ROWS = PY * PZ - BY * BZ;
    if (h < ROWS * PX) {
      const int r = h / PX;
      px = h % PX;
      if (r < ZROWS) {
        pz = r / PY;
        py = r % PY;
        if (pz >= H) pz += BZ;
      } else {
        pz = H + (r - ZROWS) / (2 * H);
        py = (r - ZROWS) % (2 * H);
        if (py >= H) py += BY;
      }
    } else {
      h -= ROWS * PX;
      px = h % (2 * H);
      if (px >= H) px += BX;
      py = H + h / (2 * H) % BY;
      pz = H + h / (2 * H) / BY;
    }
  }
};

// Where the pulls of a coordinate along one axis come from, as byte offsets
// into the arrays of f_1..f_6 (element type QS): the coordinate itself, the
// source of a population with c_a = +1 (coordinate - 1, wrapped) and of one
// with c_a = -1.  The last two count from the array of the +1 population (the
// -1 one is the next array), so that a bounce at a wall, the node itself in
// the other array, is an offset like any other.  bounce: bit 0 for c_a = +1,
// bit 1 for c_a = -1.
struct __align__(16) Axis {
  uint32_t at, plus, minus, bounce;
};

// The block's table of Axis entries, for each coordinate of the padded brick
// (x, then y, then z).  A position then costs three LDS reads and ten
// additions; wrapping its own coordinates and testing them for walls took
// about 90 vector instructions.
template <class QS, class D, int H>
__device__ inline void fill_axes(const Geo& G, int x0, int y0, int z0, Axis* tab) {
  for (int t = threadIdx.x; t < D::PX + D::PY + D::PZ; t += D::NT) {
    int v, n, stride, wall;
    if (t < D::PX) v = x0 - H + t, n = G.nx, stride = 1, wall = G.wall_x;
    else if (t < D::PX + D::PY) v = y0 - H + t - D::PX, n = G.ny, stride = G.nx, wall = G.wall_y;
    else v = z0 - H + t - D::PX - D::PY, n = G.nz, stride = G.nx * G.ny, wall = G.wall_z;
    const int m = near_axis(v, n, wall);
    const bool first = m == 0, last = m == n - 1;
    const bool bp = wall && first, bm = wall && last;
    const uint32_t next = (uint32_t)G.pitch;
    const uint32_t p = (uint32_t)((bp ? m : first ? n - 1 : m - 1) * stride) + (bp ? next : 0u);
    const uint32_t q = (uint32_t)((bm ? m : last ? 0 : m + 1) * stride) + (bm ? 0u : next);
    constexpr uint32_t sz = sizeof(QS);
    tab[t] = Axis{(uint32_t)(m * stride) * sz, p * sz, q * sz, (bp ? 1u : 0u) | (bm ? 2u : 0u)};
  }
}

// Offsets of the pulls along the axes: o[i - 1] for population i = 1..6.
__device__ inline void face_offsets(const Axis& x, const Axis& y, const Axis& z, uint32_t o[6]) {
  const uint32_t xy = x.at + y.at, yz = y.at + z.at, xz = x.at + z.at;
  o[0] = yz + x.plus;
  o[1] = yz + x.minus;
  o[2] = xz + y.plus;
  o[3] = xz + y.minus;
  o[4] = xy + z.plus;
  o[5] = xy + z.minus;
}

// rf: the f buffer from its start, ri: from the arrays of f_1..f_6
template <int P, bool PACK>
__device__ inline void pull7(__amdgpu_buffer_rsrc_t rf, __amdgpu_buffer_rsrc_t ri, uint32_t pitch, const Axis& x,
                             const Axis& y, const Axis& z, F7Raw<P, PACK>& o) {
  using S0 = typename Lat<P, PACK>::S0;
  using QS = typename F7Raw<P, PACK>::QS;
  static_assert(sizeof(S0) % sizeof(QS) == 0, "f_0 at a multiple of the others' offset");
  o.r0 = ld_off<S0>(rf, (x.at + y.at + z.at) * (uint32_t)(sizeof(S0) / sizeof(QS)), 0);
  uint32_t off[6];
  face_offsets(x, y, z, off);
#pragma unroll
  for (int i = 0; i < 6; ++i) o.r[i] = ld_off<QS>(ri, off[i], (uint32_t)(i / 2) * 2 * pitch * (uint32_t)sizeof(QS));
}

// The g of the brick's own node (PACK: g_0 and g_7 on, at half the offsets of
// the packed words).  The faces come from where f_1..f_6 do; the others, also
// stored in antipodal pairs, bounce if any of their axes does.
template <int P, bool PACK, bool WALL, int Q>
__device__ inline void pull_own_g(__amdgpu_buffer_rsrc_t rg, uint32_t pitch, const Axis& x, const Axis& y,
                                  const Axis& z, typename Lat<P, PACK>::S g[Q]) {
  using L = Lat<P, PACK>;
  using S = typename L::S;
  using QS = typename F7Raw<P, PACK>::QS;
  constexpr uint32_t half = sizeof(QS) / sizeof(S);
  const uint32_t arr = pitch * (uint32_t)sizeof(S), next = pitch * (uint32_t)sizeof(QS);
  const uint32_t n = x.at + y.at + z.at;
  g[0] = ld_off<S>(rg, n / half, 0);
  if constexpr (!PACK) {
    uint32_t off[6];
    face_offsets(x, y, z, off);
#pragma unroll
    for (int i = 0; i < 6; ++i) g[i + 1] = ld_off<S>(rg, off[i], (uint32_t)(1 + i / 2 * 2) * arr);
  }
  // sources of the diagonal velocities, without the step to the next array
  const uint32_t sx[3] = {x.minus - next, x.at, x.plus}, sy[3] = {y.minus - next, y.at, y.plus},
                 sz[3] = {z.minus - next, z.at, z.plus};
#pragma unroll
  for (int i = 7; i < Q; ++i) {
    const int cx = cq<Q>(i, 0), cy = cq<Q>(i, 1), cz = cq<Q>(i, 2);
    uint32_t at = sx[cx + 1] + sy[cy + 1] + sz[cz + 1];
    const int first = i & 1 ? i : i - 1;  // of the antipodal pair
    if constexpr (WALL) {
      uint32_t b = 0;
      if (cx != 0) b |= x.bounce & (cx > 0 ? 1u : 2u);
      if (cy != 0) b |= y.bounce & (cy > 0 ? 1u : 2u);
      if (cz != 0) b |= z.bounce & (cz > 0 ? 1u : 2u);
      at = i == first ? (b ? n + next : at) : (b ? n : at + next);
      g[i] = ld_off<S>(rg, at / half, (uint32_t)L::gslot(first) * arr);
    } else {
      g[i] = ld_off<S>(rg, at / half, (uint32_t)L::gslot(i) * arr);
    }
  }
}

// Brick lb of the lattice: its first node, bricks ordered x, y, z.
template <int BX, int BY, int BZ>
__device__ inline void brick_origin(const Geo& G, int lb, int& x0, int& y0, int& z0) {
  const int bx = (G.nx + BX - 1) / BX, by = (G.ny + BY - 1) / BY;
  x0 = lb % bx * BX;
  const int t = lb / bx;
  y0 = t % by * BY;
  z0 = t / by * BZ;
}

// The coupled step of brick lb (Q: velocities of the NSE lattice; V: kVarUnit
// or 0).
template <int P, int Q, bool WALL, int V, int BX, int BY, int BZ>
__device__ inline void brick_body(const Geo& G, const Coef<typename Prec<P>::T>& C, const Bufs& B, int cur, int lb) {
  using T = typename Prec<P>::T;
  constexpr bool PACK = packed<P, true>();
  using L = Lat<P, PACK>;
  using S = typename L::S;
  using S0 = typename L::S0;
  using QS = typename F7Raw<P, PACK>::QS;
  using D = Pad<BX, BY, BZ, 2>;
  using M1 = Pad<BX, BY, BZ, 1>;
  constexpr int NT = D::NT;
  static_assert(sizeof(T) == sizeof(QS) && sizeof(S0) == sizeof(QS), "one offset for f, f_0 and the history");
  __shared__ T sphi[D::NPHI];
  __shared__ T smu[M1::NPHI];
  __shared__ Axis tab[D::PX + D::PY + D::PZ];
  if (C.poison) {
    poison_shared(sphi, sizeof sphi);
    poison_shared(smu, sizeof smu);
    poison_shared(tab, sizeof tab);
    __syncthreads();
  }
  int x0, y0, z0;
  brick_origin<BX, BY, BZ>(G, lb, x0, y0, z0);
  fill_axes<QS, D, 2>(G, x0, y0, z0, tab);
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX % BY, tz = tid / (BX * BY);
  const bool own = x0 + tx < G.nx && y0 + ty < G.ny && z0 + tz < G.nz;
  const uint32_t pitch = (uint32_t)G.pitch, arr = pitch * (uint32_t)sizeof(T);
  const void* fin = cur ? B.f[1] : B.f[0];
  const void* gin = cur ? B.g[1] : B.g[0];
  void* fo = cur ? B.f[0] : B.f[1];
  void* go = cur ? B.g[0] : B.g[1];
  const auto rf = rsrc_at(fin), ri = rsrc_at(L::fi(fin, G.pitch)), rg = rsrc_at(gin), rh = rsrc_at(B.phiu);
  __syncthreads();

  // every load of the step: the node's own f, the f of its halo positions, g
  // and the history.  Every lane loads (a lane without a node or a position
  // takes a valid one and drops the value): a branch would leave the number
  // of loads in flight unknown, and phi would wait for the g as well (32^3
  // FP32 6.6 -> 6.1 us per step, W = 48 box with 16-bit populations 19.2 ->
  // 16.8 us).
  const Axis ax = tab[tx + 2], ay = tab[D::PX + ty + 2], az = tab[D::PX + D::PY + tz + 2];
  const uint32_t n = ax.at + ay.at + az.at;
  F7Raw<P, PACK> fr;
  pull7<P, PACK>(rf, ri, pitch, ax, ay, az, fr);
  F7Raw<P, PACK> hr[D::HPT];
  int hat[D::HPT];
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    const int h = tid + k * NT;
    int px, py, pz;
    D::pos(h < D::NHALO ? h : D::NHALO - 1, px, py, pz);
    hat[k] = px + D::PX * py + D::PXY * pz;
    pull7<P, PACK>(rf, ri, pitch, tab[px], tab[D::PX + py], tab[D::PX + D::PY + pz], hr[k]);
  }
  S gr[Q];
  T hp[3];
  pull_own_g<P, PACK, WALL, Q>(rg, pitch, ax, ay, az, gr);
#pragma unroll
  for (int a = 0; a < 3; ++a) hp[a] = ld_off<T>(rh, n, (uint32_t)a * arr);
  __builtin_amdgcn_sched_barrier(0);

  // phi of the padded brick
  T f[7];
  cvt_f7<P, PACK>(fr, f);
  const T phi = phi_of(f);
  const int pat = (tx + 2) + D::PX * (ty + 2) + D::PXY * (tz + 2);
  sphi[pat] = phi;
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    if (tid + k * NT < D::NHALO) {
      T fh[7];
      cvt_f7<P, PACK>(hr[k], fh);
      sphi[hat[k]] = phi_of(fh);
    }
  }
  __syncthreads();
  // mu of the brick (k = 0) and of a halo of one; a ghost position of a wall
  // takes its mirror image
#pragma unroll
  for (int k = 0; k <= M1::HPT; ++k) {
    const int h = tid + (k - 1) * NT;
    if (k == 0 || h < M1::NHALO) {
      int qx = tx + 1, qy = ty + 1, qz = tz + 1;
      if (k > 0) M1::pos(h, qx, qy, qz);
      int sx = qx + 1, sy = qy + 1, sz = qz + 1;
      if constexpr (WALL) {
        if (G.wall_x) sx = clamp_axis(x0 - 1 + qx, G.nx) - (x0 - 2);
        if (G.wall_y) sy = clamp_axis(y0 - 1 + qy, G.ny) - (y0 - 2);
        if (G.wall_z) sz = clamp_axis(z0 - 1 + qz, G.nz) - (z0 - 2);
      }
      const T* pc = sphi + (sx + D::PX * sy + D::PXY * sz);
      const T c0 = pc[0];
      const T lap = lap_lds<T, D::PX>(pc - D::PXY, pc, pc + D::PXY, 0);
      smu[qx + M1::PX * qy + M1::PXY * qz] = 4 * C.beta * c0 * (c0 - 1) * (c0 + 1) - C.kappa * lap;
    }
  }
  __syncthreads();
  if (!own) return;

  T g[Q];
  if constexpr (PACK) {
#pragma unroll
    for (int i = 1; i < 7; ++i) g[i] = L::hi(fr.r[i - 1]);
  }
  g[0] = (T)gr[0];
#pragma unroll
  for (int i = PACK ? 7 : 1; i < Q; ++i) g[i] = (T)gr[i];
  const T* pc = sphi + pat;
  const T* mc = smu + ((tx + 1) + M1::PX * (ty + 1) + M1::PXY * (tz + 1));
  T gphi[3];
  grad_lds<T, D::PX>(pc - D::PXY, pc, pc + D::PXY, 0, gphi);
  const T mu = mc[0];
  const T lapmu = lap_lds<T, M1::PX>(mc - M1::PXY, mc, mc + M1::PXY, 0);
  Macro<T> M;
  if constexpr (Q == 19) flow_macro19(C, g, phi, mu, gphi, lapmu, M);
  else flow_macro(C, g, phi, mu, gphi, lapmu, M);
  T dphiu[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const T pu = phi * M.u[a];
    dphiu[a] = pu - hp[a];
    st_off<T>(rh, n, (uint32_t)a * arr, pu);
  }
  collide_che(C, f, phi, mu, M.u, dphiu);
  if constexpr (Q == 19) collide_ns19(C, g, M);
  else collide_ns<false, (V & kVarUnit) != 0>(C, g, M);
  const auto wf = rsrc_at(fo), wi = rsrc_at(L::fi(fo, G.pitch)), wg = rsrc_at(go);
  constexpr uint32_t half = sizeof(QS) / sizeof(S);
  const uint32_t ng = n / half, garr = pitch * (uint32_t)sizeof(S);
  st_off<S0>(wf, n, 0, (S0)f[0]);
  st_off<S>(wg, ng, 0, (S)g[0]);
#pragma unroll
  for (int i = 1; i < 7; ++i) {
    if constexpr (PACK) st_off<uint32_t>(wi, n, (uint32_t)(i - 1) * arr, L::pack(f[i], g[i]));
    else st_off<S>(wi, n, (uint32_t)(i - 1) * arr, (S)f[i]);
  }
#pragma unroll
  for (int i = PACK ? 7 : 1; i < Q; ++i) st_off<S>(wg, ng, (uint32_t)L::gslot(i) * garr, (S)g[i]);
  if (!(all_finite(f, 7) && all_finite(g, Q))) *B.flag = 1;
}

template <int P, int Q, bool WALL, int V, int BX, int BY, int BZ>
__global__ void __launch_bounds__(BX* BY* BZ) __attribute__((amdgpu_waves_per_eu(waves_per_eu<P>())))
k_brick(Geo G, Coef<typename Prec<P>::T> C, Bufs B, int cur) {
  brick_body<P, Q, WALL, V, BX, BY, BZ>(G, C, B, cur, logical_block(blockIdx.x, gridDim.x));
}

// The CHE-only step of a brick: mu at the node only, so phi needs a halo of
// one, and the history is phi alone.
template <int P, int BX, int BY, int BZ>
__global__ void __launch_bounds__(BX* BY* BZ) __attribute__((amdgpu_waves_per_eu(waves_per_eu<P>())))
k_brick_che(Geo G, Coef<typename Prec<P>::T> C, Bufs B, int cur) {
  using T = typename Prec<P>::T;
  using L = Lat<P, false>;
  using S = typename L::S;
  using S0 = typename L::S0;
  using D = Pad<BX, BY, BZ, 1>;
  constexpr int NT = D::NT;
  static_assert(2 * (BX + BY + BZ) <= NT, "one sine per thread");
  __shared__ T sphi[D::NPHI];
  // sin(pi t / n) and sin(2 pi t / n) of the deformation flow at the brick's
  // coordinates, x then y then z
  __shared__ T sn[2][BX + BY + BZ];
  __shared__ Axis tab[D::PX + D::PY + D::PZ];
  if (C.poison) {
    poison_shared(sphi, sizeof sphi);
    poison_shared(sn, sizeof sn);
    poison_shared(tab, sizeof tab);
    __syncthreads();
  }
  int x0, y0, z0;
  brick_origin<BX, BY, BZ>(G, logical_block(blockIdx.x, gridDim.x), x0, y0, z0);
  fill_axes<S, D, 1>(G, x0, y0, z0, tab);
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX % BY, tz = tid / (BX * BY);
  const int gx = x0 + tx, gy = y0 + ty, gz = z0 + tz;
  const bool own = gx < G.nx && gy < G.ny && gz < G.nz;
  const uint32_t pitch = (uint32_t)G.pitch;
  const void* fin = cur ? B.f[1] : B.f[0];
  void* fo = cur ? B.f[0] : B.f[1];
  const auto rf = rsrc_at(fin), ri = rsrc_at(L::fi(fin, G.pitch)), rh = rsrc_at(B.phiu);
  __syncthreads();
  const Axis ax = tab[tx + 1], ay = tab[D::PX + ty + 1], az = tab[D::PX + D::PY + tz + 1];
  const uint32_t n = ax.at + ay.at + az.at;                       // f_1..f_6
  const uint32_t n0 = n * (uint32_t)(sizeof(T) / sizeof(S));      // f_0 and the history
  F7Raw<P, false> fr;
  pull7<P, false>(rf, ri, pitch, ax, ay, az, fr);
  F7Raw<P, false> hr[D::HPT];
  int hat[D::HPT];
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    const int h = tid + k * NT;
    hat[k] = -1;
    if (h < D::NHALO) {
      int px, py, pz;
      D::pos(h, px, py, pz);
      hat[k] = px + D::PX * py + D::PXY * pz;
      pull7<P, false>(rf, ri, pitch, tab[px], tab[D::PX + py], tab[D::PX + D::PY + pz], hr[k]);
    }
  }
  T phip = 0, u[3] = {0, 0, 0}, up[3] = {0, 0, 0};
  if (own) {
    phip = ld_off<T>(rh, n0, 0);
    if (C.vel_kind != MPLB_VEL_DEFORM)
      presc_u(G, C, (const T*)B.ufield, gx, gy, gz, (int)(n / (uint32_t)sizeof(S)), u, up);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (C.vel_kind == MPLB_VEL_DEFORM && tid < 2 * (BX + BY + BZ)) {
    const T pi = (T)3.14159265358979323846;
    const int w = tid / (BX + BY + BZ), k = tid % (BX + BY + BZ);
    const int c = k < BX ? x0 + k : (k < BX + BY ? y0 + k - BX : z0 + k - BX - BY);
    const int m = k < BX ? G.nx : (k < BX + BY ? G.ny : G.nz);
    const T h = (T)c / (T)m;
    sn[w][k] = w ? sin(2 * pi * h) : sin(pi * h);
  }
  T f[7];
  cvt_f7<P, false>(fr, f);
  const T phi = phi_of(f);
  const int pat = (tx + 1) + D::PX * (ty + 1) + D::PXY * (tz + 1);
  sphi[pat] = phi;
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    if (hat[k] >= 0) {
      T fh[7];
      cvt_f7<P, false>(hr[k], fh);
      sphi[hat[k]] = phi_of(fh);
    }
  }
  __syncthreads();
  if (!own) return;
  const T* pc = sphi + pat;
  const T lap = lap_lds<T, D::PX>(pc - D::PXY, pc, pc + D::PXY, 0);
  const T mu = 4 * C.beta * phi * (phi - 1) * (phi + 1) - C.kappa * lap;
  if (C.vel_kind == MPLB_VEL_DEFORM) {
    // the products in the order of PrescColumn
    const T U = C.velU;
    const T sx = sn[0][tx], s2x = sn[1][tx], sy = sn[0][BX + ty], s2y = sn[1][BX + ty];
    const T sz = sn[0][BX + BY + tz], s2z = sn[1][BX + BY + tz];
    const T a0 = 2 * U * sx * sx * s2y, a1 = -U * s2x * sy * sy, a2 = -U * s2x * s2y;
    const T b[3] = {a0 * s2z, a1 * s2z, a2 * sz * sz};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      u[k] = b[k] * C.vel_ct;
      up[k] = b[k] * C.vel_ct_prev;
    }
  }
  st_off<T>(rh, n0, 0, phi);
  T dphiu[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) dphiu[a] = phi * u[a] - phip * up[a];
  collide_che(C, f, phi, mu, u, dphiu);
  const auto wf = rsrc_at(fo), wi = rsrc_at(L::fi(fo, G.pitch));
  st_off<S0>(wf, n0, 0, (S0)f[0]);
#pragma unroll
  for (int i = 1; i < 7; ++i) st_off<S>(wi, n, (uint32_t)(i - 1) * pitch * (uint32_t)sizeof(S), (S)f[i]);
  if (!all_finite(f, 7)) *B.flag = 1;
}

// Many small lattices in one launch, as k_fused_many does it: a block finds
// its lattice in the table by its index.
template <int P, bool WALL, int V, int BX, int BY, int BZ>
__global__ void __launch_bounds__(BX* BY* BZ) __attribute__((amdgpu_waves_per_eu(waves_per_eu<P>())))
k_brick_many(const BatchItem<typename Prec<P>::T>* __restrict__ tab, int count, int flip) {
  const int b = logical_block(blockIdx.x, gridDim.x);
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) / 2;
    if (tab[mid].block0 <= b) lo = mid;
    else hi = mid - 1;
  }
  const BatchItem<typename Prec<P>::T> it = tab[lo];
  brick_body<P, 15, WALL, V, BX, BY, BZ>(it.G, it.C, it.B, it.cur0 ^ flip, b - it.block0);
}

// The brick sizes: 16 x 4 x 4, 16 x 8 x 4 and 32 x 4 x 4.
constexpr int brick_x(Bricks br) { return br == kBricksWide ? 32 : 16; }
constexpr int brick_y(Bricks br) { return br == kBricksMid ? 8 : 4; }
static_assert(brick_x(kBricksNarrow) * brick_y(kBricksNarrow) * 4 == brick_threads(kBricksNarrow) &&
                  brick_x(kBricksMid) * brick_y(kBricksMid) * 4 == brick_threads(kBricksMid) &&
                  brick_x(kBricksWide) * brick_y(kBricksWide) * 4 == brick_threads(kBricksWide),
              "one thread per node");

// the coupled bricks that brick_kind picks
constexpr bool coupled_bricks(int P, Bricks br) { return P != MPLB_F64 || br == kBricksNarrow; }

template <int P, bool WALL, Bricks BR>
hipError_t brick_impl3(int mode, const Geo& G, const Coef<typename Prec<P>::T>& C, const Bufs& B, int cur,
                       hipStream_t s) {
  constexpr int BX = brick_x(BR), BY = brick_y(BR), BZ = 4;
  const dim3 grid((unsigned)brick_blocks(G, BR)), block(brick_threads(BR));
  if (mode == MPLB_CHE_ONLY) {
    hipLaunchKernelGGL((k_brick_che<P, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
    return hipGetLastError();
  }
  if constexpr (coupled_bricks(P, BR)) {
    if (mode == MPLB_COUPLED_Q19)
      hipLaunchKernelGGL((k_brick<P, 19, WALL, 0, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
    else if (C.unit_rates)
      hipLaunchKernelGGL((k_brick<P, 15, WALL, kVarUnit, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
    else
      hipLaunchKernelGGL((k_brick<P, 15, WALL, 0, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <int P, bool WALL>
hipError_t brick_impl2(int mode, const Geo& G, const Coef<typename Prec<P>::T>& C, const Bufs& B, int cur, Bricks br,
                       hipStream_t s) {
  switch (br) {
    case kBricksWide: return brick_impl3<P, WALL, kBricksWide>(mode, G, C, B, cur, s);
    case kBricksMid: return brick_impl3<P, WALL, kBricksMid>(mode, G, C, B, cur, s);
    default: return brick_impl3<P, WALL, kBricksNarrow>(mode, G, C, B, cur, s);
  }
}

template <int P>
hipError_t brick_impl(int mode, const Geo& G, const Coef<double>& Cd, const Bufs& B, int cur, Bricks br,
                      hipStream_t s) {
  const auto C = cast_coef<typename Prec<P>::T>(Cd);
  if (G.wall_x || G.wall_y || G.wall_z) return brick_impl2<P, true>(mode, G, C, B, cur, br, s);
  return brick_impl2<P, false>(mode, G, C, B, cur, br, s);
}

template <int P, bool WALL, int V>
const void* brick_many3(Bricks br) {
  if (br == kBricksNarrow)
    return (const void*)k_brick_many<P, WALL, V, brick_x(kBricksNarrow), brick_y(kBricksNarrow), 4>;
  if constexpr (coupled_bricks(P, kBricksWide)) {
    return br == kBricksWide
               ? (const void*)k_brick_many<P, WALL, V, brick_x(kBricksWide), brick_y(kBricksWide), 4>
               : (const void*)k_brick_many<P, WALL, V, brick_x(kBricksMid), brick_y(kBricksMid), 4>;
  }
  return nullptr;
}
template <int P>
const void* brick_many2(bool wall, bool unit, Bricks br) {
  if (wall) return unit ? brick_many3<P, true, kVarUnit>(br) : brick_many3<P, true, 0>(br);
  return unit ? brick_many3<P, false, kVarUnit>(br) : brick_many3<P, false, 0>(br);
}

// Bricks pull the f of their halo once per brick, so they need the state in
// the 256 MB last-level cache; beyond it the march, which reads each
// population about once, wins.  Bytes a step reads and writes, march against
// bricks in us per step: coupled FP32 200 MB (100^3) 55.7 / 45.9, 281 MB
// (112^3) 65.3 / 56.8, 315 MB (128 x 128 x 96) 68.3 / 81.8; FP64 149 MB (72^3)
// 43.7 / 32.5, 273 MB (88^3) 58.9 / 53.7, 295 MB 60.3 / 66.1; D3Q19 FP32
// 243 MB (64 x 64 x 256) 56.0 / 47.5, 326 MB 83.9 / 94.7; CHE-only FP32
// 262 MB (160^3) 58.7 / 52.7, 349 MB 97.7 / 117.7; CHE-only FP16 283 MB
// (192^3) 90.2 / 75.9; CHE-only FP64 221 MB (120^3) 45.6 / 44.7, 268 MB (128^3)
// 49.5 / 52.1.
constexpr size_t kBrickBytes = (size_t)285000000, kBrickBytesCheF64 = (size_t)240000000;
// 16-bit populations reach that size only on lattices large enough to fill the
// chip with marching blocks.  There a march whose 64 x 8 tiles are full wins:
// 1.05 M nodes (64 x 64 x 256) 38.1 / 35.9, 1.57 M (128 x 128 x 96) 46.2 / 52.0;
// not so with partly empty tiles: 120^3 62.5 / 58.4, 112^3 52.4 / 49.9.
constexpr long long kBrickNodes16 = 1200000;

// Narrow bricks below 100 k nodes, where they put twice as many CUs to work
// (32^3 FP32 6.3 us per step against 7.2 and 7.3 with the larger ones), and for
// the coupled step in FP64, whose blocks of four waves fit a CU twice (72^3
// 32.2 / 35.0 mid / 39.4 wide).  Otherwise wide ones, whose rows are a whole
// cache line, where they cover at most 1.2 times the nodes that mid ones do
// (1.1 with 16-bit populations), else mid ones.  Mid against wide: FP32
// 64 x 64 x 256 40.1 / 36.2, 72^3 (1.2) 21.2 / 18.4, 70 x 77 x 69 (1.2) 21.6 /
// 20.5, 48 x 48 x 192 (1.33) 20.7 / 21.4; FP16 128 x 100 x 80 (0.96) 32.8 / 29.6,
// 100^3 (1.10) 33.2 / 32.0, 112 x 112 x 84 (1.14) 33.0 / 32.5, 70 x 77 x 69 (1.2)
// 17.3 / 17.9, 80^3 (1.2) 18.1 / 18.7; CHE-only FP32 128^3 29.3 / 27.1, FP64
// 64^3 9.5 / 9.0.  These are periodic boxes at the paper's rates; with walls on
// every axis and other rates mid ones gain 3-15 % against wide ones (FP32 70 x
// 77 x 69 21.1 / 21.8, FP16 100^3 32.2 / 36.0), which the rule does not look at.
Bricks brick_kind(int P, int mode, long long nodes, long long mid, long long wide) {
  if (nodes < 100000 || (mode != MPLB_CHE_ONLY && P == MPLB_F64)) return kBricksNarrow;
  const bool bits16 = P == MPLB_F32_F16 || P == MPLB_F32_BF16;
  return 10 * wide <= (mode != MPLB_CHE_ONLY && bits16 ? 11 : 12) * mid ? kBricksWide : kBricksMid;
}

// nodes that 64 x 8 marching tiles cover
long long march_nodes(const Geo& G) {
  return (long long)((G.nx + 63) / 64 * 64) * ((G.ny + 7) / 8 * 8) * G.nz;
}

// A flat lattice, of a node or five along z, say, leaves part of every brick
// empty.  Bricks are still the faster on a small one, which latency bounds; the
// march is on a large one, or in a batch of many: where the nodes that bricks
// cover, times the excess over those that marching tiles do, pass this limit
// (a lattice counts from an excess of 0.3 on).  us per step, march / bricks,
// by that product: FP32 256 x 256 (0.8 M) 11.1 / 10.2, 512 x 512 (3.1 M) 18.9 /
// 22.8, 256 x 256 x 5 (0.3 M) 27.5 / 19.6, 512 x 512 x 5 (1.3 M) 53.9 / 61.1;
// 24 together, 64 x 64 x 9 (0.4 M) 50 / 36, 64 x 64 (1.2 M) 12.5 / 13.7, 128 x
// 128 x 5 (1.9 M) 89 / 95; FP64, 64 x 64 x 5 (0.5 M) 48 / 51.
constexpr long long kFlatWork = 1000000, kFlatWorkBatchF64 = 450000;

}  // namespace

long long flat_work(const Geo& G) {
  const long long bricks = 512LL * brick_blocks(G, kBricksMid), march = march_nodes(G);
  return 10 * bricks > 13 * march ? (long long)((double)bricks * (bricks - march) / march) : 0;
}

long long flat_work_limit(int P) { return P == MPLB_F64 ? kFlatWorkBatchF64 : kFlatWork; }

int brick_blocks(const Geo& G, Bricks br) {
  const int bx = brick_x(br), by = brick_y(br);
  return ((G.nx + bx - 1) / bx) * ((G.ny + by - 1) / by) * ((G.nz + 3) / 4);
}

Shape brick_shape(const Geo& G, Bricks br) {
  const int bx = brick_x(br), by = brick_y(br);
  return Shape{kShapeBricks + (int)br - 1, bx, by, Tiling{(G.nx + bx - 1) / bx, (G.ny + by - 1) / by, 4, (G.nz + 3) / 4}};
}

Bricks step_bricks(int P, int mode, const Geo& G, const Coef<double>& C) {
  if (C.stencil7 || C.forcing28) return kBricksNone;  // the study variants are marching kernels
  const long long n = (long long)G.nx * G.ny * G.nz;
  const bool bits16 = P == MPLB_F32_F16 || P == MPLB_F32_BF16;
  const size_t bytes = fused_step_bytes(P, mode, n);
  const size_t limit = mode == MPLB_CHE_ONLY && P == MPLB_F64 ? kBrickBytesCheF64 : kBrickBytes;
  if (bytes > limit || flat_work(G) > kFlatWork) return kBricksNone;
  if (mode != MPLB_CHE_ONLY && bits16 && n > kBrickNodes16 && 10 * march_nodes(G) < 11 * n) return kBricksNone;
  return brick_kind(P, mode, n, 512LL * brick_blocks(G, kBricksMid), 512LL * brick_blocks(G, kBricksWide));
}

// In a batch, GLUPS in bricks (groups of lattices that fit the cache together)
// against the marching kernel over many: FP32 32^3 27.1 / 18.9, 48^3 24.4 /
// 22.0, 64^3 26.3 / 24.7, 96^3 25.4 / 22.2; FP64 32^3 13.6 / 9.1, 48^3 12.8 / 11.2;
// 16-bit populations 32^3 35.5 / 23.2, 48^3 35.6 / 30.3, 96^3 33.0 / 30.2.  In
// FP64 and with 16-bit populations a march whose tiles are full is the faster
// one once its lattices fill the chip: 64^3 11.1 / 12.7 and 32.5 / 38.3.
BatchUse batch_use(int P, const Geo& G) {
  const long long n = (long long)G.nx * G.ny * G.nz;
  if (fused_step_bytes(P, MPLB_COUPLED, n) > kBrickBytes) return kBatchMarch;
  return P != MPLB_F32 && 10 * march_nodes(G) < 11 * n ? kBatchMarchIfFull : kBatchBricks;
}

Bricks batch_bricks(int P, long long nodes, long long mid, long long wide) {
  return brick_kind(P, MPLB_COUPLED, nodes, mid, wide);
}

const void* brick_many_kernel(int P, bool wall, bool unit, Bricks br) {
  switch (P) {
    case MPLB_F64: return brick_many2<MPLB_F64>(wall, unit, br);
    case MPLB_F32: return brick_many2<MPLB_F32>(wall, unit, br);
    case MPLB_F32_F16: return brick_many2<MPLB_F32_F16>(wall, unit, br);
    case MPLB_F32_BF16: return brick_many2<MPLB_F32_BF16>(wall, unit, br);
    default: return nullptr;
  }
}

hipError_t launch_brick_step(int P, int mode, const Geo& G, const Coef<double>& C, const Bufs& B, int cur, Bricks br,
                             hipStream_t s) {
  switch (P) {
    case MPLB_F64: return brick_impl<MPLB_F64>(mode, G, C, B, cur, br, s);
    case MPLB_F32: return brick_impl<MPLB_F32>(mode, G, C, B, cur, br, s);
    case MPLB_F32_F16: return brick_impl<MPLB_F32_F16>(mode, G, C, B, cur, br, s);
    case MPLB_F32_BF16: return brick_impl<MPLB_F32_BF16>(mode, G, C, B, cur, br, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mplb
