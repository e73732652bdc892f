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
// and the vector-memory instructions of the halo pulls (4.0-4.5 times the
// brick's own nodes in the coupled step, 2.4-2.5 in the CHE-only one).
#pragma once

#include "common.h"
#include "device.h"
#include "launch.h"

namespace mplb {
namespace {

using namespace dev;

template <class S>
__device__ inline S ld_off(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(S) == 2) {
    return __builtin_bit_cast(S, (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0));
  } else if constexpr (sizeof(S) == 4) {
    return __builtin_bit_cast(S, (unsigned int)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  } else {
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  }
}
template <class S>
__device__ inline void st_off(__amdgpu_buffer_rsrc_t r, uint32_t off, S v) {
  if constexpr (sizeof(S) == 2) {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, off, 0, 0);
  } else if constexpr (sizeof(S) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, 0);
  } else {
    using U2 = unsigned int __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, off, 0, 0);
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

// A lattice node with the index steps to the sources of its pulls: s[a][0]
// leads to the node a population with c_a = +1 comes from (x_a - 1, wrapped),
// s[a][1] to that with c_a = -1; b likewise says that the population comes
// through a wall of axis a.
struct Node {
  int n;
  int s[3][2];
  bool b[3][2];
};

// Node of lattice position (x, y, z), at most two nodes outside the lattice.
template <bool WALL>
__device__ inline Node make_node(const Geo& G, int x, int y, int z) {
  Node d;
  x = near_axis(x, G.nx, WALL && G.wall_x);
  y = near_axis(y, G.ny, WALL && G.wall_y);
  z = near_axis(z, G.nz, WALL && G.wall_z);
  const int nxy = G.nx * G.ny;
  d.n = x + G.nx * y + nxy * z;
  d.s[0][0] = x == 0 ? G.nx - 1 : -1;
  d.s[0][1] = x == G.nx - 1 ? 1 - G.nx : 1;
  d.s[1][0] = y == 0 ? nxy - G.nx : -G.nx;
  d.s[1][1] = y == G.ny - 1 ? G.nx - nxy : G.nx;
  d.s[2][0] = z == 0 ? G.N - nxy : -nxy;
  d.s[2][1] = z == G.nz - 1 ? nxy - G.N : nxy;
  if constexpr (WALL) {
    d.b[0][0] = G.wall_x && x == 0;
    d.b[0][1] = G.wall_x && x == G.nx - 1;
    d.b[1][0] = G.wall_y && y == 0;
    d.b[1][1] = G.wall_y && y == G.ny - 1;
    d.b[2][0] = G.wall_z && z == 0;
    d.b[2][1] = G.wall_z && z == G.nz - 1;
  }
  return d;
}

// Element index of the pull of population i (velocity c) into node d, in a
// run of arrays `pitch` apart whose array `slot` holds population i and
// `oslot` the opposite one.  32 bits hold it, in bytes too: the host takes
// this kernel only for buffers below 4 GiB.
template <bool WALL>
__device__ inline uint32_t pull_at(const Node& d, uint32_t pitch, int cx, int cy, int cz, uint32_t slot,
                                   uint32_t oslot) {
  int idx = d.n;
  if (cx != 0) idx += d.s[0][cx < 0];
  if (cy != 0) idx += d.s[1][cy < 0];
  if (cz != 0) idx += d.s[2][cz < 0];
  const uint32_t at = slot * pitch + (uint32_t)idx;
  if constexpr (WALL) {
    bool b = false;
    if (cx != 0) b = b || d.b[0][cx < 0];
    if (cy != 0) b = b || d.b[1][cy < 0];
    if (cz != 0) b = b || d.b[2][cz < 0];
    return b ? oslot * pitch + (uint32_t)d.n : at;
  }
  return at;
}

template <int P, bool PACK>
struct Raw7 {
  using L = Lat<P, PACK>;
  using QS = typename std::conditional<PACK, uint32_t, typename L::S>::type;
  typename L::S0 r0;
  QS r[6];
};

// rf: the f buffer from its start, ri: from the arrays of f_1..f_6
template <int P, bool PACK, bool WALL>
__device__ inline void pull7(__amdgpu_buffer_rsrc_t rf, __amdgpu_buffer_rsrc_t ri, uint32_t pitch, const Node& d,
                             Raw7<P, PACK>& o) {
  using L = Lat<P, PACK>;
  using QS = typename Raw7<P, PACK>::QS;
  o.r0 = ld_off<typename L::S0>(rf, (uint32_t)d.n * (uint32_t)sizeof(typename L::S0));
#pragma unroll
  for (int i = 1; i < 7; ++i)
    o.r[i - 1] = ld_off<QS>(ri, pull_at<WALL>(d, pitch, c7(i, 0), c7(i, 1), c7(i, 2), i - 1, opp(i) - 1) *
                                    (uint32_t)sizeof(QS));
}

template <int P, bool PACK>
__device__ inline void cvt7(const Raw7<P, PACK>& o, typename Prec<P>::T f[7]) {
  using L = Lat<P, PACK>;
  using T = typename Prec<P>::T;
  f[0] = (T)o.r0;
#pragma unroll
  for (int i = 1; i < 7; ++i) {
    if constexpr (PACK) f[i] = L::lo(o.r[i - 1]);
    else f[i] = (T)o.r[i - 1];
  }
}

// A brick padded by H nodes on every side, and its halo positions.
template <int BX, int BY, int BZ, int H>
struct Pad {
  static constexpr int PX = BX + 2 * H, PY = BY + 2 * H, PZ = BZ + 2 * H;
  static constexpr int PXY = PX * PY, NPHI = PXY * PZ;
  static constexpr int NT = BX * BY * BZ, NHALO = NPHI - NT;
  static constexpr int HPT = (NHALO + NT - 1) / NT;

  // halo position h: H planes below and above the brick, then the frames of
  // the planes between, H rows at each end and H columns at each side
  __device__ static void pos(int h, int& px, int& py, int& pz) {
    constexpr int CAP = H * PXY, FRAME = PXY - BX * BY;
    if (h < 2 * CAP) {
      pz = h / PXY;
      const int r = h % PXY;
      py = r / PX;
      px = r % PX;
      if (pz >= H) pz += BZ;
      return;
    }
    h -= 2 * CAP;
    pz = H + h / FRAME;
    h %= FRAME;
    if (h < 2 * H * PX) {
      py = h / PX;
      px = h % PX;
      if (py >= H) py += BY;
      return;
    }
    h -= 2 * H * PX;
    py = H + h / (2 * H);
    const int c = h % (2 * H);
    px = c < H ? c : BX + c;
  }
};

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
  using D = Pad<BX, BY, BZ, 2>;
  using M1 = Pad<BX, BY, BZ, 1>;
  constexpr int NT = D::NT;
  __shared__ T sphi[D::NPHI];
  __shared__ T smu[M1::NPHI];
  if (C.poison) {
    poison_shared(sphi, sizeof sphi);
    poison_shared(smu, sizeof smu);
    __syncthreads();
  }
  int x0, y0, z0;
  brick_origin<BX, BY, BZ>(G, lb, x0, y0, z0);
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX % BY, tz = tid / (BX * BY);
  const int gx = x0 + tx, gy = y0 + ty, gz = z0 + tz;
  const bool own = gx < G.nx && gy < G.ny && gz < G.nz;
  const uint32_t pitch = (uint32_t)G.pitch;
  const void* fin = cur ? B.f[1] : B.f[0];
  const void* gin = cur ? B.g[1] : B.g[0];
  void* fo = cur ? B.f[0] : B.f[1];
  void* go = cur ? B.g[0] : B.g[1];
  const auto rf = rsrc_at(fin), ri = rsrc_at(L::fi(fin, G.pitch)), rg = rsrc_at(gin), rh = rsrc_at(B.phiu);

  // every load of the step: the node's own f, the f of its halo positions, g
  // and the history.  Every lane loads (a lane without a node or a position
  // takes a valid one and drops the value): a branch would leave the number
  // of loads in flight unknown, and phi would wait for the g as well (32^3
  // FP32 6.6 -> 6.1 us per step, W = 48 box with 16-bit populations 19.2 ->
  // 16.8 us).
  const Node me = make_node<WALL>(G, gx, gy, gz);
  Raw7<P, PACK> fr;
  pull7<P, PACK, WALL>(rf, ri, pitch, me, fr);
  Raw7<P, PACK> hr[D::HPT];
  int hat[D::HPT];
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    const int h = tid + k * NT;
    int px, py, pz;
    D::pos(h < D::NHALO ? h : D::NHALO - 1, px, py, pz);
    const int hx = x0 - 2 + px, hy = y0 - 2 + py, hz = z0 - 2 + pz;
    hat[k] = h < D::NHALO ? px + D::PX * py + D::PXY * pz : -1;
    const Node hn = make_node<WALL>(G, hx, hy, hz);
    pull7<P, PACK, WALL>(rf, ri, pitch, hn, hr[k]);
  }
  S gr[Q];
  T hp[3];
  gr[0] = ld_off<S>(rg, (uint32_t)me.n * (uint32_t)sizeof(S));
#pragma unroll
  for (int i = PACK ? 7 : 1; i < Q; ++i)
    gr[i] = ld_off<S>(rg, pull_at<WALL>(me, pitch, cq<Q>(i, 0), cq<Q>(i, 1), cq<Q>(i, 2), (uint32_t)L::gslot(i),
                                        (uint32_t)L::gslot(opp(i))) * (uint32_t)sizeof(S));
#pragma unroll
  for (int a = 0; a < 3; ++a) hp[a] = ld_off<T>(rh, (a * pitch + (uint32_t)me.n) * (uint32_t)sizeof(T));
  __builtin_amdgcn_sched_barrier(0);

  // phi of the padded brick
  T f[7];
  cvt7<P, PACK>(fr, f);
  const T phi = phi_of(f);
  sphi[(tx + 2) + D::PX * (ty + 2) + D::PXY * (tz + 2)] = phi;
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    if (hat[k] >= 0) {
      T fh[7];
      cvt7<P, PACK>(hr[k], fh);
      sphi[hat[k]] = phi_of(fh);
    }
  }
  __syncthreads();
  // mu of the brick and a halo of one; a ghost position of a wall takes its
  // mirror image
  constexpr int MPT = (M1::NPHI + NT - 1) / NT;
#pragma unroll
  for (int k = 0; k < MPT; ++k) {
    const int q = tid + k * NT;
    const int qz = q / M1::PXY, r = q % M1::PXY, qy = r / M1::PX, qx = r % M1::PX;
    int mx = x0 - 1 + qx, my = y0 - 1 + qy, mz = z0 - 1 + qz;
    if (q < M1::NPHI && mx <= G.nx && my <= G.ny && mz <= G.nz) {
      if (WALL && G.wall_x) mx = clamp_axis(mx, G.nx);
      if (WALL && G.wall_y) my = clamp_axis(my, G.ny);
      if (WALL && G.wall_z) mz = clamp_axis(mz, G.nz);
      const int at = (mx - (x0 - 2)) + D::PX * (my - (y0 - 2));
      const T* pc = sphi + D::PXY * (mz - (z0 - 2));
      const T c0 = pc[at];
      const T lap = lap_lds<T, D::PX>(pc - D::PXY, pc, pc + D::PXY, at);
      smu[q] = 4 * C.beta * c0 * (c0 - 1) * (c0 + 1) - C.kappa * lap;
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
  const int pat = (tx + 2) + D::PX * (ty + 2), mat = (tx + 1) + M1::PX * (ty + 1);
  const T* pc = sphi + D::PXY * (tz + 2);
  const T* mc = smu + M1::PXY * (tz + 1);
  T gphi[3];
  grad_lds<T, D::PX>(pc - D::PXY, pc, pc + D::PXY, pat, gphi);
  const T mu = mc[mat];
  const T lapmu = lap_lds<T, M1::PX>(mc - M1::PXY, mc, mc + M1::PXY, mat);
  Macro<T> M;
  if constexpr (Q == 19) flow_macro19(C, g, phi, mu, gphi, lapmu, M);
  else flow_macro(C, g, phi, mu, gphi, lapmu, M);
  T dphiu[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const T pu = phi * M.u[a];
    dphiu[a] = pu - hp[a];
    st_off<T>(rh, (a * pitch + (uint32_t)me.n) * (uint32_t)sizeof(T), pu);
  }
  collide_che(C, f, phi, mu, M.u, dphiu);
  if constexpr (Q == 19) collide_ns19(C, g, M);
  else collide_ns<false, (V & kVarUnit) != 0>(C, g, M);
  const auto wf = rsrc_at(fo), wi = rsrc_at(L::fi(fo, G.pitch)), wg = rsrc_at(go);
  const uint32_t n = (uint32_t)me.n;
  st_off<S0>(wf, n * (uint32_t)sizeof(S0), (S0)f[0]);
  st_off<S>(wg, n * (uint32_t)sizeof(S), (S)g[0]);
  if constexpr (PACK) {
#pragma unroll
    for (int i = 1; i < 7; ++i) st_off<uint32_t>(wi, ((i - 1) * pitch + n) * 4u, L::pack(f[i], g[i]));
  } else {
#pragma unroll
    for (int i = 1; i < 7; ++i) st_off<S>(wi, ((i - 1) * pitch + n) * (uint32_t)sizeof(S), (S)f[i]);
  }
#pragma unroll
  for (int i = PACK ? 7 : 1; i < Q; ++i)
    st_off<S>(wg, ((uint32_t)L::gslot(i) * pitch + n) * (uint32_t)sizeof(S), (S)g[i]);
  if (!(all_finite(f, 7) && all_finite(g, Q))) *B.flag = 1;
}

template <int P, int Q, bool WALL, int V, int BX, int BY, int BZ>
__global__ void __launch_bounds__(BX* BY* BZ) __attribute__((amdgpu_waves_per_eu(waves_per_eu<P>())))
k_brick(Geo G, Coef<typename Prec<P>::T> C, Bufs B, int cur) {
  brick_body<P, Q, WALL, V, BX, BY, BZ>(G, C, B, cur, logical_block(blockIdx.x, gridDim.x));
}

// The CHE-only step of a brick: mu at the node only, so phi needs a halo of
// one, and the history is phi alone.
template <int P, bool WALL, int BX, int BY, int BZ>
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
  if (C.poison) {
    poison_shared(sphi, sizeof sphi);
    poison_shared(sn, sizeof sn);
    __syncthreads();
  }
  int x0, y0, z0;
  brick_origin<BX, BY, BZ>(G, logical_block(blockIdx.x, gridDim.x), x0, y0, z0);
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX % BY, tz = tid / (BX * BY);
  const int gx = x0 + tx, gy = y0 + ty, gz = z0 + tz;
  const bool own = gx < G.nx && gy < G.ny && gz < G.nz;
  const uint32_t pitch = (uint32_t)G.pitch;
  const void* fin = cur ? B.f[1] : B.f[0];
  void* fo = cur ? B.f[0] : B.f[1];
  const auto rf = rsrc_at(fin), ri = rsrc_at(L::fi(fin, G.pitch)), rh = rsrc_at(B.phiu);
  const Node me = make_node<WALL>(G, gx, gy, gz);
  const uint32_t n = (uint32_t)me.n;
  Raw7<P, false> fr;
  pull7<P, false, WALL>(rf, ri, pitch, me, fr);
  Raw7<P, false> hr[D::HPT];
  int hat[D::HPT];
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    const int h = tid + k * NT;
    hat[k] = -1;
    if (h < D::NHALO) {
      int px, py, pz;
      D::pos(h, px, py, pz);
      const int hx = x0 - 1 + px, hy = y0 - 1 + py, hz = z0 - 1 + pz;
      if (hx <= G.nx && hy <= G.ny && hz <= G.nz) {
        hat[k] = px + D::PX * py + D::PXY * pz;
        const Node hn = make_node<WALL>(G, hx, hy, hz);
        pull7<P, false, WALL>(rf, ri, pitch, hn, hr[k]);
      }
    }
  }
  T phip = 0, u[3] = {0, 0, 0}, up[3] = {0, 0, 0};
  if (own) {
    phip = ld_off<T>(rh, n * (uint32_t)sizeof(T));
    if (C.vel_kind != MPLB_VEL_DEFORM) presc_u(G, C, (const T*)B.ufield, gx, gy, gz, me.n, u, up);
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
  cvt7<P, false>(fr, f);
  const T phi = phi_of(f);
  sphi[(tx + 1) + D::PX * (ty + 1) + D::PXY * (tz + 1)] = phi;
#pragma unroll
  for (int k = 0; k < D::HPT; ++k) {
    if (hat[k] >= 0) {
      T fh[7];
      cvt7<P, false>(hr[k], fh);
      sphi[hat[k]] = phi_of(fh);
    }
  }
  __syncthreads();
  if (!own) return;
  const int at = (tx + 1) + D::PX * (ty + 1);
  const T* pc = sphi + D::PXY * (tz + 1);
  const T lap = lap_lds<T, D::PX>(pc - D::PXY, pc, pc + D::PXY, at);
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
  st_off<T>(rh, n * (uint32_t)sizeof(T), phi);
  T dphiu[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) dphiu[a] = phi * u[a] - phip * up[a];
  collide_che(C, f, phi, mu, u, dphiu);
  const auto wf = rsrc_at(fo), wi = rsrc_at(L::fi(fo, G.pitch));
  st_off<S0>(wf, n * (uint32_t)sizeof(S0), (S0)f[0]);
#pragma unroll
  for (int i = 1; i < 7; ++i) st_off<S>(wi, ((i - 1) * pitch + n) * (uint32_t)sizeof(S), (S)f[i]);
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

template <int P, bool WALL, int BX, int BY, int BZ>
hipError_t brick_impl3(int mode, const Geo& G, const Coef<typename Prec<P>::T>& C, const Bufs& B, int cur, int blocks,
                       hipStream_t s) {
  const dim3 grid((unsigned)blocks), block(BX * BY * BZ);
  if (mode == MPLB_CHE_ONLY)
    hipLaunchKernelGGL((k_brick_che<P, WALL, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
  else if (mode == MPLB_COUPLED_Q19)
    hipLaunchKernelGGL((k_brick<P, 19, WALL, 0, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
  else if (C.unit_rates)
    hipLaunchKernelGGL((k_brick<P, 15, WALL, kVarUnit, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
  else
    hipLaunchKernelGGL((k_brick<P, 15, WALL, 0, BX, BY, BZ>), grid, block, 0, s, G, C, B, cur);
  return hipGetLastError();
}

// Bricks are 4 nodes high and deep: 16 x 4 x 4 (256 threads) or 32 x 4 x 4.
constexpr int brick_width(Bricks br) { return br == kBricksWide ? 32 : 16; }
static_assert(brick_width(kBricksNarrow) * 16 == kBrickThreadsNarrow && brick_width(kBricksWide) * 16 == kBrickThreadsWide,
              "one thread per node");

template <int P, bool WALL>
hipError_t brick_impl2(int mode, const Geo& G, const Coef<typename Prec<P>::T>& C, const Bufs& B, int cur, Bricks br,
                       hipStream_t s) {
  const int blocks = brick_blocks(G, br);
  if (br == kBricksWide) return brick_impl3<P, WALL, brick_width(kBricksWide), 4, 4>(mode, G, C, B, cur, blocks, s);
  return brick_impl3<P, WALL, brick_width(kBricksNarrow), 4, 4>(mode, G, C, B, cur, blocks, s);
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
  return br == kBricksWide ? (const void*)k_brick_many<P, WALL, V, brick_width(kBricksWide), 4, 4>
                           : (const void*)k_brick_many<P, WALL, V, brick_width(kBricksNarrow), 4, 4>;
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

// Wide bricks where they cover at most 1.2 times the nodes that narrow ones
// do: their rows are twice as long for the same halo.  FP32, narrow against
// wide: 64^3 13.5 / 12.1, 72^3 (the 1.2) 20.1 / 19.2, 100^3 48.0 / 45.9; 48^3
// (1.33) 8.6 / 10.2; CHE-only 128^3 34.0 / 29.1.  Below 100 k nodes narrow
// bricks put twice as many CUs to work (32^3 6.1 / 7.0).  The coupled step in
// FP64 keeps narrow ones, whose blocks of four waves fit a CU twice (72^3
// 32.5 / 39.0).
Bricks brick_kind(int P, int mode, long long nodes, long long narrow, long long wide) {
  if (mode != MPLB_CHE_ONLY && P == MPLB_F64) return kBricksNarrow;
  return nodes >= 100000 && 10 * wide <= 12 * narrow ? kBricksWide : kBricksNarrow;
}

}  // namespace

int brick_blocks(const Geo& G, Bricks br) {
  const int bx = brick_width(br);
  return ((G.nx + bx - 1) / bx) * ((G.ny + 3) / 4) * ((G.nz + 3) / 4);
}

Bricks step_bricks(int P, int mode, const Geo& G, const Coef<double>& C) {
  if (C.stencil7 || C.forcing28) return kBricksNone;  // the study variants are marching kernels
  const long long n = (long long)G.nx * G.ny * G.nz;
  const bool che = mode == MPLB_CHE_ONLY;
  if (fused_step_bytes(P, mode, n) > (che && P == MPLB_F64 ? kBrickBytesCheF64 : kBrickBytes)) return kBricksNone;
  if (!che && (P == MPLB_F32_F16 || P == MPLB_F32_BF16) && n > kBrickNodes16) {
    const long long tiles = (long long)((G.nx + 63) / 64 * 64) * ((G.ny + 7) / 8 * 8) * G.nz;
    if (10 * tiles < 11 * n) return kBricksNone;
  }
  return brick_kind(P, mode, n, 256LL * brick_blocks(G, kBricksNarrow), 512LL * brick_blocks(G, kBricksWide));
}

Bricks batch_bricks(int P, size_t bytes, long long nodes, const long long padded[3]) {
  if (bytes > kBrickBytes) return kBricksNone;
  if ((P == MPLB_F32_F16 || P == MPLB_F32_BF16) && nodes > kBrickNodes16) return kBricksNone;
  return brick_kind(P, MPLB_COUPLED, nodes, padded[kBricksNarrow], padded[kBricksWide]);
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
