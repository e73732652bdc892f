// Two CHE-only time steps in one kernel (part of kernels.hip's translation
// unit), for periodic lattices too large for the last-level cache.
//
// The step moves 16 words per node and does little arithmetic on them, so a
// large lattice is bound by HBM.  Here the populations between the two steps
// never leave the block: it marches along z with a 64 x TY tile, does the
// first step on the tile and a frame of two nodes around it (phi of the first
// level on a frame of three), and the second on the tile.
//
// At iteration k, between two barriers, a block
//   A  sums the pulled f of plane k into phi of level n (ring s1) and issues
//      the pulls of plane k+1;
//   D  finishes the second step of plane k-4: phi of level n+1 (ring s2) gives
//      mu, the f pulled in C collide and are stored;
//   B  collides the first step of plane k-1 on tile and frame; f*_1..f*_4 go
//      to LDS (sf), f*_0, f*_5 and f*_6 stay with their thread, since their
//      sources lie in the thread's own column;
//   C  pulls the second step's f of plane k-2 from there, on the tile and a
//      frame of one, and sums its phi.
// A thread owns a tile node and at most one frame node.  f* is rounded to the
// storage type between the steps, so the fields are those of two single steps,
// bit for bit.  The phi history is read by neighbouring blocks' frames, so the
// kernel reads one buffer and writes another, which the host swaps.
//
// 64 x 16 with 1024 threads and 158 KB of LDS is the largest tile a CU holds
// (1.5 pulls and 1.33 collisions of the first step per node).  What bounds
// it is the chain of a plane, some 4.1 us per iteration at any size and
// storage type: the vector work of 16 waves between two barriers, with the next
// plane's pulls in flight; HBM moves 3.9 TB/s.  256^3 FP32: 144 us per step, 221
// in single steps (5.0 TB/s); FP16 134 against 163.  One kernel per kind of
// velocity: with the kinds told apart inside the loop the registers spilled and
// 256^3 took 153 us.  Two iterations per round of the loop, which saves the
// copies of the queued planes, spill too: 164 us.
#pragma once

#include "common.h"
#include "device.h"
#include "launch.h"

namespace mplb {
namespace {

using namespace dev;

constexpr int kPairCUs = 256, kPairMinLz = 16, kPairRows = 16;
// more nodes than a plane has (and its bytes fit 32 bits)
constexpr uint32_t kPairPlane = 0x30000000;

// v as it would be read back after a store in type S.  The conversion stays
// here, next to the collision's last multiply-add, which the compiler joins with
// it into one rounding at the stores of a single step.
template <class S, class T>
__device__ inline T rounded(T v) {
  T r = (T)(S)v;
  if constexpr (sizeof(S) < sizeof(T)) asm volatile("" : "+v"(r));
  return r;
}

// Store into a plane of `bytes` bytes; an offset beyond them drops the store.
template <bool NT, class S>
__device__ inline void st_plane(S* base, uint32_t bytes, uint32_t off, S v) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)bytes, 0x00020000);
  constexpr int aux = NT ? 2 : 0;
  if constexpr (sizeof(S) == 2)
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, off, 0, aux);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, aux);
}

template <int P, bool NT, int TY, int VK>
__global__ void __launch_bounds__(64 * TY) __attribute__((amdgpu_waves_per_eu(waves_per_eu<P>())))
k_che_pair(Geo G, Coef<typename Prec<P>::T> C, typename Prec<P>::T ct_next, Bufs B, int cur, Tiling TL) {
  using T = typename Prec<P>::T;
  using L = Lat<P, false>;
  using S = typename L::S;
  using S0 = typename L::S0;
  constexpr int TW = 64, NTH = TW * TY;
  // the tile padded by 1, 2 and 3 nodes, and its frames
  constexpr int X1 = TW + 2, X2 = TW + 4, X3 = TW + 6;
  constexpr int N1 = X1 * (TY + 2), N2 = X2 * (TY + 4), N3 = X3 * (TY + 6);
  constexpr int E1 = N1 - NTH, E2 = N2 - NTH, E3 = N3 - NTH;
  static_assert(E3 <= NTH, "one frame node per thread");
  __shared__ T s1[6][N3];    // phi, level n, planes k-4 .. k (k+1 is written one barrier later)
  __shared__ T sf[2][4][N2];  // f*_1..f*_4 of the first step, planes k-2, k-1
  __shared__ T s2[4][N1];    // phi, level n+1, planes k-5 .. k-2
  __shared__ T sq[2][7][NTH];  // the second step's f of planes k-4 .. k-2 (thread-private)
  // sin(pi z/nz) and sin(2 pi z/nz) of this run of 64 planes and the last
  __shared__ T sz[2][64][2];
  if (C.poison) {
    poison_shared(s1, sizeof s1);
    poison_shared(sf, sizeof sf);
    poison_shared(s2, sizeof s2);
    poison_shared(sq, sizeof sq);
    poison_shared(sz, sizeof sz);
    __syncthreads();
  }
  const int lb = logical_block(blockIdx.x, gridDim.x);
  const int tile = lb % (TL.tiles_x * TL.tiles_y), seg = lb / (TL.tiles_x * TL.tiles_y);
  const int x0 = (tile % TL.tiles_x) * TW, y0 = (tile / TL.tiles_x) * TY;
  const int z0 = seg * TL.lz, z1 = min(G.nz, z0 + TL.lz);
  const int tid = threadIdx.x, tx = tid % TW, ty = tid / TW;
  const bool own = x0 + tx < G.nx && y0 + ty < G.ny;
  const void* fin = cur ? B.f[1] : B.f[0];
  void* fo = cur ? B.f[0] : B.f[1];
  const T* hin = (const T*)B.phiu;
  T* hout = (T*)B.phi;

  // node 0: the tile node, node 1: the frame node (frames of 1, 2, 3 in turn)
  int ex = 0, ey = 0;
  if (tid < E3) {
    const int r = tid < E1 ? 1 : (tid < E2 ? 2 : 3), w = TW + 2 * r;
    int i = tid - (r == 1 ? 0 : (r == 2 ? E1 : E2));
    if (i < 2 * w) {
      ex = i % w - r;
      ey = i < w ? -r : TY - 1 + r;
    } else {
      i -= 2 * w;
      ex = (i & 1) ? TW - 1 + r : -r;
      ey = i / 2 - r + 1;
    }
  }
  const int lx[2] = {tx, ex}, ly[2] = {ty, ey};
  int xy[2], xm[2], xp[2], ym[2], yp[2];  // in-plane offsets of the node and its neighbours
  int at1[2], at2[2], atf[2];
  // The frame node has phi of level n; takes the first step; has phi of level
  // n+1.  The tile node has all, also beyond the lattice, where it steps the
  // node that its position wraps to and stores nothing: every load and store of
  // the tile is issued by every lane, so that the number in flight is known and
  // the wait for the pulls is none for the stores behind them.
  bool on1 = false, first1 = false;
  PrescColumn<T> pc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int gx = x0 + lx[j], gy = y0 + ly[j];
    if (j == 1) {
      const bool need = gx <= G.nx + 2 && gy <= G.ny + 2;
      on1 = need && tid < E3;
      first1 = need && tid < E2;
    }
    const int mx = map_axis(gx, G.nx, 0), my = map_axis(gy, G.ny, 0);
    xy[j] = mx + G.nx * my;
    xm[j] = wrap1(mx - 1, G.nx) + G.nx * my;
    xp[j] = wrap1(mx + 1, G.nx) + G.nx * my;
    ym[j] = mx + G.nx * wrap1(my - 1, G.ny);
    yp[j] = mx + G.nx * wrap1(my + 1, G.ny);
    at1[j] = (lx[j] + 3) + X3 * (ly[j] + 3);
    atf[j] = (lx[j] + 2) + X2 * (ly[j] + 2);
    at2[j] = (lx[j] + 1) + X1 * (ly[j] + 1);
    if (VK == MPLB_VEL_DEFORM) pc[j].init(G, C, mx, my);
    if (VK == MPLB_VEL_ZALESAK) pc[j].a[0] = (T)my - (T)G.nx / 2;  // y - L/2
  }
  // prescribed velocity of node j in plane z (the i-th of the march) with time
  // factor ct
  auto velocity = [&](int j, int i, int z, T ct, T u[3]) {
    u[0] = u[1] = u[2] = 0;
    if constexpr (VK == MPLB_VEL_DEFORM) {
      const T* sn = sz[i / 64 % 2][i % 64];
      const T s = sn[0], s2z = sn[1];
      const T b[3] = {pc[j].a[0] * s2z, pc[j].a[1] * s2z, pc[j].a[2] * s * s};
#pragma unroll
      for (int a = 0; a < 3; ++a) u[a] = b[a] * ct;
    } else if constexpr (VK == MPLB_VEL_ZALESAK) {
      const T pi = (T)3.14159265358979323846, len = (T)G.nx;
      u[1] = (C.velU * pi / len) * (len / 2 - (T)z);
      u[2] = (C.velU * pi / len) * pc[j].a[0];
    }
  };

  F7Raw<P, false> raw[2];    // pulls in flight, plane k+1
  T fp[2][7] = {};           // f of plane k-1
  T c0[2] = {0, 0}, c5[2] = {0, 0}, c5p[2] = {0, 0};  // f*_0 of k-2, f*_5 of k-2 and k-3
  bool finite = true;        // f of both steps of the tile node's column
  const int nxy = G.nx * G.ny;
  const uint32_t out = own ? (uint32_t)xy[0] : kPairPlane;  // dropped by st_plane
  // the lattice's planes of k-2 .. k+2, wrapped
  int zk[5];
  for (int i = 0; i < 5; ++i) zk[i] = map_axis(z0 - 5 + i, G.nz, 0);
  // pulls of the plane in zk[i] (its neighbours in zk[i - 1] and zk[i + 1])
  auto issue = [&](int below, int z, int above) {
    const S0* f0 = L::f0(fin) + (size_t)z * nxy;
    const S* fi = L::fi(fin, G.pitch);
    const S* fz = fi + (size_t)z * nxy;
    const S* f5 = fi + ((size_t)4 * G.pitch + (size_t)below * nxy);
    const S* f6 = fi + ((size_t)5 * G.pitch + (size_t)above * nxy);
#pragma unroll
    for (int j = 1; j >= 0; --j) {
      if (j == 0 || on1) {
        raw[j].r0 = ld_at(f0, xy[j]);
        raw[j].r[0] = ld_at(fz, xm[j]);
        raw[j].r[1] = ld_at(fz + (size_t)G.pitch, xp[j]);
        raw[j].r[2] = ld_at(fz + (size_t)2 * G.pitch, ym[j]);
        raw[j].r[3] = ld_at(fz + (size_t)3 * G.pitch, yp[j]);
        raw[j].r[4] = ld_at(f5, xy[j]);
        raw[j].r[5] = ld_at(f6, xy[j]);
      }
    }
  };
  // Iteration k.  The stages that a segment's first and last iterations lack
  // are left out at compile time, so that the steady loop has no branch around
  // its loads.
  auto iterate = [&](int k, auto fA, auto fN, auto fB, auto fC, auto fD) {
    constexpr bool A = decltype(fA)::value, NEXT = decltype(fN)::value, DB = decltype(fB)::value,
                   DC = decltype(fC)::value, DD = decltype(fD)::value;
    const int t = k - z0 + 12;  // ring positions count from here (k >= z0 - 3)
    T fk[2][7];
    if constexpr (A) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 0 || on1) {
          cvt_f7<P, false>(raw[j], fk[j]);
          s1[t % 6][at1[j]] = phi_of(fk[j]);
        }
      }
      const int run = t - 9;
      if (VK == MPLB_VEL_DEFORM && __builtin_expect(run % 64 == 0 && tid < 128, 0)) {
        const T pi = (T)3.14159265358979323846;
        const T zh = (T)map_axis(k + tid / 2, G.nz, 0) / (T)G.nz;
        sz[run / 64 % 2][tid / 2][tid % 2] = tid % 2 ? sin(2 * pi * zh) : sin(pi * zh);
      }
    }
    // phi of level n-1 of plane k-1, which B needs
    T hp[2] = {0, 0};
    if constexpr (DB) {
      const T* h = hin + (size_t)zk[1] * nxy;
#pragma unroll
      for (int j = 1; j >= 0; --j)
        if (j == 0 || first1) hp[j] = ld_at<T>(h, xy[j]);
    }
    if constexpr (NEXT) issue(zk[2], zk[3], zk[4]);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if constexpr (DD) {
      const int z = k - 4;
      const size_t zo = (size_t)z * nxy;
      T fb[7];
#pragma unroll
      for (int i = 0; i < 7; ++i) fb[i] = sq[t % 2][i][tid];
      const T* pm = s2[(t - 5) % 4];
      const T* pm1 = s2[(t - 4) % 4];
      const T* pp = s2[(t - 3) % 4];
      const T phi = phi_of(fb);
      const T lap = lap_lds<T, X1>(pm, pm1, pp, at2[0]);
      const T mu = 4 * C.beta * phi * (phi - 1) * (phi + 1) - C.kappa * lap;
      const T phip = s1[(t - 4) % 6][at1[0]];
      T u[3], up[3], dphiu[3];
      velocity(0, t - 13, z, ct_next, u);
      velocity(0, t - 13, z, C.vel_ct, up);
      st_plane<NT>(hout + zo, nxy * (uint32_t)sizeof(T), out * (uint32_t)sizeof(T), phi);
#pragma unroll
      for (int a = 0; a < 3; ++a) dphiu[a] = __builtin_fmaf(phi, u[a], -(phip * up[a]));
      collide_che(C, fb, phi, mu, u, dphiu);
      st_plane<NT>(L::f0(fo) + zo, nxy * (uint32_t)sizeof(S0), out * (uint32_t)sizeof(S0), (S0)fb[0]);
      S* fs = L::fi(fo, G.pitch);
#pragma unroll
      for (int i = 1; i < 7; ++i)
        st_plane<NT>(fs + ((size_t)(i - 1) * G.pitch + zo), nxy * (uint32_t)sizeof(S), out * (uint32_t)sizeof(S), (S)fb[i]);
      finite = finite && all_finite(fb, 7);
    }
    T c6[2] = {0, 0}, d0[2] = {0, 0}, d5[2] = {0, 0};  // f* of plane k-1
    if constexpr (DB) {
      const int z = zk[1];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 0 || first1) {
          T f[7];
#pragma unroll
          for (int i = 0; i < 7; ++i) f[i] = fp[j][i];
          const T phi = phi_of(f);
          const T lap = lap_lds<T, X3>(s1[(t - 2) % 6], s1[(t - 1) % 6], s1[t % 6], at1[j]);
          const T mu = 4 * C.beta * phi * (phi - 1) * (phi + 1) - C.kappa * lap;
          T u[3], up[3], dphiu[3];
          velocity(j, t - 10, z, C.vel_ct, u);
          velocity(j, t - 10, z, C.vel_ct_prev, up);
#pragma unroll
          for (int a = 0; a < 3; ++a) dphiu[a] = __builtin_fmaf(phi, u[a], -(hp[j] * up[a]));
          collide_che(C, f, phi, mu, u, dphiu);
          d0[j] = rounded<S0>(f[0]);
#pragma unroll
          for (int i = 1; i < 5; ++i) sf[(t - 1) % 2][i - 1][atf[j]] = rounded<S>(f[i]);
          d5[j] = rounded<S>(f[5]);
          c6[j] = rounded<S>(f[6]);
          if (j == 0) finite = finite && all_finite(f, 7);
        }
      }
    }
    if constexpr (DC) {
      const T(*q)[N2] = sf[t % 2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 0 || tid < E1) {
          T f[7] = {c0[j], q[0][atf[j] - 1], q[1][atf[j] + 1], q[2][atf[j] - X2], q[3][atf[j] + X2], c5p[j], c6[j]};
          s2[(t - 2) % 4][at2[j]] = phi_of(f);
          if (j == 0) {
#pragma unroll
            for (int i = 0; i < 7; ++i) sq[t % 2][i][tid] = f[i];
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      c0[j] = d0[j];
      c5p[j] = c5[j];
      c5[j] = d5[j];
      if constexpr (A) {
#pragma unroll
        for (int i = 0; i < 7; ++i) fp[j][i] = fk[j][i];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) zk[i] = zk[i + 1];
    zk[4] = zk[4] + 1 == G.nz ? 0 : zk[4] + 1;
  };
  constexpr std::true_type Y{};
  constexpr std::false_type O{};
  issue(zk[1], zk[2], zk[3]);  // plane z0 - 3
  for (int k = z0 - 3; k < z0 - 1; ++k) iterate(k, Y, Y, O, O, O);
  for (int k = z0 - 1; k < z0 + 1; ++k) iterate(k, Y, Y, Y, O, O);
  for (int k = z0 + 1; k < z0 + 4; ++k) iterate(k, Y, Y, Y, Y, O);
  for (int k = z0 + 4; k < z1 + 2; ++k) iterate(k, Y, Y, Y, Y, Y);
  iterate(z1 + 2, Y, O, Y, Y, Y);
  iterate(z1 + 3, O, O, O, O, Y);
  if (own && !finite) *B.flag = 1;
}

// Work split of the pair.  A CU holds one block at a time and spends about the
// same on every plane of it, and a segment runs six planes or so more than it
// stores, so the split that costs least has the smallest rounds * (lz + 6).  A
// segment has at least two planes: the kernel's schedule needs them.
struct PairPlan {
  Tiling t;
  long long nodes;  // that the chip could step in its time
};
PairPlan pair_plan(const Geo& G, int TY) {
  PairPlan p{};
  Tiling& t = p.t;
  t.tiles_x = (G.nx + 63) / 64;
  t.tiles_y = (G.ny + TY - 1) / TY;
  const long long cols = (long long)t.tiles_x * t.tiles_y;
  long long best = 0;
  for (int want = 1; want == 1 || (G.nz + want - 1) / want >= kPairMinLz; ++want) {
    const int lz = (G.nz + want - 1) / want, nseg = (G.nz + lz - 1) / lz;
    // shorter segments cost at least (lz + 6) / lz of their planes' even share
    if (best && (double)cols * G.nz * (lz + 6) >= (double)best * lz * kPairCUs) break;
    if (G.nz - (nseg - 1) * lz < 2) continue;
    const long long cost = (cols * nseg + kPairCUs - 1) / kPairCUs * (lz + 6);
    if (best && cost >= best) continue;
    best = cost;
    t.lz = lz;
    t.nseg = nseg;
  }
  p.nodes = best * kPairCUs * 64 * TY;
  return p;
}

template <int P, bool NT>
hipError_t pair_impl2(const Geo& G, const Coef<double>& Cd, double ct_next, const Bufs& B, int cur, hipStream_t s) {
  using T = typename Prec<P>::T;
  constexpr int TY = kPairRows;
  const Tiling t = pair_plan(G, TY).t;
  void (*k)(Geo, Coef<T>, T, Bufs, int, Tiling) = k_che_pair<P, NT, TY, MPLB_VEL_ZERO>;
  if (Cd.vel_kind == MPLB_VEL_ZALESAK) k = k_che_pair<P, NT, TY, MPLB_VEL_ZALESAK>;
  if (Cd.vel_kind == MPLB_VEL_DEFORM) k = k_che_pair<P, NT, TY, MPLB_VEL_DEFORM>;
  hipLaunchKernelGGL(k, dim3((unsigned)(t.tiles_x * t.tiles_y * t.nseg)), dim3(64 * TY), 0, s, G, cast_coef<T>(Cd),
                     (T)ct_next, B, cur, t);
  return hipGetLastError();
}

template <int P>
hipError_t pair_impl(const Geo& G, const Coef<double>& C, double ct_next, const Bufs& B, int cur, hipStream_t s) {
  if (streaming_stores(P, MPLB_CHE_ONLY, fused_step_bytes(P, MPLB_CHE_ONLY, G.N)))
    return pair_impl2<P, true>(G, C, ct_next, B, cur, s);
  return pair_impl2<P, false>(G, C, ct_next, B, cur, s);
}

}  // namespace

// Periodic lattices beyond the bricks, with a velocity that is known at any
// time (a caller may change the nodes' own between steps).  In FP64 the rings
// leave LDS for 8 rows only, whose frames cost what the second step saves.
// Pairs lose where their tiles, segments and rounds leave much idle, so the
// nodes that they could step are weighed against those that the march's 64 x 8
// tiles cover.  us per step, single against pairs, by that ratio: FP32 0.91
// (256^3) 221 / 144, 0.79 (192^3) 116 / 71, 0.70 (200^3) 135 / 120, 0.57
// (1024 x 1024 x 8) 122 / 103, 0.49 (1000 x 1000 x 6) 98 / 94; 16-bit
// populations, whose single step moves 40 bytes per node instead of 64, 0.91
// 163 / 134, 0.79 (224^3) 130 / 110, 0.74 (400 x 400 x 100) 244 / 174, just
// below 0.70 (200^3) 104 / 104, 0.57 96 / 96.
bool che_pair_fits(int P, int mode, const Geo& G, const Coef<double>& C) {
  if (mode != MPLB_CHE_ONLY || G.wall_x || G.wall_y || G.wall_z || C.stencil7 || C.vel_kind == MPLB_VEL_FIELD) return false;
  if (P == MPLB_F64 || G.nz < 2 || (uint64_t)G.nx * G.ny > kPairPlane || step_bricks(P, mode, G, C) != kBricksNone) return false;
  return 100 * march_nodes(G) >= (P == MPLB_F32 ? 50 : 70) * pair_plan(G, kPairRows).nodes;
}

Shape che_pair_shape(const Geo& G) { return Shape{kShapePair, 64, kPairRows, pair_plan(G, kPairRows).t}; }

hipError_t launch_che_pair(int P, const Geo& G, const Coef<double>& C, double ct_next, const Bufs& B, int cur,
                           hipStream_t s) {
  switch (P) {
    case MPLB_F32: return pair_impl<MPLB_F32>(G, C, ct_next, B, cur, s);
    case MPLB_F32_F16: return pair_impl<MPLB_F32_F16>(G, C, ct_next, B, cur, s);
    case MPLB_F32_BF16: return pair_impl<MPLB_F32_BF16>(G, C, ct_next, B, cur, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mplb
