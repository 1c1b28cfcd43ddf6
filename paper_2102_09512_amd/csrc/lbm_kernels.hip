// HIP kernels of liblbm.so (gfx950).
//
// Fused stream-and-collide (one launch per time step)
// ---------------------------------------------------
// Populations are stored plane-major: for every plane of the march axis (z
// for D3Q27, y for D2Q9) the Q velocity slots of that plane follow each
// other, each an in-plane array (x fastest) of (f_i, g_i) pairs:
//   buf[m * ms + i * 2 ps + 2 p + s],  p = in-plane node index,
//   s = 0 for f_i, 1 for g_i.
// f_i and g_i of a node stream from the same neighbour, so one 8-byte (FP32)
// or 16-byte (FP64) access moves both: half the memory instructions of
// separate arrays, and a wavefront touches a contiguous 512-byte (FP32) or
// 1-KB (FP64) run per slot.  A work-group that marches over a few planes
// touches a few MB of address space instead of 2Q arrays a whole field
// apart, which keeps the address translation caches warm.
// Streaming is done by pull: the thread of node x reads slot i from x - c_i
// (wrapped or clamped per axis) and writes the post-collision values at x.
//
// The anomaly correction needs, at node x, the post-streaming anomaly Qt_a of
// the neighbours x +- e_a of the same step.  A work-group owns a BX x BY tile
// of an in-plane slab and marches along the last axis (z for D3Q27, y for
// D2Q9) over a chunk of planes:
//   - each thread keeps its own node's post-streaming populations in
//     registers from the plane where they are loaded to the plane where they
//     are collided; the neighbours along the march axis are the same
//     thread's previous and next planes, held in registers.  The FP32 kernel
//     is software-pipelined two planes deep: while plane m collides, the
//     loads of plane m + 2 are in flight and plane m + 1 (loaded one
//     iteration earlier) supplies the anomaly along the march axis;
//   - neighbours inside the plane are exchanged through LDS; a one-node ring
//     around the tile (the halo) is computed by the first threads of the
//     group, which pull the halo nodes' populations and form their moments
//     (these re-reads mostly hit L2: the halo is the neighbouring tile's core);
//   - one barrier per plane.
// Work-groups are mapped XCD-aware: consecutive hardware block ids go to
// different XCDs, so the logical tile order is rebuilt such that every XCD
// processes one contiguous range of tiles (neighbouring tiles share an L2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "lbm_internal.h"
#include "lbm_node.h"

// Debug build switch (liblbm_poison.so): fill the step kernel's LDS anomaly
// ring with NaN at the start and before every plane refills its half, so
// that a value read without having been written for the current plane shows
// up as NaN in the results instead of a stale neighbour value.
#ifndef LBM_POISON_LDS
#define LBM_POISON_LDS 0
#endif

namespace lbm {

__device__ inline int fix_coord(int k, int n, int bc) {
  if (bc == LBM_BC_PERIODIC) {
    k %= n;
    return k < 0 ? k + n : k;
  }
  return k < 0 ? 0 : (k > n - 1 ? n - 1 : k);
}

// fix_coord for -n <= k < 3n without a division (march-plane indices).
__device__ inline int fix_near(int k, int n, int bc) {
  if (bc == LBM_BC_PERIODIC) {
    k = k < 0 ? k + n : k;
    k = k >= n ? k - n : k;
    return k >= n ? k - n : k;
  }
  return k < 0 ? 0 : (k > n - 1 ? n - 1 : k);
}

// Element offset of population i (f_i for i < Q, g_{i-Q} for i >= Q) of
// node n (node = x + nx*(y + ny*z)).
__device__ inline long long pop_offset(const StepParams& p, int Q, int i, long long n) {
  const long long m = n / p.plane;
  const long long q = n - m * p.plane;
  const int slot = i < Q ? i : i - Q;
  return m * p.ms + (q >> 6) * p.blk + (long long)slot * p.sl + 2 * (q & 63) + (i < Q ? 0 : 1);
}

// Element offset of the (f, g) pair of slot 0 of node n; slot i's pair is
// i * p.sl further on.
__device__ inline long long pair_offset(const StepParams& p, int n) {
  const int m = n / p.plane, q = n - m * p.plane;
  return m * p.ms + (q >> 6) * p.blk + 2 * (q & 63);
}

// Byte offset of the (f, g) pair of slot 0 of in-plane node q within its
// march plane.
template <typename S>
__device__ inline unsigned inplane_bytes(const StepParams& p, int q) {
  return (unsigned)(((unsigned long long)(q >> 6) * (unsigned long long)p.blk + 2u * (unsigned)(q & 63)) * sizeof(S));
}

template <typename S>
struct StoreOf;
template <>
struct StoreOf<float> {
  using R = float;
};
template <>
struct StoreOf<double> {
  using R = double;
};

__device__ inline NodeConsts node_consts(const StepParams& p) {
  NodeConsts k;
  k.rho0 = p.rho0;
  k.T0 = p.T0;
  k.inv_Cv = p.inv_Cv;
  k.Cv = p.Cv;
  k.cv1 = p.cv1;
  k.cv2 = p.cv2;
  k.U0 = p.U0;
  k.caloric = p.caloric;
  k.Pr = p.Pr;
  k.mu0 = p.mu0;
  k.visc_exp = p.visc_exp;
  k.inv_Tref = p.inv_Tref;
  for (int a = 0; a < 3; ++a) {
    k.u0[a] = p.u0[a];
    k.P0[a] = p.P0[a];
    k.u0f[a] = p.u0f[a];
    k.P0f[a] = p.P0f[a];
    for (int c = 0; c < 3; ++c) {
      k.psi0[a][c] = p.psi0[a][c];
      k.b0[a][c] = p.b0[a][c];
      k.psi0f[a][c] = p.psi0f[a][c];
      k.b0f[a][c] = p.b0f[a][c];
    }
  }
  return k;
}

// Raw buffer access: a wave-uniform resource (base of one march plane), a
// per-lane 32-bit byte offset (the in-plane node) and a wave-uniform scalar
// offset (the population), so a load or store needs no per-lane address
// arithmetic.  Offsets past the resource's size read 0 and drop writes.
constexpr int kBufferFlags = 0x00020000;  // raw 32-bit data format (gfx9 family)
// Cache policy of the step kernel's stores: default.  (Non-temporal stores
// measured 5% slower in this kernel on gfx950.)
constexpr int kStorePolicy = 0;

__device__ inline __amdgpu_buffer_rsrc_t plane_rsrc(const void* base, long long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, kBufferFlags);
}

// One (f_i, g_i) pair per access.
template <typename S>
struct Buf;
template <>
struct Buf<float> {
  typedef float pair_t __attribute__((ext_vector_type(2)));
  static __device__ inline pair_t load(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
    return __builtin_bit_cast(pair_t, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
  }
  static __device__ inline void store(pair_t v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, vo, so, kStorePolicy);
  }
};
template <>
struct Buf<double> {
  typedef double pair_t __attribute__((ext_vector_type(2)));
  static __device__ inline pair_t load(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
    return __builtin_bit_cast(pair_t, __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0));
  }
  static __device__ inline void store(pair_t v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(V, v), r, vo, so, kStorePolicy);
  }
};

// Pull-load the 2Q populations arriving at a node.  rs[k] is the resource of
// march plane (m + k - 1) after wrap/clamp; lo[j] is the byte offset inside a
// plane of the in-plane source (y + j/3 - 1, x + j%3 - 1).  Slot i of the
// source x - c_i sits at scalar offset i * slot_bytes of plane 1 - c_m.
template <int D, typename S, typename R>
__device__ inline void pull(const __amdgpu_buffer_rsrc_t* rs, unsigned slot_bytes, const unsigned* lo, R* f, R* g) {
  constexpr int Q = lat_q(D);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int cx = vx(i);
    const int cy = (D == 3) ? vy(i) : 0;
    const int cm = (D == 3) ? vz(i) : vy(i);
    const unsigned o = lo[(1 - cy) * 3 + (1 - cx)];
    const auto v = Buf<S>::load(rs[1 - cm], o, (unsigned)i * slot_bytes);
    f[i] = (R)v.x;
    g[i] = (R)v.y;
  }
}

// Density, velocity and temperature of a node from its pulled populations,
// loaded and summed in batches of nine velocities so that few registers hold
// loaded values at a time (used for the halo node where registers are short).
template <int D, typename S, typename R>
__device__ inline NodeMoments<R> pulled_moments_batched(const __amdgpu_buffer_rsrc_t* rs, unsigned slot_bytes,
                                                        const unsigned* lo, const NodeConsts& k) {
  constexpr int Q = lat_q(D);
  double s0 = 0, j[3] = {0, 0, 0}, se = 0;
#pragma unroll
  for (int b = 0; b < Q; b += 9) {
    R f[9], g[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const int i = b + q;
      const int cx = vx(i);
      const int cy = (D == 3) ? vy(i) : 0;
      const int cm = (D == 3) ? vz(i) : vy(i);
      const auto v = Buf<S>::load(rs[1 - cm], lo[(1 - cy) * 3 + (1 - cx)], (unsigned)i * slot_bytes);
      f[q] = (R)v.x;
      g[q] = (R)v.y;
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const int i = b + q;
      const int cx = vx(i), cy = vy(i), cz = (D == 3) ? vz(i) : 0;
      s0 += f[q];
      se += g[q];
      if (cx) j[0] += cx > 0 ? f[q] : -f[q];
      if (cy) j[1] += cy > 0 ? f[q] : -f[q];
      if (cz) j[2] += cz > 0 ? f[q] : -f[q];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  NodeMoments<R> m;
  velocity_temperature<D, R>(m, s0, j, se, k);
  return m;
}

// Stand-ins for the node arithmetic in the access-pattern reference kernel
// (PAT): each keeps the values it is given live at the cost of about one
// addition per value, so that the kernel loads and stores exactly what a
// step does and computes nothing else.
template <int D, typename R>
__device__ inline NodeMoments<R> pattern_moments(const R* f, const R* g) {
  NodeMoments<R> m{};
#pragma unroll
  for (int a = 0; a < 3; ++a) m.u[a] = f[a] + g[a];
  return m;
}

// All 2Q values (the halo node and the plane before a chunk, where a step
// forms the conserved sums).
template <int D, typename R>
__device__ inline NodeMoments<R> pattern_all(const R* f, const R* g) {
  constexpr int Q = lat_q(D);
  R acc = 0;
#pragma unroll
  for (int i = 0; i < Q; ++i) acc += f[i] + g[i];
  NodeMoments<R> m{};
  m.u[0] = m.u[1] = m.u[2] = acc;
  return m;
}

template <int D, typename S, typename R>
__device__ inline NodeMoments<R> pattern_pulled(const __amdgpu_buffer_rsrc_t* rs, unsigned slot_bytes,
                                                const unsigned* lo) {
  constexpr int Q = lat_q(D);
  R acc = 0;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int cx = vx(i);
    const int cy = (D == 3) ? vy(i) : 0;
    const int cm = (D == 3) ? vz(i) : vy(i);
    const auto v = Buf<S>::load(rs[1 - cm], lo[(1 - cy) * 3 + (1 - cx)], (unsigned)i * slot_bytes);
    acc += (R)v.x + (R)v.y;
  }
  NodeMoments<R> m{};
  m.u[0] = m.u[1] = m.u[2] = acc;
  return m;
}

// One work-group's share of a step: tile lb (x fastest, then y, then the
// march chunk) of the box described by p.  CAL: the general caloric law
// (p.caloric must equal CAL); with CAL false the constant-C_v arithmetic is
// all the kernel contains.
// PAT: the access-pattern reference (same loads, stores, LDS exchange and
// barriers, no collision: the streamed populations are stored).
template <int D, bool DEV, typename S, int BX, int BY, bool CAL = false, bool PAT = false>
__device__ __forceinline__ void step_tile(const S* __restrict__ src, S* __restrict__ dst, const StepParams& p, int lb) {
  using R = typename StoreOf<S>::R;
  constexpr int Q = lat_q(D);
  constexpr int NHALO = (D == 3) ? 2 * BX + 2 * BY : 2;
  static_assert(BX * BY >= NHALO, "tile too small for its halo");
  static_assert(D == 3 || BY == 1, "D2Q9 tiles are one row");
  __shared__ R lq0[2][BY][BX + 2];                    // anomaly along in-plane axis 0 (x)
  __shared__ R lq1[2][(D == 3) ? BY + 2 : 1][BX];     // anomaly along in-plane axis 1 (y, D3Q27 only)
  // half b of the ring set to NaN by the whole work-group (debug build only;
  // the caller separates it from the next reads or writes by a barrier)
  auto poison = [&](int b) {
    constexpr int N0 = BY * (BX + 2), N1 = ((D == 3) ? BY + 2 : 1) * BX;
    const R nan = (R)__builtin_nan("");
    for (int e = threadIdx.x; e < N0; e += BX * BY) (&lq0[b][0][0])[e] = nan;
    for (int e = threadIdx.x; e < N1; e += BX * BY) (&lq1[b][0][0])[e] = nan;
  };
  if constexpr (LBM_POISON_LDS) {
    poison(0);
    poison(1);
    __syncthreads();
  }

  NodeConsts k = node_consts(p);
  k.caloric = CAL ? 1 : 0;
  if constexpr (!CAL) k.U0 = k.Cv * k.T0;  // the same value, formed from constants already held

  const int tx = lb % p.tiles_x;
  const int rest = lb / p.tiles_x;
  const int ty = (D == 3) ? rest % p.tiles_y : 0;
  const int ck = (D == 3) ? rest / p.tiles_y : rest;

  const int n0 = p.nx;
  const int n1 = (D == 3) ? p.ny : 1;
  const int nm = (D == 3) ? p.nz : p.ny;
  const int bc0 = p.bc[0], bc1 = p.bc[1], bcm = (D == 3) ? p.bc[2] : p.bc[1];
  const long long sm = p.ms;  // march-plane stride

  const int t = threadIdx.x;
  const int lx = t % BX, ly = t / BX;
  const int x0 = tx * BX, y0 = ty * BY;
  const int m0 = ck * p.chunk_len;
  const int m1 = min(m0 + p.chunk_len, nm);

  // core node of this thread (positions beyond the domain map by wrap/clamp)
  const int gx = x0 + lx, gy = y0 + ly;
  const bool active = gx < n0 && gy < n1;
  // A position outside the domain stands for the node it maps to, so the
  // neighbour offsets are taken around that node (this matters for clamping).
  int cox[3], coy[3];
  const int gxn = fix_coord(gx, n0, bc0), gyn = fix_coord(gy, n1, bc1);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    cox[j] = fix_coord(gxn + j - 1, n0, bc0);
    coy[j] = (D == 3) ? fix_coord(gyn + j - 1, n1, bc1) * p.nx : 0;
  }
  const int cnode = cox[1] + coy[1];

  // halo node of this thread, if any
  const bool has_halo = t < NHALO;
  int hx = 0, hy = 0, hslot = 0;  // hslot: 0 y-low, 1 y-high, 2 x-low, 3 x-high
  if (D == 3) {
    if (t < BX) {
      hx = x0 + t, hy = y0 - 1, hslot = 0;
    } else if (t < 2 * BX) {
      hx = x0 + t - BX, hy = y0 + BY, hslot = 1;
    } else if (t < 2 * BX + BY) {
      hx = x0 - 1, hy = y0 + t - 2 * BX, hslot = 2;
    } else {
      hx = x0 + BX, hy = y0 + t - 2 * BX - BY, hslot = 3;
    }
  } else {
    hx = (t == 0) ? x0 - 1 : x0 + BX;
    hy = 0;
    hslot = (t == 0) ? 2 : 3;
  }
  int hox[3], hoy[3];
  const int hxn = fix_coord(hx, n0, bc0), hyn = fix_coord(hy, n1, bc1);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    hox[j] = fix_coord(hxn + j - 1, n0, bc0);
    hoy[j] = (D == 3) ? fix_coord(hyn + j - 1, n1, bc1) * p.nx : 0;
  }

  // FP32 with up to 256 threads per group: two planes in flight (see the
  // header), in up to 512 registers at one wavefront per SIMD.  FP64 needs
  // twice the registers per population, and 512-thread groups have half the
  // registers per thread: one plane in flight.
  // The pattern reference holds no arithmetic state, so it keeps two planes
  // in flight for every shape: the best latency hiding the access pattern
  // allows.
  constexpr bool PF2 = PAT || (DEV && BX * BY <= 256);
  // One plane in flight in a 512-thread group (two wavefronts per SIMD, both
  // of this group): the next core loads are issued before the barrier that
  // ends a plane, so their latency overlaps the wait for the wavefronts that
  // pull halo nodes.  At one wavefront per SIMD (256 threads) issuing them at
  // the top of the plane measured faster.
  constexpr bool EARLY = !PF2 && BX * BY > 256;
  const unsigned slot_bytes = (unsigned)(p.sl * (long long)sizeof(S));
  const long long plane_bytes = sm * (long long)sizeof(S);
  // byte offsets of the 9 in-plane sources of the core and of the halo node
  unsigned clo[9], hlo[9];
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    clo[j] = inplane_bytes<S>(p, coy[j / 3] + cox[j % 3]);
    hlo[j] = inplane_bytes<S>(p, hoy[j / 3] + hox[j % 3]);
  }
  auto march_planes = [&](int m, __amdgpu_buffer_rsrc_t* rs) {
    const int mn = fix_near(m, nm, bcm);  // m0 - 1 <= m <= m1 + 1
#pragma unroll
    for (int j = 0; j < 3; ++j) rs[j] = plane_rsrc(src + (long long)fix_near(mn + j - 1, nm, bcm) * sm, plane_bytes);
  };
  // Node arithmetic (or its stand-ins in the pattern reference).
  auto anom = [&](const NodeMoments<R>& mm, int a) -> R {
    if constexpr (PAT) return mm.u[a];
    else return anomaly(mm, a, k);
  };
  auto moments = [&](const R* f, const R* g) -> NodeMoments<R> {
    if constexpr (PAT) return pattern_moments<D, R>(f, g);
    else return node_moments<D, R>(f, g, k);
  };
  auto moments_light = [&](const R* f, const R* g) -> NodeMoments<R> {
    if constexpr (PAT) return pattern_all<D, R>(f, g);
    else if constexpr (DEV) return node_moments_light<D>(f, g, k);
    else return node_moments<D, R>(f, g, k);
  };
  // The halo node's anomaly into LDS buffer buf.
  auto halo_store = [&](const NodeMoments<R>& mm, int buf) {
    if (D == 3) {
      if (hslot == 0) lq1[buf][0][t] = anom(mm, 1);
      else if (hslot == 1) lq1[buf][BY + 1][t - BX] = anom(mm, 1);
      else if (hslot == 2) lq0[buf][t - 2 * BX][0] = anom(mm, 0);
      else lq0[buf][t - 2 * BX - BY][BX + 1] = anom(mm, 0);
    } else {
      lq0[buf][0][hslot == 2 ? 0 : BX + 1] = anom(mm, 0);
    }
  };
  // ... from populations already in registers (FP32 only) ...
  auto halo_finish = [&](const R* f, const R* g, int buf) {
    if constexpr (DEV || PAT) {
      if (has_halo) halo_store(moments_light(f, g), buf);
    }
  };
  // ... or loaded now, in batches.
  auto halo_direct = [&](const __amdgpu_buffer_rsrc_t* rs, int buf) {
    if (has_halo) {
      if constexpr (PAT) halo_store(pattern_pulled<D, S, R>(rs, slot_bytes, hlo), buf);
      else halo_store(pulled_moments_batched<D, S, R>(rs, slot_bytes, hlo, k), buf);
    }
  };
  // Own node's in-plane anomalies into LDS buffer buf.
  auto core_publish = [&](const NodeMoments<R>& mm, int buf) {
    lq0[buf][ly][lx + 1] = anom(mm, 0);
    if (D == 3) lq1[buf][ly + 1][lx] = anom(mm, 1);
  };

  R qm_prev, qm_cur, qm_next;  // anomaly along the march axis at m - 1, m, m + 1
  R hf[Q], hg[Q];              // halo node populations (in flight for the next plane)
  R f0[Q], g0[Q], f1[Q], g1[Q], f2[Q], g2[Q];
  NodeMoments<R> mo0, mo1, mo2;
  // prologue: anomaly along the march axis at plane m0 - 1 (core only)
  {
    __amdgpu_buffer_rsrc_t rs[3];
    march_planes(m0 - 1, rs);
    pull<D, S, R>(rs, slot_bytes, clo, f0, g0);
    const NodeMoments<R> mm = moments_light(f0, g0);
    qm_prev = anom(mm, D - 1);
  }
  // plane m0: core populations stay in registers, in-plane anomaly to LDS
  {
    __amdgpu_buffer_rsrc_t rs[3];
    march_planes(m0, rs);
    pull<D, S, R>(rs, slot_bytes, clo, f0, g0);
    mo0 = moments(f0, g0);
    qm_cur = anom(mo0, D - 1);
    core_publish(mo0, 0);
    halo_direct(rs, 0);
  }
  {
    __amdgpu_buffer_rsrc_t rs[3];
    march_planes(m0 + 1, rs);
    if (PF2 || EARLY) pull<D, S, R>(rs, slot_bytes, clo, f1, g1);
    if (PF2 && has_halo) pull<D, S, R>(rs, slot_bytes, hlo, hf, hg);
  }
  __syncthreads();

  // One plane: collide plane m (fa, ga, ma) and finish plane m + 1 (fb, gb,
  // mb).  PF2: plane m + 1's loads were issued one plane earlier, and the
  // loads of plane m + 2 (core and halo) go into (fc, gc) before the
  // collision; the three register sets rotate through a 3-way unrolled loop.
  // One plane in flight: plane m + 1 moves into (fa, ga) once plane m is
  // stored; its core loads were issued at the end of the previous plane
  // (EARLY) or at the top of this one.
  auto plane = [&](int m, R* fa, R* ga, NodeMoments<R>& ma, R* fb, R* gb, NodeMoments<R>& mb, R* fc, R* gc) {
    const int cb = (m - m0) & 1, nb = cb ^ 1;
    const bool more = m + 1 < m1;  // plane m + 1 collides in this chunk
    if constexpr (LBM_POISON_LDS) {
      // half nb was last read by plane m - 1, which ended with a barrier
      poison(nb);
      __syncthreads();
    }
    if (PF2) {
      __amdgpu_buffer_rsrc_t rs[3];
      march_planes(more ? m + 2 : m + 1, rs);
      if (more) pull<D, S, R>(rs, slot_bytes, clo, fc, gc);
      mb = moments(fb, gb);
      qm_next = anom(mb, D - 1);
      core_publish(mb, nb);
      halo_finish(hf, hg, nb);
      if (more && has_halo) pull<D, S, R>(rs, slot_bytes, hlo, hf, hg);
    } else {
      // one plane in flight; the halo node's populations are loaded in
      // batches, so only one batch of them is live beside the two core sets
      __amdgpu_buffer_rsrc_t rs[3];
      march_planes(m + 1, rs);
      if constexpr (EARLY) {
        // the halo first: its loads then overlap the latency of plane
        // m + 1's core loads, issued before the barrier (1.3 % faster than
        // pulling it after the core moments)
        halo_direct(rs, nb);
        mb = moments(fb, gb);
        qm_next = anom(mb, D - 1);
        core_publish(mb, nb);
      } else {
        pull<D, S, R>(rs, slot_bytes, clo, fb, gb);
        mb = moments(fb, gb);
        qm_next = anom(mb, D - 1);
        core_publish(mb, nb);
        halo_direct(rs, nb);
      }
    }
    // collide plane m
    R dd[3];
    dd[0] = anomaly_derivative<R>(p.deriv, ma.u[0], lq0[cb][ly][lx], lq0[cb][ly][lx + 1], lq0[cb][ly][lx + 2]);
    if (D == 3) {
      dd[1] = anomaly_derivative<R>(p.deriv, ma.u[1], lq1[cb][ly][lx], lq1[cb][ly + 1][lx], lq1[cb][ly + 2][lx]);
      dd[2] = anomaly_derivative<R>(p.deriv, ma.u[2], qm_prev, qm_cur, qm_next);
    } else {
      dd[1] = anomaly_derivative<R>(p.deriv, ma.u[1], qm_prev, qm_cur, qm_next);
      dd[2] = (R)0;
    }
    if constexpr (PAT) fa[0] += (dd[0] + dd[1]) + dd[2];
    else collide<D, R, DEV>(fa, ga, ma, dd, k);
    if (active) {
      const __amdgpu_buffer_rsrc_t rd = plane_rsrc(dst + (long long)m * sm, plane_bytes);
      const unsigned o = inplane_bytes<S>(p, cnode);
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        typename Buf<S>::pair_t v;
        v.x = (S)fa[i];
        v.y = (S)ga[i];
        Buf<S>::store(v, rd, o, (unsigned)i * slot_bytes);
      }
    }
    if (!PF2) {
      // plane m + 1 becomes the next collision set (EARLY: plane m + 2's
      // loads go into the freed set now)
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        fa[i] = fb[i];
        ga[i] = gb[i];
      }
      ma = mb;
      if (EARLY && more) {
        __amdgpu_buffer_rsrc_t rs[3];
        march_planes(m + 2, rs);
        pull<D, S, R>(rs, slot_bytes, clo, fb, gb);
      }
    }
    __syncthreads();
    qm_prev = qm_cur;
    qm_cur = qm_next;
  };

  if (PF2) {
    // sets: plane m in 0, m + 1 in 1, m + 2 loads into 2; then rotate
    for (int m = m0; m < m1; m += 3) {
      plane(m, f0, g0, mo0, f1, g1, mo1, f2, g2);
      if (m + 1 >= m1) break;
      plane(m + 1, f1, g1, mo1, f2, g2, mo2, f0, g0);
      if (m + 2 >= m1) break;
      plane(m + 2, f2, g2, mo2, f0, g0, mo0, f1, g1);
    }
  } else {
    // plane m in set 0, plane m + 1 in flight in set 1
    for (int m = m0; m < m1; ++m) plane(m, f0, g0, mo0, f1, g1, mo1, f2, g2);
  }
}

// XCD-aware logical block: consecutive hardware block ids go round the eight
// XCDs, so logical blocks are renumbered such that each XCD runs one
// contiguous range (neighbouring tiles then share an L2).
__device__ inline int xcd_logical_block(int b, int nblocks) {
  const int q8 = nblocks >> 3, r8 = nblocks & 7, xcd = b & 7;
  return xcd * q8 + min(xcd, r8) + (b >> 3);
}

template <int D, bool DEV, typename S, int BX, int BY, bool CAL = false>
__global__ void __launch_bounds__(BX* BY) step_kernel(const S* __restrict__ src, S* __restrict__ dst,
                                                      const StepParams p) {
  step_tile<D, DEV, S, BX, BY, CAL>(src, dst, p, xcd_logical_block(blockIdx.x, p.nblocks));
}

// The access-pattern reference of step_kernel (see step_tile).
template <int D, bool DEV, typename S, int BX, int BY>
__global__ void __launch_bounds__(BX* BY) pattern_kernel(const S* __restrict__ src, S* __restrict__ dst,
                                                         const StepParams p) {
  step_tile<D, DEV, S, BX, BY, false, true>(src, dst, p, xcd_logical_block(blockIdx.x, p.nblocks));
}

// Several boxes in one launch: logical block g belongs to the last box whose
// first block is <= g; that box's current buffer (cur ^ flip) is the source.
template <int D, bool DEV, typename S, int BX, int BY>
__global__ void __launch_bounds__(BX* BY) batch_step_kernel(const BoxEntry* __restrict__ table, int nboxes,
                                                            int total_blocks, int flip) {
  const int g = xcd_logical_block(blockIdx.x, total_blocks);
  int lo = 0, hi = nboxes - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (table[mid].block_start <= g) lo = mid;
    else hi = mid - 1;
  }
  const BoxEntry& e = table[lo];
  const int par = e.cur ^ flip;
  step_tile<D, DEV, S, BX, BY>(static_cast<const S*>(e.buf[par]), static_cast<S*>(e.buf[par ^ 1]), e.p,
                               g - e.block_start);
}

// The same step with a fixed grid (a few work-groups per compute unit, sized
// by occupancy): each XCD owns one contiguous eighth of the logical tiles
// (neighbouring tiles share its L2) and its work-groups take that range's
// tiles in turn, tile rank, rank + (work-groups per XCD), ...  Every
// work-group leaves the loop when its range is done; no work-group waits
// for another.  gridDim.x is a multiple of 8.
template <int D, bool DEV, typename S, int BX, int BY>
__global__ void __launch_bounds__(BX* BY) batch_persistent_kernel(const BoxEntry* __restrict__ table, int nboxes,
                                                                  int total_blocks, int flip) {
  const int per_xcd = gridDim.x >> 3, xcd = blockIdx.x & 7, rank = blockIdx.x >> 3;
  const int lo = (int)((long long)total_blocks * xcd / 8), hi = (int)((long long)total_blocks * (xcd + 1) / 8);
  for (int g = lo + rank; g < hi; g += per_xcd) {
    int a = 0, z = nboxes - 1;
    while (a < z) {
      const int mid = (a + z + 1) >> 1;
      if (table[mid].block_start <= g) a = mid;
      else z = mid - 1;
    }
    const BoxEntry& e = table[a];
    const int par = e.cur ^ flip;
    step_tile<D, DEV, S, BX, BY>(static_cast<const S*>(e.buf[par]), static_cast<S*>(e.buf[par ^ 1]), e.p,
                                 g - e.block_start);
  }
}

// After an odd number of batched steps every box's current buffer changes.
__global__ void __launch_bounds__(64) toggle_cur_kernel(BoxEntry* __restrict__ table, int nboxes) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nboxes) table[i].cur ^= 1;
}

// ---------------------------------------------------------------------------
// Initialisation: f = f^eq, g = g^eq (minus the reference state when DEV).
// The equilibria are evaluated in FP64 for either storage, so FP32 storage
// holds each deviation rounded once.
// ---------------------------------------------------------------------------

template <int D, bool DEV, typename S>
__global__ void __launch_bounds__(256) init_kernel(const double* __restrict__ rho, const double* __restrict__ u,
                                                   const double* __restrict__ T, S* __restrict__ dst, long long N,
                                                   const StepParams p) {
  using R = double;
  constexpr int Q = lat_q(D);
  const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const NodeConsts k = node_consts(p);
  NodeMoments<R> m;
  const double r = rho[n], tt = T[n];
  m.rho = (R)r;
  m.drho = (R)(r - p.rho0);
  m.T = (R)tt;
  m.dT = (R)(tt - p.T0);
  for (int a = 0; a < 3; ++a) {
    const double ua = a < D ? u[a * N + n] : 0.0;
    m.u[a] = (R)ua;
    m.du[a] = (R)(ua - p.u0[a]);
  }
  m.omega = m.omega1 = (R)1;  // unused by the equilibria
  m.corr = (R)0;                // multiplies d = 0
  R d[3] = {0, 0, 0};
  R fe[Q], ge[Q];
  equilibria<D, R, DEV>(m, d, k, fe, ge);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    dst[pop_offset(p, Q, i, n)] = (S)fe[i];
    dst[pop_offset(p, Q, i + Q, n)] = (S)ge[i];
  }
}

// ---------------------------------------------------------------------------
// Moments of the stored populations (no streaming), FP64
// ---------------------------------------------------------------------------

// The Q (f, g) pairs of the node whose slot-0 pair is at src.
template <int D, typename S>
__device__ inline void load_pairs(const S* __restrict__ src, const StepParams& p, typename Buf<S>::pair_t* v) {
#pragma unroll
  for (int i = 0; i < lat_q(D); ++i) v[i] = *(const typename Buf<S>::pair_t*)(src + i * p.sl);
}

// Sums of a node's stored values: s0 = sum f, j = sum c f and, when se is not
// NULL, *se = sum g (in population order).
template <int D, typename P>
__device__ inline void pair_sums(const P* v, double& s0, double* j, double* se) {
  double jx = 0, jy = 0, jz = 0, e = 0;
  s0 = 0;
#pragma unroll
  for (int i = 0; i < lat_q(D); ++i) {
    const double w = (double)v[i].x;
    s0 += w;
    if (se) e += (double)v[i].y;
    const int cx = vx(i), cy = vy(i), cz = (D == 3) ? vz(i) : 0;
    if (cx) jx += cx > 0 ? w : -w;
    if (cy) jy += cy > 0 ? w : -w;
    if (cz) jz += cz > 0 ? w : -w;
  }
  j[0] = jx;
  j[1] = jy;
  j[2] = jz;
  if (se) *se = e;
}

// rho and u of a node from the sums of its stored populations (FP64).
template <int D>
__device__ inline double velocity_of(const StepParams& p, double s0, const double* j, double* u) {
  const double rho = p.rho0 + s0;
  u[0] = (p.j0[0] + j[0]) / rho;
  u[1] = (p.j0[1] + j[1]) / rho;
  u[2] = (D == 3) ? (p.j0[2] + j[2]) / rho : 0.0;
  return rho;
}

// rho, u, T and rho E of a node from the sums of its stored populations (FP64;
// Eqs. (3)-(7) without streaming).
template <int D>
__device__ inline void fields_of(const StepParams& p, double s0, const double* j, double se, double& rho, double* u,
                                 double& T, double& rhoE) {
  rho = velocity_of<D>(p, s0, j, u);
  rhoE = p.rhoE0 + se;
  const double e = rhoE / rho - 0.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);  // U(T)
  T = p.caloric ? p.T0 + caloric_step(p.Cv, p.cv1, p.cv2, p.T0, e - p.U0) : e * p.inv_Cv;
}

// Any of rho, u (nu planes) and T may be NULL.  Bound by memory: 2Q values
// read and D + 2 written per node, straight into the caller's arrays.  A
// thread reads each (f, g) pair in one access.
template <int D, typename S>
__global__ void __launch_bounds__(256) fields_kernel(const S* __restrict__ pops, double* __restrict__ rho_out,
                                                     double* __restrict__ u_out, int nu, double* __restrict__ T_out,
                                                     int N, const StepParams p) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  typename Buf<S>::pair_t v[lat_q(D)];
  load_pairs<D>(pops + pair_offset(p, n), p, v);
  double s0, j[3], se, rho, u[3], T, rhoE;
  pair_sums<D>(v, s0, j, &se);
  fields_of<D>(p, s0, j, se, rho, u, T, rhoE);
  if (rho_out) rho_out[n] = rho;
  if (u_out)
    for (int a = 0; a < nu; ++a) u_out[(long long)a * N + n] = u[a];
  if (T_out) T_out[n] = T;
}

// ---------------------------------------------------------------------------
// Reductions: wave64 shuffles, then LDS across the waves of a block, FP64
// per-block partials; a second launch, one work-group per sum, adds the
// partials in a fixed order.
// ---------------------------------------------------------------------------

// The NV sums over a work-group of NW wavefronts; sum j goes to out[j * stride].
template <int NV, int NW>
__device__ inline void block_reduce_store(double (&v)[NV], double* __restrict__ out, int stride) {
  __shared__ double red[NV][NW];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    double x = v[j];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    v[j] = x;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) red[j][wave] = v[j];
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const int j = threadIdx.x;
    double x = 0.0;
#pragma unroll
    for (int w = 0; w < NW; w += 2) x += red[j][w] + (w + 1 < NW ? red[j][w + 1] : 0.0);
    out[(long long)j * stride] = x;
  }
}

// The 21 diagnostic sums: the totals of Eqs. (3)-(5) and the statistics of
// Sec. III.D.  of_node adds the terms that need one node's fields,
// of_differences those of the central differences, from the velocities vn[k]
// of the six neighbours (x + 1, x - 1, y + 1, y - 1, z + 1, z - 1).
template <int D>
struct DiagSums {
  double mass = 0, mom[3] = {}, energy = 0, kinetic = 0, div2 = 0, cs = 0, rho2 = 0, vort2 = 0, diss = 0;
  double u2[3] = {}, du2[3] = {};
  unsigned nonfinite = 0, nonpositive = 0, nodes = 0;  // of one thread

  __device__ inline void of_node(const StepParams& p, double rho, const double* u, double T, double rhoE) {
    const bool finite = isfinite(rho) && isfinite(T) && isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]);
    mass += rho;
    energy += rhoE;
    kinetic += 0.5 * rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    double gam = p.gamma;  // C_p / C_v at T (Mayer: C_p = C_v + 1)
    if (p.caloric) {
      const double cvT = caloric_cv(p.Cv, p.cv1, p.cv2, T);
      gam = (cvT + 1.0) / cvT;
    }
    cs += sqrt(gam * T);
    rho2 += rho * rho;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      mom[a] += rho * u[a];
      u2[a] += u[a] * u[a];
    }
    nonfinite += finite ? 0u : 1u;
    nonpositive += (rho <= 0.0 || T <= 0.0) ? 1u : 0u;
    ++nodes;
  }

  __device__ inline void of_differences(double mu, const double (*vn)[3]) {
    double d[3] = {};
    d[0] = 0.5 * (vn[0][0] - vn[1][0]);
    d[1] = 0.5 * (vn[2][1] - vn[3][1]);
    if (D == 3) d[2] = 0.5 * (vn[4][2] - vn[5][2]);
    const double wz = 0.5 * (vn[0][1] - vn[1][1]) - 0.5 * (vn[2][0] - vn[3][0]);
    double wx = 0.0, wy = 0.0;
    if (D == 3) {
      wx = 0.5 * (vn[2][2] - vn[3][2]) - 0.5 * (vn[4][1] - vn[5][1]);
      wy = 0.5 * (vn[4][0] - vn[5][0]) - 0.5 * (vn[0][2] - vn[1][2]);
    }
    const double v2 = wx * wx + wy * wy + wz * wz, div = d[0] + d[1] + d[2];
    div2 += div * div;
    vort2 += v2;
    diss += mu * v2;
#pragma unroll
    for (int a = 0; a < D; ++a) du2[a] += d[a] * d[a];
  }

  // in the order of lbm_diag (see diag_from_sums)
  __device__ inline void store(double (&v)[kNumDiag]) const {
    const double all[kNumDiag] = {mass,  mom[0], mom[1], mom[2], energy, kinetic, div2,   (u2[0] + u2[1]) + u2[2],
                                  cs,    rho2,   vort2,  diss,   u2[0],  u2[1],   u2[2],  du2[0],
                                  du2[1], du2[2], (double)nonfinite, (double)nonpositive, (double)nodes};
#pragma unroll
    for (int j = 0; j < kNumDiag; ++j) v[j] = all[j];
  }
};

// The diagnostic sums straight from the stored populations.  A work-group
// takes tiles of BX x BY nodes and marches each over a chunk of planes (z for
// D3Q27, rows along y for D2Q9): every node's fields are formed once, its
// velocity goes to LDS for the in-plane differences (a one-node ring around
// the tile is formed by the first threads), and the march-axis neighbours are
// the same thread's previous and next planes.  The populations are read once,
// plus the two planes next to a chunk and the ring, whose column nodes cost a
// cache line each (64 x 8: half as many lines again as the tile's).  Bound by that
// traffic: neighbouring tiles run on one die, whose cache then serves most of a
// ring (a call with tiles dealt out over the dies in turn and in die order: 256^3
// FP32 868 and 718 us, FP64 1498 and 1267; 166x213x86 202 and 184, 332 and 304).
// Registers allow two wavefronts per SIMD (222: 35 for the sums, 54 or 108 for a
// node's loads).
template <int D, typename S, int BX, int BY>
__global__ void __launch_bounds__(BX* BY) diag_kernel(const S* __restrict__ pops, double* __restrict__ partial,
                                                         const StepParams p, const DiagGrid g) {
  constexpr int LY = (D == 3) ? BY + 2 : 1;
  constexpr int Q = lat_q(D);
  constexpr int NHALO = (D == 3) ? 2 * BX + 2 * BY : 2;
  static_assert(BX * BY >= NHALO, "tile too small for its ring");
  __shared__ double lu[2][D][LY][BX + 2];
  const int n0 = p.nx, n1 = (D == 3) ? p.ny : 1, nm = (D == 3) ? p.nz : p.ny;
  const int bc0 = p.bc[0], bc1 = p.bc[1], bcm = (D == 3) ? p.bc[2] : p.bc[1];
  const unsigned slot_bytes = (unsigned)(p.sl * (long long)sizeof(S));
  const long long plane_bytes = p.ms * (long long)sizeof(S);
  const int t = threadIdx.x, lx = t % BX, ly = t / BX;
  DiagSums<D> sums;
  const int block = xcd_logical_block(blockIdx.x, gridDim.x);
  for (int task = block; task < g.tasks; task += gridDim.x) {
    const int tx = task % g.tiles_x, r = task / g.tiles_x;
    const int ty = (D == 3) ? r % g.tiles_y : 0, ck = (D == 3) ? r / g.tiles_y : r;
    const int x0 = tx * BX, y0 = ty * BY, m0 = ck * g.chunk, m1 = min(m0 + g.chunk, nm);
    // A position beyond the domain stands for the node it maps to by wrap or
    // clamp; only the first one past each end is anybody's neighbour.
    auto in_plane = [&](int x, int y) {
      return inplane_bytes<S>(p, fix_coord(x, n0, bc0) + ((D == 3) ? fix_coord(y, n1, bc1) * n0 : 0));
    };
    const int gx = x0 + lx, gy = y0 + ly;
    const bool active = gx < n0 && gy < n1;
    const bool formed = gx <= n0 && ((D == 3) ? gy <= n1 : true);
    const unsigned core = in_plane(gx, gy);
    int hx = (t == 0) ? -1 : BX, hy = 0;  // the ring node of this thread, within the tile
    if (D == 3) {
      if (t < 2 * BX) hx = t % BX, hy = t < BX ? -1 : BY;
      else hy = (t - 2 * BX) % BY, hx = t < 2 * BX + BY ? -1 : BX;
    }
    const bool ring = t < NHALO && x0 + hx <= n0 && ((D == 3) ? y0 + hy <= n1 : true);
    const unsigned ring_off = in_plane(x0 + hx, y0 + hy);
    auto load = [&](int m, unsigned off, typename Buf<S>::pair_t* v) {
      const __amdgpu_buffer_rsrc_t rs = plane_rsrc(pops + (long long)fix_near(m, nm, bcm) * p.ms, plane_bytes);
#pragma unroll
      for (int i = 0; i < Q; ++i) v[i] = Buf<S>::load(rs, off, (unsigned)i * slot_bytes);
    };
    auto velocity = [&](int m, unsigned off, double* u) {
      typename Buf<S>::pair_t v[Q];
      double s0, j[3];
      load(m, off, v);
      pair_sums<D>(v, s0, j, nullptr);
      velocity_of<D>(p, s0, j, u);
    };
    auto publish = [&](int buf, int y, int x, const double* u) {
#pragma unroll
      for (int a = 0; a < D; ++a) lu[buf][a][(D == 3) ? y + 1 : 0][x + 1] = u[a];
    };
    // Fields of plane m: the sums of its nodes, its velocity to LDS and to u,
    // its viscosity to mu.
    auto fill = [&](int m, int buf, double* u, double& mu) {
      if (formed) {
        double s0, j[3], se, rho, T, rhoE;
        typename Buf<S>::pair_t v[Q];
        load(m, core, v);
        pair_sums<D>(v, s0, j, &se);
        fields_of<D>(p, s0, j, se, rho, u, T, rhoE);
        publish(buf, ly, lx, u);
        if (active) {
          sums.of_node(p, rho, u, T, rhoE);
          mu = (p.visc_exp == 0.0) ? p.mu0 : p.mu0 * pow(T * p.inv_Tref, p.visc_exp);
        }
      }
      if (ring) {
        double uh[3];
        velocity(m, ring_off, uh);
        publish(buf, hy, hx, uh);
      }
    };
    double up[3] = {}, uc[3] = {}, un[3] = {};  // velocity at m - 1, m, m + 1
    double mu = 0, mu_n = 0;
    if (active) {  // a one-plane chunk asks for both neighbours before the barrier
      velocity(m0 - 1, core, up);
      if (m0 + 1 == m1) velocity(m1, core, un);
    }
    fill(m0, 0, uc, mu);
    __syncthreads();
    for (int m = m0; m < m1; ++m) {
      const int cb = (m - m0) & 1;
      if (m + 1 < m1) fill(m + 1, cb ^ 1, un, mu_n);
      else if (m > m0 && active) velocity(m + 1, core, un);
      if (active) {
        double vn[6][3] = {};
        const int yy = (D == 3) ? ly + 1 : 0;
#pragma unroll
        for (int a = 0; a < D; ++a) {
          vn[0][a] = lu[cb][a][yy][lx + 2];
          vn[1][a] = lu[cb][a][yy][lx];
          if (D == 3) {
            vn[2][a] = lu[cb][a][(D == 3) ? ly + 2 : 0][lx + 1];
            vn[3][a] = lu[cb][a][(D == 3) ? ly : 0][lx + 1];
          }
          vn[D == 3 ? 4 : 2][a] = un[a];
          vn[D == 3 ? 5 : 3][a] = up[a];
        }
        sums.of_differences(mu, vn);
      }
      __syncthreads();
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        up[a] = uc[a];
        uc[a] = un[a];
      }
      mu = mu_n;
    }
  }
  double v[kNumDiag];
  sums.store(v);
  block_reduce_store<kNumDiag, BX * BY / 64>(v, partial + block, gridDim.x);
}

// The same sums for boxes so narrow that a tile would leave most of its lanes
// idle: 256 nodes in memory order, whose velocities go to LDS; a neighbour
// that is not among them is formed again from its populations.  Bound by
// those loads: a velocity costs Q pairs where the marching kernel reads LDS.
template <int D, typename S>
__global__ void __launch_bounds__(256) diag_flat_kernel(const S* __restrict__ pops, double* __restrict__ partial,
                                                        int N, const StepParams p) {
  constexpr int Q = lat_q(D);
  __shared__ double lu[D][256];
  const int t = threadIdx.x;
  const int n0 = p.nx, n1 = p.ny, n2 = (D == 3) ? p.nz : 1;
  DiagSums<D> sums;
  // Work-groups go round the eight dies: each die takes one stretch of the
  // box, whose planes its cache then serves three times (300 x 3 x 400 FP64:
  // 130 us a call against 175 with the tiles dealt out in turn).
  const int tiles = (int)(((long long)N + 255) / 256), per = (tiles + 7) / 8, die = blockIdx.x & 7;
  const int last = min((die + 1) * per, tiles);
  for (int tile = die * per + (blockIdx.x >> 3); tile < last; tile += gridDim.x >> 3) {
    const long long base = (long long)tile * 256;
    const bool active = base + t < N;
    const int n = active ? (int)(base + t) : N - 1;
    const int x = n % n0, r = n / n0, y = (D == 3) ? r % n1 : r, z = (D == 3) ? r / n1 : 0;
    double rho, u[3], T, rhoE;
    {
      typename Buf<S>::pair_t v[Q];
      double s0, j[3], se;
      load_pairs<D>(pops + pair_offset(p, n), p, v);
      pair_sums<D>(v, s0, j, &se);
      fields_of<D>(p, s0, j, se, rho, u, T, rhoE);
    }
#pragma unroll
    for (int a = 0; a < D; ++a) lu[a][t] = u[a];
    __syncthreads();
    if (active) {
      sums.of_node(p, rho, u, T, rhoE);
      const double mu = (p.visc_exp == 0.0) ? p.mu0 : p.mu0 * pow(T * p.inv_Tref, p.visc_exp);
      double vn[6][3] = {};
#pragma unroll
      for (int k = 0; k < 2 * D; ++k) {
        const int step = (k & 1) ? -1 : 1;
        int q = k < 2   ? n - x + fix_near(x + step, n0, p.bc[0])
                : k < 4 ? n + (fix_near(y + step, n1, p.bc[1]) - y) * n0
                        : n + (fix_near(z + step, n2, p.bc[2]) - z) * p.plane;
        const long long at = q - base;
        if (at >= 0 && at < 256) {
#pragma unroll
          for (int a = 0; a < D; ++a) vn[k][a] = lu[a][at];
        } else {
          typename Buf<S>::pair_t v[Q];
          double s0, j[3];
          load_pairs<D>(pops + pair_offset(p, q), p, v);
          pair_sums<D>(v, s0, j, nullptr);
          velocity_of<D>(p, s0, j, vn[k]);
        }
      }
      sums.of_differences(mu, vn);
    }
    __syncthreads();
  }
  double v[kNumDiag];
  sums.store(v);
  block_reduce_store<kNumDiag, 4>(v, partial + blockIdx.x, gridDim.x);
}

// out[j] = the sum of partial[j * nblocks ..]: one work-group per sum, so the
// partials are read side by side (one work-group for all 21 sums, each
// thread striding over them, took 11-15 us).
__global__ void __launch_bounds__(256) final_reduce_kernel(const double* __restrict__ partial, int nblocks,
                                                           double* __restrict__ out) {
  double acc[1] = {0.0};
  for (int b = threadIdx.x; b < nblocks; b += 256) acc[0] += partial[(long long)blockIdx.x * nblocks + b];
  block_reduce_store<1, 4>(acc, out + blockIdx.x, 1);
}

// Counts nodes of a candidate initial field with non-finite values or
// rho <= 0 or T <= 0 (slot 0).
template <int D>
__global__ void __launch_bounds__(256) validate_kernel(const double* __restrict__ rho, const double* __restrict__ u,
                                                       const double* __restrict__ T, double* __restrict__ partial,
                                                       long long N) {
  double acc[1] = {0.0};
  for (long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x; n < N; n += (long long)gridDim.x * blockDim.x) {
    bool ok = isfinite(rho[n]) && isfinite(T[n]) && rho[n] > 0.0 && T[n] > 0.0;
    for (int a = 0; a < D; ++a) ok = ok && isfinite(u[(long long)a * N + n]);
    acc[0] += ok ? 0.0 : 1.0;
  }
  block_reduce_store<1, 4>(acc, partial + blockIdx.x, 1);
}

__global__ void __launch_bounds__(256) copy_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                                   long long n16) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

// Checkpoints: the internal layout <-> the ABI state (2Q planes of N values,
// f then g).  Both directions are bound by memory (4 Q values moved per node
// each way).  A thread moves the (f, g) pair of a slot in one access, so the
// populations are touched once (a value at a time, the other half of every
// pair was fetched again for g: 1635 us at 256^3 FP32 against 1355 us, 5.35 TB/s,
// and 9.7 against 6.2 us for a 300^2 box).
template <int D, typename S>
__global__ void __launch_bounds__(256) pack_kernel(const S* __restrict__ pops, S* __restrict__ state, int N,
                                                   const StepParams p) {
  using pair_t = typename Buf<S>::pair_t;
  constexpr int Q = lat_q(D);
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const S* src = pops + pair_offset(p, n);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const pair_t v = *(const pair_t*)(src + i * p.sl);
    state[(long long)i * N + n] = v.x;
    state[(long long)(i + Q) * N + n] = v.y;
  }
}

template <int D, typename S>
__global__ void __launch_bounds__(256) unpack_kernel(const S* __restrict__ state, S* __restrict__ pops, int N,
                                                     const StepParams p) {
  using pair_t = typename Buf<S>::pair_t;
  constexpr int Q = lat_q(D);
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  S* dst = pops + pair_offset(p, n);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    pair_t v;
    v.x = state[(long long)i * N + n];
    v.y = state[(long long)(i + Q) * N + n];
    *(pair_t*)(dst + i * p.sl) = v;
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

template <int D, bool DEV, typename S, int BX, int BY, bool CAL = false>
static hipError_t launch_step_t(const Ctx& c, const void* src, void* dst) {
  hipLaunchKernelGGL((step_kernel<D, DEV, S, BX, BY, CAL>), dim3(c.sp.nblocks), dim3(BX * BY), 0, c.stream,
                     static_cast<const S*>(src), static_cast<S*>(dst), c.sp);
  return hipGetLastError();
}

// Estimated time of a 3-D launch, in units of one 64 x 4 tile plane.  A
// work-group marches `chunk` planes of one tile column and occupies a whole
// CU (one wavefront per SIMD for the 256-thread shapes, two for 64 x 8), so
// the launch runs in rounds of 256 work-groups.  Each chunk pays a prologue
// (the planes next to it are loaded and their moments computed before its
// first collision) worth about 8 planes in the measured chunk sweeps.  w is
// the time of one tile plane of the shape relative to 64 x 4: 32 x 8 moves
// the same nodes a little slower (1.02), 64 x 8 moves twice the nodes with
// two wavefronts per SIMD hiding more latency (1.8).
static double march_cost(const int64_t n[3], int bx, int by, int64_t chunk, double w, double pro) {
  const int64_t tiles = ((n[0] + bx - 1) / bx) * ((n[1] + by - 1) / by);
  const int64_t blocks = tiles * ((n[2] + chunk - 1) / chunk);
  return (double)((blocks + 255) / 256) * ((double)chunk + pro) * w;
}

// Per-plane cost w and chunk prologue pro (in planes) of a 3-D launch shape,
// fitted to tile and chunk sweeps: 64 x 4 (1, 8 planes), 32 x 8 (1.02, 8)
// and the 512-thread 64 x 8 (1.82, 4.45; its next plane's loads are issued
// before the per-plane barrier, which shortens its prologue: fitted to
// 256^3 in 128-plane chunks and a 256 x 256 x 32 slab in 16-plane chunks).
static double shape_prologue(int bx, int by) { return (bx == 64 && by == 8) ? 4.45 : 8.0; }

// The power-of-two chunk of 4 to 256 planes, or the whole march axis, with
// the lowest march_cost for one 3-D launch shape.  Chunks stay powers of
// two: at 80^3 and 96^3, 8- and 16-plane chunks ran up to 45% faster than
// 6-, 12- or 24-plane ones.
static int64_t best_chunk3(const int64_t n[3], int bx, int by, double w, double* cost) {
  int64_t best = 1;
  double best_cost = -1.0;
  const double pro = shape_prologue(bx, by);
  for (int64_t chunk = 4;; chunk *= 2) {
    const int64_t c = chunk < n[2] ? chunk : n[2];
    const double k = march_cost(n, bx, by, c, w, pro);
    if (best_cost < 0.0 || k < best_cost) {
      best_cost = k;
      best = c;
    }
    if (chunk >= n[2] || chunk >= 256) break;
  }
  if (cost) *cost = best_cost;
  return best;
}

int default_chunk(int D, const int64_t n[3], int bx, int by) {
  if (D == 3) return (int)best_chunk3(n, bx, by, 1.0, nullptr);
  // D2Q9: chunks short enough for about 2^17 threads in flight (1024
  // work-groups of 128; the whole 2-D field is small), between 4 and 32 rows.
  const int64_t tiles = (n[0] + bx - 1) / bx;
  int64_t chunk = n[1] * tiles * bx / (1024 * 128);
  chunk = chunk < 4 ? 4 : (chunk > 32 ? 32 : chunk);
  return (int)(chunk < n[1] ? chunk : n[1]);
}

// Two finer models of a launch, for the shapes whose results do not depend on the
// march chunk (FP64, and 64 x 8 in FP32: one plane in flight, one copy of the
// plane's arithmetic).  The first proposes a chunk, the second has to agree.
//
// The first: a work-group marches c planes of one tile column and pays p1 planes
// for its start (launch, the planes next to the chunk, its first loads); one that
// follows another on its compute unit pays less, p2.  The device holds cap2
// work-groups of the shape at a time; w2 is what a plane takes them, and w1 what
// it takes up to cap1 of them, which share no SIMD.  A round that leaves some
// compute units idle runs a little faster (`idle`; D3Q27, where memory binds).
struct ShapeModel {
  int bx, by, cap1, cap2;
  double w1, w2, p1, p2, idle;
};

static double launch_time(const ShapeModel& s, int64_t blocks, double c) {
  auto filled = [&](int64_t b) { return 1.0 - s.idle * (1.0 - std::max(0.75, (double)b / s.cap2)); };
  if (blocks <= s.cap2) return (blocks <= s.cap1 ? s.w1 : s.w2) * (c + s.p1) * filled(blocks);
  const double rounds = (double)blocks / s.cap2;
  // over many rounds a compute unit takes the next work-group as it gets free
  if (rounds > 3.0) return s.w2 * ((c + s.p1) + (rounds - 1.0) * (c + s.p2));
  const int64_t whole = blocks / s.cap2, rest = blocks % s.cap2;
  double t = s.w2 * ((c + s.p1) + (double)(whole - 1) * (c + s.p2));
  if (rest) t += (rest <= s.cap1 ? s.w1 : s.w2) * (c + s.p2) * filled(rest);
  return t;
}

// One work-group per compute unit.
static const ShapeModel kShape64x8{64, 8, 256, 256, 1.5, 1.5, 7.0, 6.0, 0.2};
static const ShapeModel kShapes3F64[] = {{64, 4, 256, 256, 1.0, 1.0, 15.0, 13.0, 0.2},
                                         {32, 8, 256, 256, 1.02, 1.02, 15.0, 13.0, 0.2}};
// Two wavefronts per SIMD; two work-groups of a compute unit share SIMDs.
static const ShapeModel kShape2F64[] = {{128, 1, 256, 1024, 1.03, 1.45, 3.0, 1.5, 0.0},
                                        {256, 1, 256, 512, 1.06, 1.43, 3.0, 1.5, 0.0}};

// The model's best of the shapes and of the chunks of at most `longest` planes
// that split the march axis evenly (longer ones gain nothing more).
static Tile best_tile(const ShapeModel* shapes, int count, const int64_t n[3], int64_t nm, int64_t longest) {
  Tile best{0, 0, 1};
  double best_time = 0.0;
  for (int k = 0; k < count; ++k) {
    const ShapeModel& s = shapes[k];
    const int64_t tiles = ((n[0] + s.bx - 1) / s.bx) * (s.by > 1 ? (n[1] + s.by - 1) / s.by : 1);
    for (int64_t c = 1; c <= longest && c <= nm; ++c) {
      const int64_t chunks = (nm + c - 1) / c;
      if ((nm + chunks - 1) / chunks != c) continue;
      const double t = launch_time(s, tiles * chunks, (double)c);
      if (!best.bx || t < best_time) {
        best_time = t;
        best = Tile{s.bx, s.by, (int)c};
      }
    }
  }
  return best;
}

// The second: the first knows nothing of memory, prices a few work-groups past
// three full rounds as a part of a round, and credits idle compute units too much:
// FP64 224^3 took 2525 us a step in 784 work-groups of 32 x 8 and 56 planes against
// 2120 in 224 of 64 x 4, and 227x150x40 358 in 152 of 64 x 4 against 312 in 760.
//
// What it knows of a launch over one or several boxes:
struct Load {
  double blocks = 0, planes = 0, lanes = 0, nodes = 0;  // planes, lanes: of all work-groups

  void add(const int64_t n[3], int D, const Tile& t) {
    const int64_t nm = D == 3 ? n[2] : n[1];
    const double tiles = (double)((n[0] + t.bx - 1) / t.bx) * (double)(D == 3 ? (n[1] + t.by - 1) / t.by : 1);
    const double groups = tiles * (double)((nm + t.chunk - 1) / t.chunk);
    blocks += groups;
    planes += groups * t.chunk;
    lanes += tiles * t.bx * t.by * (double)nm;
    nodes += (double)n[0] * (double)n[1] * (double)n[2];
  }
};

// Microseconds of a D3Q27 launch whose work-groups march c planes each, one
// work-group per compute unit.  A round takes `plane` a plane, and `crowd` more
// when all compute units march; a launch moves its planes, and `reread` planes
// next to every chunk, at `cached` to `hbm` microseconds for one plane of all 256
// tiles, in proportion to what of the two population buffers lies beyond
// `cache` MB.  The two overlap in part (a sum of powers of 1.5).
// Fitted to sweeps over 165 boxes in FP64 and 52 in FP32 from 10^4 to 1.7 10^7
// nodes: 6-7% of a launch's time.
struct MarchModel {
  int bx, by, word;
  double start, plane, crowd, cached, hbm, cache, reread, scale;

  double time(const Load& l) const {
    const double c = l.planes / l.blocks, share = l.blocks / 256.0, rounds = std::ceil(share);
    const double megabytes = l.nodes * 2 * 54 * word * 1e-6;
    const double move = cached + (hbm - cached) * std::max(0.0, 1.0 - cache / megabytes);
    const double memory = share * (c + reread) * move / std::sqrt(l.lanes / l.nodes);
    const double march = rounds * c * (plane + crowd * std::min(1.0, share)) + (rounds - 1.0) * start;
    const double both = std::cbrt(memory * std::sqrt(memory) + march * std::sqrt(march));
    return (4.0 + start + both * both) * scale;
  }
};
static const MarchModel kMarch3F64[] = {{64, 4, 8, 4.0, 5.5, 1.3, 2.7, 7.0, 120.0, 3.0, 1.0},
                                        {32, 8, 8, 4.0, 5.5, 1.3, 2.7, 7.0, 120.0, 3.0, 1.05}};
static const MarchModel kMarch64x8{64, 8, 4, 4.0, 7.0, 0.0, 4.5, 7.4, 160.0, 2.0, 1.0};

// The second model's time of a launch in a shape.
static double modelled(int precision, int bx, const Load& l) {
  return precision == LBM_FP32_DEV ? kMarch64x8.time(l) : kMarch3F64[bx == 64 ? 0 : 1].time(l);
}

// A proposal is taken where the second model finds it no slower than the base:
// of 1937 D3Q27 boxes up to 4.2 M nodes with another choice than the base, over
// both schemes, open and periodic axes and both caloric laws, four are slower by
// more than 2.5% (at most 6%), and the mean gain is 1.43 (FP64) and 1.16 (64 x 8);
// without the second model nine, by up to 16%.  Larger boxes have to gain 1.05: of
// 53 none is slower (without the second model 17, by up to 16%).  D2Q9's first
// model has none slower of 978 boxes up to 4 M nodes, at a mean gain of 1.62, and
// 15 of 100 larger ones, by up to 19%, which keep the base.
constexpr int64_t kLargeBox = 4000000;
constexpr double kGainLarge = 1.05;

// Default launch shape and march chunk (32 x 16 tiles, the 512-thread shape
// with the smallest halo ring, measured 10% slower than 64 x 8 at 256^3 FP32
// and are not compiled).  The caloric variant is compiled for one shape of each
// lattice.
// D3Q27: the shape with the lowest march_cost at its best power-of-two chunk;
// for FP64, and for 64 x 8 (the only 512-thread shape that fits 256 registers
// without spilling), refined by the models.  The 256-thread FP32 shapes keep two
// planes in flight through a plane loop unrolled three times; the compiler fuses
// products and sums a little differently in each copy, so there the rounding of a
// node follows the chunk, and a different chunk moves the results of long runs,
// and of runs with the bf16 corrector, by more than rounding (5e-5 of the
// deviations after four corrections).  On one MI355X this picks 64 x 4 / 4 at
// FP32 64^3, 64 x 8 / 16 at 128^3 and for a 256 x 256 x 32 slab, 64 x 8 / 128 at
// 256^3 (9% faster than 64 x 4 / 256 there).
// D2Q9: rows of 128, or of 256 from 1024 nodes per row (FP32: 9% faster at
// 4096^2, even at 1024^2 and 2048^2; FP64 at 1024^2: 4% faster), FP64 refined by
// the first model.  FP32 keeps two rows in flight, so its chunks stay as they are too.
// Microseconds a step, base and choice: FP64 20x25x40 64x4/4 31.4, 32x8/1 14.6;
// 190x131x110 64x4/16 600, 64x4/55 555; 800x4 128x1/4 11.2, 128x1/1 6.2; 300^2
// 128x1/4 15.1, 128x1/1 10.7; FP32 190x131x110 64x8/32 346, 64x8/22 296.
static Tile base_tile(int D, int precision, const int64_t n[3], bool caloric) {
  if (D == 2) {
    const int bx = !caloric && n[0] >= 1024 ? 256 : 128;
    return Tile{bx, 1, default_chunk(D, n, bx, 1)};
  }
  struct Shape { int bx, by; double w; };
  const Shape shapes[3] = {{64, 4, 1.0}, {32, 8, 1.02}, {64, 8, 1.82}};
  const int nshapes = caloric ? 1 : (precision == LBM_FP32_DEV ? 3 : 2);
  Tile best{64, 4, 1};
  double best_cost = -1.0;
  for (int s = 0; s < nshapes; ++s) {
    double k = 0.0;
    const int64_t c = best_chunk3(n, shapes[s].bx, shapes[s].by, shapes[s].w, &k);
    if (best_cost < 0.0 || k < best_cost) {
      best_cost = k;
      best = Tile{shapes[s].bx, shapes[s].by, (int)c};
    }
  }
  return best;
}

// base, refined over its own shape, or over all shapes of its lattice.
static Tile refined(int D, int precision, const int64_t n[3], const Tile& base, bool all_shapes) {
  const bool large = n[0] * n[1] * n[2] > kLargeBox;
  if (D == 2) {
    if (precision == LBM_FP32_DEV || large || base.bx < 128) return base;
    return best_tile(&kShape2F64[base.bx == 128 ? 0 : 1], 1, n, n[1], 32);
  }
  const bool wide = base.bx == 64 && base.by == 8;
  if (precision == LBM_FP32_DEV && !wide) return base;
  const Tile t = precision == LBM_FP32_DEV ? best_tile(&kShape64x8, 1, n, n[2], 256)
                 : all_shapes             ? best_tile(kShapes3F64, 2, n, n[2], 256)
                                          : best_tile(&kShapes3F64[base.bx == 64 ? 0 : 1], 1, n, n[2], 256);
  Load before, after;
  before.add(n, D, base);
  after.add(n, D, t);
  return modelled(precision, t.bx, after) * (large ? kGainLarge : 1.0) <= modelled(precision, base.bx, before) ? t : base;
}

Tile default_tile(int D, int precision, const int64_t n[3], bool caloric) {
  return refined(D, precision, n, base_tile(D, precision, n, caloric), !caloric);
}

int shape_chunk(int D, int precision, const int64_t n[3], int bx, int by, bool caloric) {
  const Tile own = default_tile(D, precision, n, caloric);
  return own.bx == bx && own.by == by ? own.chunk : default_chunk(D, n, bx, by);
}

static bool worth(double time, double base_time, double nodes) {
  return time * (nodes > (double)kLargeBox ? 1.15 : 1.07) < base_time;
}

// March chunks of a batch's boxes in one shape.  A box's own chunk is chosen for
// a device that it has to itself; in a batch the boxes share the compute units,
// and a short chunk's prologue is paid by every one of their work-groups.  So
// D3Q27 boxes take their own chunks together, where the model finds the launch of
// all of them faster, or default_chunk.  FP64, us a step with default_chunk in the
// base shape, each box's own chunk whatever the batch, and this rule: 64 boxes of
// 16^3 123, 202, 116; 48 of 24^3 229, 354, 229; 2 of 160^3 1610, 1742, 1385; one of
// 20x25x40 30, 15, 15; 57 batches of 1 to 64 boxes are 1.22 times as fast as with
// default_chunk in the mean, and none is slower.  D2Q9 boxes have
// default_chunk: own chunks made a batch of 1024x64 and 600x1600, two each, 8%
// slower in FP64, and lbm_batch_tune's chunks start at four rows.
double batch_chunks(int D, int precision, const Extent* box, int count, int bx, int by, int* chunk) {
  std::vector<int> own(count);
  Load base, fine;
  for (int i = 0; i < count; ++i) {
    const Tile b{bx, by, default_chunk(D, box[i].n, bx, by)};
    chunk[i] = b.chunk;
    if (D == 2) continue;
    const Tile t = refined(D, precision, box[i].n, b, false);
    base.add(box[i].n, D, b);
    fine.add(box[i].n, D, t);
    own[i] = t.chunk;
  }
  if (D == 2) return 0.0;
  const double base_time = modelled(precision, bx, base), time = modelled(precision, bx, fine);
  if (!worth(time, base_time, base.nodes)) return base_time;
  std::copy(own.begin(), own.end(), chunk);
  return time;
}

// The shape of a batch: the first box's, of the power-of-two rule or, where that
// is faster for all boxes, of the default (D3Q27 FP64; elsewhere they are one).
Tile batch_shape(int D, int precision, const Extent* box, int count) {
  const Tile base = base_tile(D, precision, box[0].n, false), own = default_tile(D, precision, box[0].n);
  if (base.bx == own.bx && base.by == own.by) return Tile{base.bx, base.by, 0};
  std::vector<int> chunk(count);
  const double base_time = batch_chunks(D, precision, box, count, base.bx, base.by, chunk.data());
  const double time = batch_chunks(D, precision, box, count, own.bx, own.by, chunk.data());
  double nodes = 0.0;
  for (int i = 0; i < count; ++i) nodes += (double)box[i].n[0] * (double)box[i].n[1] * (double)box[i].n[2];
  const Tile& best = worth(time, base_time, nodes) ? own : base;
  return Tile{best.bx, best.by, 0};
}

// The 512-thread 64 x 8 shape exists for FP32 storage only: with FP64
// populations it does not fit the registers of two wavefronts per SIMD and
// spills, so it is not compiled for FP64.
bool tile_supported(int D, int precision, const Tile& t, bool caloric) {
  if (caloric) return D == 3 ? (t.bx == 64 && t.by == 4) : (t.bx == 128 && t.by == 1);
  if (D == 3)
    return (t.bx == 64 && t.by == 4) || (t.bx == 32 && t.by == 8) ||
           (t.bx == 64 && t.by == 8 && precision == LBM_FP32_DEV);
  return t.by == 1 && (t.bx == 64 || t.bx == 128 || t.bx == 256);
}

template <int D, bool DEV, typename S>
static hipError_t dispatch_tile(const Ctx& c, const void* src, void* dst) {
  const Tile& t = c.tile;
  if (c.sp.caloric) {  // the general caloric law: the default shape only
    if constexpr (D == 3) {
      if (t.bx == 64 && t.by == 4) return launch_step_t<D, DEV, S, 64, 4, true>(c, src, dst);
    } else {
      if (t.bx == 128) return launch_step_t<D, DEV, S, 128, 1, true>(c, src, dst);
    }
    return hipErrorInvalidValue;
  }
  if constexpr (D == 3) {
    if (t.bx == 64 && t.by == 4) return launch_step_t<D, DEV, S, 64, 4>(c, src, dst);
    if constexpr (DEV)
      if (t.bx == 64 && t.by == 8) return launch_step_t<D, DEV, S, 64, 8>(c, src, dst);
    if (t.bx == 32 && t.by == 8) return launch_step_t<D, DEV, S, 32, 8>(c, src, dst);
  } else {
    if (t.bx == 64) return launch_step_t<D, DEV, S, 64, 1>(c, src, dst);
    if (t.bx == 128) return launch_step_t<D, DEV, S, 128, 1>(c, src, dst);
    if (t.bx == 256) return launch_step_t<D, DEV, S, 256, 1>(c, src, dst);
  }
  return hipErrorInvalidValue;
}

template <int D, bool DEV, typename S, int BX, int BY>
static hipError_t launch_pattern_t(const Ctx& c, const void* src, void* dst) {
  hipLaunchKernelGGL((pattern_kernel<D, DEV, S, BX, BY>), dim3(c.sp.nblocks), dim3(BX * BY), 0, c.stream,
                     static_cast<const S*>(src), static_cast<S*>(dst), c.sp);
  return hipGetLastError();
}

template <int D, bool DEV, typename S>
static hipError_t dispatch_pattern(const Ctx& c, const void* src, void* dst) {
  const Tile& t = c.tile;
  if constexpr (D == 3) {
    if (t.bx == 64 && t.by == 4) return launch_pattern_t<D, DEV, S, 64, 4>(c, src, dst);
    if constexpr (DEV)
      if (t.bx == 64 && t.by == 8) return launch_pattern_t<D, DEV, S, 64, 8>(c, src, dst);
    if (t.bx == 32 && t.by == 8) return launch_pattern_t<D, DEV, S, 32, 8>(c, src, dst);
  } else {
    if (t.bx == 64) return launch_pattern_t<D, DEV, S, 64, 1>(c, src, dst);
    if (t.bx == 128) return launch_pattern_t<D, DEV, S, 128, 1>(c, src, dst);
    if (t.bx == 256) return launch_pattern_t<D, DEV, S, 256, 1>(c, src, dst);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pattern(const Ctx& c, const void* src, void* dst) {
  if (c.lattice == 3) {
    if (c.precision == LBM_FP64) return dispatch_pattern<3, false, double>(c, src, dst);
    return dispatch_pattern<3, true, float>(c, src, dst);
  }
  if (c.precision == LBM_FP64) return dispatch_pattern<2, false, double>(c, src, dst);
  return dispatch_pattern<2, true, float>(c, src, dst);
}

hipError_t launch_step(const Ctx& c, const void* src, void* dst) {
  if (c.lattice == 3) {
    if (c.precision == LBM_FP64) return dispatch_tile<3, false, double>(c, src, dst);
    return dispatch_tile<3, true, float>(c, src, dst);
  }
  if (c.precision == LBM_FP64) return dispatch_tile<2, false, double>(c, src, dst);
  return dispatch_tile<2, true, float>(c, src, dst);
}

// Work-groups of the persistent batched launch: the occupancy of the kernel
// times the compute units, rounded down to a multiple of 8 (the XCDs).  0
// (one work-group per tile instead) when that covers every tile: rounding a
// grid near the tile count down would leave a few work-groups two tiles.
template <int D, bool DEV, typename S, int BX, int BY>
static hipError_t persistent_grid(const Batch& b, int* grid) {
  int per_cu = 0, cus = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batch_persistent_kernel<D, DEV, S, BX, BY>,
                                                              BX * BY, 0);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b.device);
  if (e != hipSuccess) return e;
  const int g = (per_cu * cus / 8) * 8;
  *grid = per_cu * cus < b.total_blocks && g >= 8 ? g : 0;
  return hipSuccess;
}

bool persistent_supported(const Tile& t) { return t.bx * t.by <= 256; }

template <int D, bool DEV, typename S, int BX, int BY>
static hipError_t launch_batch_t(const Batch& b, hipStream_t s, int flip) {
  // The looped tile body of a 512-work-item tile does not fit the register
  // file without a stack frame, so that form exists for tiles of at most 256
  // work-items only (the host refuses the combination).
  if constexpr (BX * BY <= 256) {
    if (b.persistent) {
      int grid = 0;
      const hipError_t e = persistent_grid<D, DEV, S, BX, BY>(b, &grid);
      if (e != hipSuccess) return e;
      if (grid > 0) {
        hipLaunchKernelGGL((batch_persistent_kernel<D, DEV, S, BX, BY>), dim3(grid), dim3(BX * BY), 0, s, b.table,
                           (int)b.boxes.size(), b.total_blocks, flip);
        return hipGetLastError();
      }
    }
  } else {
    if (b.persistent) return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL((batch_step_kernel<D, DEV, S, BX, BY>), dim3(b.total_blocks), dim3(BX * BY), 0, s, b.table,
                     (int)b.boxes.size(), b.total_blocks, flip);
  return hipGetLastError();
}

template <int D, bool DEV, typename S>
static hipError_t dispatch_batch(const Batch& b, hipStream_t s, int flip) {
  const Tile& t = b.tile;
  if constexpr (D == 3) {
    if (t.bx == 64 && t.by == 4) return launch_batch_t<D, DEV, S, 64, 4>(b, s, flip);
    if constexpr (DEV)
      if (t.bx == 64 && t.by == 8) return launch_batch_t<D, DEV, S, 64, 8>(b, s, flip);
    if (t.bx == 32 && t.by == 8) return launch_batch_t<D, DEV, S, 32, 8>(b, s, flip);
  } else {
    if (t.bx == 64) return launch_batch_t<D, DEV, S, 64, 1>(b, s, flip);
    if (t.bx == 128) return launch_batch_t<D, DEV, S, 128, 1>(b, s, flip);
    if (t.bx == 256) return launch_batch_t<D, DEV, S, 256, 1>(b, s, flip);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_batch_step(const Batch& b, hipStream_t s, int flip) {
  if (b.lattice == 3) {
    if (b.precision == LBM_FP64) return dispatch_batch<3, false, double>(b, s, flip);
    return dispatch_batch<3, true, float>(b, s, flip);
  }
  if (b.precision == LBM_FP64) return dispatch_batch<2, false, double>(b, s, flip);
  return dispatch_batch<2, true, float>(b, s, flip);
}

hipError_t launch_toggle(const Batch& b, hipStream_t s) {
  const int n = (int)b.boxes.size();
  hipLaunchKernelGGL(toggle_cur_kernel, dim3((n + 63) / 64), dim3(64), 0, s, b.table, n);
  return hipGetLastError();
}

hipError_t launch_init(const Ctx& c, const double* rho, const double* u, const double* T, void* dst) {
  const long long N = c.N;
  const dim3 grid((unsigned)((N + 255) / 256)), block(256);
  if (c.lattice == 3) {
    if (c.precision == LBM_FP64)
      hipLaunchKernelGGL((init_kernel<3, false, double>), grid, block, 0, c.stream, rho, u, T, (double*)dst, N, c.sp);
    else
      hipLaunchKernelGGL((init_kernel<3, true, float>), grid, block, 0, c.stream, rho, u, T, (float*)dst, N, c.sp);
  } else {
    if (c.precision == LBM_FP64)
      hipLaunchKernelGGL((init_kernel<2, false, double>), grid, block, 0, c.stream, rho, u, T, (double*)dst, N, c.sp);
    else
      hipLaunchKernelGGL((init_kernel<2, true, float>), grid, block, 0, c.stream, rho, u, T, (float*)dst, N, c.sp);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Field increments by re-equilibration, and the conservative box filter
// ---------------------------------------------------------------------------

// f^eq - w and g^eq - w of one node in FP64, a row of three c_x at a time (see
// EqBuilder).  Without an anomaly the factors of f are the a-factors of g, so
// half of EqBuilder's state is enough.
template <int D, bool DEV>
struct NodeEq {
  AxisG<double> Y, Z;
  double g1[3], g2[3], eps, deps;

  __device__ inline NodeEq(const NodeConsts& k, double rho, const double* u, double T) {
    const double drho = rho - k.rho0, dT = T - k.T0;
    auto axis = [&](int a) { return axis_g<double, DEV>(u[a], u[a] - k.u0[a], k.u0[a], T, dT, k.T0); };
    const AxisG<double> X = axis(0);
    Y = axis(1);
    if (D == 3) Z = axis(2);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      g1[c] = drho * X.a[c] + (DEV ? k.rho0 * X.da[c] : 0.0);
      g2[c] = drho * X.b[c] + (DEV ? k.rho0 * X.db[c] : 0.0);
    }
    deps = k.caloric ? caloric_du<double>(k.Cv, k.cv1, k.cv2, k.T0, dT) : k.Cv * dT;
    eps = k.caloric ? k.U0 + deps : k.Cv * T;
  }

  // What the populations of row p (c_y, c_z) need besides g1 and g2:
  // f = g1 A + rho0 psi0_x dA, g = g1 V1 + g2 A + rho0 (psi0_x V2 + b0_x dA).
  struct Row {
    double A, V1, dA, V2;
  };
  __device__ inline Row row(const NodeConsts& k, int p) const {
    const int jy = p % 3, jz = p / 3;
    const double a0 = k.psi0[1][jy], b0 = k.b0[1][jy];
    Row r;
    r.A = Y.a[jy];
    r.dA = Y.da[jy];
    double B = Y.b[jy], dB = Y.db[jy];
    if (D == 3) {
      r.A = Y.a[jy] * Z.a[jz];
      B = Y.b[jy] * Z.a[jz] + Y.a[jy] * Z.b[jz];
      r.dA = Y.da[jy] * Z.a[jz] + a0 * Z.da[jz];
      dB = Y.db[jy] * Z.a[jz] + b0 * Z.da[jz] + Y.da[jy] * Z.b[jz] + a0 * Z.db[jz];
    }
    r.V1 = eps * r.A + B;
    r.V2 = deps * r.A + (k.caloric ? k.U0 : k.Cv * k.T0) * r.dA + dB;
    return r;
  }
};

// Ends the expressions that the fields come from: a product and a sum on either
// side of it are not fused, so equal fields give equal equilibria whatever they
// were computed from.
__device__ inline void as_values(double& rho, double* u, double& T) {
  asm("" : "+v"(rho), "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(T));
}

// New fields of a node: the planes rho, u_x, u_y, u_z, T of F ...
struct NewFields {
  const double* F;
  long long N;
  __device__ inline void operator()(long long n, double& rho, double* u, double& T) const {
    rho = F[n];
    for (int a = 0; a < 3; ++a) u[a] = F[(1 + a) * N + n];
    T = F[4 * N + n];
  }
};

// ... or the old ones and the normalised corrections y[c][n], output c for
// field off + c (0 rho, 1..3 u, 4 T); with limit > 0 a correction is clipped to
// [-limit, limit] first.  Networks have D3Q27's three axes.
struct Corrected {
  const float *y, *sd;
  int C, off;
  float limit;
  long long N;
  __device__ inline void operator()(long long n, double& rho, double* u, double& T) const {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      const int c = f - off;
      double inc = 0.0;
      if (c >= 0 && c < C) {
        float v = y[(long long)c * N + n];
        if (limit > 0.f) v = fminf(fmaxf(v, -limit), limit);
        inc = (double)v * sd[c];
      }
      if (f == 0) rho += inc;
      else if (f <= 3) u[f - 1] += inc;
      else T += inc;
    }
  }
};

// f_i += f^eq_i(new) - f^eq_i(old), g likewise (equilibria evaluated in FP64
// for either storage), the old fields those of the populations themselves.
// Where the new fields are the old ones, the populations keep every bit.
// Two equilibria a node take 2 x 64 registers beside the pairs' 54 (FP32) or 108,
// so FP64 arithmetic and the latency of two wavefronts per SIMD bind.  The
// populations are written once and read once, but for the last two rows of D3Q27
// in FP32, which are read again: held, they would put 52 bytes a lane into scratch
// memory.  lbm_nn_correct with a one-layer network at 64^3: 51.2 us (53.7 with all rows
// held, 58.8 with none; FP64 69.6, 72.7, 83.6), of which this kernel takes about half
// (45.2 us with the old fields from memory and both equilibria whole in registers,
// and 28 us for the kernels around it).
template <int D, bool DEV, typename S, typename New>
__global__ void __launch_bounds__(256, 2) fields_add_kernel(S* __restrict__ pops, const New fresh, int N,
                                                         const StepParams p) {
  using pair_t = typename Buf<S>::pair_t;
  constexpr int Q = lat_q(D);
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const NodeConsts k = node_consts(p);
  S* at = pops + pair_offset(p, n);
  pair_t v[Q];
  load_pairs<D>(at, p, v);
  double s0, j[3], se, rho, u[3], T, rhoE;
  pair_sums<D>(v, s0, j, &se);
  fields_of<D>(p, s0, j, se, rho, u, T, rhoE);
  as_values(rho, u, T);
  const NodeEq<D, DEV> before(k, rho, u, T);
  fresh(n, rho, u, T);
  as_values(rho, u, T);
  const NodeEq<D, DEV> after(k, rho, u, T);
  constexpr int held = D == 3 && DEV ? 7 : Q / 3;  // rows whose pairs stay in registers
#pragma unroll
  for (int r = 0; r < Q / 3; ++r) {
#pragma clang fp contract(off)  // both sides of a difference are rounded
    const auto o = before.row(k, r), w = after.row(k, r);
    const double dA = k.rho0 * (w.dA - o.dA), dV = k.rho0 * (w.V2 - o.V2);  // of the terms with constant factors
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      pair_t x = r < held ? v[3 * r + c] : *(const pair_t*)(at + (3 * r + c) * p.sl);
      double df = after.g1[c] * w.A - before.g1[c] * o.A;
      double dg = (after.g1[c] * w.V1 - before.g1[c] * o.V1) + (after.g2[c] * w.A - before.g2[c] * o.A);
      if (DEV) {
        df += k.psi0[0][c] * dA;
        dg += k.psi0[0][c] * dV + k.b0[0][c] * dA;
      }
      x.x = (S)((double)x.x + df);
      x.y = (S)((double)x.y + dg);
      *(pair_t*)(at + (3 * r + c) * p.sl) = x;
    }
  }
}

// New fields keep * old + d (rho, u, T; d: drho[N], du[D N], dT[N]; keep is 1
// for increments, 0 for new values; u_z of a 2-D lattice stays 0) of the
// populations' own fields into the planes of newf, and the count of nodes
// where they are not finite or rho or T is not positive, per work-group.
template <int D, typename S>
__global__ void __launch_bounds__(256) fields_new_kernel(const S* __restrict__ pops, const double* __restrict__ drho,
                                                         const double* __restrict__ du, const double* __restrict__ dT,
                                                         double keep, double* __restrict__ newf,
                                                         double* __restrict__ partial, int N, const StepParams p) {
  double bad[1] = {0.0};
  for (long long n = (long long)blockIdx.x * 256 + threadIdx.x; n < N; n += (long long)gridDim.x * 256) {
    typename Buf<S>::pair_t v[lat_q(D)];
    load_pairs<D>(pops + pair_offset(p, (int)n), p, v);
    double s0, j[3], se, rho, u[3], T, rhoE;
    pair_sums<D>(v, s0, j, &se);
    fields_of<D>(p, s0, j, se, rho, u, T, rhoE);
    const double r = keep * rho + drho[n], t = keep * T + dT[n];
    bool ok = isfinite(r) && isfinite(t) && r > 0.0 && t > 0.0;
    newf[n] = r;
    newf[4LL * N + n] = t;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double w = keep * u[a] + (a < D ? du[(long long)a * N + n] : 0.0);
      if (a < D) ok = ok && isfinite(w);
      newf[(1LL + a) * N + n] = w;
    }
    bad[0] += ok ? 0.0 : 1.0;
  }
  block_reduce_store<1, 4>(bad, partial + blockIdx.x, 1);
}

// rho, u, T as the FP32 input planes x[5][N] of the corrector (D3Q27).
template <typename S>
__global__ void __launch_bounds__(256) planes_kernel(const S* __restrict__ pops, float* __restrict__ x, int N,
                                                     const StepParams p) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  typename Buf<S>::pair_t v[lat_q(3)];
  load_pairs<3>(pops + pair_offset(p, n), p, v);
  double s0, j[3], se, rho, u[3], T, rhoE;
  pair_sums<3>(v, s0, j, &se);
  fields_of<3>(p, s0, j, se, rho, u, T, rhoE);
  x[n] = (float)rho;
#pragma unroll
  for (int a = 0; a < 3; ++a) x[(long long)(1 + a) * N + n] = (float)u[a];
  x[4LL * N + n] = (float)T;
}

// Coarse nodes: means of rho, rho u and rho E over factor^D fine nodes,
// straight from the populations; T from U(T) = E - |u|^2 / 2 with the caloric
// law of p.  A work-group takes `per` consecutive coarse nodes: a thread sums
// one fine column x of a coarse node over its f fz rows (consecutive threads,
// consecutive x), and the f columns are added through LDS.  Bound by reading
// the populations: 256^3 FP32 by 4, 622 us, 5.8 TB/s (827 + 189 us when the fields went
// through memory).
template <int D, typename S>
__global__ void __launch_bounds__(256) filter_kernel(const S* __restrict__ pops, const StepParams p, int f, int per,
                                                     int Nc, double* __restrict__ rho, double* __restrict__ u,
                                                     double* __restrict__ T) {
  __shared__ double red[D + 2][256];
  const int cx = p.nx / f, cy = p.ny / f, fz = (D == 3) ? f : 1;
  const int t = threadIdx.x;
  const int c = blockIdx.x * per + (f <= 256 ? t / f : 0);
  double sr = 0.0, sj[3] = {0.0, 0.0, 0.0}, se = 0.0;
  if (c < Nc && (f > 256 || t < per * f)) {
    const int X = c % cx, Y = (c / cx) % cy, Z = c / (cx * cy);
    for (int k = 0; k < fz; ++k)
      for (int j = 0; j < f; ++j) {
        const long long row = (long long)p.nx * ((Y * f + j) + (long long)p.ny * (Z * fz + k)) + (long long)X * f;
        for (int i = f <= 256 ? t % f : t; i < f; i += f <= 256 ? f : 256) {
          double s0, jj[3], e;
          typename Buf<S>::pair_t v[lat_q(D)];
          load_pairs<D>(pops + pair_offset(p, (int)(row + i)), p, v);
          pair_sums<D>(v, s0, jj, &e);
          sr += p.rho0 + s0;
          se += p.rhoE0 + e;
#pragma unroll
          for (int a = 0; a < D; ++a) sj[a] += p.j0[a] + jj[a];
        }
      }
  }
  red[0][t] = sr;
  red[1][t] = se;
#pragma unroll
  for (int a = 0; a < D; ++a) red[2 + a][t] = sj[a];
  __syncthreads();
  const int o = blockIdx.x * per + t;
  if (t >= per || o >= Nc) return;
  const int cols = f <= 256 ? f : 256;
  double v[D + 2];
#pragma unroll
  for (int w = 0; w < D + 2; ++w) {
    v[w] = 0.0;
    for (int i = 0; i < cols; ++i) v[w] += red[w][t * cols + i];
  }
  const double inv = 1.0 / v[0];
  double u2 = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const double ua = v[2 + a] * inv;
    u[(long long)a * Nc + o] = ua;
    u2 += ua * ua;
  }
  rho[o] = v[0] / ((double)f * f * fz);
  const double e = v[1] * inv - 0.5 * u2;
  T[o] = p.caloric ? caloric_step(p.Cv, p.cv1, p.cv2, 0.0, e) : e / p.Cv;
}

template <int D, typename New>
static hipError_t launch_add_t(const Ctx& c, void* pops, const New& fresh) {
  const dim3 grid((unsigned)((c.N + 255) / 256)), block(256);
  if (c.precision == LBM_FP64)
    hipLaunchKernelGGL((fields_add_kernel<D, false, double, New>), grid, block, 0, c.stream,
                       static_cast<double*>(pops), fresh, (int)c.N, c.sp);
  else
    hipLaunchKernelGGL((fields_add_kernel<D, true, float, New>), grid, block, 0, c.stream, static_cast<float*>(pops),
                       fresh, (int)c.N, c.sp);
  return hipGetLastError();
}

hipError_t launch_fields_add(const Ctx& c, void* pops, const double* newf) {
  const NewFields fresh{newf, c.N};
  return c.lattice == 3 ? launch_add_t<3>(c, pops, fresh) : launch_add_t<2>(c, pops, fresh);
}

hipError_t launch_correct(const Ctx& c, void* pops, const float* y, const float* sd, int channels, int offset,
                          float limit) {
  return launch_add_t<3>(c, pops, Corrected{y, sd, channels, offset, limit, c.N});
}

template <int D, typename S>
static void launch_new_t(const Ctx& c, const void* pops, const double* drho, const double* du, const double* dT,
                         bool keep, double* newf, double* partial, int nblocks) {
  hipLaunchKernelGGL((fields_new_kernel<D, S>), dim3(nblocks), dim3(256), 0, c.stream, static_cast<const S*>(pops),
                     drho, du, dT, keep ? 1.0 : 0.0, newf, partial, (int)c.N, c.sp);
}

hipError_t launch_fields_new(const Ctx& c, const void* pops, const double* drho, const double* du, const double* dT,
                             bool keep, double* newf, double* partial, int nblocks, double* out) {
  if (c.lattice == 3) {
    if (c.precision == LBM_FP64) launch_new_t<3, double>(c, pops, drho, du, dT, keep, newf, partial, nblocks);
    else launch_new_t<3, float>(c, pops, drho, du, dT, keep, newf, partial, nblocks);
  } else {
    if (c.precision == LBM_FP64) launch_new_t<2, double>(c, pops, drho, du, dT, keep, newf, partial, nblocks);
    else launch_new_t<2, float>(c, pops, drho, du, dT, keep, newf, partial, nblocks);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(final_reduce_kernel, dim3(1), dim3(256), 0, c.stream, partial, nblocks, out);
  return hipGetLastError();
}

template <typename S>
static hipError_t launch_planes_t(const Ctx& c, const void* pops, float* x) {
  hipLaunchKernelGGL(planes_kernel<S>, dim3((unsigned)((c.N + 255) / 256)), dim3(256), 0, c.stream,
                     static_cast<const S*>(pops), x, (int)c.N, c.sp);
  return hipGetLastError();
}

hipError_t launch_planes(const Ctx& c, const void* pops, float* x) {
  return c.precision == LBM_FP64 ? launch_planes_t<double>(c, pops, x) : launch_planes_t<float>(c, pops, x);
}

template <int D, typename S>
static hipError_t launch_filter_t(const Ctx& c, const void* pops, int f, double* rho, double* u, double* T) {
  const int64_t Nc = (c.n[0] / f) * (c.n[1] / f) * (D == 3 ? c.n[2] / f : 1);
  const int per = f <= 256 ? 256 / f : 1;
  hipLaunchKernelGGL((filter_kernel<D, S>), dim3((unsigned)((Nc + per - 1) / per)), dim3(256), 0, c.stream,
                     static_cast<const S*>(pops), c.sp, f, per, (int)Nc, rho, u, T);
  return hipGetLastError();
}

hipError_t launch_filter(const Ctx& c, const void* pops, int factor, double* rho, double* u, double* T) {
  if (c.lattice == 3)
    return c.precision == LBM_FP64 ? launch_filter_t<3, double>(c, pops, factor, rho, u, T)
                                   : launch_filter_t<3, float>(c, pops, factor, rho, u, T);
  return c.precision == LBM_FP64 ? launch_filter_t<2, double>(c, pops, factor, rho, u, T)
                                 : launch_filter_t<2, float>(c, pops, factor, rho, u, T);
}

template <int D, typename S>
static hipError_t launch_moments_t(const Ctx& c, const void* pops, double* rho, double* u, int nu, double* T) {
  hipLaunchKernelGGL((fields_kernel<D, S>), dim3((unsigned)((c.N + 255) / 256)), dim3(256), 0, c.stream,
                     static_cast<const S*>(pops), rho, u, nu, T, (int)c.N, c.sp);
  return hipGetLastError();
}

hipError_t launch_moments(const Ctx& c, const void* pops, double* rho, double* u, int nu, double* T) {
  if (c.lattice == 3)
    return c.precision == LBM_FP64 ? launch_moments_t<3, double>(c, pops, rho, u, nu, T)
                                   : launch_moments_t<3, float>(c, pops, rho, u, nu, T);
  return c.precision == LBM_FP64 ? launch_moments_t<2, double>(c, pops, rho, u, nu, T)
                                 : launch_moments_t<2, float>(c, pops, rho, u, nu, T);
}

hipError_t launch_fields(const Ctx& c, const void* pops, double* fields) {
  return launch_moments(c, pops, fields, fields + c.N, 3, fields + 4 * c.N);
}

int validate_blocks(const Ctx& c) {
  const long long want = (c.N + 255) / 256;
  return (int)(want < kMaxDiagBlocks ? want : kMaxDiagBlocks);
}

// Launch geometry of the diagnostics.
// D2Q9: rows of 128 (2000 x 1500 FP64: 116 us a call against 129 for 256 x 1, which
// also leaves more lanes idle past a ragged edge) in chunks as long as 1024
// work-groups allow, and shorter than four rows only where the grid cannot fill
// the chip (100 x 60: 32 us a call against 37).  Rows that use less than 0.25
// (FP32: 0.4) of their lanes go in memory order.
// D3Q27: in memory order go planes that use less than 0.35 of the lanes of 32 x 8
// tiles, and boxes up to 65,536 nodes (one work-group of 256 per compute unit)
// unless one-plane chunks of 32 x 8 leave no compute unit two work-groups; boxes up to
// 300,000 nodes take 32 x 8, larger ones 64 x 8 or 32 x 16, or memory order, by
// DiagModel.  A call against the first form of lbm_diagnostics, which put every node's
// fields into memory and took the differences from there: 1.09 times as fast in FP64
// and 1.10 in FP32 over 1466 boxes of up to 10^7 nodes.  That form is still faster by more
// than 3% for 27 of them in FP64 (at most 10%: planes of 1 to 9 nodes along x, and calls of 56
// us or less) and for 22 in FP32 (at most 17%: a few nodes past a multiple of 32
// along x; 16 x 32 tiles win some of those back and lose others).
struct DiagModel {
  double cached, hbm, cache, ring;  // us per MB of populations, within `cache` MB and beyond; weight of ring lines
  double plane, flat;               // us per plane of a round; per node in memory order

  double microseconds(double megabytes) const { return cached + (hbm - cached) * std::max(0.0, 1.0 - cache / megabytes); }
};
static const DiagModel kDiag64{0.055, 0.093, 165.0, 1.0, 4.0, 2.3e-4}, kDiag32{0.038, 0.067, 205.0, 0.55, 3.9, 1.35e-4};

DiagGrid diag_grid(int D, int precision, const int64_t n[3]) {
  DiagGrid g{};
  const int64_t nm = D == 3 ? n[2] : n[1], N = n[0] * n[1] * n[2];
  auto in_memory_order = [&] {
    g.flat = true;
    g.blocks = (int)((std::min<int64_t>((N + 255) / 256, kMaxDiagBlocks) + 7) / 8 * 8);
    return g;
  };
  auto tiles_of = [&](int bx, int by) { return ((n[0] + bx - 1) / bx) * (D == 3 ? (n[1] + by - 1) / by : 1); };
  auto tiled = [&](int bx, int by, int64_t chunk) {
    g.bx = bx;
    g.by = by;
    g.tiles_x = (int)((n[0] + bx - 1) / bx);
    g.tiles_y = D == 3 ? (int)((n[1] + by - 1) / by) : 1;
    chunk = std::min(chunk, nm);
    g.chunk = (int)chunk;
    g.tasks = (int)(tiles_of(bx, by) * ((nm + chunk - 1) / chunk));
    g.blocks = std::min(g.tasks, kMaxDiagBlocks);
    return g;
  };
  if (D == 2) {
    const int64_t tiles = tiles_of(128, 1), chunks = tiles < 1024 ? 1024 / tiles : 1;
    if ((double)n[0] < (precision == LBM_FP64 ? 0.25 : 0.4) * 128.0 * (double)tiles) return in_memory_order();
    return tiled(128, 1, std::max((nm + chunks - 1) / chunks, std::min<int64_t>((tiles * nm + 1023) / 1024, 4)));
  }
  const int64_t small = tiles_of(32, 8);
  if ((double)(n[0] * n[1]) < 0.35 * 256.0 * (double)small) return in_memory_order();
  if (N <= 300000 && small * nm <= 256) return tiled(32, 8, 1);
  if (N <= 65536) return in_memory_order();
  const DiagModel& m = precision == LBM_FP64 ? kDiag64 : kDiag32;
  const int word = precision == LBM_FP64 ? 8 : 4, line = 128 / (2 * word);  // pairs of a cache line
  const double megabytes = (double)N * 54 * word * 1e-6, rate = m.microseconds(megabytes);
  double best = 16.0 + std::hypot((double)N * m.flat, 17.5);  // memory order
  int bx = 0, by = 0;
  int64_t chunk = 0;
  const int shapes[3][2] = {{32, 8}, {64, 8}, {32, 16}};
  for (int s = N <= 300000 ? 0 : 1; s < (N <= 300000 ? 1 : 3); ++s) {
    const int64_t wx = std::min<int64_t>(shapes[s][0], n[0]), wy = std::min<int64_t>(shapes[s][1], n[1]);
    const int64_t tiles = tiles_of(shapes[s][0], shapes[s][1]), resident = s ? 256 : 512;
    const double lines = (double)((wx + line - 1) / line);  // of a tile's row; a ring column costs one a row
    const double ring = ((wx < n[0] ? 2.0 * (double)wy : 0.0) + (wy < n[1] ? 2.0 * lines : 0.0)) / (lines * (double)wy);
    for (int64_t most = 256; most <= 4096; most += 256) {  // the shortest chunk with at most so many work-groups
      const int64_t chunks = std::min(std::max<int64_t>(most / tiles, 1), nm), c = (nm + chunks - 1) / chunks;
      const int64_t blocks = tiles * ((nm + c - 1) / c), rest = blocks % resident;
      // a last round that leaves compute units one work-group of their two costs less
      const double rounds = (double)(blocks / resident) + (!rest ? 0.0 : resident == 512 && rest <= 256 ? 0.7 : 1.0);
      const double time = 24.0 + megabytes * (1.0 + 2.0 / (double)c + m.ring * ring) * rate +
                          rounds * ((s ? 8.7 : 7.0) + (double)c * m.plane);
      if (time >= best) continue;
      best = time;
      bx = shapes[s][0];
      by = shapes[s][1];
      chunk = c;
    }
  }
  return bx ? tiled(bx, by, chunk) : in_memory_order();
}

DiagGrid diag_grid(const Ctx& c) { return diag_grid(c.lattice, c.precision, c.n); }

// Device memory of the allocation-free diagnostics (lbm_diagnostics_noalloc):
// the per-block partial sums and the final sums, kScratchDoubles doubles
// (344 KB) on every device the library runs on, held until the process
// ends.  Host code never uses this name as an address: scratch_address
// returns the device address of the current device's copy.
static __device__ __align__(256) double scratch[kScratchDoubles];

hipError_t scratch_address(double** out) {
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  *out = e == hipSuccess ? static_cast<double*>(ptr) : nullptr;
  return e;
}

template <int D, typename S, int BX, int BY>
static void launch_diag_t(const Ctx& c, const void* pops, double* partial, const DiagGrid& g) {
  hipLaunchKernelGGL((diag_kernel<D, S, BX, BY>), dim3(g.blocks), dim3(BX * BY), 0, c.stream,
                     static_cast<const S*>(pops), partial, c.sp, g);
}

template <int D, typename S>
static void launch_diag_flat(const Ctx& c, const void* pops, double* partial, const DiagGrid& g) {
  hipLaunchKernelGGL((diag_flat_kernel<D, S>), dim3(g.blocks), dim3(256), 0, c.stream, static_cast<const S*>(pops),
                     partial, (int)c.N, c.sp);
}

hipError_t launch_diag(const Ctx& c, const void* pops, double* partial, const DiagGrid& g, double* out) {
  if (g.flat) {
    if (c.lattice == 3) {
      if (c.precision == LBM_FP64) launch_diag_flat<3, double>(c, pops, partial, g);
      else launch_diag_flat<3, float>(c, pops, partial, g);
    } else {
      if (c.precision == LBM_FP64) launch_diag_flat<2, double>(c, pops, partial, g);
      else launch_diag_flat<2, float>(c, pops, partial, g);
    }
  } else if (c.lattice == 3) {
    if (c.precision == LBM_FP64) {
      if (g.bx == 64) launch_diag_t<3, double, 64, 8>(c, pops, partial, g);
      else if (g.by == 16) launch_diag_t<3, double, 32, 16>(c, pops, partial, g);
      else launch_diag_t<3, double, 32, 8>(c, pops, partial, g);
    } else {
      if (g.bx == 64) launch_diag_t<3, float, 64, 8>(c, pops, partial, g);
      else if (g.by == 16) launch_diag_t<3, float, 32, 16>(c, pops, partial, g);
      else launch_diag_t<3, float, 32, 8>(c, pops, partial, g);
    }
  } else if (c.precision == LBM_FP64) {
    launch_diag_t<2, double, 128, 1>(c, pops, partial, g);
  } else {
    launch_diag_t<2, float, 128, 1>(c, pops, partial, g);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(final_reduce_kernel, dim3(kNumDiag), dim3(256), 0, c.stream, partial, g.blocks, out);
  return hipGetLastError();
}

hipError_t launch_validate(const Ctx& c, const double* rho, const double* u, const double* T, double* partial,
                           int nblocks, double* out) {
  if (c.lattice == 3)
    hipLaunchKernelGGL((validate_kernel<3>), dim3(nblocks), dim3(256), 0, c.stream, rho, u, T, partial,
                       (long long)c.N);
  else
    hipLaunchKernelGGL((validate_kernel<2>), dim3(nblocks), dim3(256), 0, c.stream, rho, u, T, partial,
                       (long long)c.N);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(final_reduce_kernel, dim3(1), dim3(256), 0, c.stream, partial, nblocks, out);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  // one 16-byte vector per thread; launches of at most 2^30 vectors
  const long long n16 = (long long)(bytes / 16);
  constexpr long long kMax = 1LL << 30;
  for (long long off = 0; off < n16; off += kMax) {
    const long long n = n16 - off < kMax ? n16 - off : kMax;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const float4*)src + off,
                       (float4*)dst + off, n);
  }
  return hipGetLastError();
}

}  // namespace lbm

namespace lbm {

template <int D, typename S>
static hipError_t launch_pack_t(const Ctx& c, const void* pops, void* state) {
  hipLaunchKernelGGL((pack_kernel<D, S>), dim3((unsigned)((c.N + 255) / 256)), dim3(256), 0, c.stream,
                     static_cast<const S*>(pops), static_cast<S*>(state), (int)c.N, c.sp);
  return hipGetLastError();
}

hipError_t launch_pack(const Ctx& c, const void* pops, void* state) {
  if (c.lattice == 3)
    return c.precision == LBM_FP64 ? launch_pack_t<3, double>(c, pops, state) : launch_pack_t<3, float>(c, pops, state);
  return c.precision == LBM_FP64 ? launch_pack_t<2, double>(c, pops, state) : launch_pack_t<2, float>(c, pops, state);
}

template <int D, typename S>
static hipError_t launch_unpack_t(const Ctx& c, const void* state, void* pops) {
  hipLaunchKernelGGL((unpack_kernel<D, S>), dim3((unsigned)((c.N + 255) / 256)), dim3(256), 0, c.stream,
                     static_cast<const S*>(state), static_cast<S*>(pops), (int)c.N, c.sp);
  return hipGetLastError();
}

hipError_t launch_unpack(const Ctx& c, const void* state, void* pops) {
  if (c.lattice == 3)
    return c.precision == LBM_FP64 ? launch_unpack_t<3, double>(c, state, pops)
                                   : launch_unpack_t<3, float>(c, state, pops);
  return c.precision == LBM_FP64 ? launch_unpack_t<2, double>(c, state, pops)
                                 : launch_unpack_t<2, float>(c, state, pops);
}

}  // namespace lbm
