// Finite-difference time step of the damped acoustic wave equation:
//   next = [2 m cur - (m - a) prev + dt^2 L cur] / (m + a),   a = eta dt / 2,
// L the 8th-order Laplacian with the field taken as zero outside the grid.
// Forward and adjoint sweeps use the same step (the operator is symmetric).
//
// Three kernels share one per-cell arithmetic (axis_sum / cell_update), so their
// results are bitwise identical:
//   k_stencil_simple  one thread per cell, neighbours from global memory
//                     (small and thin grids, large 2D grids; the reference for
//                     the others)
//   k_stencil2d_steps 2D: up to four steps per launch
//   k_stencil3d_tiled 3D: a TX x TY column tile per workgroup marches through
//                     a z-chunk; the planes z .. z+4 (with a 4-cell x/y halo)
//                     sit in a ring of LDS planes, and the z neighbours in a
//                     9-deep register queue per column.  Every access is a
//                     16-byte vector of consecutive x cells.
#include <algorithm>
#include <type_traits>

#include "step_common.h"

namespace rtm {

// The fused multiply-adds of the step are spelled out: left to the compiler,
// which product of a sum is contracted depends on the code around it, and the
// kernels that share this arithmetic would differ in the last bit.
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}

// c1 (p1 + m1) + c2 (p2 + m2) + c3 (p3 + m3) + c4 (p4 + m4), fixed order
template <typename T>
__device__ __forceinline__ T axis_sum(const StepArgs<T> &a, T p1, T m1, T p2, T m2, T p3,
                                      T m3, T p4, T m4) {
  T s = fma_t(a.c1, p1 + m1, a.c2 * (p2 + m2));
  s = fma_t(a.c3, p3 + m3, s);
  return fma_t(a.c4, p4 + m4, s);
}

// n / d; for FP32 a hardware reciprocal refined by one Newton step and one
// residual correction (Markstein's scheme), within an ulp of the IEEE
// quotient for the normal, well-scaled operands of the update (slowness
// squared plus damping), in fewer instructions than the IEEE sequence
template <typename T>
__device__ __forceinline__ T quot(T n, T d) {
  return n / d;
}
template <>
__device__ __forceinline__ float quot<float>(float n, float d) {
  float r = __builtin_amdgcn_rcpf(d);
  r = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
  const float q = n * r;
  return __builtin_fmaf(__builtin_fmaf(-d, q, n), r, q);
}

template <typename T>
__device__ __forceinline__ T cell_update(const StepArgs<T> &a, T u, T up, T m, T lap, T damp) {
  const T v = fma_t(u, T(2) * m, -((m - damp) * up));
  return quot(fma_t(a.dt2, lap, v), m + damp);
}

// The folded injection: the sum of weight x value over the entries of cell
// (z, y, x), in the order of k_inject; false where the cell has none.
template <typename T>
__device__ __forceinline__ bool inj_sum(const InjMap<T> &j, int z, int y, int x, T &acc) {
  acc = T(0);
  if (z < j.z0 || z >= j.z1 || y < j.y0 || y >= j.y1 || x < j.x0 || x >= j.x1) return false;
  const int v = j.map[((int64_t)(z - j.z0) * (j.y1 - j.y0) + (y - j.y0)) * (j.x1 - j.x0) + x - j.x0];
  if (v >= 0) {
    acc += j.vals[v];
  } else if (v < -1) {
    const int c = -2 - v;
    for (int e = j.ioff[c]; e < j.ioff[c + 1]; ++e) acc = fma_t(j.iw[e], j.vals[j.ipt[e]], acc);
  }
  return v != -1;
}
// what the injection adds to the new level (`mpa` = m + damping)
template <typename T>
__device__ __forceinline__ T inj_term(const StepArgs<T> &a, T acc, T mpa) {
  return a.dt2 * acc / mpa;
}

// ---------------------------------------------------------------------------
// one thread per cell
// ---------------------------------------------------------------------------
template <typename T, int NDIM>
__global__ __launch_bounds__(256) void k_stencil_simple(StepArgs<T> a, InjMap<T> inj) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;  // N < 2^31
  if (i >= (uint32_t)a.N) return;
  const uint32_t zy = i / (uint32_t)a.nx;
  const int x = (int)(i - zy * (uint32_t)a.nx);
  const int z = (int)(zy / (uint32_t)a.ny);
  const int y = (int)(zy - (uint32_t)z * (uint32_t)a.ny);
  const T *u = a.cur;
  auto U = [&](int zz, int yy, int xx) -> T {
    return (zz >= 0 && zz < a.nz && yy >= 0 && yy < a.ny && xx >= 0 && xx < a.nx)
               ? u[((int64_t)zz * a.ny + yy) * a.nx + xx]
               : T(0);
  };
  const T c = u[i];
  const T lz = axis_sum(a, U(z + 1, y, x), U(z - 1, y, x), U(z + 2, y, x), U(z - 2, y, x),
                        U(z + 3, y, x), U(z - 3, y, x), U(z + 4, y, x), U(z - 4, y, x));
  const T lx = axis_sum(a, U(z, y, x + 1), U(z, y, x - 1), U(z, y, x + 2), U(z, y, x - 2),
                        U(z, y, x + 3), U(z, y, x - 3), U(z, y, x + 4), U(z, y, x - 4));
  T lap;
  if constexpr (NDIM == 3) {
    const T ly = axis_sum(a, U(z, y + 1, x), U(z, y - 1, x), U(z, y + 2, x), U(z, y - 2, x),
                          U(z, y + 3, x), U(z, y - 3, x), U(z, y + 4, x), U(z, y - 4, x));
    lap = (fma_t(a.cc, c, lz) + ly) + lx;
  } else {
    lap = fma_t(a.cc, c, lz) + lx;
  }
  const T damp = sponge_a(a, z, y, x);
  T v = cell_update(a, c, a.prev[i], a.m[i], lap, damp);
  T acc;
  if (inj.map && inj_sum(inj, z, y, x, acc)) v += inj_term(a, acc, a.m[i] + damp);
  a.next[i] = v;
}

// ---------------------------------------------------------------------------
// 2D: several steps per launch
// ---------------------------------------------------------------------------
// A workgroup (NW waves) advances a tile of TX x TZ cells by up to kSteps2D
// steps: the tile with a halo of four cells per step (64 x EZ cells) is loaded
// once, each step computes the cells that the remaining ones still need (the
// region shrinks by four on each side), and every level's tile goes to the
// ring.  A lane owns one x column of rows w, w + NW, ... (wave w): its cells'
// two levels, model and damping stay in registers, the current level sits in
// LDS for the neighbours, double buffered, one barrier per step.  Cells
// outside the grid stay zero.  The arithmetic per cell is k_stencil_simple's,
// and the halo's cells get the same injection as their owners give them, so
// levels are the same bit for bit.
// Bound: a 2D step's levels stay in the caches; a launch per step is bound by
// the launch and one chain of loads, this kernel by the chains of its steps
// (16 waves per workgroup: the more rows in flight, the better) and, on large
// grids, by the halo's arithmetic (2.6 times the tile's).  us per step, one
// launch per step -> four steps per launch: 221 x 221 3.4 -> 1.9 (FP64 3.5 ->
// 2.3), 301 x 901 4.8 -> 3.6 (6.1 -> 5.4), 600 x 1000 7.3 -> 5.4 (8.7 -> 7.9),
// 1200 x 2000 20.5 -> 17.4 (24.3 -> 24.9: FP64 keeps the launch per step there).
constexpr int kSteps2D = kMaxSteps2D;

// The halo is loaded and mostly computed whether one step follows or four, so
// the fewer steps a launch has (short probe blocks, the end of one), the
// smaller the grid up to which it is worth it.  us per step, a thread per cell
// against this kernel:
//   1 step   221 x 221 7.0 / 5.9 (FP64 7.0 / 6.5), 300 x 500 7.0 / 7.6
//            (7.9 / 10.2), 1200 x 2000 23 / 44
//   2 steps  600 x 1000 11.1 / 9.1 (11.5 / 12.1; 400 x 600 8.4 / 7.2),
//            1500 x 1300 20 / 23 (27 / 29)
//   3 steps  1200 x 2000 23 / 22 (1500 x 1300 27 / 24), 2400 x 4000 73 / 79
//   4 steps  2400 x 4000 73 / 69, 4000 x 8000 232 / 231, 8000 x 16000 921 / 937
template <typename T>
bool stencil2d_multi(int64_t N, int nsteps) {
  static const int64_t below[2][kSteps2D] = {{64000, 1000000, 4000000, 16000000},
                                             {64000, 250000, 2000000, 2000000}};
  return nsteps >= 1 && nsteps <= kSteps2D && N < below[sizeof(T) == 8][nsteps - 1];
}
template bool stencil2d_multi<float>(int64_t, int);
template bool stencil2d_multi<double>(int64_t, int);
template <typename T, int TZ, int NW>
__global__ __launch_bounds__(64 * NW) void k_stencil2d_steps(StepArgs<T> a, InjMap<T> inj,
                                                         int64_t vstride, T *ring, int64_t ld,
                                                         int R, int s, int nsteps, int ntx) {
  constexpr int H = 4 * kSteps2D;
  constexpr int TX = 64 - 2 * H;
  constexpr int EZ = TZ + 2 * H;
  constexpr int NR = EZ / NW;
  static_assert(EZ % NW == 0, "whole rows per wave");
  __shared__ T lds[2][EZ * 64 + 8];  // 4 cells of slack at both ends
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const int x = (b % ntx) * TX - H + lane;
  const int zt = (b / ntx) * TZ - H;
  auto level = [&](int j) { return ring + (int64_t)((j + 1) % R) * ld; };
  const T *c0 = level(s), *p0 = level(s - 1);
  T cu[NR], pv[NR], mm[NR], damp[NR];
  int iv[NR];  // the folded injection's map entry
  bool in[NR], any[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const int r = w + NW * k, z = zt + r;
    in[k] = x >= 0 && x < a.nx && z >= 0 && z < a.nz;
    const int64_t i = in[k] ? (int64_t)z * a.nx + x : 0;
    cu[k] = in[k] ? c0[i] : T(0);
    pv[k] = in[k] ? p0[i] : T(0);
    mm[k] = in[k] ? a.m[i] : T(1);
    damp[k] = sponge_a(a, z, 0, x);
    iv[k] = -1;
    if (inj.map && in[k] && z >= inj.z0 && z < inj.z1 && x >= inj.x0 && x < inj.x1)
      iv[k] = inj.map[(int64_t)(z - inj.z0) * (inj.x1 - inj.x0) + x - inj.x0];
    any[k] = __any(iv[k] != -1);
    lds[0][4 + r * 64 + lane] = cu[k];
  }
  __syncthreads();
  const T *vals = inj.vals;
  for (int j = 0; j < nsteps; ++j) {
    const int e = 4 * (j + 1);  // cells the region has shrunk to on each side
    const T *L = &lds[j & 1][4];
    T *Ln = &lds[(j + 1) & 1][4];
    T *out = level(s + 1 + j);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int r = w + NW * k, z = zt + r;
      if (r < e || r >= EZ - e) continue;  // wave-uniform
      T acc = T(0);
      const int v = iv[k];
      if (any[k]) {  // wave-uniform
        if (v >= 0) {
          acc += vals[v];
        } else if (v < -1) {
          for (int q = inj.ioff[-2 - v]; q < inj.ioff[-1 - v]; ++q)
            acc = fma_t(inj.iw[q], vals[inj.ipt[q]], acc);
        }
      }
      const T *row = L + r * 64 + lane;
      const T c = cu[k];
      const T lz = axis_sum(a, row[64], row[-64], row[128], row[-128], row[192], row[-192],
                            row[256], row[-256]);
      const T lx = axis_sum(a, row[1], row[-1], row[2], row[-2], row[3], row[-3], row[4], row[-4]);
      const T lap = fma_t(a.cc, c, lz) + lx;
      T nv = cell_update(a, c, pv[k], mm[k], lap, damp[k]);
      if (any[k] && v != -1) nv += inj_term(a, acc, mm[k] + damp[k]);
      nv = in[k] ? nv : T(0);
      pv[k] = c;
      cu[k] = nv;
      Ln[r * 64 + lane] = nv;
      if (in[k] && r >= H && r < H + TZ && lane >= H && lane < H + TX)
        out[(int64_t)z * a.nx + x] = nv;
    }
    vals += vstride;
    __syncthreads();
  }
}

// steps s .. s + nsteps - 1 of a 2D sweep (nsteps <= kSteps2D <= R - 2); inj:
// the folded injection of step s, whose values advance by vstride per step
template <typename T>
hipError_t launch_stencil2d(const StepArgs<T> &a, const InjMap<T> &inj, int64_t vstride, T *ring,
                            int64_t ld, int R, int s, int nsteps, hipStream_t st) {
  constexpr int TX = 64 - 8 * kSteps2D;
  const int ntx = (a.nx + TX - 1) / TX;
  auto go = [&](auto kern, int tz, int nw) {
    hipLaunchKernelGGL(kern, dim3(ntx * ((a.nz + tz - 1) / tz)), dim3(64 * nw), 0, st, a, inj,
                       vstride, ring, ld, R, s, nsteps, ntx);
  };
  // tiles of 16 rows: 8 need more halo, 32 leave CUs idle; FP64, whose halo
  // arithmetic weighs more, 32 once those fill the chip (301 x 901: 5.4
  // against 5.9)
  if (sizeof(T) == 8 && ntx * ((a.nz + 31) / 32) >= 256) go(k_stencil2d_steps<T, 32, 16>, 32, 16);
  else go(k_stencil2d_steps<T, 16, 16>, 16, 16);
  return hipGetLastError();
}
template hipError_t launch_stencil2d<float>(const StepArgs<float> &, const InjMap<float> &, int64_t,
                                            float *, int64_t, int, int, int, hipStream_t);
template hipError_t launch_stencil2d<double>(const StepArgs<double> &, const InjMap<double> &,
                                             int64_t, double *, int64_t, int, int, int,
                                             hipStream_t);

// ---------------------------------------------------------------------------
// 3D LDS plane ring + z-marching register queue
// ---------------------------------------------------------------------------
// A thread owns VX = 16 / sizeof(T) consecutive x cells of RY rows, so every
// access to the levels, the model and LDS is one 16-byte vector.
template <typename T>
struct V16 {
  static constexpr int n = 16 / (int)sizeof(T);
  typedef T type __attribute__((ext_vector_type(16 / sizeof(T))));
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Raw buffer over one plane (or nothing: `bytes` = 0): reads at or past the
// end return zero and stores there are dropped, so a cell outside the grid
// takes the offset kOff (a per-thread constant) and a plane outside the grid
// an empty buffer; neither needs a branch or per-load arithmetic.
constexpr uint32_t kOff = kPlaneBytes;  // past the end of any plane (see plane_fits)
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const T *p, uint32_t bytes) {
  // gfx9 buffer descriptor word 3: 32-bit data format, no swizzle
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float bload1(__amdgpu_buffer_rsrc_t r, uint32_t o, float) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)o, 0, 0));
}
__device__ __forceinline__ double bload1(__amdgpu_buffer_rsrc_t r, uint32_t o, double) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)o, 0, 0));
}
__device__ __forceinline__ void bstore1(__amdgpu_buffer_rsrc_t r, uint32_t o, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (int)o, 0, 0);
}
__device__ __forceinline__ void bstore1(__amdgpu_buffer_rsrc_t r, uint32_t o, double v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)o, 0, 0);
}

// Where one thread's vector of a plane sits: `full` its byte offset, or kOff;
// with RAG (rows whose length is no multiple of VX) a vector that the row's
// end cuts has full = kOff and its first np cells at `part`.
struct VOff {
  uint32_t full = kOff, part = kOff;
  int np = 0;
};
template <typename T, bool RAG>
__device__ __forceinline__ VOff vec_off(int ny, int nx, int y, int x) {
  constexpr int VX = V16<T>::n;
  VOff v;
  if (y < 0 || y >= ny || x < 0 || x >= nx) return v;
  const uint32_t o = ((uint32_t)y * (uint32_t)nx + (uint32_t)x) * (uint32_t)sizeof(T);
  if (!RAG || x + VX <= nx) {
    v.full = o;
  } else {
    v.part = o;
    v.np = nx - x;
  }
  return v;
}
template <typename T, bool NT, bool RAG>
__device__ __forceinline__ typename V16<T>::type vload(__amdgpu_buffer_rsrc_t r, const VOff &o) {
  typedef typename V16<T>::type V;
  V v = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, (int)o.full, 0, NT ? 2 : 0));
  if constexpr (RAG) {
    if (o.np > 0) {  // only the waves that hold a row's end
#pragma unroll
      for (int c = 0; c < V16<T>::n - 1; ++c)
        v[c] = bload1(r, c < o.np ? o.part + c * (uint32_t)sizeof(T) : kOff, T(0));
    }
  }
  return v;
}
template <typename T, bool NT, bool RAG>
__device__ __forceinline__ void vstore(__amdgpu_buffer_rsrc_t r, const VOff &o,
                                       typename V16<T>::type v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)o.full, 0,
                                         NT ? 2 : 0);
  if constexpr (RAG) {
    if (o.np > 0) {
#pragma unroll
      for (int c = 0; c < V16<T>::n - 1; ++c)
        bstore1(r, c < o.np ? o.part + c * (uint32_t)sizeof(T) : kOff, v[c]);
    }
  }
}

// Bound: beyond the caches by HBM (16 bytes per cell-update; 384 x 512 x 512
// 261 us, 6.2 TB/s, where the copy kernel reaches 5.9-6.4), before that by the
// latency of a step.  43 VALU instructions per cell-update (81 with one cell
// per thread and lane-wise LDS reads, where vector issue bound the step as
// much as HBM did: 286-318 us at 384 x 512 x 512, 188-255 at 320 x 448 x 448
// now 173, 27 at 128^3 now 8.8).
// One column tile (bx, by) over planes [z0, z1) of one level.  EPI adds a
// cell-local epilogue for the exact comparator: EPI_D2 writes the second time
// difference of the step, EPI_CORR subtracts (stored u_tt) x (new level) from
// a gradient.
// The tile's planes (with their 4-cell x / y halo) pass through a ring of six
// LDS planes: a plane is written when it is the lead plane z + 4 (its own
// cells are the fronts of the register queue then) and read four planes later,
// when it is the current one, so a tile's halo loads and its neighbours'
// interior loads of a plane are issued close together in time (they meet in
// L2) and no register waits for a halo.  Six slots make one barrier per plane
// enough: the slot written before barrier i was last read before barrier
// i - 1.  Six planes per loop trip turn the slots into immediate LDS offsets
// and most moves of the register queue into renames.
// LDS rows are TX cells (the x halo sits apart), so that the four rows of a
// wave's 16-byte accesses fall on consecutive 16-byte chunks: no conflicts.
// rev: march the chunk from z1 - 1 down to z0 instead of up (same per-cell
// arithmetic: the z terms pair z + j with z - j in a commutative sum, so the
// levels are bitwise the same either way).  Sweeps alternate the direction
// from step to step, so that a step starts on the planes the previous step
// touched last (still in the memory-side cache).
template <typename T, int TX, int TYT, int RY, bool NT, int EPI, bool RAG>
__device__ __forceinline__ void tiled_body(const StepArgs<T> &a, const InjMap<T> &inj, int bx,
                                           int by, int z0, int z1, const EpiArgs<T> &e, bool rev) {
  typedef typename V16<T>::type V;
  constexpr int VX = V16<T>::n;                  // cells per vector
  constexpr int GX = TX / VX;                    // threads along x
  constexpr int NTH = GX * TYT;
  constexpr int TY = TYT * RY;
  constexpr int XV = 4 / VX;                     // vectors of one side's x halo
  constexpr int NYH = 8 * GX;                    // y-halo vectors of a plane
  constexpr int NH = NYH + TY * 2 * XV;          // all halo vectors
  constexpr int KH = (NH + NTH - 1) / NTH;       // per thread
  constexpr int XH = (TY + 8) * TX;              // LDS: rows of TX cells, then x halos [TY][8]
  constexpr int PS = XH + TY * 8;                // LDS cells of a plane
  constexpr int SLOTS = 6;
  __shared__ __attribute__((aligned(16))) T lds[SLOTS * PS];

  const int tid = threadIdx.x;
  const int tx = tid % GX;
  const int ty = tid / GX;
  const int x0 = bx * TX, y0 = by * TY;
  const int x = x0 + tx * VX;
  const int64_t sp = (int64_t)a.ny * a.nx;
  const uint32_t pbytes = (uint32_t)(sp * (int64_t)sizeof(T));

  VOff own[RY];
  T fyx[RY][VX];  // dy^2 + dx^2 of the sponge (small integers, exact)
  int lown[RY], lxl[RY][XV], lxr[RY][XV];  // LDS cells: own vector, x neighbours
#pragma unroll
  for (int j = 0; j < RY; ++j) {
    const int r = ty + j * TYT;
    own[j] = vec_off<T, RAG>(a.ny, a.nx, y0 + r, x);
    const int dy = a.ny > 1 ? sponge_depth(y0 + r, a.ny, a.nb) : 0;
#pragma unroll
    for (int c = 0; c < VX; ++c) {
      const int dx = sponge_depth(x + c, a.nx, a.nb);
      fyx[j][c] = T(dy * dy + dx * dx);
    }
    lown[j] = (r + 4) * TX + tx * VX;
#pragma unroll
    for (int p = 0; p < XV; ++p) {
      const int xl = tx * VX - 4 + p * VX, xr = tx * VX + VX + p * VX;
      lxl[j][p] = xl < 0 ? XH + r * 8 + xl + 4 : (r + 4) * TX + xl;
      lxr[j][p] = xr >= TX ? XH + r * 8 + 4 + xr - TX : (r + 4) * TX + xr;
    }
  }
  // halo vectors of this thread: y-halo rows first, then the x halos
  VOff ho[KH];
  int lh[KH];
  bool hon[KH];
#pragma unroll
  for (int k = 0; k < KH; ++k) {
    const int t = tid + NTH * k;
    hon[k] = t < NH;
    if (t < NYH) {
      const int hr = t / GX, row = hr < 4 ? hr : TY + hr;
      ho[k] = vec_off<T, RAG>(a.ny, a.nx, y0 - 4 + row, x0 + (t % GX) * VX);
      lh[k] = row * TX + (t % GX) * VX;
    } else {
      const int u = t - NYH, row = u / (2 * XV), p = u % (2 * XV);
      const int xc = p < XV ? x0 - 4 + p * VX : x0 + TX + (p - XV) * VX;
      ho[k] = hon[k] ? vec_off<T, RAG>(a.ny, a.nx, y0 + row, xc) : VOff();
      lh[k] = XH + row * 8 + p * VX;
    }
  }

  const int dz = rev ? -1 : 1;
  const int zs = rev ? z1 - 1 : z0;
  const int n = z1 - z0;
  auto plane = [&](const T *f, int z) {
    return plane_rsrc(f + (int64_t)z * sp, (z >= 0 && z < a.nz) ? pbytes : 0u);
  };
  V q[RY][9], front[RY], hv[KH], pv[RY], mv[RY], es[RY], eg[RY];
  // folded injection: only tiles over its box look
  const bool itile = inj.map && x0 < inj.x1 && x0 + TX > inj.x0 && y0 < inj.y1 && y0 + TY > inj.y0;
  auto ldhalo = [&](__amdgpu_buffer_rsrc_t r, V *h) {
#pragma unroll
    for (int k = 0; k < KH; ++k)
      if (KH == 1 || (k + 1) * NTH <= NH || hon[k]) h[k] = vload<T, false, RAG>(r, ho[k]);
  };
  auto sthalo = [&](T *L, const V *h) {
#pragma unroll
    for (int k = 0; k < KH; ++k)
      if ((k + 1) * NTH <= NH || hon[k]) *reinterpret_cast<V *>(L + lh[k]) = h[k];
  };
  // operands of plane z that only its own cells need
  auto ldcell = [&](int z) {
    const __amdgpu_buffer_rsrc_t rp = plane(a.prev, z), rm = plane(a.m, z);
#pragma unroll
    for (int j = 0; j < RY; ++j) {
      pv[j] = vload<T, NT, RAG>(rp, own[j]);
      mv[j] = vload<T, NT, RAG>(rm, own[j]);
    }
    if constexpr (EPI == EPI_CORR) {
      const __amdgpu_buffer_rsrc_t rs = plane(e.s, z), rg = plane((const T *)e.g, z);
#pragma unroll
      for (int j = 0; j < RY; ++j) {
        es[j] = vload<T, NT, RAG>(rs, own[j]);
        eg[j] = vload<T, false, RAG>(rg, own[j]);
      }
    }
  };
  // the march's first nine planes; planes zs .. zs + 3 dz go to slots 0 .. 3
  {
    V h[4][KH];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const __amdgpu_buffer_rsrc_t r = plane(a.cur, zs + dz * (k - 4));
#pragma unroll
      for (int j = 0; j < RY; ++j) q[j][k] = vload<T, false, RAG>(r, own[j]);
      if (k >= 4) ldhalo(r, h[k - 4]);
    }
    const __amdgpu_buffer_rsrc_t r = plane(a.cur, zs + 4 * dz);
#pragma unroll
    for (int j = 0; j < RY; ++j) front[j] = vload<T, false, RAG>(r, own[j]);
    ldhalo(r, hv);
    ldcell(zs);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
      for (int j = 0; j < RY; ++j)
        *reinterpret_cast<V *>(lds + d * PS + lown[j]) = q[j][4 + d];
      sthalo(lds + d * PS, h[d]);
    }
  }

  // plane i of the chunk (i mod 6 = S), queue entry k of it in q[.][S + k - 9 at
  // most]: entries advance by one plane per step inside a trip of the loop
  int z = zs;
  auto step = [&](auto Sc, int i) {
    constexpr int S = decltype(Sc)::value;
    constexpr int W = (S + 4) % SLOTS;
    V pvc[RY], mvc[RY], esc[RY], egc[RY];
#pragma unroll
    for (int j = 0; j < RY; ++j) {
      q[j][(S + 8) % 9] = front[j];
      *reinterpret_cast<V *>(lds + W * PS + lown[j]) = front[j];
      pvc[j] = pv[j];
      mvc[j] = mv[j];
      if constexpr (EPI == EPI_CORR) {
        esc[j] = es[j];
        egc[j] = eg[j];
      }
    }
    sthalo(lds + W * PS, hv);
    if (i + 1 < n) {  // the next step's loads
      const __amdgpu_buffer_rsrc_t r = plane(a.cur, z + 5 * dz);
#pragma unroll
      for (int j = 0; j < RY; ++j) front[j] = vload<T, false, RAG>(r, own[j]);
      ldhalo(r, hv);
      ldcell(z + dz);
    }
    __syncthreads();
    const T *L = lds + S * PS;
    const int d = sponge_depth(z, a.nz, a.nb);
    const T fz = T(d * d);
    const __amdgpu_buffer_rsrc_t ro = plane(a.next, z);
#pragma unroll
    for (int j = 0; j < RY; ++j) {
      auto Q = [&](int k) -> const V & { return q[j][(S + k) % 9]; };
      V yn[8];  // rows -4 .. -1, 1 .. 4
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        yn[k] = *reinterpret_cast<const V *>(L + lown[j] + (k - 4) * TX);
        yn[4 + k] = *reinterpret_cast<const V *>(L + lown[j] + (k + 1) * TX);
      }
      T w[8 + VX];  // x - 4 .. x + VX + 3
#pragma unroll
      for (int p = 0; p < XV; ++p) {
        const V l = *reinterpret_cast<const V *>(L + lxl[j][p]);
        const V r = *reinterpret_cast<const V *>(L + lxr[j][p]);
#pragma unroll
        for (int c = 0; c < VX; ++c) {
          w[p * VX + c] = l[c];
          w[4 + VX + p * VX + c] = r[c];
        }
      }
#pragma unroll
      for (int c = 0; c < VX; ++c) w[4 + c] = Q(4)[c];
      V out, d2;
#pragma unroll
      for (int c = 0; c < VX; ++c) {
        const T u = Q(4)[c];
        const T lz = axis_sum(a, Q(5)[c], Q(3)[c], Q(6)[c], Q(2)[c], Q(7)[c], Q(1)[c], Q(8)[c],
                              Q(0)[c]);
        const T ly = axis_sum(a, yn[4][c], yn[3][c], yn[5][c], yn[2][c], yn[6][c], yn[1][c],
                              yn[7][c], yn[0][c]);
        const T lx = axis_sum(a, w[c + 5], w[c + 3], w[c + 6], w[c + 2], w[c + 7], w[c + 1],
                              w[c + 8], w[c]);
        const T lap = (fma_t(a.cc, u, lz) + ly) + lx;
        out[c] = cell_update(a, u, pvc[j][c], mvc[j][c], lap, sponge_mul(a.kd, fz + fyx[j][c]));
        if constexpr (EPI == EPI_D2)
          d2[c] = (fma_t(T(-2), u, out[c]) + pvc[j][c]) * e.inv_dt2;
        if constexpr (EPI == EPI_CORR) d2[c] = fma_t(-esc[j][c], out[c], egc[j][c]);
      }
      if (itile && z >= inj.z0 && z < inj.z1) {
#pragma unroll
        for (int c = 0; c < VX; ++c) {
          T acc;
          if (inj_sum(inj, z, y0 + ty + j * TYT, x + c, acc)) {
            const T t = inj_term(a, acc, mvc[j][c] + sponge_mul(a.kd, fz + fyx[j][c]));
            out[c] += t;
            if constexpr (EPI == EPI_D2) d2[c] = fma_t(t, e.inv_dt2, d2[c]);
            if constexpr (EPI == EPI_CORR) d2[c] = fma_t(-esc[j][c], t, d2[c]);
          }
        }
      }
      vstore<T, NT, RAG>(ro, own[j], out);
      if constexpr (EPI == EPI_D2) vstore<T, NT, RAG>(plane(e.d2, z), own[j], d2);
      if constexpr (EPI == EPI_CORR) vstore<T, false, RAG>(plane(e.g, z), own[j], d2);
    }
    z += dz;
  };
  for (int i = 0; i < n;) {
    step(std::integral_constant<int, 0>(), i);
    if (++i == n) break;
    step(std::integral_constant<int, 1>(), i);
    if (++i == n) break;
    step(std::integral_constant<int, 2>(), i);
    if (++i == n) break;
    step(std::integral_constant<int, 3>(), i);
    if (++i == n) break;
    step(std::integral_constant<int, 4>(), i);
    if (++i == n) break;
    step(std::integral_constant<int, 5>(), i);
    ++i;
    // a trip moved the queue by six entries: back to entry k in q[k]
#pragma unroll
    for (int j = 0; j < RY; ++j) {
      V t[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) t[k] = q[j][(6 + k) % 9];
#pragma unroll
      for (int k = 0; k < 9; ++k) q[j][k] = t[k];
    }
  }
}

template <typename T, int TX, int TYT, int RY, bool NT, int EPI, bool RAG>
__global__ __launch_bounds__(TX / V16<T>::n *TYT) void k_stencil3d_tiled(
    StepArgs<T> a, InjMap<T> inj, int ntx, int nty, int nzc, int zchunk, EpiArgs<T> e, int rev) {
  // XCD-aware order: consecutive hardware block ids go round-robin over the 8
  // XCDs; give each XCD a contiguous run of tiles so halo re-reads hit its L2.
  const int nblk = ntx * nty * nzc;
  int b = blockIdx.x;
  b = xcd_block(b, nblk);
  const int bx = b % ntx;
  const int by = (b / ntx) % nty;
  const int bz = rev ? nzc - 1 - b / (ntx * nty) : b / (ntx * nty);
  const int z0 = bz * zchunk;
  tiled_body<T, TX, TYT, RY, NT, EPI, RAG>(a, inj, bx, by, z0, min(z0 + zchunk, a.nz), e, rev != 0);
}

// Several shots (independent grids, one ring each) in one launch: entry e of
// the tile table names the shot and the tile; the shot's step arguments come
// from a device table (level pointers rebuilt from the step index s).
template <typename T, int TX, int TYT, int RY, bool NT, bool RAG>
__global__ __launch_bounds__(TX / V16<T>::n *TYT) void k_stencil3d_batched(
    const ShotStep<T> *__restrict__ shots, const ShotIO<T> *__restrict__ io, int mapped,
    const int4 *__restrict__ tiles, int ntiles, int s, int n, int rev) {
  int b = blockIdx.x;
  b = xcd_block(b, ntiles);
  const int4 t = tiles[b];  // (shot, bx | by << 16, z0, z1)
  StepArgs<T> a = shots[t.x].a;
  const ShotStep<T> &sh = shots[t.x];
  a.cur = sh.ring + (int64_t)(((s + 1) % sh.R)) * sh.ld;
  a.prev = sh.ring + (int64_t)(((s + sh.R) % sh.R)) * sh.ld;
  a.next = sh.ring + (int64_t)(((s + 2) % sh.R)) * sh.ld;
  InjMap<T> inj;
  if (mapped) {
    inj = io[t.x].map;
    inj.vals = io[t.x].inj + (int64_t)n * io[t.x].n_inj;
  }
  tiled_body<T, TX, TYT, RY, NT, EPI_NONE, RAG>(a, inj, t.y & 0xffff, t.y >> 16, t.z, t.w,
                                               EpiArgs<T>{}, rev != 0);
}

template <typename T, int TX, int TYT, int RY, bool NT, int EPI = EPI_NONE>
static void launch_tiled(const StepArgs<T> &a, const InjMap<T> &inj, int nzc, hipStream_t st,
                         const EpiArgs<T> &e = EpiArgs<T>{}, int rev = 0) {
  constexpr int TY = TYT * RY;
  constexpr int NTH = TX / V16<T>::n * TYT;
  const int ntx = (a.nx + TX - 1) / TX;
  const int nty = (a.ny + TY - 1) / TY;
  const int zchunk = (a.nz + nzc - 1) / nzc;
  nzc = (a.nz + zchunk - 1) / zchunk;
  if (a.nx % V16<T>::n == 0)
    hipLaunchKernelGGL((k_stencil3d_tiled<T, TX, TYT, RY, NT, EPI, false>), dim3(ntx * nty * nzc),
                       dim3(NTH), 0, st, a, inj, ntx, nty, nzc, zchunk, e, rev);
  else
    hipLaunchKernelGGL((k_stencil3d_tiled<T, TX, TYT, RY, NT, EPI, true>), dim3(ntx * nty * nzc),
                       dim3(NTH), 0, st, a, inj, ntx, nty, nzc, zchunk, e, rev);
}

// z chunks of a tile shape: the fewest (of at least `minp` planes) that give
// `target` workgroups of 256 threads' worth
static int z_split(int nz, int64_t tiles, int threads, int target, int minp) {
  const int64_t want = (int64_t)target * 256 / threads;
  return (int)std::max<int64_t>(
      1, std::min<int64_t>((want + tiles - 1) / tiles, std::max(1, nz / minp)));
}

// The shortest z chunks worth their warm-up, by the bytes of a level (all
// shots together): us per step with chunks of 1 / 2 / 4 / 6 / 8 planes: 64^3
// 4.0 / 5.1 / 5.9 / 7.7 / 8.3 (one thread per cell 5.8); 100^3 8.4 / 7.2 / 7.7 /
// 8.3 / 9.6; 128^3 10.8 / 9.3 / 8.9 / 10.4 / 9.9; 160^3 19.8 / 16.0 / 14.6 /
// 14.0 / 15.0; 200^3 39 / 31 / 27.5 / 26.9 / 26.7.  Loads two or three planes
// ahead instead of one changed none of them by more than 0.2.
int min_planes(int64_t bytes) {
  return bytes < 1600000 ? 1 : bytes < 6000000 ? 2 : bytes < 12000000 ? 4 : 6;
}

// tiled variants: id -> tile (x cells x y rows), threads
//   1: 64 x 16, 256     2: 64 x 32, 512     3: 64 x 32, 256 (two rows each)
//   4: 64 x 8, 128      5: 32 x 32, 256     6: 128 x 8, 256
//   7 .. 10, 12: as 1 .. 4, 6, non-temporal    11, 13: as 12
// (FP64: half as many rows).  11 and 13 once stood for 64 x 16 and 64 x 32
// non-temporal tiles of other kernels, 13 the fastest at 384 x 512 x 512 (289);
// 12 is at least as fast as either was on every grid measured (268-293 there;
// 300^3 94-111 against 114-148, 320 x 448 x 447 222-250 against 236-308), tiles
// of 32 x 32 and 32 x 16 were not (310-334 and 359-372, 137-151 and 111-115,
// 377-389 and 307-315).
struct TileShape {
  int tx, ty, threads;
};
template <typename T>
static TileShape tile_shape(int variant) {
  static const TileShape k[6] = {{64, 16, 256}, {64, 32, 512}, {64, 32, 256},
                                 {64, 8, 128},  {32, 32, 256}, {128, 8, 256}};
  TileShape t = k[(tiled_kernel(variant) - 1) % 6];
  t.ty /= (int)sizeof(T) / 4;
  return t;
}

// Automatic choice of the kernel and its z chunks (us per step, F32 unless
// said; v: the variant).
//   Grids below kSimpleCells run one thread per cell.  Bare steps cross near
//   100 K cells (tiled / thread per cell: 101 K cells 4.8 / 4.8, 124 K 4.2 / 5.0,
//   150 K 4.5 / 5.2, 64^3 4.7 / 6.0; FP64 101 K 5.0 / 5.1, 201 K 5.0 / 6.2), adjoint
//   steps near 200 K, as a folded injection waits for one cell's entries per
//   thread, not four's (receivers on a plane: 148 K cells 5.4 / 4.9, 201 K 5.4 /
//   5.5; every seventh off the grid: 6.1 / 5.2 and 6.5 / 5.4): the line between.
//   So do grids that would leave four fifths of the tiles' lanes idle (FP64,
//   and F32 in brackets, thread per cell against tiled): 300 x 300 x 20, 31 %
//   of the lanes, 27 against 25 (23, 16); 1000 x 16 x 16, 25 %, 8.3 against
//   9.6 (6.7, 7.3); 64 x 2000 x 8, 12 %, 18 against 29 (15, 19); 400 x 400 x 4
//   13 against 33 (11, 21); 3000 x 300 x 1 16 against 181 (13, 93).
//   While the four arrays of a step (16 N bytes) stay near the 256 MB
//   memory-side cache, ordinary loads and short chunks on 64 x 16 tiles: a
//   chunk re-reads eight planes, but they hit the caches, and a step is a chain
//   of waits, one per plane (min_planes).  200^3: 26.9 against 38.3
//   non-temporal; 300^3: 96 against 103.  FP64: 96 x 90 x 110 9.8, 128^3 13.4
//   (one thread per cell 15.8 and 28); 300^3 166 non-temporal, 200 not.
//   Beyond that the levels stream from HBM: non-temporal, 64 x 32 tiles.  If
//   one or more whole chunks per column fill nearly all 256 CUs with one
//   workgroup each, they are the chunks, else 16 planes.  Against that, 128 x 8
//   tiles with their best split: 384 x 512 x 512 (2 chunks) 254 / 256 (16-plane
//   chunks 288), 256 x 512 x 512 159 / 163, 320 x 448 x 448 170 / 183, 300 x 300 x
//   512 116 / 125, 352 x 384 x 384 140 / 136, 512 x 400 x 400 270 / 272, 400^3 209 /
//   206, 300 x 400 x 400 155 / 150, 384 x 448 x 512 261 / 251.
//   F32 rows that are no multiple of the vector cut a cache line at every
//   tile's edge.  128-cell tiles have half as many edges and stream (320 x 448
//   x 447: 236; 64 x 32 ordinary 261, non-temporal 274; 260 x 320 x 501 152,
//   157), as long as they cover at most a seventh more columns than 64-cell
//   tiles; else two rows per thread and twice the workgroups (320 x 600 x 257:
//   189, 204, 128-cell tiles 207; 500 x 800 x 131: 215, 224, 253).  FP64 rows:
//   64 x 16 tiles, ordinary.
constexpr int64_t kSimpleCells = 150000;
template <typename T>
static int auto_variant(const StepArgs<T> &a, int *nzc) {
  constexpr int F = sizeof(T) / 4;
  const int64_t lanes = (int64_t)((a.nx + 63) / 64 * 64) * ((a.ny + 16 / F - 1) / (16 / F) * (16 / F));
  if (a.N < kSimpleCells || lanes > 5 * (int64_t)a.ny * a.nx) return kStencilSimple;
  const bool stream = 4 * a.N * (int64_t)sizeof(T) > kStreamBytes;
  const bool ragged = a.nx % V16<T>::n != 0;
  const bool edges = stream && ragged && sizeof(T) == 4;
  const bool wide = edges && (a.nx + 127) / 128 * 14 <= (a.nx + 63) / 64 * 8;
  const int v = !stream ? 1 : edges ? (wide ? 12 : 3) : ragged ? 2 : 8;
  const TileShape t = tile_shape<T>(v);
  const int64_t tiles = (int64_t)((a.nx + t.tx - 1) / t.tx) * ((a.ny + t.ty - 1) / t.ty);
  if (!stream) {
    *nzc = z_split(a.nz, tiles, t.threads, kAutoBlocks, min_planes(a.N * (int)sizeof(T)));
  } else if (edges) {
    *nzc = z_split(a.nz, tiles, t.threads, wide ? kAutoBlocks : 2 * kAutoBlocks, 6);
  } else {
    const int c = (int)std::min<int64_t>(256 / tiles, a.nz / 16);
    *nzc = c >= 1 && c * tiles >= 230 && !ragged ? c : std::max(1, a.nz / 16);
  }
  return v;
}

template <typename T>
bool stencil_tiled(int ndim, int nz, int ny, int nx, int variant) {
  if (ndim != 3 || !plane_fits(ny, nx, sizeof(T))) return false;
  StepArgs<T> a{};
  a.nz = nz;
  a.ny = ny;
  a.nx = nx;
  a.N = (int64_t)nz * ny * nx;
  int nzc;
  return (variant < 0 ? auto_variant(a, &nzc) : variant) != kStencilSimple;
}
template bool stencil_tiled<float>(int, int, int, int, int);
template bool stencil_tiled<double>(int, int, int, int, int);

template <typename T>
hipError_t launch_stencil(int ndim, const StepArgs<T> &a, const InjMap<T> &inj, int variant,
                          int target_blocks, hipStream_t st, int rev) {
  constexpr int F = sizeof(T) / 4;
  const EpiArgs<T> e{};
  int nzc = 1;
  const bool rule = variant < 0;
  if (ndim != 3 || !plane_fits(a.ny, a.nx, sizeof(T))) {
    variant = kStencilSimple;
  } else if (rule) {
    variant = auto_variant(a, &nzc);
  }
  if (variant != kStencilSimple && (!rule || target_blocks != kAutoBlocks)) {
    const TileShape t = tile_shape<T>(variant);
    nzc = z_split(a.nz, (int64_t)((a.nx + t.tx - 1) / t.tx) * ((a.ny + t.ty - 1) / t.ty),
                  t.threads, target_blocks, 4);
  }
  switch (tiled_kernel(variant)) {
    case kStencilSimple: {
      const unsigned nblk = (unsigned)((a.N + 255) / 256);
      if (ndim == 3)
        hipLaunchKernelGGL((k_stencil_simple<T, 3>), dim3(nblk), dim3(256), 0, st, a, inj);
      else
        hipLaunchKernelGGL((k_stencil_simple<T, 2>), dim3(nblk), dim3(256), 0, st, a, inj);
      break;
    }
    case 2: launch_tiled<T, 64, 32 / F, 1, false>(a, inj, nzc, st, e, rev); break;
    case 3: launch_tiled<T, 64, 16 / F, 2, false>(a, inj, nzc, st, e, rev); break;
    case 4: launch_tiled<T, 64, 8 / F, 1, false>(a, inj, nzc, st, e, rev); break;
    case 5: launch_tiled<T, 32, 32 / F, 1, false>(a, inj, nzc, st, e, rev); break;
    case 6: launch_tiled<T, 128, 8 / F, 1, false>(a, inj, nzc, st, e, rev); break;
    case 7: launch_tiled<T, 64, 16 / F, 1, true>(a, inj, nzc, st, e, rev); break;
    case 8: launch_tiled<T, 64, 32 / F, 1, true>(a, inj, nzc, st, e, rev); break;
    case 9: launch_tiled<T, 64, 16 / F, 2, true>(a, inj, nzc, st, e, rev); break;
    case 10: launch_tiled<T, 64, 8 / F, 1, true>(a, inj, nzc, st, e, rev); break;
    case 12: launch_tiled<T, 128, 8 / F, 1, true>(a, inj, nzc, st, e, rev); break;
    default: launch_tiled<T, 64, 16 / F, 1, false>(a, inj, nzc, st, e, rev); break;
  }
  return hipGetLastError();
}

template hipError_t launch_stencil<float>(int, const StepArgs<float> &, const InjMap<float> &, int,
                                          int, hipStream_t, int);
template hipError_t launch_stencil<double>(int, const StepArgs<double> &, const InjMap<double> &,
                                           int, int, hipStream_t, int);

// Stencil step with an exact-comparator epilogue (3D F32, 64 x 16 tiles with
// the z split of the plain step's rule).  Returns hipErrorInvalidValue for
// grids the tiled kernel does not serve, so the caller falls back to the
// separate kernels.
template <typename T>
hipError_t launch_stencil_epi(int ndim, const StepArgs<T> &a, const InjMap<T> &inj, int variant,
                              int target_blocks, int epi, const EpiArgs<T> &e, hipStream_t st,
                              int rev) {
  if (ndim != 3 || sizeof(T) != 4 || variant == kStencilSimple ||
      !plane_fits(a.ny, a.nx, sizeof(T)))
    return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 4) {
    const bool stream = 4 * a.N * (int64_t)sizeof(T) > kStreamBytes;
    const bool nt = variant < 0 ? stream && a.nx % V16<T>::n == 0 : variant >= 7;
    const int64_t tiles = (int64_t)((a.nx + 63) / 64) * ((a.ny + 15) / 16);
    const int nzc = z_split(a.nz, tiles, 256, target_blocks,
                            stream ? 16 : min_planes(a.N * (int)sizeof(T)));
    if (epi == EPI_D2) {
      if (nt) launch_tiled<T, 64, 16, 1, true, EPI_D2>(a, inj, nzc, st, e, rev);
      else launch_tiled<T, 64, 16, 1, false, EPI_D2>(a, inj, nzc, st, e, rev);
    } else if (epi == EPI_CORR) {
      if (nt) launch_tiled<T, 64, 16, 1, true, EPI_CORR>(a, inj, nzc, st, e, rev);
      else launch_tiled<T, 64, 16, 1, false, EPI_CORR>(a, inj, nzc, st, e, rev);
    } else {
      return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}
template hipError_t launch_stencil_epi<float>(int, const StepArgs<float> &, const InjMap<float> &,
                                              int, int, int, const EpiArgs<float> &, hipStream_t,
                                              int);
template hipError_t launch_stencil_epi<double>(int, const StepArgs<double> &,
                                               const InjMap<double> &, int, int, int,
                                               const EpiArgs<double> &, hipStream_t, int);

// Injection whose increment d = dt^2 acc / (m + a) also updates an
// exact-comparator epilogue output: EPI_D2 adds d / dt^2 to the stored u_tt,
// EPI_CORR subtracts s * d from the gradient.
template <typename T>
__global__ __launch_bounds__(256) void k_inject_epi(StepArgs<T> a, PointTables<T> pt,
                                                    const T *__restrict__ vals, T *field, int epi,
                                                    EpiArgs<T> e) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= pt.ncell) return;
  T acc = T(0);
  for (int j = pt.ioff[c]; j < pt.ioff[c + 1]; ++j) acc += pt.iw[j] * vals[pt.ipt[j]];
  const int64_t i = pt.icell[c];
  const int x = (int)(i % a.nx);
  const int64_t zy = i / a.nx;
  const int y = (int)(zy % a.ny);
  const int z = (int)(zy / a.ny);
  const T d = a.dt2 * acc / (a.m[i] + sponge_a(a, z, y, x));
  field[i] += d;
  if (epi == EPI_D2) e.d2[i] += d * e.inv_dt2;
  if (epi == EPI_CORR) e.g[i] -= e.s[i] * d;
}

template <typename T>
hipError_t launch_inject_epi(const StepArgs<T> &a, const PointTables<T> &pt, const T *vals,
                             T *field, int epi, const EpiArgs<T> &e, hipStream_t st) {
  if (pt.ncell <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_inject_epi<T>), dim3((pt.ncell + 255) / 256), dim3(256), 0, st, a, pt,
                     vals, field, epi, e);
  return hipGetLastError();
}
template hipError_t launch_inject_epi<float>(const StepArgs<float> &, const PointTables<float> &,
                                             const float *, float *, int, const EpiArgs<float> &,
                                             hipStream_t);
template hipError_t launch_inject_epi<double>(const StepArgs<double> &,
                                              const PointTables<double> &, const double *,
                                              double *, int, const EpiArgs<double> &,
                                              hipStream_t);

// ---------------------------------------------------------------------------
// autotuning helpers: a deterministic test pattern and a bitwise comparison
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_pattern(T *p, int64_t n, uint32_t seed, T scale) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * 256) {
    uint32_t h = (uint32_t)i * 2654435761u ^ seed;  // Knuth multiplicative hash
    h ^= h >> 15;
    h *= 2246822519u;
    h ^= h >> 13;
    p[i] = scale * (T)((int32_t)(h & 0xffff) - 32768) / T(32768);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_count_diff(const T *a, const T *b, int64_t n,
                                                    unsigned long long *count) {
  unsigned long long c = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * 256)
    c += (a[i] != b[i]) ? 1ull : 0ull;
  if (c) atomicAdd(count, c);
}

template <typename T>
hipError_t launch_pattern(T *p, int64_t n, uint32_t seed, T scale, hipStream_t st) {
  hipLaunchKernelGGL((k_pattern<T>), dim3(4096), dim3(256), 0, st, p, n, seed, scale);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_count_diff(const T *a, const T *b, int64_t n, unsigned long long *count,
                             hipStream_t st) {
  hipLaunchKernelGGL((k_count_diff<T>), dim3(4096), dim3(256), 0, st, a, b, n, count);
  return hipGetLastError();
}
template hipError_t launch_pattern<float>(float *, int64_t, uint32_t, float, hipStream_t);
template hipError_t launch_pattern<double>(double *, int64_t, uint32_t, double, hipStream_t);
template hipError_t launch_count_diff<float>(const float *, const float *, int64_t,
                                             unsigned long long *, hipStream_t);
template hipError_t launch_count_diff<double>(const double *, const double *, int64_t,
                                              unsigned long long *, hipStream_t);

// ---------------------------------------------------------------------------
// point injection (after the step) and sampling
// ---------------------------------------------------------------------------
// field[cell] += dt^2 * (sum_j w_j vals[pt_j]) / (m + a): the source term of
// the step added once the stencil part of the update is done.
template <typename T>
__global__ __launch_bounds__(256) void k_inject(StepArgs<T> a, PointTables<T> pt,
                                                const T *__restrict__ vals, T *field) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= pt.ncell) return;
  T acc = T(0);
  for (int j = pt.ioff[c]; j < pt.ioff[c + 1]; ++j) acc += pt.iw[j] * vals[pt.ipt[j]];
  const int64_t i = pt.icell[c];
  const int x = (int)(i % a.nx);
  const int64_t zy = i / a.nx;
  const int y = (int)(zy % a.ny);
  const int z = (int)(zy / a.ny);
  field[i] += a.dt2 * acc / (a.m[i] + sponge_a(a, z, y, x));
}

// A block's levels are all in the ring when it ends, so one launch samples
// them (a launch per step cost 4.6 us of a 128^3 step's 18).
template <typename T>
__global__ __launch_bounds__(256) void k_sample_block(PointTables<T> pt, const T *__restrict__ ring,
                                                      const T *__restrict__ ring2, int64_t ld,
                                                      int R, int s0, int dir, T *__restrict__ out) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= pt.npts) return;
  const int t = blockIdx.y;
  const int64_t slot = (int64_t)((s0 + t + 2) % R) * ld;  // level s0 + 1 + t
  const T *f = ring + slot, *f2 = ring2 ? ring2 + slot : nullptr;
  T s = T(0);
  for (int j = pt.soff[p]; j < pt.soff[p + 1]; ++j) {
    const T v = f2 ? f[pt.sidx[j]] + f2[pt.sidx[j]] : f[pt.sidx[j]];
    s = fma_t(pt.sw[j], v, s);
  }
  out[(int64_t)t * dir * pt.npts + p] = s;
}

template <typename T>
hipError_t launch_inject(const StepArgs<T> &a, const PointTables<T> &pt, const T *vals, T *field,
                         hipStream_t st) {
  if (pt.ncell <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_inject<T>), dim3((pt.ncell + 255) / 256), dim3(256), 0, st, a, pt, vals,
                     field);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sample_block(const PointTables<T> &pt, const T *ring, const T *ring2, int64_t ld,
                               int R, int s0, int kb, int dir, T *out, hipStream_t st) {
  if (pt.npts <= 0 || kb <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_sample_block<T>), dim3((pt.npts + 255) / 256, kb), dim3(256), 0, st, pt,
                     ring, ring2, ld, R, s0, dir, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// batched shots
// ---------------------------------------------------------------------------
template <typename T>
hipError_t launch_stencil_batched(const ShotStep<T> *shots, const ShotIO<T> *io, bool mapped,
                                  const int4 *tiles, int ntiles, int s, int n, int variant,
                                  bool ragged, bool wide, hipStream_t st, int rev) {
  if (ntiles <= 0) return hipSuccess;
  const bool nt = variant >= 7;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(ntiles), dim3(256), 0, st, shots, io, (int)mapped, tiles,
                       ntiles, s, n, rev);
  };
  if (wide) {
    if (nt) go(k_stencil3d_batched<T, 128, 8, 1, true, true>);
    else go(k_stencil3d_batched<T, 128, 8, 1, false, true>);
  } else if (ragged) {
    if (nt) go(k_stencil3d_batched<T, 64, 16, 1, true, true>);
    else go(k_stencil3d_batched<T, 64, 16, 1, false, true>);
  } else {
    if (nt) go(k_stencil3d_batched<T, 64, 16, 1, true, false>);
    else go(k_stencil3d_batched<T, 64, 16, 1, false, false>);
  }
  return hipGetLastError();
}

// level s+1 of shot sh
template <typename T>
__device__ __forceinline__ T *next_level(const ShotStep<T> &sh, int s) {
  return sh.ring + (int64_t)((s + 2) % sh.R) * sh.ld;
}

template <typename T>
__global__ __launch_bounds__(256) void k_inject_batched(const ShotStep<T> *__restrict__ shots,
                                                        const ShotIO<T> *__restrict__ io,
                                                        BatchPoints<T> pt, int s, int n) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= pt.ncell) return;
  const int sh = pt.ishot[c];
  const T *vals = io[sh].inj + (int64_t)n * io[sh].n_inj;
  T acc = T(0);
  for (int j = pt.ioff[c]; j < pt.ioff[c + 1]; ++j) acc += pt.iw[j] * vals[pt.ipt[j]];
  const StepArgs<T> &a = shots[sh].a;
  const int64_t i = pt.icell[c];
  const int x = (int)(i % a.nx);
  const int64_t zy = i / a.nx;
  const int y = (int)(zy % a.ny);
  const int z = (int)(zy / a.ny);
  T *field = next_level(shots[sh], s);
  field[i] += a.dt2 * acc / (a.m[i] + sponge_a(a, z, y, x));
}

template <typename T>
__global__ __launch_bounds__(256) void k_sample_batched(const ShotStep<T> *__restrict__ shots,
                                                        const ShotIO<T> *__restrict__ io,
                                                        BatchPoints<T> pt, int s0) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= pt.npts) return;
  const int sh = pt.sshot[p];
  if (!io[sh].out) return;
  const int n = s0 + blockIdx.y;
  const T *field = next_level(shots[sh], n);
  T v = T(0);
  for (int j = pt.soff[p]; j < pt.soff[p + 1]; ++j) v = fma_t(pt.sw[j], field[pt.sidx[j]], v);
  io[sh].out[(int64_t)n * io[sh].n_smp + pt.slocal[p]] = v;
}

template <typename T>
hipError_t launch_inject_batched(const ShotStep<T> *shots, const ShotIO<T> *io,
                                 const BatchPoints<T> &pt, int s, int n, hipStream_t st) {
  if (pt.ncell <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_inject_batched<T>), dim3((pt.ncell + 255) / 256), dim3(256), 0, st, shots,
                     io, pt, s, n);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_sample_batched(const ShotStep<T> *shots, const ShotIO<T> *io,
                                 const BatchPoints<T> &pt, int s0, int kb, hipStream_t st) {
  if (pt.npts <= 0 || kb <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_sample_batched<T>), dim3((pt.npts + 255) / 256, kb), dim3(256), 0, st,
                     shots, io, pt, s0);
  return hipGetLastError();
}
template hipError_t launch_stencil_batched<float>(const ShotStep<float> *, const ShotIO<float> *,
                                                  bool, const int4 *, int, int, int, int, bool,
                                                  bool, hipStream_t, int);
template hipError_t launch_inject_batched<float>(const ShotStep<float> *, const ShotIO<float> *,
                                                 const BatchPoints<float> &, int, int,
                                                 hipStream_t);
template hipError_t launch_sample_batched<float>(const ShotStep<float> *, const ShotIO<float> *,
                                                 const BatchPoints<float> &, int, int,
                                                 hipStream_t);

template hipError_t launch_inject<float>(const StepArgs<float> &, const PointTables<float> &,
                                         const float *, float *, hipStream_t);
template hipError_t launch_inject<double>(const StepArgs<double> &, const PointTables<double> &,
                                          const double *, double *, hipStream_t);
template hipError_t launch_sample_block<float>(const PointTables<float> &, const float *,
                                               const float *, int64_t, int, int, int, int, float *,
                                               hipStream_t);
template hipError_t launch_sample_block<double>(const PointTables<double> &, const double *,
                                                const double *, int64_t, int, int, int, int,
                                                double *, hipStream_t);

}  // namespace rtm
