// romap_kernels.hip -- gfx950 kernels of one training step of RO-MAP's
// per-object radiance fields (arXiv 2304.05735, Sec. V).
//
// One step over every object of a launch:
//   k_raygen       draw rays in each object's detection boxes, classify them by
//                  the instance mask, back-project into the object frame, clip
//                  to the 3D box (Sec. V-B)                        [FP32, exact];
//                  MLP weights -> MFMA operand images (FP32 and BF16)
//   k_encode_fwd   multiresolution hash-grid gather, one (object, level) table
//                  at a time; advances the Adam step
//   k_field        fused per-ray MLP (MFMA) + volume rendering (Eq. 6) + loss
//                  (Eq. 7-11) + adjoint, activations recomputed in the backward
//                  half, wavefront prefix scans for transmittance
//   k_reduce       per-object MLP gradient and loss from the work-item records;
//                  Adam on the MLP weights
//   k_bin_scatter  encoding adjoint -> (entry, value) records sorted into bins
//                  of table regions
//   k_bin_acc      region sums in LDS; Adam on the region's table entries
//   k_bin_finish   Adam on regions summed by several workgroups
//
// Adam is dense: every parameter of every object of the step is updated each
// step, each where its gradient is complete, so the gradient itself is never
// written in a training step.
//
// Precision: the ray / sample-position / cell / hash path is IEEE FP32 with no
// contraction (this file is built with -ffp-contract=off; FMAs are written
// out where wanted), so positions and indices are reproducible bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <math.h>
#include <stdint.h>

#include "romap_device.h"

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef float rm_f2v __attribute__((ext_vector_type(2)));
typedef float rm_f4v __attribute__((ext_vector_type(4), aligned(8)));

// ---------------------------------------------------------------------------
// small helpers

// Philox4x32-10 (Salmon et al., SC'11): the counter-based generator behind
// every random draw, so a draw depends only on (seed, object, step, ray).
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                     uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int rnd = 0; rnd < 10; ++rnd) {
    const uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
    const uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));

// FP32 -> BF16 with round to nearest, ties to even (gfx950 v_cvt_pk_bf16_f32)
__device__ inline uint32_t pack_bf16x2(float x, float y) {
  const floatx2_t v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// FP32 -> BF16, round to nearest even (integer form, for the weight images)
__device__ inline uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Orders this wave's LDS traffic: every lane's earlier LDS accesses are
// complete before any lane's later ones (cross-lane exchange inside a wave).
// Orders a wave's LDS writes before its later LDS reads of other lanes' data
// (and reads before later writes): the LDS executes one wave's operations in
// issue order, so only the compiler must keep them in program order; the
// hardware waits where a read's result is used.
__device__ inline void wave_lds_sync() { asm volatile("" ::: "memory"); }

// Wave-wide scans in registers with DPP (no LDS round trips): row shifts
// build the scan inside each 16-lane row, row broadcasts carry the row
// totals across.  Lanes a shift reads from outside the row (or the wave)
// read 0.
template <int CTRL, int ROWM = 0xf, int BANKM = 0xf, bool BC = true>
__device__ inline float dppf(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWM, BANKM, BC));
}

__device__ inline float readlane_f(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// inclusive prefix sum over the 64 lanes
__device__ inline float wave_incl_prefix(float x) {
  x += dppf<0x111>(x);                   // row_shr:1
  x += dppf<0x112>(x);                   // row_shr:2
  x += dppf<0x114>(x);                   // row_shr:4
  x += dppf<0x118>(x);                   // row_shr:8
  x += dppf<0x142, 0xa, 0xf, false>(x);  // row_bcast:15 into rows 1 and 3
  x += dppf<0x143, 0xc, 0xf, false>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}

__device__ inline float wave_sum(float x) { return readlane_f(wave_incl_prefix(x), 63); }

// exclusive suffix sum over the 64 lanes (sum over lanes > lane)
__device__ inline float wave_excl_suffix(float x, int lane) {
  x += dppf<0x101>(x);  // row_shl:1
  x += dppf<0x102>(x);  // row_shl:2
  x += dppf<0x104>(x);  // row_shl:4
  x += dppf<0x108>(x);  // row_shl:8: inclusive suffix inside the row
  const float t1 = readlane_f(x, 16), t2 = readlane_f(x, 32), t3 = readlane_f(x, 48);
  const int row = lane >> 4;
  x += row == 0 ? (t1 + t2) + t3 : (row == 1 ? t2 + t3 : (row == 2 ? t3 : 0.0f));
  return dppf<0x130>(x);  // wave_shl:1: the next lane's inclusive suffix
}

// integer inclusive prefix sum over the 64 lanes (same steps)
template <int CTRL, int ROWM = 0xf, int BANKM = 0xf, bool BC = true>
__device__ inline int dppi(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWM, BANKM, BC);
}

// the values of lane ^ 1, of the even and of the odd lane of a pair of lanes
__device__ inline float pair_swap(float x) { return dppf<0xB1>(x); }  // quad_perm:[1,0,3,2]
__device__ inline uint32_t pair_even(uint32_t x) { return (uint32_t)dppi<0xA0>((int)x); }
__device__ inline uint32_t pair_odd(uint32_t x) { return (uint32_t)dppi<0xF5>((int)x); }

__device__ inline int wave_incl_prefix_i(int x) {
  x += dppi<0x111>(x);
  x += dppi<0x112>(x);
  x += dppi<0x114>(x);
  x += dppi<0x118>(x);
  x += dppi<0x142, 0xa, 0xf, false>(x);
  x += dppi<0x143, 0xc, 0xf, false>(x);
  return x;
}

// exclusive prefix without the subtraction: shift the inclusive scan by one lane
__device__ inline float wave_excl_prefix(float x, int lane) {
  return dppf<0x138>(wave_incl_prefix(x));  // wave_shr:1
}

// Quotient a / b for a in [0, b], rounded as IEEE division rounds it, with
// r = 1 / b rounded to nearest: two corrections of a r by its remainder (the
// first brings the quotient within one unit, from where the second rounds
// correctly because the remainder is exact and r correctly rounded).  Holds
// where nothing underflows: b within 2^-60 .. 2^60 (400 M random and edge
// operands: none differs).  5 instructions against 11 of the division.
__device__ inline float div_fixed(float a, float b, float r) {
  float q = a * r;
  q = fmaf(fmaf(-q, b, a), r, q);
  return fmaf(fmaf(-q, b, a), r, q);
}

// Unit-cube coordinates of an object-frame point: p = (x + a) / 2a clamped to
// [0, 1] (clamped before dividing, which gives the same values: division is
// monotonic, and a NaN clamps to 0 either way).  inv: 1 / 2a, or zeros for a
// box outside div_fixed's range, where 2a may be infinite: then a clamped
// x + a may be too, and the quotient, a NaN, is clamped to 0.
__device__ inline void unit_pos(const float x[3], const float* half, const float* inv, float p[3]) {
  float n[3], w[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    w[k] = half[k] + half[k];
    n[k] = __builtin_amdgcn_fmed3f(x[k] + half[k], 0.0f, w[k]);
  }
  if (inv[0] != 0.0f) {
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k] = div_fixed(n[k], w[k], inv[k]);
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) p[k] = __builtin_amdgcn_fmed3f(n[k] / w[k], 0.0f, 1.0f);
  }
}

// What a sample's position needs of its ray.
struct RayGeo {
  float o[3], d[3], tn, delta;
  uint32_t flags;
};

// Position of sample i of a ray in the unit cube of the object's box:
// d_i = t_n + (i + 1/2) delta, x = o + d_i d, p = (x + a) / 2a, clamped.
template <class Ray>
__device__ inline void sample_pos(const Ray& R, int i, const float* half, const float* inv,
                                  float p[3]) {
  const float di = R.tn + ((float)i + 0.5f) * R.delta;
  float x[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) x[k] = R.o[k] + di * R.d[k];
  unit_pos(x, half, inv, p);
}

// A table that no kernel of the launch writes, read at an index that is
// uniform in the wave: through the scalar cache (a plain pointer would make
// vector loads of them, as the kernel's own stores might alias it).
template <class T>
using cptr = const __attribute__((address_space(4))) T*;
template <class T>
__device__ inline cptr<T> as_const(const T* p) {
  return (cptr<T>)(uintptr_t)p;
}

// Device memory behind a pointer that was itself read from memory (without
// this the compiler makes flat accesses, which also wait for the LDS).
template <class T>
using gptr = __attribute__((address_space(1))) T*;
template <class T>
__device__ inline gptr<T> as_global(T* p) {
  return (gptr<T>)(uintptr_t)p;
}

__device__ inline RayGeo ray_uniform(const RayRec* rays, int ray) {
  const cptr<RayRec> q = as_const(rays + ray);
  RayGeo g;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    g.o[k] = q->o[k];
    g.d[k] = q->d[k];
  }
  g.tn = q->tn;
  g.delta = q->delta;
  g.flags = q->flags;
  return g;
}

// The ray of each lane of a wave that covers samples k .. k + 63 (k uniform, a
// multiple of 64) from ray ray0's first: one ray, or with 32 samples per ray
// two, chosen by lane.  Rays past the launch's n_rays read the last one.
template <int NS>
__device__ inline RayGeo wave_ray(const RayRec* rays, int n_rays, int ray0, int k, int lane) {
  const int ray = ray0 + k / NS;
  RayGeo g = ray_uniform(rays, ray < n_rays ? ray : n_rays - 1);
  if constexpr (NS < 64) {
    const RayGeo h = ray_uniform(rays, ray + 1 < n_rays ? ray + 1 : n_rays - 1);
    const bool up = lane >= NS;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      g.o[k] = up ? h.o[k] : g.o[k];
      g.d[k] = up ? h.d[k] : g.d[k];
    }
    g.tn = up ? h.tn : g.tn;
    g.delta = up ? h.delta : g.delta;
    g.flags = up ? h.flags : g.flags;
  }
  return g;
}

// Occupancy skip: 64^3 bits over the unit cube, bit x + 64 y + 4096 z of cell
// floor(64 p) (clamped).  A sample in a clear cell has density 0.
__device__ inline bool occupied(const uint32_t* occ, const float p[3]) {
  if (!occ) return true;
  int c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    int ci = (int)floorf(p[k] * 64.0f);
    c[k] = ci < 0 ? 0 : (ci > 63 ? 63 : ci);
  }
  const int bit = c[0] + 64 * c[1] + 4096 * c[2];
  return (as_global(occ)[bit >> 5] >> (bit & 31)) & 1u;
}

__device__ inline bool ray_active(uint32_t flags) {
  return (flags & RM_F_HIT) && (flags & RM_F_CLS) != RM_CLS_OCCLUDER;
}

struct Cell {
  uint32_t c[3];
  float f[3];
};

__device__ inline void make_cell(const float p[3], uint32_t N, Cell& cl) {
  const float Nf = (float)N;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float g = p[k] * Nf;  // p in [0, 1]: g in [0, N]
    const float c = __builtin_amdgcn_fmed3f(floorf(g), 0.0f, Nf - 1.0f);
    cl.c[k] = (uint32_t)(int)c;
    cl.f[k] = g - c;
  }
}

// Index of corner b (bit0 x, bit1 y, bit2 z) of a cell within its level:
// dense 1:1 when the level fits its table, else the spatial hash of the
// multiresolution hash encoding (primes 1, 2654435761, 805459861) mod T.
__device__ inline uint32_t corner_index(const Cell& cl, int b, uint32_t N, uint32_t T,
                                        bool hashed) {
  const uint32_t vx = cl.c[0] + (uint32_t)(b & 1);
  const uint32_t vy = cl.c[1] + (uint32_t)((b >> 1) & 1);
  const uint32_t vz = cl.c[2] + (uint32_t)((b >> 2) & 1);
  if (hashed) return (vx ^ (vy * 2654435761u) ^ (vz * 805459861u)) & (T - 1u);
  const uint32_t n1 = N + 1u;
  return vx + vy * n1 + vz * n1 * n1;
}

__device__ inline float corner_weight(const Cell& cl, int b) {
  const float wx = (b & 1) ? cl.f[0] : 1.0f - cl.f[0];
  const float wy = (b & 2) ? cl.f[1] : 1.0f - cl.f[1];
  const float wz = (b & 4) ? cl.f[2] : 1.0f - cl.f[2];
  return (wx * wy) * wz;
}

// All 8 corner indices of a cell, with the products shared between corners:
// (c + 1) * P = c * P + P mod 2^32 for the hash, and the dense index of
// corner b is the cell's index plus b's offsets.  Same values as corner_index
// for slot b ^ flip: flip = 0 gives the corners in order b, flip = the
// cell's coordinate parities gives parity slots (slot q is the corner whose
// vertex has parities q, the same slot in every cell sharing that vertex).
__device__ inline void cell_corners(const Cell& cl, uint32_t N, uint32_t T, bool hashed,
                                    uint32_t idx[8], uint32_t flip = 0u) {
  // per axis, the two vertex offsets in slot order
  const uint32_t fx = flip & 1u, fy = (flip >> 1) & 1u, fz = (flip >> 2) & 1u;
  if (hashed) {
    const uint32_t xa = cl.c[0], ya = cl.c[1] * 2654435761u, za = cl.c[2] * 805459861u;
    const uint32_t xb = xa + 1u, yb = ya + 2654435761u, zb = za + 805459861u;
    const uint32_t x0 = fx ? xb : xa, x1 = fx ? xa : xb;
    const uint32_t y0 = fy ? yb : ya, y1 = fy ? ya : yb;
    const uint32_t z0 = fz ? zb : za, z1 = fz ? za : zb;
    const uint32_t m = T - 1u;
    idx[0] = (x0 ^ y0 ^ z0) & m;
    idx[1] = (x1 ^ y0 ^ z0) & m;
    idx[2] = (x0 ^ y1 ^ z0) & m;
    idx[3] = (x1 ^ y1 ^ z0) & m;
    idx[4] = (x0 ^ y0 ^ z1) & m;
    idx[5] = (x1 ^ y0 ^ z1) & m;
    idx[6] = (x0 ^ y1 ^ z1) & m;
    idx[7] = (x1 ^ y1 ^ z1) & m;
  } else {
    const uint32_t n1 = N + 1u, n2 = n1 * n1;
    const uint32_t b0 = cl.c[0] + cl.c[1] * n1 + cl.c[2] * n2;
    const uint32_t ox[2] = {fx, 1u - fx}, oy[2] = {fy * n1, (1u - fy) * n1},
                   oz[2] = {fz * n2, (1u - fz) * n2};
#pragma unroll
    for (int b = 0; b < 8; ++b) idx[b] = b0 + ox[b & 1] + oy[(b >> 1) & 1] + oz[b >> 2];
  }
}

// All 8 trilinear weights, (wx * wy) * wz as corner_weight, sharing wx * wy,
// in the slots of cell_corners with the same flip.
__device__ inline void cell_weights(const Cell& cl, float w[8], uint32_t flip = 0u) {
  const float gx = 1.0f - cl.f[0], gy = 1.0f - cl.f[1], gz = 1.0f - cl.f[2];
  const float wx[2] = {(flip & 1u) ? cl.f[0] : gx, (flip & 1u) ? gx : cl.f[0]};
  const float wy[2] = {(flip & 2u) ? cl.f[1] : gy, (flip & 2u) ? gy : cl.f[1]};
  const float wz[2] = {(flip & 4u) ? cl.f[2] : gz, (flip & 4u) ? gz : cl.f[2]};
  float wxy[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) wxy[q] = wx[q & 1] * wy[q >> 1];
#pragma unroll
  for (int b = 0; b < 8; ++b) w[b] = wxy[b & 3] * wz[b >> 2];
}

// the cell's coordinate parities (bit k: c_k & 1)
__device__ inline uint32_t cell_parity(const Cell& cl) {
  return (cl.c[0] & 1u) | ((cl.c[1] & 1u) << 1) | ((cl.c[2] & 1u) << 2);
}

__device__ inline int find_sobj(const StepObj* so, int n, int r) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (so[mid].ray_begin <= r) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Back-projection of pixel (u, v) and clipping to the box [-a, a]:
// pinhole camera, pixel centres at +0.5, unit direction, slab test.
__device__ inline void pixel_ray(const float* M, const float* c, float fx, float fy, float cx,
                                 float cy, int u, int v, const float* half, RayRec& R, int NS) {
  const float x = (((float)u + 0.5f) - cx) / fx;
  const float y = (((float)v + 0.5f) - cy) / fy;
  float dd[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) dd[k] = (M[3 * k + 0] * x + M[3 * k + 1] * y) + M[3 * k + 2];
  const float n = sqrtf((dd[0] * dd[0] + dd[1] * dd[1]) + dd[2] * dd[2]);
  float tmin = -INFINITY, tmax = INFINITY;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    R.d[k] = dd[k] / n;
    R.o[k] = c[k];
    const float inv = 1.0f / R.d[k];
    const float t0 = (-half[k] - R.o[k]) * inv;
    const float t1 = (half[k] - R.o[k]) * inv;
    tmin = fmaxf(tmin, fminf(t0, t1));
    tmax = fminf(tmax, fmaxf(t0, t1));
  }
  const float tn = fmaxf(tmin, 0.0f);
  const bool hit = tmax > tn;
  R.tn = tn;
  R.delta = hit ? (tmax - tn) / (float)NS : 0.0f;
  R.flags = hit ? RM_F_HIT : 0u;
}

// ---------------------------------------------------------------------------
// MLP weights -> MFMA operand images.  For a GEMM Out(M x 16 samples) =
// A(M x K) X(K x 16), operand element (t, q, r, lane) is
// A[16t + lane%16][16q + 4(lane/16) + r]; the FP32 image orders it
// ((t Q + q) 4 + r) 64 + lane (one 16x16x4 operand per 64 contiguous values),
// the BF16 image ((t Q + q) 64 + lane) 4 + r (one 16x16x16 operand per lane)
// when K = 16, and for K a multiple of 32 ((t C + c) 64 + lane) 8 + q8 with
// A[16t + lane%16][32c + (q8 < 4 ? 4g + q8 : 16 + 4g + q8 - 4)], g = lane/16
// (one 16x16x32 operand per lane, in the slot order of Mma<1>).
// Operands 8 + 2(k-1) and 9 + 2(k-1) are the k-th hidden-to-hidden matrix of
// a deeper density MLP (nh hidden layers) and its transpose.
__device__ inline float mlp_A(const float* W, int din, int nh, int gemm, int m, int k) {
  const float* W1 = W;
  const float* Wh = W1 + RM_HIDDEN * din;
  const float* W2 = Wh + (nh - 1) * RM_HH;
  const float* W3 = W2 + RM_DOUT * RM_HIDDEN;
  const float* W4 = W3 + RM_HIDDEN * RM_GEO;
  switch (gemm) {
    case 0: return k < din ? W1[m * din + k] : 0.0f;                 // F1 64 x K1
    case 1: return W2[m * RM_HIDDEN + k];                             // F2 16 x 64
    case 2: return k >= 1 ? W3[m * RM_GEO + (k - 1)] : 0.0f;          // F3 64 x 16
    case 3: return m < 3 ? W4[m * RM_HIDDEN + k] : 0.0f;              // F4 16 x 64
    case 4: return k < 3 ? W4[k * RM_HIDDEN + m] : 0.0f;              // B4 64 x 16
    case 5: return m >= 1 ? W3[k * RM_GEO + (m - 1)] : 0.0f;          // B3 16 x 64
    case 6: return W2[k * RM_HIDDEN + m];                             // B2 64 x 16
    case 7: return m < din ? W1[k * din + m] : 0.0f;                  // B1 K1 x 64
    default: {
      const float* H = Wh + ((gemm - 8) >> 1) * RM_HH;
      return (gemm & 1) ? H[k * RM_HIDDEN + m] : H[m * RM_HIDDEN + k];  // Wh_k^T, Wh_k
    }
  }
}

// Work item j of the packing: operand j % P of object j / P of the launch, in
// RM_PACK_SPLIT parts.  Run by the workgroups of the ray kernels past those of
// the rays (the two have nothing in common but their place in a step: as a
// kernel of its own, eight workgroups per object, it took 8 us of every call).
#define RM_PACK_SPLIT 4
__device__ inline void pack_weights(const StepArgs& a, int j, int K1) {
  const int part = j % RM_PACK_SPLIT, op = j / RM_PACK_SPLIT;
  const int nh = a.mlp_layers, nops = 8 + 2 * (nh - 1);
  const int so = op / nops, gm = op % nops;
  const ObjStatic& ob = a.objs[a.sobj[so].obj];
  const float* W = (a.params_override ? a.params_override : ob.params) + ob.P_grid;
  const int din = ob.din;
  const int Ms[8] = {64, 16, 64, 16, 64, 16, 64, K1};
  const int Ks[8] = {K1, 64, 16, 64, 16, 64, 16, 64};
  const int offs[8] = {RM_OFF_F1, RM_OFF_F2, RM_OFF_F3, RM_OFF_F4,
                       RM_OFF_B4, RM_OFF_B3, RM_OFF_B2, RM_OFF_B1};
  const int64_t stride = RM_WPACK_NH(nh);
  const int M = gm < 8 ? Ms[gm] : RM_HIDDEN, K = gm < 8 ? Ks[gm] : RM_HIDDEN, Q = K / 16;
  const int off = gm < 8 ? offs[gm] : RM_OFF_HF(1) + (gm - 8) * RM_HH;
  float* o32 = a.wpack32 + so * stride + off;
  uint16_t* o16 = a.wpack16 + so * stride + off;
  const int per = M * K / RM_PACK_SPLIT;  // M K is a multiple of 1024
  for (int j = part * per + threadIdx.x; j < (part + 1) * per; j += blockDim.x) {
    {  // FP32 image
      const int lane = j & 63, r = (j >> 6) & 3, tq = j >> 8;
      const int q = tq % Q, t = tq / Q;
      o32[j] = mlp_A(W, din, nh, gm, 16 * t + (lane & 15), 16 * q + 4 * (lane >> 4) + r);
    }
    if (K % 32 == 0) {  // BF16 image of a 16x16x32 operand (slot order of Mma<1>)
      const int q8 = j & 7, lane = (j >> 3) & 63, tc = j >> 9, C = K / 32;
      const int c = tc % C, t = tc / C, g = lane >> 4;
      const int col = 32 * c + (q8 < 4 ? 4 * g + q8 : 16 + 4 * g + (q8 - 4));
      o16[j] = f2bf(mlp_A(W, din, nh, gm, 16 * t + (lane & 15), col));
    } else {  // BF16 image of a 16x16x16 operand
      const int r = j & 3, lane = (j >> 2) & 63, tq = j >> 8;
      const int q = tq % Q, t = tq / Q;
      o16[j] = f2bf(mlp_A(W, din, nh, gm, 16 * t + (lane & 15), 16 * q + 4 * (lane >> 4) + r));
    }
  }
}

// ---------------------------------------------------------------------------
// K1: ray draw, classification, back-projection, box clipping (Sec. V-B)
template <int NS>
__global__ __launch_bounds__(256) void k_raygen(StepArgs a, int K1) {
  const int nb = (a.n_rays + 255) / 256;
  if ((int)blockIdx.x >= nb) return pack_weights(a, blockIdx.x - nb, K1);
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= a.n_rays) return;
  const int si = find_sobj(a.sobj, a.n_sobj, r);
  const StepObj so = a.sobj[si];
  const ObjStatic& ob = a.objs[so.obj];
  const int local = r - so.ray_begin;
  const uint32_t step = (uint32_t)a.state[so.obj].step;
  uint32_t x[4];
  philox4x32_10(step, (uint32_t)local, 0u, 0u, a.seed_lo ^ (uint32_t)ob.id, a.seed_hi, x);
  const int64_t q = (int64_t)(((uint64_t)x[0] * (uint64_t)ob.n_cand) >> 32);
  int lo = 0, hi = ob.n_kf - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ob.kfs[mid].cand_begin <= q) lo = mid; else hi = mid - 1;
  }
  const KfRef& kr = ob.kfs[lo];
  const int64_t lq = q - kr.cand_begin;
  const int u = kr.x0 + (int)(lq % kr.w);
  const int v = kr.y0 + (int)(lq / kr.w);
  const KfDev kf = a.kfs[kr.kf];
  float crand[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) crand[j] = (float)(x[j + 1] >> 8) * (1.0f / 16777216.0f);
  const int64_t pix = (int64_t)v * kf.W + u;
  const int m = kf.mask[pix];
  const uint32_t cls = (m == ob.instance) ? RM_CLS_OBJECT : (m == 0 ? RM_CLS_BACKGROUND : RM_CLS_OCCLUDER);
  RayRec R;
  pixel_ray(kr.M, kr.c, kf.fx, kf.fy, kf.cx, kf.cy, u, v, ob.half, R, NS);
  R.flags |= cls;
  R.D = 0.0f;
  if (cls == RM_CLS_BACKGROUND) {
#pragma unroll
    for (int j = 0; j < 3; ++j) R.tgt[j] = crand[j];
  } else {
#pragma unroll
    for (int j = 0; j < 3; ++j) R.tgt[j] = (float)kf.rgb[3 * pix + j] / 255.0f;
  }
  if (cls == RM_CLS_OBJECT && kf.depth) {
    const float z = kf.depth[pix];
    if (z > 0.0f && isfinite(z)) {
      // camera z -> distance along the ray, the quantity of Eq. 8
      const float xn = (((float)u + 0.5f) - kf.cx) / kf.fx;
      const float yn = (((float)v + 0.5f) - kf.cy) / kf.fy;
      R.D = z * sqrtf((xn * xn + yn * yn) + 1.0f);
      R.flags |= RM_F_DEPTH;
    }
  }
  R.obj = so.obj;
  R.out = r;
  R.pad1 = 0;
  a.rays[r] = R;
  if (a.dbg_kfuv) {
    a.dbg_kfuv[3 * r + 0] = lo;
    a.dbg_kfuv[3 * r + 1] = u;
    a.dbg_kfuv[3 * r + 2] = v;
  }
}

// Rays of n_pix pixels of a camera from pix0 on, for rendering (class "object",
// no target).
struct CamArgs {
  float M[9], c[3];
  float fx, fy, cx, cy;
  int W, pix0;
};

// The pixels whose ray misses the box get their outputs here; the others are
// appended to the ray records (*n_hit counts them; their order, wave by wave,
// depends on timing, the outputs do not), so that the gather and the field
// kernel run over hits alone.
template <int NS>
__global__ __launch_bounds__(256) void k_camera_rays(StepArgs a, CamArgs ca, int n_pix, int* n_hit,
                                                     int K1) {
  const int nb = (n_pix + 255) / 256;
  if ((int)blockIdx.x >= nb) return pack_weights(a, blockIdx.x - nb, K1);
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = r < n_pix;
  const int p = ca.pix0 + (in ? r : n_pix - 1);
  const int obj = a.sobj[0].obj;
  RayRec R;
  pixel_ray(ca.M, ca.c, ca.fx, ca.fy, ca.cx, ca.cy, p % ca.W, p / ca.W, a.objs[obj].half, R, NS);
  const bool hit = in && (R.flags & RM_F_HIT);
  if (in && !hit) {
    if (a.out_rgb) a.out_rgb[3 * (int64_t)p] = a.out_rgb[3 * (int64_t)p + 1] = a.out_rgb[3 * (int64_t)p + 2] = 0.0f;
    if (a.out_depth) a.out_depth[p] = 0.0f;
    if (a.out_tend) a.out_tend[p] = a.out_opacity ? 0.0f : 1.0f;
  }
  const uint64_t m = __ballot(hit);
  if (m == 0ull) return;
  const int lane = threadIdx.x & 63;
  int first = 0;
  if (lane == 0) first = atomicAdd(n_hit, __popcll(m));
  first = __builtin_amdgcn_readfirstlane(first);
  if (!hit) return;
  R.flags |= RM_CLS_OBJECT;
  R.tgt[0] = R.tgt[1] = R.tgt[2] = 0.0f;
  R.D = 0.0f;
  R.obj = obj;
  R.out = p;
  R.pad1 = 0;
  a.rays[first + __popcll(m & ((1ull << lane) - 1ull))] = R;
}

// caller-given rays (o, d, t_near, t_far) in the object frame
template <int NS>
__global__ __launch_bounds__(256) void k_user_rays(StepArgs a, const float* rays, int K1) {
  const int nb = (a.n_rays + 255) / 256;
  if ((int)blockIdx.x >= nb) return pack_weights(a, blockIdx.x - nb, K1);
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= a.n_rays) return;
  const float* q = rays + 8 * (int64_t)r;
  RayRec R;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    R.o[k] = q[k];
    R.d[k] = q[3 + k];
  }
  const float tn = q[6], tf = q[7];
  const bool hit = tf > tn;
  R.tn = tn;
  R.delta = hit ? (tf - tn) / (float)NS : 0.0f;
  R.flags = (hit ? RM_F_HIT : 0u) | RM_CLS_OBJECT;
  R.tgt[0] = R.tgt[1] = R.tgt[2] = 0.0f;
  R.D = 0.0f;
  R.obj = a.sobj[0].obj;
  R.out = r;
  R.pad1 = 0;
  a.rays[r] = R;
}

// Occupancy skip: the live samples of every ray, one bit each (one word per 64
// samples, the low half of one for 32), tested once here for the gather's 16
// levels, the field kernel and the binning.  Launched when an object of the
// launch has occupancy bits.
template <int NS>
__global__ __launch_bounds__(256) void k_live(StepArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t n = (int64_t)a.n_rays * NS, stride = (int64_t)gridDim.x * 256;
  for (int64_t k = (int64_t)blockIdx.x * 256 + (threadIdx.x - lane); k < n; k += stride) {
    const int64_t s = k + lane;
    const int ray = (int)(s / NS);
    bool on = false;
    if (ray < a.n_rays) {
      const RayRec& R = a.rays[ray];
      if (ray_active(R.flags)) {
        const ObjStatic& ob = a.objs[R.obj];
        on = true;
        if (ob.occ) {
          float p[3];
          sample_pos(R, (int)(s % NS), ob.half, ob.inv2a, p);
          on = occupied(ob.occ, p);
        }
      }
    }
    const uint64_t m = __ballot(on);
    if constexpr (NS >= 64) {
      if (lane == 0) a.live[(int64_t)ray * a.live_step + (s % NS) / 64] = m;
    } else {
      if ((lane & 31) == 0 && ray < a.n_rays)
        a.live[(int64_t)ray * a.live_step] = (lane & 32) ? m >> 32 : m & 0xFFFFFFFFull;
    }
  }
}

// ---------------------------------------------------------------------------
// K2: encoding forward.  One workgroup per block of RM_SCAT_WG samples of one
// (object, level) pair, blocks ordered object by object and level by level
// within an object, so the chip sweeps one table at a time; the object and
// level are uniform in a workgroup.  Each wave takes chunks of 64 samples, whose
// ray (and everything else that is uniform) comes through the scalar cache, so
// that the vector memory path serves the table alone.  Fine levels are bound
// by line fills from the L2: 65536 rays x 64 samples on one hashed level of
// 2^19 entries take 83 us (210 G lines/s, of 265 G/s that random loads reach on
// this chip) against 94 with one lane per corner pair; coarse dense levels by
// instruction issue: 24 us against 40.  16 levels of 16..1024 cells: 930 us
// against 1112.

// Features of the 8 corners of each lane's cell, in the slots of cell_corners
// with `flip`, on a dense level: the two corners of an x-pair are neighbouring
// entries, the lower at c_x, and one 16-byte load brings both.  Lanes that
// are not `live` read the cell at the origin.
__device__ inline void gather_dense(const gptr<const char> G, const Cell& cl, uint32_t N, bool live,
                                    uint32_t flip, float2 g[8]) {
  const uint32_t n1 = N + 1u, n2 = n1 * n1;
  const uint32_t b0 = live ? cl.c[0] + cl.c[1] * n1 + cl.c[2] * n2 : 0u;
  const uint32_t y0 = (flip & 2u) ? n1 : 0u, z0 = (flip & 4u) ? n2 : 0u;
  const uint32_t b1 = b0 + z0, b2 = b0 + (n2 - z0), y1 = n1 - y0;
  const uint32_t row[4] = {b1 + y0, b1 + y1, b2 + y0, b2 + y1};
  rm_f4v v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = *(gptr<const rm_f4v>)(G + (row[q] << 3));
  const bool up = flip & 1u;  // the lower entry is slot 1 of the pair
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    g[2 * q].x = up ? v[q][2] : v[q][0];
    g[2 * q].y = up ? v[q][3] : v[q][1];
    g[2 * q + 1].x = up ? v[q][0] : v[q][2];
    g[2 * q + 1].y = up ? v[q][1] : v[q][3];
  }
}

// The same on a hashed level.  x enters the hash with factor 1, so the two
// entries of an x-pair differ in the trailing ones of c_x and the bit above
// and lie in the same 128 B line 15 times in 16.  Two neighbouring lanes load
// the two corners of one lane's pair in one instruction, which then asks for
// 32 lines and not 64 (line fills from the L2, 2.3 clocks each per CU, bound
// this kernel on the fine levels): first the pairs of the even lanes' samples
// (A), then those of the odd lanes' (B).  Indices are kept as byte offsets.
// Every lane of the wave takes part; lanes that are not `live` read entry 0.
template <bool FLIP>
__device__ inline void gather_hashed(const gptr<const char> G, const Cell& cl, uint32_t T, bool live,
                                     uint32_t flip, uint32_t odd, float2 g[8]) {
  const uint32_t ya = cl.c[1] * (2654435761u << 3), za = cl.c[2] * (805459861u << 3);
  const uint32_t yb = ya + (2654435761u << 3), zb = za + (805459861u << 3);
  const uint32_t y0 = FLIP && (flip & 2u) ? yb : ya, y1 = FLIP && (flip & 2u) ? ya : yb;
  const uint32_t z0 = FLIP && (flip & 4u) ? zb : za, z1 = FLIP && (flip & 4u) ? za : zb;
  const uint32_t yz[4] = {y0 ^ z0, y1 ^ z0, y0 ^ z1, y1 ^ z1};
  // x of this lane's corner: slot `odd` of the cell of lane A or B
  const uint32_t ca = pair_even(cl.c[0]), cb = pair_odd(cl.c[0]);
  const uint32_t xa = (ca + (FLIP ? (odd ^ ca) & 1u : odd)) << 3;
  const uint32_t xb = (cb + (FLIP ? (odd ^ cb) & 1u : odd)) << 3;
  const uint32_t m = live ? (T - 1u) << 3 : 0u, ma = pair_even(m), mb = pair_odd(m);
  rm_f2v va[4], vb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) va[q] = *(gptr<const rm_f2v>)(G + ((xa ^ pair_even(yz[q])) & ma));
#pragma unroll
  for (int q = 0; q < 4; ++q) vb[q] = *(gptr<const rm_f2v>)(G + ((xb ^ pair_odd(yz[q])) & mb));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    // exchanged with every lane active, then chosen
    const float2 sa = make_float2(pair_swap(va[q][0]), pair_swap(va[q][1]));
    const float2 sb = make_float2(pair_swap(vb[q][0]), pair_swap(vb[q][1]));
    g[2 * q].x = odd ? sb.x : va[q][0];
    g[2 * q].y = odd ? sb.y : va[q][1];
    g[2 * q + 1].x = odd ? vb[q][0] : sa.x;
    g[2 * q + 1].y = odd ? vb[q][1] : sa.y;
  }
}

// Live samples of the 64 from sample k (a multiple of 64) of ray ray0 on, one
// bit each (k_live); all ones where nothing is skipped.  Rays past the
// launch's read the last one's.
template <int NS>
__device__ inline uint64_t live_word(const StepArgs& a, int ray0, int k) {
  if (!a.live) return ~0ull;
  const int ray = ray0 + k / NS;
  const cptr<uint64_t> q = as_const(a.live);
  if constexpr (NS >= 64) {
    return q[(int64_t)(ray < a.n_rays ? ray : a.n_rays - 1) * a.live_step + (k % NS) / 64];
  } else {
    const uint64_t lo = q[(int64_t)(ray < a.n_rays ? ray : a.n_rays - 1) * a.live_step];
    const uint64_t hi = q[(int64_t)(ray + 1 < a.n_rays ? ray + 1 : a.n_rays - 1) * a.live_step];
    return (lo & 0xFFFFFFFFull) | (hi << 32);
  }
}

// Sample block j of a launch: from the table, or of one object by arithmetic
// (its pairs all have a.one_nb blocks), so that a call on one object uploads
// no table that grows with its rays.
__device__ inline BinBlock block_of(const StepArgs& a, int j) {
  BinBlock b;
  if (a.one_nb) {
    b.pair = j / a.one_nb;
    b.blk = j - b.pair * a.one_nb;
  } else {
    const cptr<BinBlock> q = as_const(a.bblocks + j);
    b.pair = q->pair;
    b.blk = q->blk;
  }
  return b;
}

// One level's encoding of the samples at p (unit cube) of a wave's live lanes,
// added up in slot order; all lanes of the wave call it.
__device__ inline void encode_wave(const gptr<const char> G, uint32_t N, uint32_t T, bool hashed,
                                   bool touch, bool live, const float p[3], uint32_t odd, float& ex,
                                   float& ey) {
  Cell cl;
  make_cell(p, N, cl);  // valid indices for every lane: p is clamped
  float2 g[8];
  float w[8];
  if (hashed && !touch) {
    gather_hashed<false>(G, cl, T, live, 0u, odd, g);
    cell_weights(cl, w);
  } else {
    // on levels where consecutive samples of a ray touch, parity slots: a
    // vertex two lanes share is then loaded by one instruction at one address
    const uint32_t flip = touch ? cell_parity(cl) : 0u;
    if (hashed) gather_hashed<true>(G, cl, T, live, flip, odd, g);
    else gather_dense(G, cl, N, live, flip, g);
    cell_weights(cl, w, flip);
  }
  float x = 0.0f, y = 0.0f;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    x = fmaf(w[b], g[b].x, x);
    y = fmaf(w[b], g[b].y, y);
  }
  ex = live ? x : 0.0f;
  ey = live ? y : 0.0f;
}

template <int NS>
__global__ __launch_bounds__(512) void k_encode_fwd(StepArgs a) {
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t j = gtid; j < a.n_regions; j += (int64_t)gridDim.x * blockDim.x)
    a.bin_count[j] = 0;  // fresh fill counters for the binned scatter of this pass
  // Training steps: each object's Adam step advances, after the ray draw, which
  // uses the step as its counter, and before any Adam update.
  if (a.fuse_adam && gtid < a.n_sobj) {
    ObjState* st = a.state + a.sobj[gtid].obj;
    const int kk = st->step + 1;
    st->step = kk;
    st->bc1 = (float)(1.0 - pow((double)a.beta1, (double)kk));
    st->bc2 = (float)(1.0 - pow((double)a.beta2, (double)kk));
  }
  // Workgroup i runs on XCD i mod 8; numbered so that each XCD takes a
  // contiguous range of (object, level) blocks, a level's table is gathered
  // by one XCD at a time and stays in its L2: the L2 hit rate goes from 0.67
  // to 0.93 and the lines fetched beyond the L2 from 2.8 to 0.5 GB per step
  // on the 24-object workload.  The kernel alone is no faster (the XCDs' ranges
  // differ in cost), but the bandwidth it no longer takes goes to the other
  // object group's kernels: 1.812 -> 1.800 ms per step when this was built.
  const int per_xcd = (a.n_bblocks + 7) >> 3;
  const int jw = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
  if (jw >= a.n_bblocks) return;
  const BinBlock bb = block_of(a, jw);
  const int blk = bb.blk;
  const cptr<BinPair> bp = as_const(a.bpairs + bb.pair);
  const cptr<ObjStatic> ob = as_const(a.objs + bp->obj);
  const int ray0 = bp->ray_begin + (int)((int64_t)blk * RM_SCAT_WG / NS);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int waves = (int)blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const uint32_t odd = lane & 1;
  const float* Gp = (a.params_override ? a.params_override : ob->params) + bp->off;
  const gptr<const char> G = as_global((const char*)Gp);
  const float half[3] = {ob->half[0], ob->half[1], ob->half[2]};
  const float inv[3] = {ob->inv2a[0], ob->inv2a[1], ob->inv2a[2]};
  const uint32_t N = bp->N, T = bp->T;
  const bool touch = bp->touch, hashed = bp->hashed;
  const int64_t left = bp->n_samples - (int64_t)blk * RM_SCAT_WG;  // samples from here on
  const int n = left < RM_SCAT_WG ? (int)left : RM_SCAT_WG;
  const int64_t at = (int64_t)bp->l * a.S + bp->s_begin + (int64_t)blk * RM_SCAT_WG;
  RayGeo Rn = wave_ray<NS>(a.rays, a.n_rays, ray0, 64 * wave, lane);
  for (int k = 64 * wave; k < n; k += 64 * waves) {
    const RayGeo R = Rn;
    // the next chunk's ray, in flight during this one
    Rn = wave_ray<NS>(a.rays, a.n_rays, ray0, k + 64 * waves, lane);
    const bool act = k + lane < n && ray_active(R.flags);
    const bool live = act && ((live_word<NS>(a, ray0, k) >> lane) & 1ull);
    if (__ballot(live) == 0ull) continue;  // nothing reads a chunk without live samples
    float p[3];
    sample_pos(R, (k + lane) & (NS - 1), half, inv, p);
    float ex, ey;  // zero for a skipped sample
    encode_wave(G, N, T, hashed, touch, live, p, odd, ex, ey);
    if (!act) continue;
    if (a.e_bf16)  // the BF16 MLP reads the encoding rounded to BF16, nothing else
      ((uint32_t*)a.e + at + k)[lane] = pack_bf16x2(ex, ey);
    else
      (a.e + at + k)[lane] = make_float2(ex, ey);
  }
}

// One Adam update of parameter p with gradient g (moments m, v; bias
// corrections bc1, bc2 of the step).
__device__ inline void adam1(float& p, float& m, float& v, float g, const StepArgs& a, float bc1,
                             float bc2) {
  m = a.beta1 * m + (1.0f - a.beta1) * g;
  v = a.beta2 * v + (1.0f - a.beta2) * (g * g);
  p -= a.lr * (m / bc1) / (sqrtf(v / bc2) + a.eps);
}

// Adam on the two features of the table entry at float offset off, with
// gradient (gx, gy); the object's step has been advanced by the gather kernel.
__device__ inline void adam_entry(const ObjStatic& ob, int64_t off, float gx, float gy,
                                  const StepArgs& a, float bc1, float bc2) {
  float2 p = *(float2*)(ob.params + off), m = *(float2*)(ob.m + off), v = *(float2*)(ob.v + off);
  adam1(p.x, m.x, v.x, gx, a, bc1, bc2);
  adam1(p.y, m.y, v.y, gy, a, bc1, bc2);
  *(float2*)(ob.params + off) = p;
  *(float2*)(ob.m + off) = m;
  *(float2*)(ob.v + off) = v;
}

// ---------------------------------------------------------------------------
// K6: encoding backward, grad[idx_b] += w_b * de for the 8 corners of every
// sample, as a binned scatter.  Float atomics on a table cost per cache line
// an instruction touches, and on the fine levels no two samples of a ray
// share a cell, so direct atomics are bound by one line per corner.  Instead
// the (entry, value) records are sorted into regions of 2^region_bits entries,
// and workgroups per region sum them in LDS and update the region of the
// gradient with coalesced memory operations:
//   k_bin_scatter  per block of samples: rank the records per region, reserve
//                  space in the regions' bins, write them out sorted by region
//                  (a full bin falls back to atomics)
//   k_bin_acc      K workgroups per region: LDS sums, then the gradient
//                  region is updated (plain stores when K = 1 -- the gradient
//                  is zero on entry -- atomics on consecutive entries
//                  otherwise, and read-modify-write if the bin overflowed)
// The bins' fill counters are zeroed by the gather kernel of the same pass.

// Two formats of records, by level.
//
// Corner record (8 B): the two feature values of one corner, each rounded to
// nearest at 17 mantissa bits (a change of at most 2^-18 of the value; the
// sums are then taken to about 2^-38 of an entry's largest term), with the
// entry's index within its region (RM_RB_BITS <= 12 bits) in the 6 mantissa
// bits freed in each.  Zero stays zero, infinities and NaNs keep their class.
//
// Pair record (12 B, BinPair::pairs): an x-pair of corners on a hashed level.
// Its two entries differ by XOR with 2^kind - 1 (x enters the hash with
// factor 1: the trailing ones of c_x and the bit above) and lie in the same
// region, and their values are (1 - s) A and s A with s <= 1/2 the smaller of
// the pair's two x weights.  Held: A (both features, 18 mantissa bits) and s
// (20), the index of the entry that takes 1 - s in 5 + 5 + 1 freed bits, kind
// in 2 freed bits of s and its two top bits (clear, as 0 <= s <= 1/2).  Each
// value is off by at most 2^-19 + 2^-21 of itself.
static_assert(RM_RB_BITS == 11, "a pair record holds 11 index bits");

__device__ inline uint32_t rec_round(float x) { return (__float_as_uint(x) + 0x20u) & ~0x3Fu; }

__device__ inline float2 rec_pack(float2 v, uint32_t e) {
  return make_float2(__uint_as_float(rec_round(v.x) | (e & 0x3Fu)),
                     __uint_as_float(rec_round(v.y) | ((e >> 6) & 0x3Fu)));
}

__device__ inline uint32_t rec_entry(float x, float y) {
  return (__float_as_uint(x) & 0x3Fu) | ((__float_as_uint(y) & 0x3Fu) << 6);
}

__device__ inline float rec_value(float x) { return __uint_as_float(__float_as_uint(x) & ~0x3Fu); }

struct PairRec {
  float ax, ay, s;
};

__device__ inline PairRec pair_pack(float ax, float ay, uint32_t sw, uint32_t e) {
  PairRec r;
  r.ax = __uint_as_float(((__float_as_uint(ax) + 0x10u) & ~0x1Fu) | (e & 0x1Fu));
  r.ay = __uint_as_float(((__float_as_uint(ay) + 0x10u) & ~0x1Fu) | ((e >> 5) & 0x1Fu));
  r.s = __uint_as_float(sw | ((e >> 10) & 1u));
  return r;
}

// the s word without its index bit: s rounded, and kind (1..11)
__device__ inline uint32_t pair_sword(float s, uint32_t kind) {
  return ((__float_as_uint(s) + 4u) & ~7u) | ((kind & 3u) << 1) | ((kind >> 2) << 30);
}

__device__ inline void pair_entries(const PairRec& r, uint32_t& e, uint32_t& o) {
  const uint32_t x = __float_as_uint(r.ax), y = __float_as_uint(r.ay), w = __float_as_uint(r.s);
  e = (x & 0x1Fu) | ((y & 0x1Fu) << 5) | ((w & 1u) << 10);
  const uint32_t kind = ((w >> 1) & 3u) | ((w >> 30) << 2);
  o = e ^ ((1u << kind) - 1u);
}

__device__ inline float pair_s(const PairRec& r) {
  return __uint_as_float(__float_as_uint(r.s) & 0x3FFFFFF8u);
}

__device__ inline float pair_a(float x) { return __uint_as_float(__float_as_uint(x) & ~0x1Fu); }

// Stores of data that no kernel reads back while it could still be in the
// L2 (corner records, read by the next kernel after the whole scatter;
// parameters and moments after their Adam update): written past the L2's
// allocation (measured: the accumulation that follows runs 6 % faster).
__device__ inline void nt_store2(float2* p, float2 v) {
  rm_f2v w;
  w[0] = v.x;
  w[1] = v.y;
  __builtin_nontemporal_store(w, (rm_f2v*)p);
}
typedef int rm_i3v __attribute__((ext_vector_type(3), aligned(4)));

// Shared corners of consecutive samples.  Cells c and n = c + d share a
// vertex only if |d| <= 1 on every axis; corner b of c (vertex c + bits(b))
// is then a corner of n where d is 0, or where d = +1 and bit b is 1, or
// d = -1 and bit b is 0.
__device__ inline uint32_t shared_corners(int c0, int c1, int c2, int n0, int n1, int n2) {
  const int d0 = n0 - c0, d1 = n1 - c1, d2 = n2 - c2;
  if (abs(d0) > 1 || abs(d1) > 1 || abs(d2) > 1) return 0u;
  const uint32_t m = (uint32_t)(d0 != 0) | ((uint32_t)(d1 != 0) << 1) | ((uint32_t)(d2 != 0) << 2);
  const uint32_t up = (uint32_t)(d0 > 0) | ((uint32_t)(d1 > 0) << 1) | ((uint32_t)(d2 > 0) << 2);
  uint32_t r = 0u;
#pragma unroll
  for (int b = 0; b < 8; ++b) r |= (uint32_t)(((uint32_t)b & m) == up) << b;
  return r;
}

// Parity slots: slot q of a cell holds its corner b = q ^ pc, pc the
// cell's coordinate parities (bit k: c_k & 1), so slot q is the corner whose
// vertex has parities q, and a vertex takes the same slot in every cell it
// is a corner of.  Corner b and corner b ^ 1 stay an x-pair.

// bit b of the result is bit b ^ m of x (8 bits)
__device__ inline uint32_t xor_permute_bits(uint32_t x, uint32_t m) {
  if (m & 1u) x = ((x & 0x55u) << 1) | ((x >> 1) & 0x55u);
  if (m & 2u) x = ((x & 0x33u) << 2) | ((x >> 2) & 0x33u);
  if (m & 4u) x = ((x & 0x0Fu) << 4) | ((x >> 4) & 0x0Fu);
  return x;
}

// the value of lane + O (undefined past the wave's last lane)
template <int O>
__device__ inline int lane_down(int x) {
  if constexpr (O == 1) return dppi<0x130>(x);  // wave_shl:1
  else return __shfl_down(x, O, 64);
}

template <int O>
__device__ inline float lane_down_f(float x) {
  return __int_as_float(lane_down<O>(__float_as_int(x)));
}

// One step of a segmented suffix sum over chains of lanes, in parity slots.
// Bit q of open says that the sum in v[q] covers lanes lane .. lane + O - 1
// of its vertex's chain and the chain goes on; the sum of lane + O (the
// same slot there) is added and the chain's end there carried over.
// Returns false, adding nothing, once no chain of the wave is open.
template <int O>
__device__ inline bool chain_step(float2 v[8], uint32_t& open) {
  if (__ballot(open != 0u) == 0ull) return false;
  float2 y[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) y[q] = make_float2(lane_down_f<O>(v[q].x), lane_down_f<O>(v[q].y));
  const uint32_t yo = (uint32_t)lane_down<O>((int)open);
#pragma unroll
  for (int q = 0; q < 8; ++q)
    if ((open >> q) & 1u) {
      v[q].x += y[q].x;
      v[q].y += y[q].y;
    }
  open &= yo;
  return true;
}

// Exclusive scan of cnt[0..n) into at[0..n).x by a whole block of WG threads
// (n / WG entries each); returns the total to every thread.  at[j].y of the thread's
// own entry (n <= WG) is set to y.
template <int WG>
__device__ inline int block_exclusive_scan(const int* cnt, int2* at, int n, int y, int* s_wsum) {
  constexpr int NW = WG / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n + WG - 1) / WG;  // contiguous entries per thread
  const int j0 = tid * per;
  int mine = 0;
  for (int j = j0; j < j0 + per && j < n; ++j) mine += cnt[j];
  const int inc = wave_incl_prefix_i(mine);
  if (lane == 63) s_wsum[wave] = inc;
  __syncthreads();
  int woff = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    woff += w < wave ? s_wsum[w] : 0;
    tot += s_wsum[w];
  }
  int run = woff + inc - mine;
  if (per == 1) {
    if (tid < n) at[tid] = make_int2(run, y);
  } else {
    for (int j = j0; j < j0 + per && j < n; ++j) {
      at[j].x = run;
      run += cnt[j];
    }
  }
  __syncthreads();
  return tot;
}

// One block: RM_SCAT_WG samples of one (object, level) pair, up to 4 pair or 8
// corner records each.  The records are ranked per region in LDS, each
// region's share of the block is reserved in its bin with one global atomic,
// and the records, sorted by region through LDS with their slots, are written
// out with consecutive lanes on consecutive slots.  Records beyond a bin's
// capacity go to the gradient directly (atomics).  The order of records
// inside a bin depends on timing; the fixed-point region sums do not.
//
// A pair record halves the ranking, staging and storing of two corner records
// and takes 12 B for their 16: vector instructions of a block 43.9 M -> 27.7 M
// on 4096 rays x 64 samples x 16 levels, 83 -> 74 us; 24 objects 467 -> 383 us.
// What bounds it then is writing short runs: stores kept in the L2, where the
// next block of the same XCD completes the lines.
// Staging: 32 KB, so that four blocks fit a CU: all pair records, and
// RM_STAGE_CORNERS corner records (a block's further ones, on levels where
// hardly any merge, are stored straight to their slots).  Four blocks also
// leave a thread 64 registers: 4 of them spill (16 B of scratch a lane).
template <int NS, int RB>
__global__ __launch_bounds__(RM_SCAT_WG) __attribute__((amdgpu_waves_per_eu(8))) void k_bin_scatter(
    StepArgs a) {
  // dynamic LDS: staging of the sorted records, then two per-region arrays of
  // a.bin_max_R entries
  extern __shared__ __align__(16) char dyn[];
  int2* rg = (int2*)(dyn + RM_STAGE_BYTES);  // first staging position; first slot reserved
  int* lcnt = (int*)(rg + a.bin_max_R);      // records of the block per region
  __shared__ int s_wsum[RM_SCAT_WG / 64];
  // Workgroup i runs on XCD i mod 8: numbered so that each XCD takes a
  // contiguous range of blocks, the blocks of a pair then reserve space in
  // that pair's bins from one XCD and fill them in block order (measured:
  // this kernel 3 % and the accumulation that reads the bins 6 % faster
  // than with consecutive blocks spread over the XCDs).
  const int per_xcd = (a.n_bblocks + 7) >> 3;
  const int jb = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
  if (jb >= a.n_bblocks) return;
  const BinBlock bb = block_of(a, a.bb_begin + jb);
  const int blk = bb.blk;
  const cptr<BinPair> bp = as_const(a.bpairs + bb.pair);
  const cptr<ObjStatic> ob = as_const(a.objs + bp->obj);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = bp->R, cap = bp->cap;
  constexpr uint32_t em = (1u << RB) - 1u;  // entry within its region
  for (int r = tid; r < R; r += RM_SCAT_WG) lcnt[r] = 0;
  const int64_t k0 = (int64_t)blk * RM_SCAT_WG;
  const int ray0 = bp->ray_begin + (int)(k0 / NS);
  const uint64_t lw = live_word<NS>(a, ray0, 64 * wave);
  const bool in = k0 + tid < bp->n_samples && ((lw >> lane) & 1ull);
  const int64_t at = (int64_t)bp->l * a.S + bp->s_begin + k0;
  const float2 g = in ? (a.de + at)[tid] : make_float2(0.0f, 0.0f);
  const RayGeo ray = wave_ray<NS>(a.rays, a.n_rays, ray0, 64 * wave, lane);
  const float half[3] = {ob->half[0], ob->half[1], ob->half[2]};
  const float inv[3] = {ob->inv2a[0], ob->inv2a[1], ob->inv2a[2]};
  const uint32_t N = bp->N, T = bp->T;
  const bool hashed = bp->hashed, pairs = bp->pairs, merge = bp->merge;
  float* gl = (a.grad_override ? a.grad_override : ob->grad) + bp->off;
  float* rec = a.rec + bp->rec_base;
  int* const bin_count = a.bin_count + bp->bin_base;
  __syncthreads();
  const bool has = in && ray_active(ray.flags) && (g.x != 0.0f || g.y != 0.0f);
  Cell cl;
  {
    float p[3];
    sample_pos(ray, (64 * wave + lane) & (NS - 1), half, inv, p);
    make_cell(p, N, cl);
  }
  // Reserves the block's share of each bin after the ranking; with at most
  // one region per thread the reservations are in flight through the scan
  // (the barriers wait for LDS operations only).
  auto place = [&]() {
    __syncthreads();
    int mine = 0;
    const bool one = R <= RM_SCAT_WG;
    if (one && tid < R && lcnt[tid]) mine = atomicAdd(&bin_count[tid], lcnt[tid]);
    if (!one)
      for (int r = tid; r < R; r += RM_SCAT_WG)
        rg[r].y = lcnt[r] ? atomicAdd(&bin_count[r], lcnt[r]) : 0;
    return block_exclusive_scan<RM_SCAT_WG>(lcnt, rg, R, mine, s_wsum);
  };
  if (pairs) {
    uint32_t idx[4];
    float2 av[4];
    int rank[4];
    float s = 0.0f;  // the smaller x weight
    const uint32_t m = T - 1u;
    if (has) {
      const uint32_t ya = cl.c[1] * 2654435761u, za = cl.c[2] * 805459861u;
      const uint32_t yb = ya + 2654435761u, zb = za + 805459861u;
      const bool up = cl.f[0] > 0.5f;  // the corner at c_x + 1 takes the larger weight
      const uint32_t x = cl.c[0] + (up ? 1u : 0u);
      idx[0] = (x ^ ya ^ za) & m;
      idx[1] = (x ^ yb ^ za) & m;
      idx[2] = (x ^ ya ^ zb) & m;
      idx[3] = (x ^ yb ^ zb) & m;
      const float gy = 1.0f - cl.f[1], gz = 1.0f - cl.f[2];
      const float w[4] = {gy * gz, cl.f[1] * gz, gy * cl.f[2], cl.f[1] * cl.f[2]};
#pragma unroll
      for (int q = 0; q < 4; ++q) av[q] = make_float2(w[q] * g.x, w[q] * g.y);
      s = up ? 1.0f - cl.f[0] : cl.f[0];
#pragma unroll
      for (int q = 0; q < 4; ++q) rank[q] = atomicAdd(&lcnt[idx[q] >> RB], 1);
    }
    const int n = place();
    int4* stage = (int4*)dyn;  // slot within the pair's records, then the record
    if (has) {
      const uint32_t diff = (cl.c[0] ^ (cl.c[0] + 1u)) & m;  // 2^kind - 1
      const uint32_t sw = pair_sword(s, (uint32_t)__popc(diff));
      int2 b[4];  // all four first: one LDS round trip
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = rg[idx[q] >> RB];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int slot = b[q].y + rank[q];
        const PairRec r = pair_pack(av[q].x, av[q].y, sw, idx[q] & em);
        const bool fits = slot < cap;
        stage[b[q].x + rank[q]] =
            make_int4(fits ? (int)(idx[q] >> RB) * cap + slot : -1, __float_as_int(r.ax),
                      __float_as_int(r.ay), __float_as_int(r.s));
        if (!fits) {  // bin full: direct atomics of the unrounded values (only slower)
          const uint32_t o = idx[q] ^ diff;
          unsafeAtomicAdd(gl + 2 * (int64_t)idx[q], (1.0f - s) * av[q].x);
          unsafeAtomicAdd(gl + 2 * (int64_t)idx[q] + 1, (1.0f - s) * av[q].y);
          unsafeAtomicAdd(gl + 2 * (int64_t)o, s * av[q].x);
          unsafeAtomicAdd(gl + 2 * (int64_t)o + 1, s * av[q].y);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = tid + u * RM_SCAT_WG;
      if (j < n) {
        const int4 v = stage[j];
        // kept in the L2 (past it, runs of 12-byte records cost partial line
        // writes: 97 us against 73 on 4096 rays x 64 samples, 16 levels)
        if (v.x >= 0) {
          rm_i3v w;
          w[0] = v.y;
          w[1] = v.z;
          w[2] = v.w;
          *(rm_i3v*)(rec + 3 * (int64_t)v.x) = w;
        }
      }
    }
    return;
  }
  float2 v[8];
  // in parity slots where corners are merged
  const uint32_t flip = merge ? cell_parity(cl) : 0u;
  {
    float w[8];
    cell_weights(cl, w, flip);
#pragma unroll
    for (int b = 0; b < 8; ++b)
      v[b] = has ? make_float2(w[b] * g.x, w[b] * g.y) : make_float2(0.0f, 0.0f);
  }
  uint32_t keep = has ? 0xFFu : 0u;  // bit b: corner b is written as a record
  if (merge) {
    // Consecutive samples of a ray (consecutive lanes) share corners where
    // their cells touch, and runs of samples share a whole cell.  A vertex's
    // occurrences along the ray form a chain of lanes linked corner to
    // corner; every chain is summed into its first lane (a segmented suffix
    // sum by doubling, at most 6 steps, in parity slots so that a vertex
    // keeps its slot from lane to lane), which alone writes the record.  A
    // sample without records (a zero adjoint, or skipped by the occupancy
    // test) breaks the chains through it.
    const int c0 = has ? (int)cl.c[0] : -2, c1 = has ? (int)cl.c[1] : -2,
              c2 = has ? (int)cl.c[2] : -2;
    // the next lane's values (wave_shl:1), read by every lane of the wave
    const int nh = dppi<0x130>(has ? 1 : 0);
    const int n0 = dppi<0x130>(c0), n1 = dppi<0x130>(c1), n2 = dppi<0x130>(c2);
    const bool next_in = has && (lane & (NS < 64 ? NS - 1 : 63)) != (NS < 64 ? NS - 1 : 63) && nh != 0;
    uint32_t open = next_in ? xor_permute_bits(shared_corners(c0, c1, c2, n0, n1, n2), flip) : 0u;
    // vertices the previous lane's chains continue into are summed there
    // (wave_shr:1; lane 0 reads 0: no chain comes in)
    keep &= ~(uint32_t)dppi<0x138>((int)open);
    if (chain_step<1>(v, open))
      if (chain_step<2>(v, open))
        if (chain_step<4>(v, open))
          if (chain_step<8>(v, open))
            if (chain_step<16>(v, open)) chain_step<32>(v, open);
  }
  uint32_t idx[8];
  int rank[8];
  cell_corners(cl, N, T, hashed, idx, flip);
  if (keep) {
    // an x-pair of corners in one region takes both ranks with one atomic
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool k0 = (keep >> (2 * q)) & 1u, k1 = (keep >> (2 * q + 1)) & 1u;
      const uint32_t r0 = idx[2 * q] >> RB, r1 = idx[2 * q + 1] >> RB;
      if (k0 && k1 && r0 == r1) {
        rank[2 * q] = atomicAdd(&lcnt[r0], 2);
        rank[2 * q + 1] = rank[2 * q] + 1;
      } else {
        if (k0) rank[2 * q] = atomicAdd(&lcnt[r0], 1);
        if (k1) rank[2 * q + 1] = atomicAdd(&lcnt[r1], 1);
      }
    }
  }
  const int n = place();
  float2* s_val = (float2*)dyn;                       // RM_STAGE_CORNERS
  int* s_slot = (int*)(s_val + RM_STAGE_CORNERS);     // RM_STAGE_CORNERS
  if (keep) {
    int2 b[8];  // all eight first: one LDS round trip
#pragma unroll
    for (int q = 0; q < 8; ++q) b[q] = rg[idx[q] >> RB];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if ((keep >> q) & 1u) {
        const int j = b[q].x + rank[q], slot = b[q].y + rank[q];
        const int at = (int)(idx[q] >> RB) * cap + slot;
        const float2 r = rec_pack(v[q], idx[q] & em);
        const bool fits = slot < cap;
        if (j < RM_STAGE_CORNERS) {
          s_val[j] = r;
          s_slot[j] = fits ? at : -1;
        } else if (fits) {
          nt_store2((float2*)rec + at, r);
        }
        if (!fits) {  // bin full: direct atomics (correct, only slower)
          unsafeAtomicAdd(gl + 2 * (int64_t)idx[q], v[q].x);
          unsafeAtomicAdd(gl + 2 * (int64_t)idx[q] + 1, v[q].y);
        }
      }
  }
  __syncthreads();
  const int ns = n < RM_STAGE_CORNERS ? n : RM_STAGE_CORNERS;
  for (int j = tid; j < ns; j += RM_SCAT_WG) {
    const int slot = s_slot[j];
    if (slot >= 0) nt_store2((float2*)rec + slot, s_val[j]);
  }
}

// Region sums are taken in LDS as 64-bit fixed point: float atomics in LDS
// run about 24 times slower than integer ones on this chip.  A first pass
// takes, per entry, the largest binary exponent of its records (an integer
// max); the second adds every record scaled by 2^(RM_FX_BITS - that
// exponent), rounded to an integer (|term| < 2^(RM_FX_BITS + 1)), so each
// term is kept to 2^-RM_FX_BITS of the entry's largest one -- finer than an
// FP32 rounding of the sum -- and the sum is exact and independent of order.
// Up to 2^(62 - RM_FX_BITS) records per entry and workgroup fit.

// biased FP32 exponent field of |v| (0 for zero and subnormals)
__device__ inline uint32_t exp_field(float v) { return (__float_as_uint(v) >> 23) & 0xffu; }

// 2^k as a double, k within the normal range
__device__ inline double pow2d(int k) { return __longlong_as_double((long long)(k + 1023) << 52); }

// The double whose product with a term is the term's fixed-point integer,
// for an entry whose largest exponent field is e: 2^(RM_FX_BITS + 127 - e).
__device__ inline double fx_scale(uint32_t e) {
  return pow2d(RM_FX_BITS + 127 - (int)(e > 1u ? e : 1u));  // |v| < 2^(e - 126)
}

// v sc rounded to an integer (nearest, ties to even) and added: adding
// 1.5 2^52 leaves the integer in the low mantissa bits (|v sc| < 2^39).
__device__ inline void fx_add1(unsigned long long* acc, float v, double sc) {
  const double x = fma((double)v, sc, 6755399441055744.0);
  atomicAdd(acc, (unsigned long long)__double_as_longlong(x) - 0x4338000000000000ull);
}

__device__ inline void fx_add(unsigned long long* acc, const uint32_t* emax, uint32_t e, float vx,
                              float vy) {
  const double sc = fx_scale(emax[e]);
  fx_add1(&acc[e], vx, sc);
  fx_add1(&acc[RM_RB + e], vy, sc);
}

__device__ inline void rec_max(uint32_t* emax, float x, float y) {
  atomicMax(&emax[rec_entry(x, y)], max(exp_field(x), exp_field(y)));
}

__device__ inline void rec_add(unsigned long long* acc, const uint32_t* emax, float x, float y) {
  fx_add(acc, emax, rec_entry(x, y), rec_value(x), rec_value(y));
}

// Pair records: of the products that pair_add takes (a sum of the factors'
// exponents may be one above, and would cost the sums a bit).
__device__ inline void pair_max(uint32_t* emax, const PairRec& r) {
  uint32_t e, o;
  pair_entries(r, e, o);
  const float s = pair_s(r), t = 1.0f - s, ax = pair_a(r.ax), ay = pair_a(r.ay);
  atomicMax(&emax[e], max(exp_field(t * ax), exp_field(t * ay)));
  atomicMax(&emax[o], max(exp_field(s * ax), exp_field(s * ay)));
}

__device__ inline void pair_add(unsigned long long* acc, const uint32_t* emax, const PairRec& r) {
  uint32_t e, o;
  pair_entries(r, e, o);
  const float s = pair_s(r), t = 1.0f - s, ax = pair_a(r.ax), ay = pair_a(r.ay);
  const uint32_t m0 = emax[e], m1 = emax[o];
  const double c0 = fx_scale(m0), c1 = fx_scale(m1);
  fx_add1(&acc[e], t * ax, c0);
  fx_add1(&acc[RM_RB + e], t * ay, c0);
  fx_add1(&acc[o], s * ax, c1);
  fx_add1(&acc[RM_RB + o], s * ay, c1);
}

// Record i of a bin.
template <bool PAIRS>
struct Rec;
template <>
struct Rec<false> {
  float2 v;
  __device__ inline void load(const float* rec, int i) { v = ((const float2*)rec)[i]; }
  __device__ inline void largest(uint32_t* emax) const { rec_max(emax, v.x, v.y); }
  __device__ inline void add(unsigned long long* acc, const uint32_t* emax) const {
    rec_add(acc, emax, v.x, v.y);
  }
  __device__ inline void opaque() { asm volatile("" : "+v"(v.x), "+v"(v.y)); }
};
template <>
struct Rec<true> {
  PairRec v;
  __device__ inline void load(const float* rec, int i) {
    const rm_i3v w = *(const rm_i3v*)(rec + 3 * (int64_t)i);
    v = PairRec{__int_as_float(w[0]), __int_as_float(w[1]), __int_as_float(w[2])};
  }
  __device__ inline void largest(uint32_t* emax) const { pair_max(emax, v); }
  __device__ inline void add(unsigned long long* acc, const uint32_t* emax) const {
    pair_add(acc, emax, v);
  }
  __device__ inline void opaque() { asm volatile("" : "+v"(v.ax), "+v"(v.ay), "+v"(v.s)); }
};

// Sums records [i0, i1) of a bin into acc, in units of 2^(emax - 127 -
// RM_FX_BITS) of each entry; both start cleared, and a barrier follows.
// Consecutive lanes take consecutive records.  The first NR records of each
// thread stay in registers from the first pass to the second: a share of up
// to NR * RM_ACC_WG records is read once (the shares of all workgroups in
// flight do not fit in the L2 between the passes).
template <bool PAIRS>
__device__ inline void sum_records(const float* rec, int i0, int i1, uint32_t* emax,
                                   unsigned long long* acc) {
  constexpr int NR = PAIRS ? RM_ACC_PAIRS : RM_ACC_CORNERS;
  const int b = i0 + (int)threadIdx.x;
  Rec<PAIRS> c[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k)
    if (b + k * RM_ACC_WG < i1) c[k].load(rec, b + k * RM_ACC_WG);
  // pass 1: largest exponent per entry
#pragma unroll
  for (int k = 0; k < NR; ++k)
    if (b + k * RM_ACC_WG < i1) c[k].largest(emax);
  constexpr int U = 4;  // further records, four in flight per lane
  for (int i = b + NR * RM_ACC_WG; i < i1; i += U * RM_ACC_WG) {
    Rec<PAIRS> x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * RM_ACC_WG < i1) x[u].load(rec, i + u * RM_ACC_WG);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * RM_ACC_WG < i1) x[u].largest(emax);
  }
  __syncthreads();
  // pass 2: fixed-point sums (records beyond the registers are read again).
  // The records pass through an empty statement, so that no field decoded in
  // the first pass is kept in further registers.
#pragma unroll
  for (int k = 0; k < NR; ++k) c[k].opaque();
#pragma unroll
  for (int k = 0; k < NR; ++k)
    if (b + k * RM_ACC_WG < i1) c[k].add(acc, emax);
  for (int i = b + NR * RM_ACC_WG; i < i1; i += U * RM_ACC_WG) {
    Rec<PAIRS> x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * RM_ACC_WG < i1) x[u].load(rec, i + u * RM_ACC_WG);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * RM_ACC_WG < i1) x[u].add(acc, emax);
  }
}

// Bound by memory: 24 B per parameter and the records, 4.9 TB/s of the 5.2 TB/s
// that a large copy reaches (135 M parameters in 24 objects: 802 us with
// corner records alone, 4.3 TB/s of Adam operands; 820 us beside the L2's
// write-back of the pair records, which the binning no longer waits for).
__global__ __launch_bounds__(RM_ACC_WG) void k_bin_acc(StepArgs a) {
  __shared__ uint32_t emax[RM_RB];
  // the first feature's sums, then the second's: interleaved, the adds of one
  // feature would use half of the banks
  __shared__ unsigned long long acc[2 * RM_RB];
  const cptr<Bin> bn = as_const(a.bins + a.bin_begin + blockIdx.x);
  const int region = bn->region, k_of = bn->k;
  const cptr<BinPair> bp = as_const(a.bpairs + bn->pair);
  const int cap = bp->cap, K = bp->K;
  const bool pairs = bp->pairs;
  const cptr<ObjStatic> ob = as_const(a.objs + bp->obj);
  const cptr<ObjState> state = as_const(a.state + bp->obj);
  const float bc1 = state->bc1, bc2 = state->bc2;
  int n = as_const(a.bin_count + bp->bin_base)[region];
  const bool spilled = n > cap;  // some records went to the gradient directly
  n = spilled ? cap : n;
  // this workgroup's share of the bin: [i0, i1), multiples of 4 but the end
  const int per = ((n + K - 1) / K + 3) & ~3;
  const int i0 = k_of * per;
  const int i1 = (i0 + per < n) ? i0 + per : n;
  // The sole workgroup of a region (K = 1) applies a training step's Adam
  // update to all of the region's entries, even with no records; shared
  // regions are finished by k_bin_finish.
  const bool adam_here = a.fuse_adam && K == 1;
  if (i0 >= i1 && !adam_here) return;  // empty share: nothing to add
  // entries of this region (a dense level's last region is partial)
  const int rsize = 1 << a.region_bits;
  const int64_t e0 = (int64_t)region * rsize;
  const int64_t rem = (int64_t)bp->T - e0;
  const int ne = rem < rsize ? (int)rem : rsize;
  const int64_t off0 = bp->off + 2 * e0;  // float offset of the region
  // Adam operands of this thread's entries, loaded now so that they arrive
  // while the records are summed
  constexpr int EPT = RM_RB / RM_ACC_WG;
  const gptr<rm_f2v> Pp = as_global((rm_f2v*)(ob->params + off0));
  const gptr<rm_f2v> Pm = as_global((rm_f2v*)(ob->m + off0));
  const gptr<rm_f2v> Pv = as_global((rm_f2v*)(ob->v + off0));
  rm_f2v ap[EPT], am[EPT], av[EPT];
  if (adam_here) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int e = threadIdx.x + k * RM_ACC_WG;
      if (e < ne) {
        ap[k] = Pp[e];
        am[k] = Pm[e];
        av[k] = Pv[e];
      }
    }
  }
  for (int e = threadIdx.x; e < rsize; e += RM_ACC_WG) {
    emax[e] = 0u;
    acc[e] = 0ull;
    acc[RM_RB + e] = 0ull;
  }
  __syncthreads();
  const float* rec = a.rec + bp->rec_base + (int64_t)region * cap * (pairs ? 3 : 2);
  if (pairs)
    sum_records<true>(rec, i0, i1, emax, acc);
  else
    sum_records<false>(rec, i0, i1, emax, acc);
  __syncthreads();
  const gptr<rm_f2v> g = as_global((rm_f2v*)((a.grad_override ? a.grad_override : ob->grad) + off0));
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int e = threadIdx.x + k * RM_ACC_WG;
    if (e >= ne) break;
    const uint32_t em = emax[e];
    const long long sx = (long long)acc[e], sy = (long long)acc[RM_RB + e];
    float dx = 0.0f, dy = 0.0f;
    if (em == 0xffu) {  // an Inf or NaN among the records
      dx = dy = __int_as_float(0x7fc00000);
    } else if (sx != 0 || sy != 0) {
      const double isc = pow2d((int)(em > 1u ? em : 1u) - 127 - RM_FX_BITS);
      dx = (float)((double)sx * isc);
      dy = (float)((double)sy * isc);
    }
    if (adam_here) {  // the entry's gradient is complete: update, keep g zero
      if (spilled) {
        const rm_f2v x = g[e];
        dx += x[0];
        dy += x[1];
        g[e] = rm_f2v{0.0f, 0.0f};
      }
      float p0 = ap[k][0], m0 = am[k][0], v0 = av[k][0], p1 = ap[k][1], m1 = am[k][1], v1 = av[k][1];
      adam1(p0, m0, v0, dx, a, bc1, bc2);
      adam1(p1, m1, v1, dy, a, bc1, bc2);
      __builtin_nontemporal_store(rm_f2v{p0, p1}, Pp + e);
      __builtin_nontemporal_store(rm_f2v{m0, m1}, Pm + e);
      __builtin_nontemporal_store(rm_f2v{v0, v1}, Pv + e);
      continue;
    }
    if (em == 0u && sx == 0 && sy == 0) continue;  // untouched (or only zeros)
    if (K == 1) {
      // sole writer: onto a zero region, or the scatter's overflow atomics
      rm_f2v x = {dx, dy};
      if (spilled) {
        const rm_f2v y = g[e];
        x[0] += y[0];
        x[1] += y[1];
      }
      g[e] = x;
    } else {  // shared region: atomics on consecutive entries
      float* d = (float*)(uintptr_t)(g + e);
      unsafeAtomicAdd(d, dx);
      unsafeAtomicAdd(d + 1, dy);
    }
  }
}

// Training steps: Adam on the entries of regions that several workgroups
// summed into the gradient (and leaves it zero for the next step).
__global__ __launch_bounds__(RM_FIN_WG) void k_bin_finish(StepArgs a) {
  const Fin f = a.fins[blockIdx.x];
  const BinPair bp = a.bpairs[f.pair];
  const int oi = a.sobj[bp.so].obj;
  const ObjStatic& ob = a.objs[oi];
  const int rsize = 1 << a.region_bits;
  const int64_t e0 = (int64_t)f.region * rsize;
  const int64_t rem = (int64_t)ob.T_l[bp.l] - e0;
  const int ne = rem < rsize ? (int)rem : rsize;
  const int e = f.sub * RM_FIN_WG + threadIdx.x;
  if (e >= ne) return;
  const int64_t off = ob.off[bp.l] + 2 * (e0 + e);
  float2* g = (float2*)(ob.grad + off);
  const float2 x = *g;
  *g = make_float2(0.0f, 0.0f);
  adam_entry(ob, off, x.x, x.y, a, a.state[oi].bc1, a.state[oi].bc2);
}

// ---------------------------------------------------------------------------
// K4: fused per-ray field kernel.
//
// A wave owns one ray at a time; its N samples are processed in blocks of 16.
// Activations are kept transposed, [feature][sample], as 16x16 MFMA result
// fragments (lane = sample column, 4 feature rows per lane), which are
// directly the B operands of the next layer: every forward and input-adjoint
// GEMM chains in registers.  Weight gradients contract over samples and need
// the [feature][sample] tiles in LDS (per-wave staging).
//
// PREC 0: FP32 MFMA 16x16x4.  PREC 1: BF16 MFMA 16x16x16, FP32 accumulation.
template <int PREC>
struct Mma;

template <>
struct Mma<0> {
  typedef float wtype;
  static constexpr int STRIDE = 17;  // staging row stride (floats)
  template <int M, int K>
  __device__ static inline void gemm(const float* wA, const floatx4* X, floatx4* Out, int lane) {
    constexpr int Q = K / 16;
#pragma unroll
    for (int t = 0; t < M / 16; ++t) {
      floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int q = 0; q < Q; ++q) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[((t * Q + q) * 4 + r) * 64 + lane],
                                                    X[q][r], acc, 0, 0, 0);
      }
      Out[t] = acc;
    }
  }
  __device__ static inline void stage(float* buf, const floatx4* F, int nf, int lane) {
    const int g = lane >> 4, n = lane & 15;
    for (int f = 0; f < nf; ++f) {
#pragma unroll
      for (int r = 0; r < 4; ++r) buf[(16 * f + 4 * g + r) * STRIDE + n] = F[f][r];
    }
  }
  // acc[t][u] += G^T(16t.., 16 samples) X(16 samples, 16u..)
  template <int MG, int MX>
  __device__ static inline void dw(const float* gb, const float* xb, floatx4* acc, int lane) {
    const int i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < MG / 16; ++t)
#pragma unroll
      for (int u = 0; u < MX / 16; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[t * (MX / 16) + u] = __builtin_amdgcn_mfma_f32_16x16x4f32(
              gb[(16 * t + i) * STRIDE + 4 * c + g], xb[(16 * u + i) * STRIDE + 4 * c + g],
              acc[t * (MX / 16) + u], 0, 0, 0);
  }
};

__device__ inline bf16x4_t cvt_bf16x4(floatx4 v) { return __builtin_convertvector(v, bf16x4_t); }

// PREC 1 operands.  A contraction over K >= 32 runs as 16x16x32 MFMAs whose K
// slots are ordered so that two consecutive [feature][sample] result
// fragments (features 32c..32c+15 and 32c+16..32c+31) are, concatenated per
// lane, its B operand: lane (g, n) feeds slots 8g..8g+7 = features
// 32c + 4g + 0..3 and 32c + 16 + 4g + 0..3 of sample n; the weight image
// holds A in the same slot order (pack_weights).  K = 16 runs as 16x16x16.
template <>
struct Mma<1> {
  typedef uint16_t wtype;
  static constexpr int STRIDE = 20;  // staging row stride (bf16), keeps 8-byte alignment
  // Out(M x 16 samples) = A(M x K) X(K x 16), X given as BF16 fragments
  template <int M, int K>
  __device__ static inline void gemm_b(const uint16_t* wA, const bf16x4_t* xb, floatx4* Out,
                                       int lane) {
    if constexpr (K % 32 == 0) {
      constexpr int C = K / 32;
      bf16x8_t x8[C];
#pragma unroll
      for (int c = 0; c < C; ++c)
        x8[c] = __builtin_shufflevector(xb[2 * c], xb[2 * c + 1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int t = 0; t < M / 16; ++t) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const bf16x8_t av = *(const bf16x8_t*)(wA + ((t * C + c) * 64 + lane) * 8);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, x8[c], acc, 0, 0, 0);
        }
        Out[t] = acc;
      }
    } else {
      constexpr int Q = K / 16;
#pragma unroll
      for (int t = 0; t < M / 16; ++t) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const shortx4 av = *(const shortx4*)(wA + ((t * Q + q) * 64 + lane) * 4);
          acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
              av, __builtin_bit_cast(shortx4, xb[q]), acc, 0, 0, 0);
        }
        Out[t] = acc;
      }
    }
  }
  template <int M, int K>
  __device__ static inline void gemm(const uint16_t* wA, const floatx4* X, floatx4* Out,
                                     int lane) {
    bf16x4_t xb[K / 16];
#pragma unroll
    for (int q = 0; q < K / 16; ++q) xb[q] = cvt_bf16x4(X[q]);
    gemm_b<M, K>(wA, xb, Out, lane);
  }
  __device__ static inline void stage_b(uint16_t* buf, const bf16x4_t* F, int nf, int lane) {
    const int g = lane >> 4, n = lane & 15;
    for (int f = 0; f < nf; ++f) {
      const shortx4 v = __builtin_bit_cast(shortx4, F[f]);
#pragma unroll
      for (int r = 0; r < 4; ++r) buf[(16 * f + 4 * g + r) * STRIDE + n] = (uint16_t)v[r];
    }
  }
  __device__ static inline void stage(uint16_t* buf, const floatx4* F, int nf, int lane) {
    const int g = lane >> 4, n = lane & 15;
    for (int f = 0; f < nf; ++f) {
      const shortx4 v = __builtin_bit_cast(shortx4, cvt_bf16x4(F[f]));
#pragma unroll
      for (int r = 0; r < 4; ++r) buf[(16 * f + 4 * g + r) * STRIDE + n] = (uint16_t)v[r];
    }
  }
  template <int MG, int MX>
  __device__ static inline void dw(const uint16_t* gb, const uint16_t* xb, floatx4* acc,
                                   int lane) {
    const int i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < MG / 16; ++t) {
      const shortx4 av = *(const shortx4*)(gb + (16 * t + i) * STRIDE + 4 * g);
#pragma unroll
      for (int u = 0; u < MX / 16; ++u) {
        const shortx4 bv = *(const shortx4*)(xb + (16 * u + i) * STRIDE + 4 * g);
        acc[t * (MX / 16) + u] =
            __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc[t * (MX / 16) + u], 0, 0, 0);
      }
    }
  }
  // Tiles of 32 samples (two 16-sample blocks side by side): rows of
  // STRIDE2 values, 16-byte aligned, so a lane reads 8 consecutive samples.
  static constexpr int STRIDE2 = 40;
  __device__ static inline void stage_b2(uint16_t* buf, const bf16x4_t* F, int nf, int lane,
                                         int col0) {
    const int g = lane >> 4, n = lane & 15;
    for (int f = 0; f < nf; ++f) {
      const shortx4 v = __builtin_bit_cast(shortx4, F[f]);
#pragma unroll
      for (int r = 0; r < 4; ++r) buf[(16 * f + 4 * g + r) * STRIDE2 + col0 + n] = (uint16_t)v[r];
    }
  }
  // dW += G X^T over 32 samples, one 16x16x32 MFMA per output tile: lane
  // (i, g) holds samples 8g .. 8g+7 of row i of both operands (the same
  // order of the contracted index on both sides)
  template <int MG, int MX>
  __device__ static inline void dw32(const uint16_t* gb, const uint16_t* xb, floatx4* acc,
                                     int lane) {
    const int i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < MG / 16; ++t) {
      const bf16x8_t av = *(const bf16x8_t*)(gb + (16 * t + i) * STRIDE2 + 8 * g);
#pragma unroll
      for (int u = 0; u < MX / 16; ++u) {
        const bf16x8_t bv = *(const bf16x8_t*)(xb + (16 * u + i) * STRIDE2 + 8 * g);
        acc[t * (MX / 16) + u] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[t * (MX / 16) + u], 0, 0, 0);
      }
    }
  }
};

// ReLU of FP32 pre-activations, rounded to BF16: rounding to nearest
// commutes with max(x, 0), and a BF16 value read as int16 is negative exactly
// when its sign bit is set, so one packed 16-bit integer max does two units.
__device__ inline bf16x4_t relu_b(floatx4 x) {
  const shortx4 v = __builtin_bit_cast(shortx4, cvt_bf16x4(x));
  const shortx4 z = {0, 0, 0, 0};
  return __builtin_bit_cast(bf16x4_t, __builtin_elementwise_max(v, z));
}

// An FP32 adjoint rounded to BF16 and kept where the unit's ReLU output h
// (BF16, >= 0) is positive: min(h, 1) * 0xFFFF as 16-bit lanes is the mask.
// (op_sel_hi:[1,0]: the high lane also reads the constant's low half, which
// is where an inline constant of a packed instruction sits.)
__device__ inline bf16x4_t mask_b(floatx4 d, bf16x4_t h) {
  const uint2 hb = __builtin_bit_cast(uint2, h);
  uint32_t m0, m1;
  asm("v_pk_min_u16 %0, %1, 1 op_sel_hi:[1,0]" : "=v"(m0) : "v"(hb.x));
  asm("v_pk_min_u16 %0, %1, 1 op_sel_hi:[1,0]" : "=v"(m1) : "v"(hb.y));
  asm("v_pk_mul_lo_u16 %0, %1, -1 op_sel_hi:[1,0]" : "=v"(m0) : "v"(m0));
  asm("v_pk_mul_lo_u16 %0, %1, -1 op_sel_hi:[1,0]" : "=v"(m1) : "v"(m1));
  const uint2 db = __builtin_bit_cast(uint2, cvt_bf16x4(d));
  return __builtin_bit_cast(bf16x4_t, make_uint2(db.x & m0, db.y & m1));
}

__device__ inline void relu4(floatx4* F, int n) {
  for (int f = 0; f < n; ++f) {
#pragma unroll
    for (int r = 0; r < 4; ++r) F[f][r] = F[f][r] > 0.0f ? F[f][r] : 0.0f;
  }
}

__device__ inline float sigmoidf_(float z) { return 1.0f / (1.0f + expf(-z)); }

// Loads the encoding of 16 samples (s0 .. s0+15) as K1/16 fragments:
// fragment q, register r, lane (g, n) = feature 16q + 4g + r of sample s0 + n,
// feature f = level f/2, component f%2 of the [L][S] float2 buffer.
template <int K1>
__device__ inline void load_e(const float2* e, int64_t S, int64_t s, int L, int g, floatx4* E) {
#pragma unroll
  for (int q = 0; q < K1 / 16; ++q) {
    const int l0 = 8 * q + 2 * g, l1 = l0 + 1;
    const float2 v0 = l0 < L ? e[(int64_t)l0 * S + s] : make_float2(0.0f, 0.0f);
    const float2 v1 = l1 < L ? e[(int64_t)l1 * S + s] : make_float2(0.0f, 0.0f);
    E[q][0] = v0.x;
    E[q][1] = v0.y;
    E[q][2] = v1.x;
    E[q][3] = v1.y;
  }
}

// The same fragments from the BF16 pairs of an e_bf16 buffer (bits as stored).
template <int K1>
__device__ inline void load_e_b(const uint32_t* e, int64_t S, int64_t s, int L, int g,
                                bf16x4_t* E) {
#pragma unroll
  for (int q = 0; q < K1 / 16; ++q) {
    const int l0 = 8 * q + 2 * g, l1 = l0 + 1;
    const uint32_t v0 = l0 < L ? e[(int64_t)l0 * S + s] : 0u;
    const uint32_t v1 = l1 < L ? e[(int64_t)l1 * S + s] : 0u;
    E[q] = __builtin_bit_cast(bf16x4_t, (uint64_t)v0 | ((uint64_t)v1 << 32));
  }
}

// NH: hidden layers of the density MLP (1, or 2 and 3 for the model-size
// study); the deeper variants run one wave per SIMD (their 64 x 64 weight
// gradients are accumulated in registers).  The work-item record shares LDS
// with the weights, which are no longer read when it is written, and a layer's
// two staged tiles follow each other, so that two FP32 workgroups fit a CU
// (one before: 97 KB; 4096 rays x 64 samples 138 -> 112 us).
// FWD: colour, depth and T_end only (RM_MODE_FORWARD): without the backward
// half's registers and operands several waves share a SIMD and hide the
// layers' latency (the same rays: FP32 44 -> 32 us).  At 128 samples its two
// words of a ray's live mask, indexed by block, lie in 32 B of scratch a lane.
template <int PREC, int NS, int K1, int NH, bool FWD>
#ifndef RM_FIELD_BF16_WAVES
#define RM_FIELD_BF16_WAVES 2
#endif
__global__ __launch_bounds__(RM_WG) __attribute__((
    amdgpu_waves_per_eu(FWD ? (PREC == 0 && K1 == 32 ? 3 : NH > 2 ? 2 : NH > 1 ? 3 : 4) : NH > 1 ? 1 : (PREC == 1 ? RM_FIELD_BF16_WAVES : 2)))) void k_field(StepArgs a) {
  typedef Mma<PREC> MM;
  typedef typename MM::wtype wt;
  constexpr int NB = NS / 16;             // 16-sample blocks per ray
  constexpr int SPL = NS > 64 ? NS / 64 : 1;  // samples per lane in the composite
  // staged rows of a wave: a layer's adjoint and input (64 + K1, 64 + 16, or
  // 64 + 64 of a hidden-to-hidden layer)
  constexpr int ROWS = NH > 1 ? 128 : 64 + K1;
  constexpr int KQ = K1 / 16;
  // a ray's encodings stay in registers from the forward to the backward
  // pass when they fit (NS <= 64, one hidden layer), else the backward reads
  // them again
  constexpr bool KEEP_E = !FWD && NH == 1 && NB * KQ <= 8 && (PREC == 0 || RM_FIELD_BF16_WAVES < 3);
  constexpr int NBK = KEEP_E ? NB : 1;
  constexpr int WP = RM_WPACK_NH(NH);
  // a forward pass of one hidden layer needs the forward operands only
  constexpr int WUSED = FWD && NH == 1 ? RM_OFF_B4 : WP;
  constexpr int RL = RM_REC_LOSS_NH(NH);
  constexpr int WBYTES = WUSED * (int)sizeof(wt), RBYTES = FWD ? 0 : (RL + 4) * 4;
  // records combined at the end: one per wave where they leave two workgroups
  // to a CU (66 KB)
  constexpr int NREC = NH == 1 ? 4 : 1;
  // BF16 with one hidden layer: activations kept as rounded BF16 pairs
  constexpr bool PACKED = PREC == 1 && NH == 1;

  // BF16 with one hidden layer stages tiles of 32 samples (pairs of blocks)
  constexpr int STR = PACKED ? Mma<1>::STRIDE2 : MM::STRIDE;
  constexpr int STAGE = FWD ? 8 : ROWS * STR;  // elements a wave stages
  constexpr int UBYTES = WBYTES + 4 * STAGE * (int)sizeof(wt) + 4 * NS * 16;
  // LDS: the weights, each wave's stage and ray; at the end the records
  __shared__ __align__(16) char s_raw[UBYTES > NREC * RBYTES ? UBYTES : NREC * RBYTES];
  wt* s_w = (wt*)s_raw;
  wt* s_stage = (wt*)(s_raw + WBYTES);
  float* s_rv = (float*)(s_raw + WBYTES + 4 * STAGE * (int)sizeof(wt));

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, n = lane & 15;
  Item it;
  if (a.one_nb) {  // one object: by arithmetic, as block_of
    it.so = 0;
    it.ray_begin = (int)blockIdx.x * a.one_rpi;
    it.n_rays = a.n_rays - it.ray_begin < a.one_rpi ? a.n_rays - it.ray_begin : a.one_rpi;
  } else {
    it = a.items[blockIdx.x];
  }
  const StepObj so = a.sobj[it.so];
  const ObjStatic& ob = a.objs[so.obj];
  const int L = ob.L, din = ob.din;
  const int64_t S = a.S;
  const float invB = 1.0f / (float)so.n_rays;
  const int mode = a.mode;

  {  // weights of this object into LDS (16-byte copies)
    const floatx4* src = (const floatx4*)((PREC ? (const void*)(a.wpack16 + (int64_t)it.so * WP)
                                                : (const void*)(a.wpack32 + (int64_t)it.so * WP)));
    floatx4* dst = (floatx4*)s_w;
    constexpr int NV = WBYTES / 16;
    // up to ten loads in flight, then their stores: one round trip to the L2
    // (64 items of 4 rays: kernel 19.8 -> 18.6 us; 24 objects 178 -> 175)
    constexpr int DEEP = NV / RM_WG < 10 ? (NV + RM_WG - 1) / RM_WG : 10;
#pragma unroll
    for (int j0 = 0; j0 < NV; j0 += DEEP * RM_WG) {
      floatx4 t[DEEP];
#pragma unroll
      for (int u = 0; u < DEEP; ++u) {
        const int j = j0 + u * RM_WG + tid;
        t[u] = src[j < NV ? j : NV - 1];
      }
#pragma unroll
      for (int u = 0; u < DEEP; ++u)
        if (j0 + u * RM_WG + tid < NV) dst[j0 + u * RM_WG + tid] = t[u];
    }
  }
  __syncthreads();

  const wt* wF1 = s_w + RM_OFF_F1;
  const wt* wF2 = s_w + RM_OFF_F2;
  const wt* wF3 = s_w + RM_OFF_F3;
  const wt* wF4 = s_w + RM_OFF_F4;
  const wt* wB4 = s_w + RM_OFF_B4;
  const wt* wB3 = s_w + RM_OFF_B3;
  const wt* wB2 = s_w + RM_OFF_B2;
  const wt* wB1 = s_w + RM_OFF_B1;
  wt* gbuf = s_stage + wave * STAGE;           // a layer's adjoint, then its input
  wt* x16 = gbuf + 16 * STR;          // after an adjoint of 16 rows
  wt* x64 = gbuf + 64 * STR;          // after one of 64
  float* rv = s_rv + wave * (NS * 4);
  // encodings: FP32 fragments, or with the BF16 MLP the stored BF16 pairs as
  // they are (the MLP reads nothing else of them)
  typedef typename std::conditional<PREC == 1, bf16x4_t, floatx4>::type etype;
  auto load_enc = [&](int64_t s, etype* E) {
    if constexpr (PREC == 1)
      load_e_b<K1>((const uint32_t*)a.e, S, s, L, g, E);
    else
      load_e<K1>(a.e, S, s, L, g, E);
  };
  auto gemm_e = [&](const etype* E, floatx4* H) {
    if constexpr (PREC == 1)
      MM::template gemm_b<64, K1>(wF1, E, H, lane);
    else
      MM::template gemm<64, K1>(wF1, E, H, lane);
  };

  floatx4 acc1[4 * KQ], acc2[4], acc3[4], acc4[4];
  floatx4 accH[NH > 1 ? NH - 1 : 1][16];  // hidden-to-hidden weight gradients
#pragma unroll
  for (int j = 0; j < 4 * KQ; ++j) acc1[j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < (NH > 1 ? NH - 1 : 1); ++k)
#pragma unroll
    for (int j = 0; j < 16; ++j) accH[k][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc2[j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    acc3[j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    acc4[j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  float loss_w = 0.0f;

  for (int rr = wave; rr < it.n_rays; rr += 4) {
    const int ray = __builtin_amdgcn_readfirstlane(it.ray_begin + rr);
    const RayRec R = a.rays[ray];
    if (!ray_active(R.flags)) {
      if (FWD && lane == 0) {
        const int64_t o = R.out;
        if (a.out_rgb) a.out_rgb[3 * o] = a.out_rgb[3 * o + 1] = a.out_rgb[3 * o + 2] = 0.0f;
        if (a.out_depth) a.out_depth[o] = 0.0f;
        if (a.out_tend) a.out_tend[o] = a.out_opacity ? 0.0f : 1.0f;
      }
      continue;
    }
    const int64_t sray = (int64_t)ray * NS;
    // live samples: a block of 16 without any is passed over
    constexpr int LW = NS > 64 ? NS / 64 : 1;
    uint64_t lw[LW];
#pragma unroll
    for (int j = 0; j < LW; ++j) lw[j] = a.live ? as_const(a.live)[(int64_t)ray * a.live_step + j] : ~0ull;
    auto block_live = [&](int b) {
      return ((lw[LW > 1 ? b / 4 : 0] >> (16 * (LW > 1 ? b % 4 : b))) & 0xFFFFull) != 0ull;
    };

    // ---- forward: sigma, colour of every sample ----
    etype EK[NBK][KQ];
#pragma unroll(KEEP_E ? NB : 1)
    for (int b = 0; b < NB; ++b) {
      etype E[KQ];
      floatx4 H1[4], Y[1], H2[4], Z[1];
      if (!block_live(b)) {
        if (g == 0) *(floatx4*)(rv + (16 * b + n) * 4) = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (KEEP_E) {
#pragma unroll
          for (int q = 0; q < KQ; ++q) EK[KEEP_E ? b : 0][q] = etype{};
        }
        continue;
      }
      load_enc(sray + 16 * b + n, E);
      if (KEEP_E) {
#pragma unroll
        for (int q = 0; q < KQ; ++q) EK[KEEP_E ? b : 0][q] = E[q];
      }
      if constexpr (PACKED) {  // activations as rounded BF16 pairs
        bf16x4_t H1b[4], Yb[1], H2b[4];
        gemm_e(E, H1);
#pragma unroll
        for (int f = 0; f < 4; ++f) H1b[f] = relu_b(H1[f]);
        MM::template gemm_b<16, 64>(wF2, H1b, Y, lane);
        Yb[0] = cvt_bf16x4(Y[0]);
        MM::template gemm_b<64, 16>(wF3, Yb, H2, lane);
#pragma unroll
        for (int f = 0; f < 4; ++f) H2b[f] = relu_b(H2[f]);
        MM::template gemm_b<16, 64>(wF4, H2b, Z, lane);
      } else {
        gemm_e(E, H1);
        relu4(H1, 4);
#pragma unroll
        for (int k = 1; k < NH; ++k) {  // deeper density MLP: H1 <- ReLU(Wh_k H1)
          floatx4 Hn[4];
          MM::template gemm<64, 64>(s_w + RM_OFF_HF(k), H1, Hn, lane);
          relu4(Hn, 4);
#pragma unroll
          for (int f = 0; f < 4; ++f) H1[f] = Hn[f];
        }
        MM::template gemm<16, 64>(wF2, H1, Y, lane);
        MM::template gemm<64, 16>(wF3, Y, H2, lane);
        relu4(H2, 4);
        MM::template gemm<16, 64>(wF4, H2, Z, lane);
      }
      if (g == 0) {
        float* q = rv + (16 * b + n) * 4;
        q[0] = Y[0][0];
        q[1] = Z[0][0];  // colour logits: the adjoint needs sigmoid(-z) as well
        q[2] = Z[0][1];
        q[3] = Z[0][2];
      }
    }
    wave_lds_sync();

    // ---- volume rendering (Eq. 6) and its adjoint; lane = sample ----
    {
      const uint32_t cls = R.flags & RM_F_CLS;
      const bool bg = (mode == RM_MODE_TRAIN) && cls == RM_CLS_BACKGROUND;
      const bool valid = lane * SPL < NS;
      float y0[SPL], c[SPL][3], zc[SPL][3], sig[SPL], tau[SPL], dist[SPL], w[SPL], Sx[SPL];
      float lane_tau = 0.0f, lane_sig = 0.0f;
#pragma unroll
      for (int j = 0; j < SPL; ++j) {
        const int i = lane * SPL + j;
        if (valid) {
          const float* q = rv + i * 4;
          y0[j] = q[0];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            zc[j][k] = q[1 + k];
            c[j][k] = sigmoidf_(zc[j][k]);
          }
          const bool live = (lw[LW > 1 ? i / 64 : 0] >> (i & 63)) & 1ull;
          sig[j] = live ? expf(fminf(y0[j], 15.0f)) : 0.0f;
          if (!live) y0[j] = 16.0f;  // no density adjoint either
          tau[j] = sig[j] * R.delta;
          dist[j] = R.tn + ((float)i + 0.5f) * R.delta;
        } else {
          y0[j] = 0.0f;
          c[j][0] = c[j][1] = c[j][2] = 0.0f;
          zc[j][0] = zc[j][1] = zc[j][2] = 0.0f;
          sig[j] = tau[j] = dist[j] = 0.0f;
        }
        lane_tau += tau[j];
        lane_sig += sig[j];
      }
      const float P = wave_excl_prefix(lane_tau, lane);
      float run = P;
      float lc[3] = {0.0f, 0.0f, 0.0f}, ld = 0.0f;
#pragma unroll
      for (int j = 0; j < SPL; ++j) {
        Sx[j] = run;
        const float T = expf(-run);
        const float alpha = -expm1f(-tau[j]);
        w[j] = valid ? T * alpha : 0.0f;
        run += tau[j];
        lc[0] = fmaf(w[j], c[j][0], lc[0]);
        lc[1] = fmaf(w[j], c[j][1], lc[1]);
        lc[2] = fmaf(w[j], c[j][2], lc[2]);
        ld = fmaf(w[j], dist[j], ld);
      }
      float Ch[3];
      Ch[0] = wave_sum(lc[0]);
      Ch[1] = wave_sum(lc[1]);
      Ch[2] = wave_sum(lc[2]);
      const float Dh = wave_sum(ld);
      const float Stot = wave_sum(lane_tau);
      const float Tend = expf(-Stot);

      if constexpr (FWD) {
        if (lane == 0) {
          const int64_t o = R.out;
          if (a.out_rgb) {
            a.out_rgb[3 * o] = Ch[0];
            a.out_rgb[3 * o + 1] = Ch[1];
            a.out_rgb[3 * o + 2] = Ch[2];
          }
          if (a.out_depth) a.out_depth[o] = Dh;
          if (a.out_tend) a.out_tend[o] = a.out_opacity ? 1.0f - Tend : Tend;
        }
        continue;
      } else {
      float gC[3], gD = 0.0f, gT = 0.0f, dens = 0.0f;
      if (mode == RM_MODE_TRAIN) {
        // Eq. 7-11: squared colour error against the image (object rays) or
        // against the random colour with residual transmittance (background
        // rays), L1 depth term, density term on every background sample.
        float Co[3], l = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          Co[k] = bg ? fmaf(Tend, R.tgt[k], Ch[k]) : Ch[k];
          const float df = Co[k] - R.tgt[k];
          l = fmaf(df, df, l);
          gC[k] = 2.0f * df * invB;
        }
        if (!bg && (R.flags & RM_F_DEPTH)) {
          const float dd = Dh - R.D;
          l += a.lambda_depth * fabsf(dd);
          gD = a.lambda_depth * (dd > 0.0f ? 1.0f : (dd < 0.0f ? -1.0f : 0.0f)) * invB;
        }
        if (bg) {
          l += a.lambda_density * wave_sum(lane_sig);
          dens = a.lambda_density * invB;
        }
        loss_w += l * invB;
      } else {  // RM_MODE_ADJOINT
#pragma unroll
        for (int k = 0; k < 3; ++k) gC[k] = a.adj_rgb ? a.adj_rgb[3 * ray + k] : 0.0f;
        gD = a.adj_depth ? a.adj_depth[ray] : 0.0f;
        gT = a.adj_tend ? a.adj_tend[ray] : 0.0f;
      }
      // suffix sums  sum_{j > i} w_j c_j  and  sum_{j > i} w_j d_j
      const float Qc0 = wave_excl_suffix(lc[0], lane);
      const float Qc1 = wave_excl_suffix(lc[1], lane);
      const float Qc2 = wave_excl_suffix(lc[2], lane);
      const float Qd = wave_excl_suffix(ld, lane);
      float sc[3] = {Qc0, Qc1, Qc2}, sd = Qd;
      float bgterm = 0.0f;
      if (bg) bgterm = Tend * (gC[0] * R.tgt[0] + gC[1] * R.tgt[1] + gC[2] * R.tgt[2]);
#pragma unroll
      for (int j = SPL - 1; j >= 0; --j) {
        const int i = lane * SPL + j;
        const float Tn = expf(-(Sx[j] + tau[j]));
        float dtau = gC[0] * (Tn * c[j][0] - sc[0]) + gC[1] * (Tn * c[j][1] - sc[1]) +
                     gC[2] * (Tn * c[j][2] - sc[2]) + gD * (Tn * dist[j] - sd) - bgterm -
                     gT * Tend;
        const float dsig = dtau * R.delta + dens;
        sc[0] = fmaf(w[j], c[j][0], sc[0]);
        sc[1] = fmaf(w[j], c[j][1], sc[1]);
        sc[2] = fmaf(w[j], c[j][2], sc[2]);
        sd = fmaf(w[j], dist[j], sd);
        if (valid) {
          float* q = rv + i * 4;
          q[0] = y0[j] < 15.0f ? dsig * sig[j] : 0.0f;
#pragma unroll
          // sigmoid'(z) = sigmoid(z) sigmoid(-z): no cancellation where c rounds to 1
          for (int k = 0; k < 3; ++k) q[1 + k] = w[j] * gC[k] * c[j][k] * sigmoidf_(-zc[j][k]);
        }
      }
      }
    }
    if constexpr (!FWD) {
    wave_lds_sync();

    // ---- backward: recompute activations per block, adjoints, dW ----
    if constexpr (PACKED) {
      // BF16, one hidden layer: blocks in pairs, so that each weight
      // gradient is one product over 32 samples (half the LDS round trips
      // and MFMA instructions of per-block products); activations recomputed
      // and rounded as in the forward, adjoints rounded once and used by
      // both their MFMA and their staging
#pragma unroll(KEEP_E ? NB / 2 : 1)
      for (int bp = 0; bp < NB; bp += 2) {
        if (!block_live(bp) && !block_live(bp + 1)) continue;
        bf16x4_t E2[2][KQ], H1b[2][4], Yb[2][1], H2b[2][4], dZb[2][1], dH2b[2][4], dYb[2][1],
            dH1b[2][4];
        float dy0[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int b = bp + h;
          if (KEEP_E) {
#pragma unroll
            for (int q = 0; q < KQ; ++q) E2[h][q] = EK[KEEP_E ? b : 0][q];
          } else {
            load_enc(sray + 16 * b + n, E2[h]);
          }
          floatx4 P[4], Yf[1];
          gemm_e(E2[h], P);
#pragma unroll
          for (int f = 0; f < 4; ++f) H1b[h][f] = relu_b(P[f]);
          MM::template gemm_b<16, 64>(wF2, H1b[h], Yf, lane);
          Yb[h][0] = cvt_bf16x4(Yf[0]);
          MM::template gemm_b<64, 16>(wF3, Yb[h], P, lane);
#pragma unroll
          for (int f = 0; f < 4; ++f) H2b[h][f] = relu_b(P[f]);
          floatx4 dz = {0.0f, 0.0f, 0.0f, 0.0f};
          dy0[h] = 0.0f;
          if (g == 0) {
            const float* q = rv + (16 * b + n) * 4;
            dy0[h] = q[0];
            dz = floatx4{q[1], q[2], q[3], 0.0f};
          }
          dZb[h][0] = cvt_bf16x4(dz);
        }
        // colour head: dW4 += dZ^T H2, dH2 = W4^T dZ masked by ReLU
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          MM::stage_b2(gbuf, dZb[h], 1, lane, 16 * h);
          MM::stage_b2(x16, H2b[h], 4, lane, 16 * h);
        }
        wave_lds_sync();
        MM::template dw32<16, 64>(gbuf, x16, acc4, lane);
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          floatx4 P[4];
          MM::template gemm_b<64, 16>(wB4, dZb[h], P, lane);
#pragma unroll
          for (int f = 0; f < 4; ++f) dH2b[h][f] = mask_b(P[f], H2b[h][f]);
        }
        // dW3 += dH2^T Y, dY = W3^T dH2 (+ density adjoint in row 0)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          MM::stage_b2(gbuf, dH2b[h], 4, lane, 16 * h);
          MM::stage_b2(x64, Yb[h], 1, lane, 16 * h);
        }
        wave_lds_sync();
        MM::template dw32<64, 16>(gbuf, x64, acc3, lane);
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          floatx4 dYf[1];
          MM::template gemm_b<16, 64>(wB3, dH2b[h], dYf, lane);
          if (g == 0) dYf[0][0] += dy0[h];
          dYb[h][0] = cvt_bf16x4(dYf[0]);
        }
        // dW2 += dY^T H1, dH1 = W2^T dY masked
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          MM::stage_b2(gbuf, dYb[h], 1, lane, 16 * h);
          MM::stage_b2(x16, H1b[h], 4, lane, 16 * h);
        }
        wave_lds_sync();
        MM::template dw32<16, 64>(gbuf, x16, acc2, lane);
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          floatx4 P[4];
          MM::template gemm_b<64, 16>(wB2, dYb[h], P, lane);
#pragma unroll
          for (int f = 0; f < 4; ++f) dH1b[h][f] = mask_b(P[f], H1b[h][f]);
        }
        // dW1 += dH1^T E, dE = W1^T dH1
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          MM::stage_b2(gbuf, dH1b[h], 4, lane, 16 * h);
          MM::stage_b2(x64, E2[h], KQ, lane, 16 * h);
        }
        wave_lds_sync();
        MM::template dw32<64, K1>(gbuf, x64, acc1, lane);
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          floatx4 dEf[KQ];
          MM::template gemm_b<K1, 64>(wB1, dH1b[h], dEf, lane);
          const int64_t s = sray + 16 * (bp + h) + n;
#pragma unroll
          for (int q = 0; q < KQ; ++q) {
            const int l0 = 8 * q + 2 * g, l1 = l0 + 1;
            if (l0 < L) a.de[(int64_t)l0 * S + s] = make_float2(dEf[q][0], dEf[q][1]);
            if (l1 < L) a.de[(int64_t)l1 * S + s] = make_float2(dEf[q][2], dEf[q][3]);
          }
        }
      }
      continue;
    }
#pragma unroll(KEEP_E ? NB : 1)
    for (int b = 0; b < NB; ++b) {
      if (!block_live(b)) continue;
      const int64_t s = sray + 16 * b + n;
      etype E[KQ];
      floatx4 HH[NH][4], Y[1], H2[4];
      floatx4* H1 = HH[NH - 1];  // the last hidden layer of the density MLP
      if (KEEP_E) {
#pragma unroll
        for (int q = 0; q < KQ; ++q) E[q] = EK[KEEP_E ? b : 0][q];
      } else {
        load_enc(s, E);
      }
      gemm_e(E, HH[0]);
      relu4(HH[0], 4);
#pragma unroll
      for (int k = 1; k < NH; ++k) {
        MM::template gemm<64, 64>(s_w + RM_OFF_HF(k), HH[k - 1], HH[k], lane);
        relu4(HH[k], 4);
      }
      MM::template gemm<16, 64>(wF2, H1, Y, lane);
      MM::template gemm<64, 16>(wF3, Y, H2, lane);
      relu4(H2, 4);
      floatx4 dZ[1], dH2[4], dY[1], dH1[4], dE[KQ];
      float dy0 = 0.0f;
      if (g == 0) {
        const float* q = rv + (16 * b + n) * 4;
        dy0 = q[0];
        dZ[0] = floatx4{q[1], q[2], q[3], 0.0f};
      } else {
        dZ[0] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      }
      // colour head: dW4 += dZ^T H2, dH2 = W4^T dZ masked by ReLU
      MM::stage(gbuf, dZ, 1, lane);
      MM::stage(x16, H2, 4, lane);
      wave_lds_sync();
      MM::template dw<16, 64>(gbuf, x16, acc4, lane);
      wave_lds_sync();
      MM::template gemm<64, 16>(wB4, dZ, dH2, lane);
#pragma unroll
      for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) dH2[f][r] = H2[f][r] > 0.0f ? dH2[f][r] : 0.0f;
      // dW3 += dH2^T Y, dY = W3^T dH2 (+ density adjoint in row 0)
      MM::stage(gbuf, dH2, 4, lane);
      MM::stage(x64, Y, 1, lane);
      wave_lds_sync();
      MM::template dw<64, 16>(gbuf, x64, acc3, lane);
      wave_lds_sync();
      MM::template gemm<16, 64>(wB3, dH2, dY, lane);
      if (g == 0) dY[0][0] += dy0;
      // dW2 += dY^T H1, dH1 = W2^T dY masked
      MM::stage(gbuf, dY, 1, lane);
      MM::stage(x16, H1, 4, lane);
      wave_lds_sync();
      MM::template dw<16, 64>(gbuf, x16, acc2, lane);
      wave_lds_sync();
      MM::template gemm<64, 16>(wB2, dY, dH1, lane);
#pragma unroll
      for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) dH1[f][r] = H1[f][r] > 0.0f ? dH1[f][r] : 0.0f;
      // deeper density MLP, last layer first: dWh_k += dH^T H_{k-1},
      // dH <- Wh_k^T dH masked by ReLU
#pragma unroll
      for (int k = NH - 1; k >= 1; --k) {
        MM::stage(gbuf, dH1, 4, lane);
        MM::stage(x64, HH[k - 1], 4, lane);
        wave_lds_sync();
        MM::template dw<64, 64>(gbuf, x64, accH[k - 1], lane);
        wave_lds_sync();
        floatx4 dP[4];
        MM::template gemm<64, 64>(s_w + RM_OFF_HB(k), dH1, dP, lane);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
          for (int r = 0; r < 4; ++r) dH1[f][r] = HH[k - 1][f][r] > 0.0f ? dP[f][r] : 0.0f;
      }
      // dW1 += dH^T E, dE = W1^T dH  (dH of the first hidden layer)
      MM::stage(gbuf, dH1, 4, lane);
      if constexpr (PREC == 1)
        MM::stage_b(x64, E, KQ, lane);
      else
        MM::stage(x64, E, KQ, lane);
      wave_lds_sync();
      MM::template dw<64, K1>(gbuf, x64, acc1, lane);
      wave_lds_sync();
      MM::template gemm<K1, 64>(wB1, dH1, dE, lane);
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        const int l0 = 8 * q + 2 * g, l1 = l0 + 1;
        if (l0 < L) a.de[(int64_t)l0 * S + s] = make_float2(dE[q][0], dE[q][1]);
        if (l1 < L) a.de[(int64_t)l1 * S + s] = make_float2(dE[q][2], dE[q][3]);
      }
    }
    }
  }

  // ---- work-item record: weight gradients in parameter order, and loss ----
  // Each wave stores its partial sums in a record of its own in LDS, and the
  // four are summed on the way out; with a deeper MLP, whose records do not
  // fit, the waves add to one record in turn.  Either way in the waves' order
  // (deterministic, and the same sums).  In turn, each add waiting for its
  // read, this was 6-8 us of every item: kernel 25 -> 20 us (64 items of 4 rays
  // x 32 samples), FP32 4096 rays x 64 samples 112 -> 104, BF16 24 objects x
  // 1050 rays 203 -> 178, 12 objects x 2500 rays x 128 samples 432 -> 387.
  if constexpr (!FWD) {
    const int oh = RM_HIDDEN * din, o2 = oh + (NH - 1) * RM_HH, o3 = o2 + RM_DOUT * RM_HIDDEN,
              o4 = o3 + RM_HIDDEN * RM_GEO;
    __syncthreads();  // the record overwrites the weights: every wave is done
    float* s_rec = (float*)(s_raw + (NREC == 4 ? wave : 0) * RBYTES);
#pragma unroll
    for (int turn = 0; turn < RM_WG / 64 / NREC; ++turn) {
      if (NREC == 4 || wave == turn) {
        const bool first = turn == 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 4 * g + r;
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < KQ; ++u) {
              const int m = 16 * t + row, k = 16 * u + n;
              if (k < din) {
                float* d = &s_rec[m * din + k];
                *d = first ? acc1[t * KQ + u][r] : *d + acc1[t * KQ + u][r];
              }
            }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float* d = &s_rec[o2 + row * RM_HIDDEN + 16 * u + n];
            *d = first ? acc2[u][r] : *d + acc2[u][r];
          }
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (n >= 1) {
              float* d = &s_rec[o3 + (16 * t + row) * RM_GEO + (n - 1)];
              *d = first ? acc3[t][r] : *d + acc3[t][r];
            }
          if (row < 3)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              float* d = &s_rec[o4 + row * RM_HIDDEN + 16 * u + n];
              *d = first ? acc4[u][r] : *d + acc4[u][r];
            }
#pragma unroll
          for (int k = 0; k < NH - 1; ++k)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt)
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                float* d = &s_rec[oh + k * RM_HH + (16 * tt + row) * RM_HIDDEN + 16 * u + n];
                *d = first ? accH[k][tt * 4 + u][r] : *d + accH[k][tt * 4 + u][r];
              }
        }
        if (lane == 0) s_rec[RL] = first ? loss_w : s_rec[RL] + loss_w;
      }
      __syncthreads();
    }
    float* rec = a.partials + (int64_t)blockIdx.x * RM_REC_STRIDE_NH(NH);
    static_assert(RL % 4 == 0, "the loss stands alone");
    for (int j = 4 * tid; j < RL + 4; j += 4 * RM_WG) {
      floatx4 x = *(const floatx4*)(s_raw + 4 * j);
#pragma unroll
      for (int q = 1; q < NREC; ++q) x += *(const floatx4*)(s_raw + q * RBYTES + 4 * j);
      *(floatx4*)(rec + j) = x;
    }
  }
}

// ---------------------------------------------------------------------------
// K5: per-object MLP gradient and loss from the work-item records, summed in
// a fixed order (deterministic); in a training step the MLP's Adam update is
// applied here, else the gradient is written.  A block owns 32 record columns
// (column RM_REC_LOSS_NH is the loss), read 4 per lane: eight lanes take a
// 128-byte line of an item's record, and the 32 such runs of lanes sum
// interleaved 32nds of the items, then combine in LDS.  Bound by the records'
// read; with 256 columns to a block, one object's launch was 17 blocks of four
// waves, too few for it (512 items: 24 us, now 5; beside the other half's
// kernels 6 objects 48 -> 23, 24 objects 35 -> 22; 64 columns: 27 and 21, and
// 16: 24 and 24).
__global__ __launch_bounds__(RM_RED_WG) void k_reduce(StepArgs a) {
  constexpr int LPI = RM_RED_COLS / 4, NQ = RM_RED_WG / LPI;
  constexpr int PW = 64 / LPI;  // runs side by side in a wave
  static_assert(PW >= 4, "one lane per column at the end");
  __shared__ float4 s_part[NQ][LPI];
  const StepObj so = a.sobj[blockIdx.y];
  const ObjStatic& ob = a.objs[so.obj];
  const int nm = (int)(ob.P - ob.P_grid);
  const int col = threadIdx.x % LPI, part = threadIdx.x / LPI;
  const int j0 = blockIdx.x * RM_RED_COLS + 4 * col;  // 4 columns per lane (the stride is a multiple of 4)
  float4 s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) s[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const int stride = RM_REC_STRIDE_NH(a.mlp_layers), rloss = RM_REC_LOSS_NH(a.mlp_layers);
  if (j0 < stride) {
    // run w of lanes sums items w, w + NQ, ...: four per lane in flight, each
    // into its own partial sum (a fixed order: deterministic)
    const float* rec = a.partials + j0;
    for (int it = so.item_begin + part; it < so.item_end; it += 4 * NQ) {
      float4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        x[u] = it + u * NQ < so.item_end ? *(const float4*)(rec + (int64_t)(it + u * NQ) * stride)
                                         : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s[u].x += x[u].x; s[u].y += x[u].y; s[u].z += x[u].z; s[u].w += x[u].w;
      }
    }
  }
  s_part[part][col] = make_float4((s[0].x + s[1].x) + (s[2].x + s[3].x),
                                  (s[0].y + s[1].y) + (s[2].y + s[3].y),
                                  (s[0].z + s[1].z) + (s[2].z + s[3].z),
                                  (s[0].w + s[1].w) + (s[2].w + s[3].w));
  __syncthreads();
  if (threadIdx.x >= 64) return;
  float4 t = s_part[part][col];
#pragma unroll
  for (int w = 1; w < NQ / PW; ++w) {  // fixed order: deterministic
    const float4 u = s_part[PW * w + part][col];
    t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
  }
  // the runs together, then lane (part, col) takes column 4 col + part
  float tv[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int m = LPI; m < 64; m *= 2) tv[c] += __shfl_xor(tv[c], m);
  }
  if (part >= 4) return;
  const float g = part == 0 ? tv[0] : part == 1 ? tv[1] : part == 2 ? tv[2] : tv[3];
  const int j = j0 + part;
  float* gdst = a.grad_override ? a.grad_override : ob.grad;
  if (j < nm) {
    const int64_t o = ob.P_grid + j;
    if (a.fuse_adam) {  // training step: the MLP gradient is complete here
      adam1(ob.params[o], ob.m[o], ob.v[o], g, a, a.state[so.obj].bc1, a.state[so.obj].bc2);
    } else {
      gdst[o] = g;
    }
  } else if (j == rloss && a.mode == RM_MODE_TRAIN) {
    ObjState* st = a.state + so.obj;
    st->loss_acc += g;
    st->n_loss += 1;
  }
}

// ---------------------------------------------------------------------------
// Density of an object's field at normalised positions in [0,1]^3: encoding
// and density head in FP32.  A workgroup of four waves takes 64 points, one
// per lane: each wave encodes a quarter of the levels and then computes a
// quarter of every layer's units, exchanged through LDS, so that a call of
// 100 k points has six waves per SIMD instead of one and a half with a thread
// per point (207 -> 85 us at 16 levels of 2^18; 65^3 corners 208 -> 63 us).
// Every sum runs in the order of its index.  Random points are bound by lines
// from beyond the L2 (16 tables are swept at once), a grid by both.
#define RM_DENS_WG 256

// One layer's 16 units of this wave: out[unit][lane] = ReLU(W row . in), in[k]
// for k < K from LDS (stride 64), rows of W at `row` floats each.
__device__ __forceinline__ void dens_layer(const float* W, int row, int K, const float* in, float* out,
                                  int wave, int lane) {
  const cptr<float> w = as_const(W);
  float s[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.0f;
  for (int k0 = 0; k0 < K; k0 += 16) {
    float x[16];
    if (k0 + 16 <= K) {
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = in[64 * (k0 + k) + lane];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const cptr<float> q = w + (16 * wave + r) * row + k0;
#pragma unroll
        for (int k = 0; k < 16; ++k) s[r] = fmaf(q[k], x[k], s[r]);
      }
    } else {
      for (int k = k0; k < K; ++k) {
        const float xk = in[64 * k + lane];
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = fmaf(w[(16 * wave + r) * row + k], xk, s[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) out[64 * (16 * wave + r) + lane] = s[r] > 0.0f ? s[r] : 0.0f;
}

// Density at point p of each lane of wave 0 (all four waves pass the same
// points; lanes that are not `live` get no meaningful value).  buf_e, buf_h:
// LDS (RM_DENS_LDS).
template <bool DEEP>
__device__ __forceinline__ float density_block(const ObjStatic* objs, int obj, const float p[3], bool live,
                                      float* buf_e, float* buf_h) {
  const cptr<ObjStatic> ob = as_const(objs + obj);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int L = ob->L, din = ob->din;
  const float* params = ob->params;
  const uint32_t hm = ob->hashed_mask;
  for (int l = wave; l < L; l += 4) {
    float ex, ey;
    encode_wave(as_global((const char*)(params + ob->off[l])), ob->N_l[l], ob->T_l[l], (hm >> l) & 1u,
                false, live, p, (uint32_t)lane & 1u, ex, ey);
    buf_e[64 * (2 * l) + lane] = ex;
    buf_e[64 * (2 * l + 1) + lane] = ey;
  }
  __syncthreads();
  const float* W = params + ob->P_grid;
  dens_layer(W, din, din, buf_e, buf_h, wave, lane);
  W += RM_HIDDEN * din;
  __syncthreads();
  float* in = buf_h;
  if (DEEP) {
    float* out = buf_e;
    for (int k = 1; k < ob->mlp_layers; ++k) {
      dens_layer(W, RM_HIDDEN, RM_HIDDEN, in, out, wave, lane);
      W += RM_HH;
      __syncthreads();
      float* t = in;
      in = out;
      out = t;
    }
  }
  float y0 = 0.0f;
  if (wave == 0) {
    const cptr<float> w2 = as_const((const float*)W);
#pragma unroll
    for (int h = 0; h < RM_HIDDEN; ++h) y0 = fmaf(w2[h], in[64 * h + lane], y0);
  }
  return expf(fminf(y0, 15.0f));
}

// LDS of a density workgroup: the encoding's buffer also holds every second
// hidden layer of a deeper MLP
#define RM_DENS_LDS(DEEP)                                                             \
  __shared__ float s_e[64 * ((DEEP) ? RM_HIDDEN : 2 * RM_MAX_LEVELS)];                \
  __shared__ float s_h[64 * RM_HIDDEN]

template <bool DEEP>
__global__ __launch_bounds__(RM_DENS_WG) __attribute__((amdgpu_waves_per_eu(6)))
void k_query_density(const ObjStatic* objs, int obj,
                                                              const float* xyz, int64_t n,
                                                              float* sigma) {
  RM_DENS_LDS(DEEP);
  const int64_t t = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
  const bool live = t < n;
  const int64_t i = live ? t : n - 1;
  const float x[3] = {xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]};
  const cptr<ObjStatic> ob = as_const(objs + obj);
  const float half[3] = {ob->half[0], ob->half[1], ob->half[2]};
  const float inv[3] = {ob->inv2a[0], ob->inv2a[1], ob->inv2a[2]};
  float p[3];
  unit_pos(x, half, inv, p);
  const float s = density_block<DEEP>(objs, obj, p, live, s_e, s_h);
  if (threadIdx.x < 64 && live) sigma[t] = s;
}

// ---------------------------------------------------------------------------
// Meshing: marching cubes (Lorensen & Cline) over a (res+1)^3 corner grid,
// x fastest, corner (i, j, k) at lo + (hi - lo) * (i, j, k) / res.

__device__ inline float grid_coord(float lo, float hi, int g, int res) {
  return lo + (hi - lo) * ((float)g / (float)res);
}

// density of an object at the corners of a grid over its box
template <bool DEEP>
__global__ __launch_bounds__(RM_DENS_WG) __attribute__((amdgpu_waves_per_eu(6))) void k_density_grid(const ObjStatic* objs, int obj, int res,
                                                             float* grid) {
  RM_DENS_LDS(DEEP);
  // workgroup i runs on XCD i mod 8: each XCD takes a contiguous range of the
  // grid, whose neighbouring corners share table lines
  const uint32_t n1 = (uint32_t)res + 1u, n = n1 * n1 * n1;
  const uint32_t nb = (n + 63u) / 64u, per_xcd = (nb + 7u) >> 3;
  const uint32_t b = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
  if (b >= nb) return;
  const uint32_t t = b * 64u + (threadIdx.x & 63u);
  const bool live = t < n;
  const uint32_t i = live ? t : n - 1u;
  const cptr<ObjStatic> ob = as_const(objs + obj);
  const float half[3] = {ob->half[0], ob->half[1], ob->half[2]};
  const float inv[3] = {ob->inv2a[0], ob->inv2a[1], ob->inv2a[2]};
  const int g[3] = {(int)(i % n1), (int)((i / n1) % n1), (int)(i / (n1 * n1))};
  float x[3], p[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] = grid_coord(-half[a], half[a], g[a], res);
  unit_pos(x, half, inv, p);
  const float s = density_block<DEEP>(objs, obj, p, live, s_e, s_h);
  if (threadIdx.x < 64 && live) grid[t] = s;
}

// case of cell c and its 8 corner values
__device__ inline int mc_cell(const MeshArgs& m, int64_t c, float v[8], int g0[3]) {
  const int64_t n1 = m.res + 1;
  g0[0] = (int)(c % m.res);
  g0[1] = (int)((c / m.res) % m.res);
  g0[2] = (int)(c / ((int64_t)m.res * m.res));
  int mask = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int64_t gi = (g0[0] + (k & 1)) + n1 * ((g0[1] + ((k >> 1) & 1)) + n1 * (g0[2] + (k >> 2)));
    v[k] = m.grid[gi];
    mask |= (v[k] > m.iso ? 1 : 0) << k;
  }
  return mask;
}

__global__ __launch_bounds__(256) void k_mc_count(MeshArgs m) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= (int64_t)m.res * m.res * m.res) return;
  float v[8];
  int g0[3];
  m.cnt[c] = m.ntri[mc_cell(m, c, v, g0)];
}

// exclusive scan of cnt[0 .. n) in blocks of RM_MC_SCAN (in place); block totals to bsum
__global__ __launch_bounds__(256) void k_mc_scan_blocks(int* cnt, int64_t n, int* bsum) {
  __shared__ int s_w[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t b0 = (int64_t)blockIdx.x * RM_MC_SCAN + 4 * tid;  // 4 consecutive per thread
  int x[4], mine = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x[k] = b0 + k < n ? cnt[b0 + k] : 0;
    mine += x[k];
  }
  int inc = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  int off = 0;
  for (int w = 0; w < wave; ++w) off += s_w[w];
  int run = off + inc - mine;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (b0 + k < n) cnt[b0 + k] = run;
    run += x[k];
  }
  if (tid == 255) bsum[blockIdx.x] = off + inc;
}

// exclusive scan of the block totals (nb <= 4 * 1024) in one block; total to bsum[nb]
__global__ __launch_bounds__(1024) void k_mc_scan_totals(int* bsum, int nb) {
  __shared__ int s_w[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int x[4], mine = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x[k] = 4 * tid + k < nb ? bsum[4 * tid + k] : 0;
    mine += x[k];
  }
  int inc = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  int off = 0, tot = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) off += s_w[w];
    tot += s_w[w];
  }
  int run = off + inc - mine;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (4 * tid + k < nb) bsum[4 * tid + k] = run;
    run += x[k];
  }
  if (tid == 0) bsum[nb] = tot;
}

__global__ __launch_bounds__(256) void k_mc_emit(MeshArgs m) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= (int64_t)m.res * m.res * m.res) return;
  float v[8];
  int g0[3];
  const int mask = mc_cell(m, c, v, g0);
  const int nt = m.ntri[mask];
  if (nt == 0) return;
  const int64_t base = (int64_t)m.cnt[c] + m.bsum[c / RM_MC_SCAN];
  for (int t = 0; t < nt; ++t) {
    if (base + t >= m.max_tris) return;
    float* o = m.out + 9 * (base + t);
    for (int q = 0; q < 3; ++q) {
      const int e = m.tris[16 * mask + 3 * t + q];
      const int ca = m.edge_a[e], cb = m.edge_b[e];
      const float s = (m.iso - v[ca]) / (v[cb] - v[ca]);
      float x[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float xa = grid_coord(m.lo[a], m.hi[a], g0[a] + ((ca >> a) & 1), m.res);
        const float xb = grid_coord(m.lo[a], m.hi[a], g0[a] + ((cb >> a) & 1), m.res);
        x[a] = xa + s * (xb - xa);
      }
      if (m.world) {  // box pose: x_w = R x + t
#pragma unroll
        for (int a = 0; a < 3; ++a)
          o[3 * q + a] = ((m.R[3 * a] * x[0] + m.R[3 * a + 1] * x[1]) + m.R[3 * a + 2] * x[2]) + m.t[a];
      } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) o[3 * q + a] = x[a];
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_debug_encode(const ObjStatic* objs, int obj,
                                                      const float* pts, int64_t n, uint32_t* idx,
                                                      float* feat) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const ObjStatic& ob = objs[obj];
  const float p[3] = {pts[3 * t], pts[3 * t + 1], pts[3 * t + 2]};
  for (int l = 0; l < ob.L; ++l) {
    Cell cl;
    make_cell(p, ob.N_l[l], cl);
    const bool hashed = (ob.hashed_mask >> l) & 1u;
    const float* G = ob.params + ob.off[l];
    float ex = 0.0f, ey = 0.0f;
    for (int b = 0; b < 8; ++b) {
      const uint32_t id = corner_index(cl, b, ob.N_l[l], ob.T_l[l], hashed);
      const float w = corner_weight(cl, b);
      if (idx) idx[(t * ob.L + l) * 8 + b] = id;
      ex = fmaf(w, G[2 * (int64_t)id], ex);
      ey = fmaf(w, G[2 * (int64_t)id + 1], ey);
    }
    if (feat) {
      feat[(t * ob.L + l) * 2] = ex;
      feat[(t * ob.L + l) * 2 + 1] = ey;
    }
  }
}

// parameter initialisation: grid U(-1e-4, 1e-4), MLP Glorot-uniform, each
// value drawn from Philox with counter (index, kind, 0xFFFFFFFF, 0)
__global__ __launch_bounds__(256) void k_init_params(float* params, int64_t P_grid, int din,
                                                     int nh, uint32_t k0, uint32_t k1) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n1 = (int64_t)RM_HIDDEN * din, nhh = n1 + (int64_t)(nh - 1) * RM_HH;
  const int64_t n2 = nhh + RM_DOUT * RM_HIDDEN;
  const int64_t n3 = n2 + RM_HIDDEN * RM_GEO, n4 = n3 + 3 * RM_HIDDEN;
  if (i >= P_grid + n4) return;
  uint32_t kind;
  float lim;
  if (i < P_grid) {
    kind = 0u;
    lim = 1e-4f;
  } else {
    const int64_t j = i - P_grid;
    if (j < n1) { kind = 1u; lim = sqrtf(6.0f / (float)(RM_HIDDEN + din)); }
    else if (j < nhh) { kind = 5u; lim = sqrtf(6.0f / (float)(2 * RM_HIDDEN)); }
    else if (j < n2) { kind = 2u; lim = sqrtf(6.0f / (float)(RM_DOUT + RM_HIDDEN)); }
    else if (j < n3) { kind = 3u; lim = sqrtf(6.0f / (float)(RM_HIDDEN + RM_GEO)); }
    else { kind = 4u; lim = sqrtf(6.0f / (float)(3 + RM_HIDDEN)); }
  }
  uint32_t x[4];
  philox4x32_10((uint32_t)i, kind, 0xFFFFFFFFu, 0u, k0, k1, x);
  const float u = (float)(x[0] >> 8) * (1.0f / 16777216.0f);
  params[i] = (2.0f * u - 1.0f) * lim;
}

// sample positions of a launch's rays (inspection)
template <int NS>
__global__ __launch_bounds__(256) void k_debug_positions(StepArgs a, float* pos) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= a.S) return;
  const RayRec R = a.rays[s / NS];
  float p[3] = {0.0f, 0.0f, 0.0f};
  if (R.flags & RM_F_HIT) sample_pos(R, (int)(s % NS), a.objs[R.obj].half, a.objs[R.obj].inv2a, p);
  pos[3 * s] = p[0];
  pos[3 * s + 1] = p[1];
  pos[3 * s + 2] = p[2];
}

// clears the per-object loss accumulators of a launch's objects
__global__ void k_reset_loss(StepArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n_sobj) return;
  ObjState* st = a.state + a.sobj[i].obj;
  st->loss_acc = 0.0f;
  st->n_loss = 0;
}

// occupancy refresh: bit = density at the cell centre > threshold; a
// workgroup covers 64 consecutive cells, whose two words come from a ballot
template <bool DEEP>
__global__ __launch_bounds__(RM_DENS_WG) __attribute__((amdgpu_waves_per_eu(6))) void k_occ_update(const ObjStatic* objs, int obj,
                                                           uint32_t* bits, float threshold) {
  RM_DENS_LDS(DEEP);
  const int lane = threadIdx.x & 63;
  // workgroup i runs on XCD i mod 8: contiguous ranges of cells, as in k_density_grid
  const int b = (int)(blockIdx.x & 7u) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int cell = b * 64 + lane;  // < 64^3, grid exact
  const float p[3] = {((float)(cell & 63) + 0.5f) / 64.0f,
                      ((float)((cell >> 6) & 63) + 0.5f) / 64.0f,
                      ((float)(cell >> 12) + 0.5f) / 64.0f};
  const float s = density_block<DEEP>(objs, obj, p, true, s_e, s_h);
  if (threadIdx.x >= 64) return;
  const uint64_t m = __ballot(s > threshold);
  if (lane < 2) bits[(cell >> 5) + lane] = (uint32_t)(m >> (32 * lane));
}

__global__ void k_fill(float* x, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

// ---------------------------------------------------------------------------
// launchers

static inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

// A launch takes fewer than 2^32 work-items: kernels that may have more run
// over their work in rounds, or in several launches, of this many.
constexpr int64_t kMaxWorkItems = int64_t(1) << 28;

#define RM_NS_SWITCH(NS, CALL)              \
  switch (NS) {                             \
    case 32: { constexpr int NSC = 32; CALL; break; }   \
    case 64: { constexpr int NSC = 64; CALL; break; }   \
    case 128: { constexpr int NSC = 128; CALL; break; } \
    default: return hipErrorInvalidValue;   \
  }

// Workgroups of a ray kernel: the rays', then the packing's (K1 = 0: none).
static inline unsigned ray_blocks(const StepArgs& a, int n, int K1) {
  const unsigned pack = K1 ? a.n_sobj * (8 + 2 * (a.mlp_layers - 1)) * RM_PACK_SPLIT : 0;
  return cdiv(n, 256) + pack;
}

hipError_t rm_launch_raygen(const StepArgs& a, int NS, int K1, hipStream_t st) {
  if (a.n_rays <= 0) return hipSuccess;
  if (a.mlp_layers < 1 || a.mlp_layers > RM_MAX_MLP_LAYERS) return hipErrorInvalidValue;
  RM_NS_SWITCH(NS, (k_raygen<NSC><<<ray_blocks(a, a.n_rays, K1), 256, 0, st>>>(a, K1)));
  return hipGetLastError();
}

hipError_t rm_launch_encode_fwd(const StepArgs& a, int NS, int block, hipStream_t st) {
  if (a.n_bblocks <= 0) return hipSuccess;
  const int64_t live = std::min((int64_t)a.n_rays * NS, kMaxWorkItems);
  if (a.live) RM_NS_SWITCH(NS, (k_live<NSC><<<cdiv(live, 256), 256, 0, st>>>(a)));
  // workgroups rounded up to whole rounds of the 8 XCDs
  RM_NS_SWITCH(NS, (k_encode_fwd<NSC><<<8 * ((a.n_bblocks + 7) / 8), block, 0, st>>>(a)));
  return hipGetLastError();
}

// The region size is a constant of the instance: as a value read at run time,
// the binning of 24 objects x 2048 rays took 419 us instead of 387.
#define RM_RB_SWITCH(RB, CALL)                        \
  switch (RB) {                                       \
    case 9: { constexpr int RBC = 9; CALL; break; }   \
    case 10: { constexpr int RBC = 10; CALL; break; } \
    case 11: { constexpr int RBC = 11; CALL; break; } \
    default: return hipErrorInvalidValue;             \
  }

hipError_t rm_launch_bin_scatter(const StepArgs& a, const BinGroup& g, int NS, hipStream_t st) {
  if (g.bb_end <= g.bb_begin) return hipSuccess;
  const size_t lds = RM_STAGE_BYTES + (size_t)a.bin_max_R * (sizeof(int2) + sizeof(int));
  if (lds > 65536) {  // beyond the default dynamic LDS limit (tables of 2^22+ entries)
    hipError_t e0 = hipSuccess;
    RM_RB_SWITCH(a.region_bits,
                 RM_NS_SWITCH(NS, (e0 = hipFuncSetAttribute((const void*)k_bin_scatter<NSC, RBC>,
                                                            hipFuncAttributeMaxDynamicSharedMemorySize,
                                                            (int)lds))));
    if (e0 != hipSuccess) return e0;
  }
  StepArgs b = a;
  b.bb_begin = g.bb_begin;
  b.n_bblocks = g.bb_end - g.bb_begin;  // the group's blocks
  const dim3 grid(8 * ((b.n_bblocks + 7) / 8));
  RM_RB_SWITCH(a.region_bits,
               RM_NS_SWITCH(NS, (k_bin_scatter<NSC, RBC><<<grid, RM_SCAT_WG, lds, st>>>(b))));
  return hipGetLastError();
}

hipError_t rm_launch_bin_acc(const StepArgs& a, const BinGroup& g, hipStream_t st) {
  if (g.bin_end <= g.bin_begin) return hipSuccess;
  StepArgs b = a;
  b.bin_begin = g.bin_begin;
  k_bin_acc<<<g.bin_end - g.bin_begin, RM_ACC_WG, 0, st>>>(b);
  return hipGetLastError();
}

template <int PREC, int K1, int NH>
static hipError_t launch_field_k(const StepArgs& a, int NS, hipStream_t st) {
  if (a.mode == RM_MODE_FORWARD) {
    RM_NS_SWITCH(NS, (k_field<PREC, NSC, K1, NH, true><<<a.n_items, RM_WG, 0, st>>>(a)));
  } else {
    RM_NS_SWITCH(NS, (k_field<PREC, NSC, K1, NH, false><<<a.n_items, RM_WG, 0, st>>>(a)));
  }
  return hipGetLastError();
}

template <int NH>
static hipError_t launch_field_nh(const StepArgs& a, int NS, int K1, int prec, hipStream_t st) {
  if (K1 == 16)
    return prec ? launch_field_k<1, 16, NH>(a, NS, st) : launch_field_k<0, 16, NH>(a, NS, st);
  if (K1 == 32)
    return prec ? launch_field_k<1, 32, NH>(a, NS, st) : launch_field_k<0, 32, NH>(a, NS, st);
  return hipErrorInvalidValue;
}

hipError_t rm_launch_field(const StepArgs& a, int NS, int K1, int prec, hipStream_t st) {
  if (a.n_items <= 0) return hipSuccess;
  switch (a.mlp_layers) {
    case 1: return launch_field_nh<1>(a, NS, K1, prec, st);
    case 2: return launch_field_nh<2>(a, NS, K1, prec, st);
    case 3: return launch_field_nh<3>(a, NS, K1, prec, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t rm_launch_reduce(const StepArgs& a, hipStream_t st) {
  if (a.n_sobj <= 0) return hipSuccess;
  dim3 grid(cdiv(RM_REC_LOSS_NH(a.mlp_layers) + 1, RM_RED_COLS), a.n_sobj);
  k_reduce<<<grid, RM_RED_WG, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t rm_launch_bin_finish(const StepArgs& a, hipStream_t st) {
  if (a.n_fins <= 0 || !a.fuse_adam) return hipSuccess;
  k_bin_finish<<<a.n_fins, RM_FIN_WG, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t rm_launch_camera_rays(const StepArgs& a, int NS, const float* M, const float* c,
                                 float fx, float fy, float cx, float cy, int W, int pix0,
                                 int n_pix, int* n_hit, int K1, hipStream_t st) {
  if (n_pix <= 0) return hipSuccess;
  if (a.mlp_layers < 1 || a.mlp_layers > RM_MAX_MLP_LAYERS) return hipErrorInvalidValue;
  CamArgs ca;
  for (int k = 0; k < 9; ++k) ca.M[k] = M[k];
  for (int k = 0; k < 3; ++k) ca.c[k] = c[k];
  ca.fx = fx;
  ca.fy = fy;
  ca.cx = cx;
  ca.cy = cy;
  ca.W = W;
  ca.pix0 = pix0;
  RM_NS_SWITCH(NS, (k_camera_rays<NSC><<<ray_blocks(a, n_pix, K1), 256, 0, st>>>(a, ca, n_pix, n_hit, K1)));
  return hipGetLastError();
}

hipError_t rm_launch_user_rays(const StepArgs& a, int NS, const float* rays, int K1,
                               hipStream_t st) {
  if (a.n_rays <= 0) return hipSuccess;
  if (a.mlp_layers < 1 || a.mlp_layers > RM_MAX_MLP_LAYERS) return hipErrorInvalidValue;
  RM_NS_SWITCH(NS, (k_user_rays<NSC><<<ray_blocks(a, a.n_rays, K1), 256, 0, st>>>(a, rays, K1)));
  return hipGetLastError();
}

hipError_t rm_launch_query_density(const ObjStatic* objs, int obj, int nh, const float* xyz,
                                   int64_t n, float* sigma, hipStream_t st) {
  constexpr int64_t per = kMaxWorkItems / (RM_DENS_WG / 64);  // points of a launch
  for (; n > 0; n -= per, xyz += 3 * per, sigma += per) {
    const int64_t m = std::min(n, per);
    const unsigned nb = cdiv(m, 64);
    if (nh > 1) k_query_density<true><<<nb, RM_DENS_WG, 0, st>>>(objs, obj, xyz, m, sigma);
    else k_query_density<false><<<nb, RM_DENS_WG, 0, st>>>(objs, obj, xyz, m, sigma);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t rm_launch_density_grid(const ObjStatic* objs, int obj, int nh, int res, float* grid,
                                  hipStream_t st) {
  const int64_t n1 = res + 1;
  const unsigned nb = 8 * cdiv(cdiv(n1 * n1 * n1, 64), 8);  // whole rounds of the 8 XCDs
  if (nh > 1) k_density_grid<true><<<nb, RM_DENS_WG, 0, st>>>(objs, obj, res, grid);
  else k_density_grid<false><<<nb, RM_DENS_WG, 0, st>>>(objs, obj, res, grid);
  return hipGetLastError();
}

hipError_t rm_launch_mc_count(const MeshArgs& m, hipStream_t st) {
  const int64_t nc = (int64_t)m.res * m.res * m.res;
  k_mc_count<<<cdiv(nc, 256), 256, 0, st>>>(m);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nb = (int)cdiv(nc, RM_MC_SCAN);
  k_mc_scan_blocks<<<nb, 256, 0, st>>>(m.cnt, nc, m.bsum);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_mc_scan_totals<<<1, 1024, 0, st>>>(m.bsum, nb);
  return hipGetLastError();
}

hipError_t rm_launch_mc_emit(const MeshArgs& m, hipStream_t st) {
  const int64_t nc = (int64_t)m.res * m.res * m.res;
  k_mc_emit<<<cdiv(nc, 256), 256, 0, st>>>(m);
  return hipGetLastError();
}

hipError_t rm_launch_debug_encode(const ObjStatic* objs, int obj, const float* p, int64_t n,
                                  uint32_t* idx, float* feat, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_debug_encode<<<cdiv(n, 256), 256, 0, st>>>(objs, obj, p, n, idx, feat);
  return hipGetLastError();
}

hipError_t rm_launch_init(float* params, int64_t P_grid, int din, int nh, uint32_t k0,
                          uint32_t k1, hipStream_t st) {
  const int64_t n = P_grid + (int64_t)RM_HIDDEN * din + (int64_t)(nh - 1) * RM_HH +
                    RM_DOUT * RM_HIDDEN + RM_HIDDEN * RM_GEO + 3 * RM_HIDDEN;
  k_init_params<<<cdiv(n, 256), 256, 0, st>>>(params, P_grid, din, nh, k0, k1);
  return hipGetLastError();
}

hipError_t rm_launch_debug_positions(const StepArgs& a, int NS, float* pos, hipStream_t st) {
  if (a.S <= 0) return hipSuccess;
  RM_NS_SWITCH(NS, (k_debug_positions<NSC><<<cdiv(a.S, 256), 256, 0, st>>>(a, pos)));
  return hipGetLastError();
}

hipError_t rm_launch_reset_loss(const StepArgs& a, hipStream_t st) {
  if (a.n_sobj <= 0) return hipSuccess;
  k_reset_loss<<<cdiv(a.n_sobj, 64), 64, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t rm_launch_occ_update(const ObjStatic* objs, int obj, int nh, uint32_t* bits,
                                float threshold, hipStream_t st) {
  constexpr int nb = 64 * 64 * 64 / 64;
  if (nh > 1) k_occ_update<true><<<nb, RM_DENS_WG, 0, st>>>(objs, obj, bits, threshold);
  else k_occ_update<false><<<nb, RM_DENS_WG, 0, st>>>(objs, obj, bits, threshold);
  return hipGetLastError();
}

hipError_t rm_launch_fill(float* x, int64_t n, float v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_fill<<<cdiv(n, 256), 256, 0, st>>>(x, n, v);
  return hipGetLastError();
}
