// The register file of the adjoints: values and upstream gradients of a
// genome's nodes in v[TN_RF_FILE] .. v255, addressed with a uniform index, for
// one, two or four tiles of 64 evaluations per wavefront (lane = evaluation);
// and the folded sums of a wavefront. Shared by tn_backward, the CPPN query and
// the CPPN adjoint.
#pragma once

#include "fwd_core.hpp"

namespace tn {

// First VGPR of the file; the compiler keeps the ones below (sin's argument
// reduction needs the room). Kernels carry
// __attribute__((amdgpu_num_vgpr(TN_RF_FILE / 2))): the attribute counts half
// of the unified VGPR budget.
#define TN_RF_FILE 64
constexpr int kRfFileRows = 256 - TN_RF_FILE;

// Makes the compiler count the file in the kernel's VGPR allocation.
__device__ __forceinline__ void rf_file_reserve() { asm volatile("" ::: "v255"); }

// d act / dz at this lane, from the stored value v (and z when needed).
__device__ __forceinline__ float act_slope(int act, float v, float z) {
  switch (act) {
    case TN_ACT_IDENTITY: return 1.0f;
    case TN_ACT_SIGMOID: return v * (1.0f - v);
    case TN_ACT_TANH: return fmaf(-v, v, 1.0f);
    case TN_ACT_RELU: return v > 0.0f ? 1.0f : 0.0f;
    case TN_ACT_SIN: return cosf(z);
    case TN_ACT_GAUSSIAN: return -2.0f * z * v;
    default: return z > 0.0f ? 1.0f : (z < 0.0f ? -1.0f : 0.0f);  // abs
  }
}

__device__ __forceinline__ bool slope_needs_z(int act) {
  return act == TN_ACT_SIN || act == TN_ACT_GAUSSIAN || act == TN_ACT_ABS;
}

// act_slope of K values, for activations whose slope follows from the value.
template <int K>
__device__ __forceinline__ void act_slopes_v(int act, const float (&v)[K], float (&d)[K]) {
  if (act == TN_ACT_TANH) {
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] = act_slope(TN_ACT_TANH, v[k], 0.0f);
  } else if (act == TN_ACT_IDENTITY) {
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] = 1.0f;
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k)
      d[k] = act == TN_ACT_SIGMOID ? act_slope(TN_ACT_SIGMOID, v[k], 0.0f)
                                   : act_slope(TN_ACT_RELU, v[k], 0.0f);
  }
}

// act_slope of K values, one branch for all of them.
template <int K>
__device__ __forceinline__ void act_slopes(int act, const float (&v)[K], const float (&z)[K],
                                           float (&d)[K]) {
  if (!slope_needs_z(act)) {
    act_slopes_v<K>(act, v, d);
  } else if (act == TN_ACT_SIN) {
    // one cosine at a time: the reduction of a large argument takes many
    // registers
    float zz[K];
#pragma unroll
    for (int k = 0; k < K; ++k) zz[k] = z[k];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      d[k] = act_slope(TN_ACT_SIN, v[k], zz[k]);
      asm volatile("" : "+v"(d[k]), "+v"(zz[(k + 1) % K]));
    }
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      d[k] = act == TN_ACT_GAUSSIAN ? act_slope(TN_ACT_GAUSSIAN, v[k], z[k])
                                    : act_slope(TN_ACT_ABS, v[k], z[k]);
    }
  }
}

// Rows of four sums that a computed node with ne in-edges takes (its bias and
// its in-edges).
__device__ __forceinline__ int sum_rows(int ne) { return (ne + 4) / 4; }

// Files of K tiles, kRfFileRows / K rows each; V[r] of tile k is register
// v(TN_RF_FILE + kRfFileRows / K * k + r), G[r] the one after it. One index window each.
template <int K>
struct Files;
template <>
struct Files<1> {
  // V[r] := v
  static __device__ __forceinline__ void set_v(int r, const float (&v)[1]) {
    asm volatile(
        "s_set_gpr_idx_on %1, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v64, %0\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "s"(r)
        : "m0");
  }
  // V[r] := v, G[r] := 0
  static __device__ __forceinline__ void set_vg(int r, const float (&v)[1]) {
    asm volatile(
        "s_set_gpr_idx_on %1, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v64, %0\n\t"
        "v_mov_b32 v65, 0\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "s"(r)
        : "m0");
  }
  // t := V[r]
  static __device__ __forceinline__ void get_v(int r, float (&t)[1]) {
    asm volatile(
        "s_set_gpr_idx_on %1, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v64\n\t"
        "s_set_gpr_idx_off"
        : "=v"(t[0])
        : "s"(r)
        : "m0");
  }
  // s += w * V[r]
  static __device__ __forceinline__ void fma_v(float (&s)[1], float w, int r) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(SRC1)\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32 %0, %1, v64\n\t"
        "s_set_gpr_idx_off"
        : "+v"(s[0])
        : "s"(w), "s"(r)
        : "m0");
  }
  // g := G[r], v := V[r]
  static __device__ __forceinline__ void get_gv(int r, float (&g)[1], float (&v)[1]) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v65\n\t"
        "v_mov_b32 %1, v64\n\t"
        "s_set_gpr_idx_off"
        : "=v"(g[0]), "=v"(v[0])
        : "s"(r)
        : "m0");
  }
  // G[r] += a * w (one indexed read-modify-write per tile)
  static __device__ __forceinline__ void fma_g(int r, const float (&a)[1], float w) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(SRC2,DST)\n\t"
        "s_nop 1\n\t"
        "v_fma_f32 v65, %0, %1, v65\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(a[0]), "s"(w), "s"(r)
        : "m0");
  }
  // sum of a * V[r] over the tiles
  static __device__ __forceinline__ float dot_v(int r, const float (&a)[1]) {
    float t;
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mul_f32 %0, v64, %1\n\t"
        "s_set_gpr_idx_off"
        : "=&v"(t)
        : "v"(a[0]), "s"(r)
        : "m0");
    return t;
  }
  // the same, and G[r] += a * w (one indexed read-modify-write per tile)
  static __device__ __forceinline__ float dot_v_fma_g(int r, const float (&a)[1], float w) {
    float t;
    asm volatile(
        "s_set_gpr_idx_on %3, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mul_f32 %0, v64, %1\n\t"
        "s_set_gpr_idx_off\n\t"
        "s_set_gpr_idx_on %3, gpr_idx(SRC2,DST)\n\t"
        "s_nop 1\n\t"
        "v_fma_f32 v65, %1, %2, v65\n\t"
        "s_set_gpr_idx_off"
        : "=&v"(t)
        : "v"(a[0]), "s"(w), "s"(r)
        : "m0");
    return t;
  }
};
template <>
struct Files<2> {
  static __device__ __forceinline__ void set_v(int r, const float (&v)[2]) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v64, %0\n\t"
        "v_mov_b32 v160, %1\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "v"(v[1]), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void set_vg(int r, const float (&v)[2]) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v64, %0\n\t"
        "v_mov_b32 v160, %1\n\t"
        "v_mov_b32 v65, 0\n\t"
        "v_mov_b32 v161, 0\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "v"(v[1]), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void get_v(int r, float (&t)[2]) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v64\n\t"
        "v_mov_b32 %1, v160\n\t"
        "s_set_gpr_idx_off"
        : "=v"(t[0]), "=v"(t[1])
        : "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void fma_v(float (&s)[2], float w, int r) {
    asm volatile(
        "s_set_gpr_idx_on %3, gpr_idx(SRC1)\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32 %0, %2, v64\n\t"
        "v_fmac_f32 %1, %2, v160\n\t"
        "s_set_gpr_idx_off"
        : "+v"(s[0]), "+v"(s[1])
        : "s"(w), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void get_gv(int r, float (&g)[2], float (&v)[2]) {
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v65\n\t"
        "v_mov_b32 %1, v161\n\t"
        "v_mov_b32 %2, v64\n\t"
        "v_mov_b32 %3, v160\n\t"
        "s_set_gpr_idx_off"
        : "=v"(g[0]), "=v"(g[1]), "=v"(v[0]), "=v"(v[1])
        : "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void fma_g(int r, const float (&a)[2], float w) {
    asm volatile(
        "s_set_gpr_idx_on %3, gpr_idx(SRC2,DST)\n\t"
        "s_nop 1\n\t"
        "v_fma_f32 v65, %0, %2, v65\n\t"
        "v_fma_f32 v161, %1, %2, v161\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(a[0]), "v"(a[1]), "s"(w), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ float dot_v(int r, const float (&a)[2]) {
    float t;
    asm volatile(
        "s_set_gpr_idx_on %3, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mul_f32 %0, v64, %1\n\t"
        "v_fmac_f32 %0, v160, %2\n\t"
        "s_set_gpr_idx_off"
        : "=&v"(t)
        : "v"(a[0]), "v"(a[1]), "s"(r)
        : "m0");
    return t;
  }
  static __device__ __forceinline__ float dot_v_fma_g(int r, const float (&a)[2], float w) {
    float t;
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mul_f32 %0, v64, %1\n\t"
        "v_fmac_f32 %0, v160, %2\n\t"
        "s_set_gpr_idx_off\n\t"
        "s_set_gpr_idx_on %4, gpr_idx(SRC2,DST)\n\t"
        "s_nop 1\n\t"
        "v_fma_f32 v65, %1, %3, v65\n\t"
        "v_fma_f32 v161, %2, %3, v161\n\t"
        "s_set_gpr_idx_off"
        : "=&v"(t)
        : "v"(a[0]), "v"(a[1]), "s"(w), "s"(r)
        : "m0");
    return t;
  }
};
template <>
struct Files<4> {
  static __device__ __forceinline__ void set_v(int r, const float (&v)[4]) {
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v64, %0\n\t"
        "v_mov_b32 v112, %1\n\t"
        "v_mov_b32 v160, %2\n\t"
        "v_mov_b32 v208, %3\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void set_vg(int r, const float (&v)[4]) {
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v64, %0\n\t"
        "v_mov_b32 v112, %1\n\t"
        "v_mov_b32 v160, %2\n\t"
        "v_mov_b32 v208, %3\n\t"
        "v_mov_b32 v65, 0\n\t"
        "v_mov_b32 v113, 0\n\t"
        "v_mov_b32 v161, 0\n\t"
        "v_mov_b32 v209, 0\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void get_v(int r, float (&t)[4]) {
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v64\n\t"
        "v_mov_b32 %1, v112\n\t"
        "v_mov_b32 %2, v160\n\t"
        "v_mov_b32 %3, v208\n\t"
        "s_set_gpr_idx_off"
        : "=v"(t[0]), "=v"(t[1]), "=v"(t[2]), "=v"(t[3])
        : "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void fma_v(float (&s)[4], float w, int r) {
    asm volatile(
        "s_set_gpr_idx_on %5, gpr_idx(SRC1)\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32 %0, %4, v64\n\t"
        "v_fmac_f32 %1, %4, v112\n\t"
        "v_fmac_f32 %2, %4, v160\n\t"
        "v_fmac_f32 %3, %4, v208\n\t"
        "s_set_gpr_idx_off"
        : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3])
        : "s"(w), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void get_gv(int r, float (&g)[4], float (&v)[4]) {
    asm volatile(
        "s_set_gpr_idx_on %8, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v65\n\t"
        "v_mov_b32 %1, v113\n\t"
        "v_mov_b32 %2, v161\n\t"
        "v_mov_b32 %3, v209\n\t"
        "v_mov_b32 %4, v64\n\t"
        "v_mov_b32 %5, v112\n\t"
        "v_mov_b32 %6, v160\n\t"
        "v_mov_b32 %7, v208\n\t"
        "s_set_gpr_idx_off"
        : "=v"(g[0]), "=v"(g[1]), "=v"(g[2]), "=v"(g[3]), "=v"(v[0]), "=v"(v[1]), "=v"(v[2]), "=v"(v[3])
        : "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void fma_g(int r, const float (&a)[4], float w) {
    asm volatile(
        "s_set_gpr_idx_on %5, gpr_idx(SRC2,DST)\n\t"
        "s_nop 1\n\t"
        "v_fma_f32 v65, %0, %4, v65\n\t"
        "v_fma_f32 v113, %1, %4, v113\n\t"
        "v_fma_f32 v161, %2, %4, v161\n\t"
        "v_fma_f32 v209, %3, %4, v209\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "s"(w), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ float dot_v(int r, const float (&a)[4]) {
    float t;
    asm volatile(
        "s_set_gpr_idx_on %5, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mul_f32 %0, v64, %1\n\t"
        "v_fmac_f32 %0, v112, %2\n\t"
        "v_fmac_f32 %0, v160, %3\n\t"
        "v_fmac_f32 %0, v208, %4\n\t"
        "s_set_gpr_idx_off"
        : "=&v"(t)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "s"(r)
        : "m0");
    return t;
  }
  static __device__ __forceinline__ float dot_v_fma_g(int r, const float (&a)[4], float w) {
    float t;
    asm volatile(
        "s_set_gpr_idx_on %6, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mul_f32 %0, v64, %1\n\t"
        "v_fmac_f32 %0, v112, %2\n\t"
        "v_fmac_f32 %0, v160, %3\n\t"
        "v_fmac_f32 %0, v208, %4\n\t"
        "s_set_gpr_idx_off\n\t"
        "s_set_gpr_idx_on %6, gpr_idx(SRC2,DST)\n\t"
        "s_nop 1\n\t"
        "v_fma_f32 v65, %1, %5, v65\n\t"
        "v_fma_f32 v113, %2, %5, v113\n\t"
        "v_fma_f32 v161, %3, %5, v161\n\t"
        "v_fma_f32 v209, %4, %5, v209\n\t"
        "s_set_gpr_idx_off"
        : "=&v"(t)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "s"(w), "s"(r)
        : "m0");
    return t;
  }
};

// A file of values alone: kShortFileRows registers from v[TN_RF_SHORT] on, shared
// by K tiles. 128 registers with the compiler's, so four wavefronts fit a SIMD.
#define TN_RF_SHORT 48
constexpr int kShortFileRows = 128 - TN_RF_SHORT;
__device__ __forceinline__ void short_file_reserve() { asm volatile("" ::: "v127"); }
template <int K>
struct ShortFiles;
template <>
struct ShortFiles<2> {
  static __device__ __forceinline__ void set_v(int r, const float (&v)[2]) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v48, %0\n\t"
        "v_mov_b32 v88, %1\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "v"(v[1]), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void get_v(int r, float (&t)[2]) {
    asm volatile(
        "s_set_gpr_idx_on %2, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v48\n\t"
        "v_mov_b32 %1, v88\n\t"
        "s_set_gpr_idx_off"
        : "=v"(t[0]), "=v"(t[1])
        : "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void fma_v(float (&s)[2], float w, int r) {
    asm volatile(
        "s_set_gpr_idx_on %3, gpr_idx(SRC1)\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32 %0, %2, v48\n\t"
        "v_fmac_f32 %1, %2, v88\n\t"
        "s_set_gpr_idx_off"
        : "+v"(s[0]), "+v"(s[1])
        : "s"(w), "s"(r)
        : "m0");
  }
};
template <>
struct ShortFiles<4> {
  static __device__ __forceinline__ void set_v(int r, const float (&v)[4]) {
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(DST)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 v48, %0\n\t"
        "v_mov_b32 v68, %1\n\t"
        "v_mov_b32 v88, %2\n\t"
        "v_mov_b32 v108, %3\n\t"
        "s_set_gpr_idx_off"
        : 
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void get_v(int r, float (&t)[4]) {
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
        "s_nop 1\n\t"
        "v_mov_b32 %0, v48\n\t"
        "v_mov_b32 %1, v68\n\t"
        "v_mov_b32 %2, v88\n\t"
        "v_mov_b32 %3, v108\n\t"
        "s_set_gpr_idx_off"
        : "=v"(t[0]), "=v"(t[1]), "=v"(t[2]), "=v"(t[3])
        : "s"(r)
        : "m0");
  }
  static __device__ __forceinline__ void fma_v(float (&s)[4], float w, int r) {
    asm volatile(
        "s_set_gpr_idx_on %5, gpr_idx(SRC1)\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32 %0, %4, v48\n\t"
        "v_fmac_f32 %1, %4, v68\n\t"
        "v_fmac_f32 %2, %4, v88\n\t"
        "v_fmac_f32 %3, %4, v108\n\t"
        "s_set_gpr_idx_off"
        : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3])
        : "s"(w), "s"(r)
        : "m0");
  }
};

// a + b folded across the wavefront's halves: lanes 0..31 hold a's sums of
// lanes l and l + 32, lanes 32..63 b's.
__device__ __forceinline__ float fold32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Likewise across 16 lanes: rows 0 and 2 of 16 lanes hold a's sums of rows
// (0, 1) and (2, 3), rows 1 and 3 b's.
__device__ __forceinline__ float fold16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Four sums as quarters of 16 lanes: quarter q holds sum kQuarter[q].
__device__ __forceinline__ float fold4(float t0, float t1, float t2, float t3) {
  return fold16(fold32(t0, t1), fold32(t2, t3));
}
__device__ __forceinline__ int sum_of_quarter(int q) { return (q >> 1) | ((q & 1) << 1); }

}  // namespace tn
