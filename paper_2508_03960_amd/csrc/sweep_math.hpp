// Device helpers of the grouped sweeps: table reads, group-sum adds and the
// in-place arithmetic of one operation.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbs {

__device__ __forceinline__ void cmul(float &ar, float &ai, float br, float bi) {
    const float r = ar * br - ai * bi;
    ai = ar * bi + ai * br;
    ar = r;
}

__device__ __forceinline__ void ld4(const float4 *p, int64_t i, float v[4]) {
    const float4 t = p[i];
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
}
__device__ __forceinline__ void ld4i(const int4 *p, int64_t i, int v[4]) {
    const int4 t = p[i];
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
}

// Table gathers and group-sum atomics through the global address space (the
// pointers come out of op descriptors and would otherwise be flat accesses).
typedef const __attribute__((address_space(1))) float *global_f32_ptr;
__device__ __forceinline__ float4 gather_row(const float4 *tab, int g) {
    global_f32_ptr p = (global_f32_ptr)(tab + g);
    return make_float4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ float2 gather_row(const float2 *tab, int g) {
    global_f32_ptr p = (global_f32_ptr)(tab + g);
    return make_float2(p[0], p[1]);
}
// Table reads at a 32-bit byte offset from a wave-uniform base: the address
// needs no VALU work (scalar base, vector offset).
__device__ __forceinline__ global_f32_ptr at_bytes(const void *tab, uint32_t off) {
    return (global_f32_ptr)((const __attribute__((address_space(1))) char *)tab + off);
}
__device__ __forceinline__ float4 gather_at(const float4 *tab, uint32_t off) {
    global_f32_ptr p = at_bytes(tab, off);
    return make_float4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ float2 gather_at(const float2 *tab, uint32_t off) {
    global_f32_ptr p = at_bytes(tab, off);
    return make_float2(p[0], p[1]);
}
__device__ __forceinline__ void group_add(double *p, double v) {
    __builtin_amdgcn_global_atomic_fadd_f64((__attribute__((address_space(1))) double *)p, v);
}

// Wave-uniform read of a table that no kernel writes while it runs: through
// the constant address space, so a uniform index becomes one scalar load.
typedef const __attribute__((address_space(4))) float *const_f32_ptr;
__device__ __forceinline__ float4 uniform_row(const float4 *tab, int g) {
    const_f32_ptr p = (const_f32_ptr)(tab + g);
    return make_float4(p[0], p[1], p[2], p[3]);
}

__device__ __forceinline__ void store_pair(double2 *p, double x, double y) {
    __attribute__((address_space(1))) double *q = (__attribute__((address_space(1))) double *)p;
    q[0] = x;
    q[1] = y;
}

// An op descriptor is the same for every lane: read it through the constant
// address space so that it arrives in scalar registers.
typedef const __attribute__((address_space(4))) uint64_t *const_u64_ptr;
template <class T>
__device__ __forceinline__ T load_desc(const T *ops, int o) {
    static_assert(sizeof(T) % 8 == 0, "descriptors are read as 64-bit words");
    uint64_t w[sizeof(T) / 8];
    const_u64_ptr p = (const_u64_ptr)(ops + o);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 8); ++i) w[i] = p[i];
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// v = v * a + b, the result in v's own register.  The compiler's accumulating
// FMA form would land it in b's register instead, and the state then needs a
// copy back on every pass of the op loop.
__device__ __forceinline__ void fma_inplace(float &v, float a, float b) {
    asm("v_fma_f32 %0, %0, %1, %2" : "+v"(v) : "v"(a), "v"(b));
}

// v = v * a - b in v's own register.
__device__ __forceinline__ void fms_inplace(float &v, float a, float b) {
    asm("v_fma_f32 %0, %0, %1, -%2" : "+v"(v) : "v"(a), "v"(b));
}

// (ar + i ai) <- (ar + i ai)(br + i bi) with the results in ar's and ai's own
// registers, so that a value the loop carries needs no copy.
__device__ __forceinline__ void cmul_inplace(float &ar, float &ai, float br, float bi) {
    const float t = ai * bi, u = ar * bi;
    fma_inplace(ai, br, u);
    fms_inplace(ar, br, t);
}

// rf_apply on the state divided by M0 (see sweep_body): the affine part b
// adds as it is.
__device__ __forceinline__ void rf_apply_ratio(const float4 &r0, const float4 &r1, const float4 &r2, float &mx,
                                               float &my, float &mz) {
    const float px = fmaf(r0.y, my, fmaf(r0.z, mz, r0.w));
    const float py = fmaf(r1.x, mx, fmaf(r1.z, mz, r1.w));
    const float pz = fmaf(r2.x, mx, fmaf(r2.y, my, r2.w));
    fma_inplace(mx, r0.x, px);
    fma_inplace(my, r1.y, py);
    fma_inplace(mz, r2.z, pz);
}

// Row of T applied after the transverse factor f = fr + i fi: the row acting
// on (f (mx + i my)) equals the folded row acting on (mx + i my).
__device__ __forceinline__ void fold_row(float4 &r, float fr, float fi) {
    const float t = r.y * fi, u = r.x * fi;
    fma_inplace(r.x, fr, t);
    fms_inplace(r.y, fr, u);
}

}  // namespace gbs
