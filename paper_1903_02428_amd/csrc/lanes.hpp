// One lane's share of a feature row: 16-byte vectors (4 fp32 or 8 bf16) where
// rows are 16-byte aligned, single elements otherwise; arithmetic in fp32.
#pragma once

#include "common.hpp"

#include <type_traits>

namespace pyg {

// ------------------------------------------------------- lane vector types
template <typename T, bool VEC> struct Lane;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <> struct Lane<float, true> {  // 4 x fp32 = 16 B
    using R = float4;
    static constexpr int N = 4;
    __device__ static R load(const float *p) { return *reinterpret_cast<const R *>(p); }
    __device__ static R load_nt(const float *p) {
        const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
        return make_float4(v.x, v.y, v.z, v.w);
    }
    __device__ static R zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ static float get(const R &r, int e) { return e == 0 ? r.x : e == 1 ? r.y : e == 2 ? r.z : r.w; }
    __device__ static void store(float *p, const float (&v)[N]) { *reinterpret_cast<R *>(p) = make_float4(v[0], v[1], v[2], v[3]); }
};
template <> struct Lane<uint16_t, true> {  // 8 x bf16 = 16 B
    using R = uint4;
    static constexpr int N = 8;
    __device__ static R load(const uint16_t *p) { return *reinterpret_cast<const R *>(p); }
    __device__ static R load_nt(const uint16_t *p) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    __device__ static R zero() { return make_uint4(0, 0, 0, 0); }
    __device__ static float get(const R &r, int e) {
        const uint32_t w = (e >> 1) == 0 ? r.x : (e >> 1) == 1 ? r.y : (e >> 1) == 2 ? r.z : r.w;
        return (e & 1) ? __uint_as_float(w & 0xFFFF0000u) : __uint_as_float(w << 16);
    }
    __device__ static void store(uint16_t *p, const float (&v)[N]) {
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = uint32_t(f32_to_bf16_rne(v[2 * i])) | (uint32_t(f32_to_bf16_rne(v[2 * i + 1])) << 16);
        *reinterpret_cast<R *>(p) = make_uint4(o[0], o[1], o[2], o[3]);
    }
};
template <> struct Lane<float, false> {
    using R = float;
    static constexpr int N = 1;
    __device__ static R load(const float *p) { return *p; }
    __device__ static R load_nt(const float *p) { return __builtin_nontemporal_load(p); }
    __device__ static R zero() { return 0.f; }
    __device__ static float get(const R &r, int) { return r; }
    __device__ static void store(float *p, const float (&v)[N]) { *p = v[0]; }
};
template <> struct Lane<uint16_t, false> {
    using R = uint16_t;
    static constexpr int N = 1;
    __device__ static R load(const uint16_t *p) { return *p; }
    __device__ static R load_nt(const uint16_t *p) { return __builtin_nontemporal_load(p); }
    __device__ static R zero() { return 0; }
    __device__ static float get(const R &r, int) { return bf16_bits_to_f32(r); }
    __device__ static void store(uint16_t *p, const float (&v)[N]) { *p = f32_to_bf16_rne(v[0]); }
};

// Stores one lane's EP results of a row: in the row dtype T, or as fp32
// (OF32: partial rows of source blocks, folded later).
template <typename T, bool VEC, bool OF32>
__device__ __forceinline__ void store_out(void *out, int64_t idx, const float (&v)[Lane<T, VEC>::N]) {
    constexpr int EP = Lane<T, VEC>::N;
    if constexpr (OF32) {
        float *o = static_cast<float *>(out) + idx;
        if constexpr (VEC) {
#pragma unroll
            for (int k = 0; k < EP / 4; ++k)
                reinterpret_cast<float4 *>(o)[k] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
        } else {
            o[0] = v[0];
        }
    } else {
        Lane<T, VEC>::store(static_cast<T *>(out) + idx, v);
    }
}

template <typename T>
__device__ __forceinline__ float ld(const T *p, int64_t i) {
    if constexpr (sizeof(T) == 2) return bf16_bits_to_f32(reinterpret_cast<const uint16_t *>(p)[i]);
    else return p[i];
}

template <typename T>
__device__ __forceinline__ void st(T *p, int64_t i, float v) {
    if constexpr (sizeof(T) == 2) reinterpret_cast<uint16_t *>(p)[i] = f32_to_bf16_rne(v);
    else p[i] = v;
}

// V consecutive elements of p as floats / stored from floats: V = 4 is one
// 16-byte fp32 or 8-byte bf16 vector, V = 8 one 16-byte bf16 vector or two
// fp32 ones (the caller checks alignment).
template <typename T, int V>
__device__ __forceinline__ void ldv(const T *p, float (&o)[V]) {
    if constexpr (V == 1) {
        o[0] = ld(p, 0);
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int h = 0; h < V / 4; ++h) {
            const float4 v = reinterpret_cast<const float4 *>(p)[h];
            o[4 * h] = v.x, o[4 * h + 1] = v.y, o[4 * h + 2] = v.z, o[4 * h + 3] = v.w;
        }
    } else if constexpr (V == 4) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        o[0] = bf16_bits_to_f32(v.x & 0xFFFFu), o[1] = bf16_bits_to_f32(v.x >> 16);
        o[2] = bf16_bits_to_f32(v.y & 0xFFFFu), o[3] = bf16_bits_to_f32(v.y >> 16);
    } else {
        const uint4 v = *reinterpret_cast<const uint4 *>(p);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int h = 0; h < 4; ++h)
            o[2 * h] = bf16_bits_to_f32(w[h] & 0xFFFFu), o[2 * h + 1] = bf16_bits_to_f32(w[h] >> 16);
    }
}

template <typename T, int V>
__device__ __forceinline__ void stv(T *p, const float (&o)[V]) {
    if constexpr (V == 1) {
        st(p, 0, o[0]);
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int h = 0; h < V / 4; ++h)
            reinterpret_cast<float4 *>(p)[h] = make_float4(o[4 * h], o[4 * h + 1], o[4 * h + 2], o[4 * h + 3]);
    } else {
        uint32_t w[V / 2];
#pragma unroll
        for (int h = 0; h < V / 2; ++h)
            w[h] = uint32_t(f32_to_bf16_rne(o[2 * h])) | (uint32_t(f32_to_bf16_rne(o[2 * h + 1])) << 16);
        if constexpr (V == 4)
            *reinterpret_cast<uint2 *>(p) = make_uint2(w[0], w[1]);
        else
            *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

}  // namespace pyg
