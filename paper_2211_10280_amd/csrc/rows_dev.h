// A row of an embedding table or of a gradient held by one wave, for the forward pass and the segmented reduction.
#pragma once
#include "dev_common.h"
#include "kernels.h"

// A row of D elements held by one wave.  NQ float4 registers per lane (lane l owns chunks l, l+64, ...,
// bounds-checked against D/4) and, if TAIL, one more float per lane for the elements from 256*NQ on (at
// most 64 of them).  The second form is for dimensions just above a multiple of 256 -- D = 300 is
// 256 + 44 -- where a float4 that only 11 lanes use would cost every lane four registers per row; with
// one float instead, twice as many rows fit in flight at the same occupancy.
// LoadedRow is such a row as it comes from memory (a bf16 row not yet widened), WaveRow one in fp32 that
// arithmetic is done on.  Rows that are loaded several at a time are kept as LoadedRow until they are
// used, so that all loads of a batch are issued before the first wait.
template <typename T, int NQ, bool TAIL>
struct LoadedRow {
    typename Raw4<T>::type q[NQ];
    T t;

    __device__ __forceinline__ void load(const T *row, int D, int lane)
    {
        const int C4 = TAIL ? NQ * WAVE : (D >> 2);
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const int c = lane + WAVE * it;
            zero_raw(q[it]);
            if (c < C4) q[it] = ldraw(row + 4 * c);
        }
        if (TAIL) {
            const int e = 4 * WAVE * NQ + lane;
            t = (e < D) ? row[e] : (T)0;
        }
    }
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) zero_raw(q[it]);
        t = (T)0;
    }
    __device__ __forceinline__ float4 chunk(int it) const { return widen4(q[it]); }
    __device__ __forceinline__ float tail() const { return widen1(t); }
};

template <int NQ, bool TAIL>
struct WaveRow {
    float4 q[NQ];
    float t;

    __device__ __forceinline__ float4 chunk(int it) const { return q[it]; }
    __device__ __forceinline__ float tail() const { return t; }
    template <typename T>
    __device__ __forceinline__ void load(const T *row, int D, int lane)
    {
        LoadedRow<T, NQ, TAIL> r;
        r.load(row, D, lane);
        widen(r);
    }
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) q[it] = make_float4(0.f, 0.f, 0.f, 0.f);
        t = 0.f;
    }
    template <typename T>
    __device__ __forceinline__ void widen(const LoadedRow<T, NQ, TAIL> &r)
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) q[it] = r.chunk(it);
        t = TAIL ? r.tail() : 0.f;
    }
    template <typename R>
    __device__ __forceinline__ float dot(const R &o) const
    {
        float s = 0.f;
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const float4 v = o.chunk(it);
            s = fmaf(q[it].x, v.x, s);
            s = fmaf(q[it].y, v.y, s);
            s = fmaf(q[it].z, v.z, s);
            s = fmaf(q[it].w, v.w, s);
        }
        if (TAIL) s = fmaf(t, o.tail(), s);
        return s;
    }
    template <typename R>
    __device__ __forceinline__ void axpy(float a, const R &x)
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const float4 v = x.chunk(it);
            q[it].x = fmaf(a, v.x, q[it].x);
            q[it].y = fmaf(a, v.y, q[it].y);
            q[it].z = fmaf(a, v.z, q[it].z);
            q[it].w = fmaf(a, v.w, q[it].w);
        }
        if (TAIL) t = fmaf(a, x.tail(), t);
    }
    // element e of the row goes to dst[e]; dst has room for every lane's registers
    __device__ __forceinline__ void spill(float *dst, int lane) const
    {
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const int e = (lane + WAVE * it) * 4;
            dst[e + 0] = q[it].x;
            dst[e + 1] = q[it].y;
            dst[e + 2] = q[it].z;
            dst[e + 3] = q[it].w;
        }
        if (TAIL) dst[4 * WAVE * NQ + lane] = t;
    }
    // the row to D floats in global memory; STREAM: around the caches
    template <bool STREAM>
    __device__ __forceinline__ void store(float *row, int D, int lane) const
    {
        const int C4 = TAIL ? NQ * WAVE : (D >> 2);
#pragma unroll
        for (int it = 0; it < NQ; ++it) {
            const int c = lane + WAVE * it;
            if (c < C4) {
                if (STREAM) st4s(row + 4 * c, q[it]);
                else st4(row + 4 * c, q[it]);
            }
        }
        if (TAIL) {
            const int e = 4 * WAVE * NQ + lane;
            if (e < D) {
                if (STREAM) __builtin_nontemporal_store(t, (GLOBAL_AS float *)(row + e));
                else row[e] = t;
            }
        }
    }
};
