// Device side of the projector gather (see kb.hip): one workgroup's part,
// shared by the stencil kernels, which carry it as extra workgroups of their
// launch, and by the batched gather.
#pragma once

#include "rsg_internal.h"

namespace rsg {
namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

template <class T> struct V4;
template <> struct V4<double> { using type = d4_t; };
template <> struct V4<float> { using type = f4_t; };

// Row of the accumulator element r held by lane group hi = l / 16.
__device__ __forceinline__ int acc_row(double, int hi, int r) { return hi + 4 * r; }
__device__ __forceinline__ int acc_row(float, int hi, int r) { return 4 * hi + r; }

__device__ __forceinline__ d4_t mfma16(double a, double b, d4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4_t mfma16(float a, float b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Gather for one (atom, 16-column tile, support chunk) by NW waves: the
// support of 4-entry groups is cut into nchunk contiguous chunks; a chunk's
// groups are dealt to kGatherSlots slots (slot j takes groups j, j + 16, ...
// in ascending order, one accumulator each), a wave owns kGatherSlots / NW
// slots, and the slots' products are added in slot order.  With one chunk the
// result goes to D scaled by h^3; with several, each chunk's sum goes to the
// partial buffer P and the scatter adds the chunks in order.  Either way the
// result depends neither on timing nor on NW.  Up to 4 slots of 4 groups are
// in flight per wave: their index loads, then their data loads, then the
// MFMAs; groups past the end count zero.  red: kGatherSlots * 64 values of LDS.
constexpr int kGatherSlots = 16;
template <int NW, class Tin, class Tc>
__device__ __forceinline__ void gather_tile(const Tin *__restrict__ in, int64_t ldo, int64_t ncols,
                                            const int4 at, int a, int ct,
                                            const int32_t *__restrict__ idx,
                                            const Tc *__restrict__ p, Tc h3, Tc *__restrict__ D,
                                            Tc *red, int chunk, int nchunk, Tc *__restrict__ P) {
    using V = typename V4<Tc>::type;
    constexpr int GU = 4, SPW = kGatherSlots / NW, SB = SPW < 4 ? SPW : 4;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int lo = l & 15, hi = l >> 4;
    const int64_t col = (int64_t)ct * 16 + lo;
    const bool cok = col < ncols;
    const Tin *inc = in + (cok ? (col >> 1) * ldo + (col & 1) : 0);
    const int ngall = at.y >> 2;
    const int per = (ngall + nchunk - 1) / nchunk;
    const int g0 = min(ngall, chunk * per);
    const int ngroups = min(ngall, g0 + per);
#pragma unroll 1
    for (int s0 = 0; s0 < SPW; s0 += SB) {
        V acc[SB];
#pragma unroll
        for (int j = 0; j < SB; ++j) acc[j] = V{0, 0, 0, 0};
        for (int g = g0 + w * SPW + s0; g < ngroups; g += GU * kGatherSlots) {
            int32_t ix[SB][GU];
            Tc bv[SB][GU], av[SB][GU];
#pragma unroll
            for (int j = 0; j < SB; ++j)
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    const int gq = g + j + u * kGatherSlots;
                    const int64_t e = (int64_t)at.x + 4 * (gq < ngroups ? gq : g) + hi;
                    ix[j][u] = idx[e];
                    bv[j][u] = lo < 4 && gq < ngroups ? p[e * 4 + lo] : (Tc)0;
                }
#pragma unroll
            for (int j = 0; j < SB; ++j)
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    const bool on = cok && g + j + u * kGatherSlots < ngroups;
                    av[j][u] = on ? (Tc)inc[2 * (int64_t)ix[j][u]] : (Tc)0;
                }
#pragma unroll
            for (int j = 0; j < SB; ++j)
#pragma unroll
                for (int u = 0; u < GU; ++u) acc[j] = mfma16(av[j][u], bv[j][u], acc[j]);
        }
#pragma unroll
        for (int j = 0; j < SB; ++j)
            if (lo < 4)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[(w * SPW + s0 + j) * 64 + (hi * 4 + lo) * 4 + r] = acc[j][r];
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int t = threadIdx.x, r = t & 3, i = (t >> 2) & 3, h = t >> 4;
        Tc v = red[t];
#pragma unroll
        for (int k = 1; k < kGatherSlots; ++k) v += red[k * 64 + t];
        const int64_t c = (int64_t)ct * 16 + acc_row(Tc(0), h, r);
        if (c < ncols) {
            if (nchunk == 1)
                D[((int64_t)a * 4 + i) * ncols + c] = h3 * v;
            else
                P[(((int64_t)a * 4 + i) * nchunk + chunk) * ncols + c] = v;
        }
    }
}

}  // namespace
}  // namespace rsg
