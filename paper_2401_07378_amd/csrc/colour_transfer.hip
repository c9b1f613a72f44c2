// Colour transfer by NNS-EMD (Sec. IV-D): k-means palettes of two 8-bit RGB
// images, NNS-EMD from the reference palette to the source palette, and the
// source recoloured through the per-consumer barycentric map of the plan.
//
// The palette reduction is Lloyd iteration with every step made exactly
// reproducible, so its result does not depend on thread order:
//   start      centroid k = colour of pixel floor(k P / K)
//   assign     argmin_k sum_c (p_c - C_kc)^2 in FP64, channels in order, no
//              fused multiply-add, ties to the smallest k: an FP32 scan finds
//              the best two and the FP64 distances decide when the two are
//              within the scan's error bound (km_assign)
//   accumulate integer channel sums and counts per cluster: 64-bit integer
//              atomics, first into a per-workgroup LDS table, then one
//              global add per cluster and workgroup -- integer sums are the
//              same in any order
//   update     C_kc = S_kc / n_k (FP64, correctly rounded); an empty cluster
//              keeps its centroid
// The palettes become colour histograms: bin colour C / 255 and mass
// n_k / P, both rounded once from FP64 to FP32.  Recolouring writes
// round-half-even(255 T) clamped to 0..255 for each channel of the pixel's
// bin, or keeps the pixel when its bin received no flow.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "internal.hpp"
#include "point_search.hpp"

namespace nnsemd {
namespace {

constexpr int kKmThreads = 256;

__global__ __launch_bounds__(kKmThreads) void km_init(const uint8_t* __restrict__ px, int64_t P, int K,
                                                      double* __restrict__ C, unsigned long long* __restrict__ S) {
    const int k = blockIdx.x * kKmThreads + threadIdx.x;
    if (k >= K) return;
    const int64_t src = (int64_t)k * P / K;
#pragma unroll
    for (int c = 0; c < 3; ++c) C[k * 3 + c] = (double)px[src * 3 + c];
#pragma unroll
    for (int c = 0; c < 4; ++c) S[k * 4 + c] = 0ull;
}

// One assignment step: every pixel to its nearest centroid; the cluster
// sums and counts of this assignment are accumulated into S (zero on entry).
// The scan is FP32 on the matrix cores, as the point search's (ps::nns_tiles):
// with c = centroid - 128 rounded to FP32 and p = pixel - 128 (exact), a
// 16 x 16 block of keys ||c||^2 - 2 c.p is one v_mfma_f32_16x16x4_f32.
// |c|, |p| <= 128 per channel, so ||c||^2 and every partial sum stay below
// 2^18; the roundings of c (2^-18 each, times at most 4 * 128), of ||c||^2
// (three) and of the chain (three) total less than 0.013 + 6 * 2^-7 < 0.06 per
// key.  A second key more than 0.25 above the best one therefore cannot be the
// FP64 argmin or tie with it; otherwise the wavefront compares every centroid
// in FP64 with the definition's operations, ties to the smallest index.
// Bound: the matrix pipe (32 cycles per 256 keys).  Two 1024 x 1024 images,
// 256 bins, 11 passes each: the whole call 2480 -> 1255 us (FP64 distances to
// every centroid before; held to 128 registers, else the products land in
// accumulation registers and are copied: 1322 us).
constexpr int kKmGroups = 4;  // 64-pixel groups of a wavefront
__host__ __device__ inline int km_pad(int K) { return (K + 15) & ~15; }
__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(4))) void km_assign(const uint8_t* __restrict__ px, int64_t P, int K,
                                                        const double* __restrict__ C,
                                                        unsigned long long* __restrict__ S,
                                                        int32_t* __restrict__ assign) {
#pragma clang fp contract(off)
    extern __shared__ __align__(16) char km_lds[];
    const int Kp = km_pad(K);
    float* rec = reinterpret_cast<float*>(km_lds);                                 // Kp x 4: c, ||c||^2
    double* cs = reinterpret_cast<double*>(km_lds + 16 * (size_t)Kp);              // K x 3
    unsigned* acc = reinterpret_cast<unsigned*>(km_lds + 16 * (size_t)Kp + 24 * (size_t)K);  // K x 4
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, row = lane >> 4, comp = 3 - row;
    for (int k = tid; k < Kp; k += kKmThreads) {
        float f0 = 0.f, f1 = 0.f, f2 = 0.f, nn = INFINITY;  // padding: key +inf
        if (k < K) {
            const double c0 = C[3 * k], c1 = C[3 * k + 1], c2 = C[3 * k + 2];
            cs[3 * k] = c0;
            cs[3 * k + 1] = c1;
            cs[3 * k + 2] = c2;
            f0 = (float)(c0 - 128.0);
            f1 = (float)(c1 - 128.0);
            f2 = (float)(c2 - 128.0);
            nn = fmaf(f2, f2, fmaf(f1, f1, f0 * f0));
        }
        reinterpret_cast<float4*>(rec)[k] = make_float4(f0, f1, f2, nn);
    }
    for (int e = tid; e < 4 * K; e += kKmThreads) acc[e] = 0u;
    __syncthreads();
    const float* ap = rec + 4 * col + comp;
    for (int g = 0; g < kKmGroups; ++g) {
        const int64_t q0 = ((int64_t)blockIdx.x * kKmGroups + g) * kKmThreads + 64 * wave;
        if (q0 >= P) break;  // wavefront-uniform
        float bv[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t p = min(q0 + 16 * t + col, P - 1);
            bv[t] = comp == 3 ? 1.f : -2.f * (float)((int)px[p * 3 + (comp == 3 ? 0 : comp)] - 128);
        }
        const int64_t p = min(q0 + lane, P - 1);
        const int r = px[p * 3], gr = px[p * 3 + 1], b = px[p * 3 + 2];
        ps::Top2 best[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) best[t] = {INFINITY, INFINITY, 0x7fffffff};
#pragma unroll 2
        for (int s0 = 0; s0 < Kp; s0 += 16) {
            const float av = ap[4 * s0];
            ps::f32x4 key[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                key[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[t], (ps::f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float o = best[t].b1;
                const float m = __builtin_amdgcn_fmed3f(o, key[t][0], key[t][1]);
                const float n = fminf(o, fminf(key[t][0], key[t][1]));
                const float q = __builtin_amdgcn_fmed3f(n, key[t][2], key[t][3]);
                best[t].b2 = fminf(best[t].b2, fminf(m, q));
                best[t].b1 = fminf(n, fminf(key[t][2], key[t][3]));
                best[t].code = best[t].b1 < o ? s0 + 4 * row : best[t].code;
            }
        }
        const ps::Top2 w = ps::swap_merge<16>(ps::swap_merge<32>(best[0], best[2]), ps::swap_merge<32>(best[1], best[3]));
        // the winning four records once more: the first that holds the best
        const float f0 = -2.f * (float)(r - 128), f1 = -2.f * (float)(gr - 128), f2 = -2.f * (float)(b - 128);
        const int c0 = min(w.code, Kp - 4);
        int at = c0;
#pragma unroll
        for (int v = 3; v >= 0; --v) {
            const float4 q = reinterpret_cast<const float4*>(rec)[c0 + v];
            at = fmaf(q.x, f0, fmaf(q.y, f1, fmaf(q.z, f2, q.w))) == w.b1 ? c0 + v : at;
        }
        unsigned long long open = __ballot(q0 + lane < P && !(w.b2 - w.b1 > 0.25f));
        while (open != 0ull) {  // wavefront-uniform: one pixel at a time, 64 centroids a step
            const int who = __ffsll(open) - 1;
            open &= open - 1;
            const double dr = (double)__shfl(r, who), dg = (double)__shfl(gr, who), db = (double)__shfl(b, who);
            double bd = INFINITY;
            int bk = 0x7fffffff;
            for (int k = lane; k < K; k += 64) {
                const double t0 = dr - cs[3 * k], t1 = dg - cs[3 * k + 1], t2 = db - cs[3 * k + 2];
                double d = 0.0;
                d = d + t0 * t0;
                d = d + t1 * t1;
                d = d + t2 * t2;
                if (d < bd) {
                    bd = d;
                    bk = k;
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const double cd = __shfl_xor(bd, o);
                const int ck = __shfl_xor(bk, o);
                if (cd < bd || (cd == bd && ck < bk)) {
                    bd = cd;
                    bk = ck;
                }
            }
            at = lane == who ? bk : at;
        }
        if (q0 + lane < P) {
            assign[p] = at;
            atomicAdd(&acc[4 * at], (unsigned)r);
            atomicAdd(&acc[4 * at + 1], (unsigned)gr);
            atomicAdd(&acc[4 * at + 2], (unsigned)b);
            atomicAdd(&acc[4 * at + 3], 1u);
        }
    }
    __syncthreads();
    for (int e = tid; e < 4 * K; e += kKmThreads)
        if (acc[e] != 0u) atomicAdd(&S[e], (unsigned long long)acc[e]);
}

// Update from the sums of the last assignment, then clear them for the next.
__global__ __launch_bounds__(kKmThreads) void km_update(int K, double* __restrict__ C,
                                                        unsigned long long* __restrict__ S) {
    const int k = blockIdx.x * kKmThreads + threadIdx.x;
    if (k >= K) return;
    const unsigned long long n = S[k * 4 + 3];
    if (n > 0ull) {
#pragma unroll
        for (int c = 0; c < 3; ++c) C[k * 3 + c] = (double)S[k * 4 + c] / (double)n;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) S[k * 4 + c] = 0ull;
}

// Palette histogram from the final assignment's counts.
__global__ __launch_bounds__(kKmThreads) void km_palette(int K, int64_t P, const double* __restrict__ C,
                                                         const unsigned long long* __restrict__ S,
                                                         float* __restrict__ pts, float* __restrict__ mass) {
    const int k = blockIdx.x * kKmThreads + threadIdx.x;
    if (k >= K) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) pts[k * 3 + c] = (float)(C[k * 3 + c] / 255.0);
    mass[k] = (float)((double)S[k * 4 + 3] / (double)P);
}

__global__ __launch_bounds__(kKmThreads) void recolour_kernel(const uint8_t* __restrict__ px,
                                                              const int32_t* __restrict__ assign, int64_t P,
                                                              const double* __restrict__ T,
                                                              uint8_t* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * kKmThreads + threadIdx.x;
    if (p >= P) return;
    const double* t = T + (int64_t)assign[p] * 3;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (isnan(t[c])) {
            out[p * 3 + c] = px[p * 3 + c];
            continue;
        }
        double v = rint(255.0 * t[c]);
        v = v < 0.0 ? 0.0 : (v > 255.0 ? 255.0 : v);
        out[p * 3 + c] = (uint8_t)v;
    }
}

}  // namespace

size_t kmeans_lds_bytes(int K) { return 16 * (size_t)km_pad(K) + (24 + 16) * (size_t)K; }

int launch_kmeans(const uint8_t* px, int64_t P, int K, int iters, double* C, unsigned long long* S,
                  int32_t* assign, float* pts, float* mass, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const unsigned kb = (unsigned)((K + kKmThreads - 1) / kKmThreads);
    const unsigned pb = (unsigned)((P + kKmThreads * kKmGroups - 1) / (kKmThreads * kKmGroups));
    const size_t lds = kmeans_lds_bytes(K);
    if (lds > 48 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)km_assign, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(km_init, dim3(kb), dim3(kKmThreads), 0, st, px, P, K, C, S);
    for (int it = 0; it <= iters; ++it) {
        hipLaunchKernelGGL(km_assign, dim3(pb), dim3(kKmThreads), lds, st, px, P, K, C, S, assign);
        if (it < iters) hipLaunchKernelGGL(km_update, dim3(kb), dim3(kKmThreads), 0, st, K, C, S);
    }
    hipLaunchKernelGGL(km_palette, dim3(kb), dim3(kKmThreads), 0, st, K, P, C, S, pts, mass);
    return (int)hipGetLastError();
}

int launch_recolour(const uint8_t* px, const int32_t* assign, int64_t P, const double* T, uint8_t* out,
                    void* stream) {
    const unsigned pb = (unsigned)((P + kKmThreads - 1) / kKmThreads);
    hipLaunchKernelGGL(recolour_kernel, dim3(pb), dim3(kKmThreads), 0, (hipStream_t)stream, px, assign, P, T, out);
    return (int)hipGetLastError();
}

}  // namespace nnsemd
