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
//              within the scan's error bound (km_assign); small images with
//              small palettes take the FP64 distances alone
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

#include <algorithm>

#include "internal.hpp"
#include "point_search.hpp"

namespace nnsemd {
namespace {

constexpr int kKmThreads = 256;

constexpr int kKmMax = 1024;       // centroids
__host__ __device__ inline int km_pad(int K) { return (K + 15) & ~15; }

// Search records of the centroids (one workgroup, thread k holds centroid k):
// c - 128 rounded to FP32 and its squared norm, the norm +inf for the padding
// and for a centroid that equals one of smaller index: that one wins every tie,
// so the later one never gets a pixel.  Images with a flat background start
// with many equal centroids, and those stay (an empty cluster keeps its
// centroid); with finite keys they would leave every background pixel open in
// every pass (two 1024 x 1024 images, three quarters white, 10 update steps:
// K = 16 5570 us so, 752 with this; K = 256 7730 and 1209; FP64 distances to
// every centroid, before the scan, took 1075 and 2425).  look: whether there may
// be equal ones; they meet in a hash table (at most half full, linear probing,
// so every probe ends).  Not made (RECORDS false) where the centroids themselves
// are compared (km_assign_direct).
__device__ void km_records(int K, bool look, double c0, double c1, double c2, float4* __restrict__ rec) {
#pragma clang fp contract(off)
    __shared__ double cc[3 * kKmMax];
    __shared__ int owner[2 * kKmMax], lowest[2 * kKmMax];
    const int k = threadIdx.x;
    const int bits = 33 - __builtin_clz(max(K - 1, 1));  // 2^bits >= 2 K
    const int slots = 1 << bits;
    int slot = 0;
    if (look) {  // workgroup-uniform
        for (int e = k; e < slots; e += (int)blockDim.x) {
            owner[e] = -1;
            lowest[e] = 0x7fffffff;
        }
        if (k < K) {
            cc[3 * k] = c0;
            cc[3 * k + 1] = c1;
            cc[3 * k + 2] = c2;
        }
        __syncthreads();
        if (k < K) {
            uint64_t h = (uint64_t)__double_as_longlong(c0) * 0x9e3779b97f4a7c15ull;
            h = (h ^ (h >> 29) ^ (uint64_t)__double_as_longlong(c1)) * 0x9e3779b97f4a7c15ull;
            h = (h ^ (h >> 29) ^ (uint64_t)__double_as_longlong(c2)) * 0x9e3779b97f4a7c15ull;
            slot = (int)(h >> (64 - bits));
            for (int probe = 0; probe < slots; ++probe) {
                int o = atomicCAS(&owner[slot], -1, k);
                if (o < 0) o = k;
                if (cc[3 * o] == c0 && cc[3 * o + 1] == c1 && cc[3 * o + 2] == c2) break;
                slot = (slot + 1) & (slots - 1);
            }
            atomicMin(&lowest[slot], k);
        }
        __syncthreads();
    }
    if (k < km_pad(K)) {
        float f0 = 0.f, f1 = 0.f, f2 = 0.f, nn = INFINITY;
        if (k < K) {
            f0 = (float)(c0 - 128.0);
            f1 = (float)(c1 - 128.0);
            f2 = (float)(c2 - 128.0);
            if (!look || lowest[slot] == k) nn = fmaf(f2, f2, fmaf(f1, f1, f0 * f0));
        }
        rec[k] = make_float4(f0, f1, f2, nn);
    }
}

template <bool RECORDS>
__global__ __launch_bounds__(kKmMax) void km_init(const uint8_t* __restrict__ px, int64_t P, int K,
                                                  double* __restrict__ C, unsigned long long* __restrict__ S,
                                                  float4* __restrict__ rec) {
    const int k = threadIdx.x;
    double c[3] = {0.0, 0.0, 0.0};
    if (k < K) {
        const int64_t src = (int64_t)k * P / K;
#pragma unroll
        for (int t = 0; t < 3; ++t) C[k * 3 + t] = c[t] = (double)px[src * 3 + t];
#pragma unroll
        for (int t = 0; t < 4; ++t) S[k * 4 + t] = 0ull;
    }
    if constexpr (RECORDS) km_records(K, true, c[0], c[1], c[2], rec);
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
// 256 bins, 11 passes each: the whole call 2480 -> 1234 us (FP64 distances to
// every centroid before; held to 128 registers, else the products land in
// accumulation registers and are copied: 1322 us).
// Open pixels (second key within 0.25): few of a wavefront's 64 are settled one
// after the other by the whole wavefront, more of them side by side, each lane
// comparing the centroids within 0.25 of its own pixel's best.  The line is
// where the two take as long, about 8 instructions a centroid against 90 and 14
// per 64 centroids a pixel (512 x 512, five levels a channel, K = 256: one by one
// 4200 us, with the line 741; the smooth images above have few open pixels).
constexpr int kKmGroups = 4;  // most 64-pixel groups of a wavefront
__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(4))) void km_assign(const uint8_t* __restrict__ px, int64_t P, int K, int groups,
                                                        const double* __restrict__ C,
                                                        const float4* __restrict__ records,
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
    for (int k = tid; k < Kp; k += kKmThreads) reinterpret_cast<float4*>(rec)[k] = records[k];
    for (int e = tid; e < 3 * K; e += kKmThreads) cs[e] = C[e];
    for (int e = tid; e < 4 * K; e += kKmThreads) acc[e] = 0u;
    __syncthreads();
    const float* ap = rec + 4 * col + comp;
    for (int g = 0; g < groups; ++g) {
        const int64_t q0 = ((int64_t)blockIdx.x * groups + g) * kKmThreads + 64 * wave;
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
        // the winning four records once more: the first that holds the best (a
        // pixel for which none does is open)
        const float f0 = -2.f * (float)(r - 128), f1 = -2.f * (float)(gr - 128), f2 = -2.f * (float)(b - 128);
        auto key32 = [](const float4& q, float g0, float g1, float g2) {
            return fmaf(q.x, g0, fmaf(q.y, g1, fmaf(q.z, g2, q.w)));
        };
        auto key64 = [&](int k, double dr, double dg, double db) {
            const double t0 = dr - cs[3 * k], t1 = dg - cs[3 * k + 1], t2 = db - cs[3 * k + 2];
            double d = 0.0;
            d = d + t0 * t0;
            d = d + t1 * t1;
            d = d + t2 * t2;
            return d;
        };
        const int c0 = min(w.code, Kp - 4);
        int at = -1;
#pragma unroll
        for (int v = 3; v >= 0; --v) at = key32(reinterpret_cast<const float4*>(rec)[c0 + v], f0, f1, f2) == w.b1 ? c0 + v : at;
        const bool mine = q0 + lane < P && (at < 0 || !(w.b2 - w.b1 > 0.25f));
        const float lim = at < 0 ? INFINITY : w.b1 + 0.25f;
        unsigned long long open = __ballot(mine);
        if (__popcll(open) * (90 + 14 * ((K + 63) / 64)) > 8 * K) {
            const double dr = (double)r, dg = (double)gr, db = (double)b;
            double bd = INFINITY;
            int bk = at;
#pragma unroll 4
            for (int k = 0; k < K; ++k) {
                if (mine && key32(reinterpret_cast<const float4*>(rec)[k], f0, f1, f2) <= lim) {
                    const double d = key64(k, dr, dg, db);
                    if (d < bd) {
                        bd = d;
                        bk = k;
                    }
                }
            }
            at = bk;
            open = 0ull;
        }
        while (open != 0ull) {  // wavefront-uniform: one pixel at a time, 64 centroids a step
            const int who = __ffsll(open) - 1;
            open &= open - 1;
            const int ro = __builtin_amdgcn_readlane(r, who), go = __builtin_amdgcn_readlane(gr, who),
                      bo = __builtin_amdgcn_readlane(b, who);
            const float lo = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lim), who));
            const float o0 = -2.f * (float)(ro - 128), o1 = -2.f * (float)(go - 128), o2 = -2.f * (float)(bo - 128);
            double bd = INFINITY;
            int bk = 0x7fffffff;
            for (int k = lane; k < K; k += 64) {
                if (key32(reinterpret_cast<const float4*>(rec)[k], o0, o1, o2) <= lo) {
                    const double d = key64(k, (double)ro, (double)go, (double)bo);
                    if (d < bd) {
                        bd = d;
                        bk = k;
                    }
                }
            }
            // the few lanes that compared any: the smallest, ties to the smallest index
            unsigned long long has = __ballot(bk != 0x7fffffff);
            double sd = INFINITY;
            int sk = 0x7fffffff;
            while (has != 0ull) {
                const int l = __ffsll(has) - 1;
                has &= has - 1;
                const double cd = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(bd), l),
                                                   __builtin_amdgcn_readlane(__double2loint(bd), l));
                const int ck = __builtin_amdgcn_readlane(bk, l);
                if (cd < sd || (cd == sd && ck < sk)) {
                    sd = cd;
                    sk = ck;
                }
            }
            at = lane == who ? sk : at;
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

// The same step for small images with small palettes: one pixel per thread,
// every centroid in FP64.  A pass there is a chain of latencies (stage, compare,
// add), which is shorter without the scan, the merge and the settling.  The line
// (K <= 64, fewer than 512 workgroups): whole call, 10 update steps, direct
// against scan: 64 x 64 pixels, K = 16 176 and 210 us; 300 x 300, K = 32 263 and
// 279, K = 64 303 and 293; 200 x 200 half white, K = 64 257 and 275;
// 512 x 512, K = 16 512 and 407.
constexpr int kKmDirectMax = 64;
__global__ __launch_bounds__(kKmThreads) void km_assign_direct(const uint8_t* __restrict__ px, int64_t P, int K,
                                                               const double* __restrict__ C,
                                                               unsigned long long* __restrict__ S,
                                                               int32_t* __restrict__ assign) {
#pragma clang fp contract(off)
    __shared__ double cs[3 * kKmDirectMax];
    __shared__ unsigned acc[4 * kKmDirectMax];
    const int tid = threadIdx.x;
    for (int e = tid; e < 3 * K; e += kKmThreads) cs[e] = C[e];
    for (int e = tid; e < 4 * K; e += kKmThreads) acc[e] = 0u;
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * kKmThreads + tid;
    if (p < P) {
        const int pr = px[p * 3], pg = px[p * 3 + 1], pb = px[p * 3 + 2];
        const double r = (double)pr, g = (double)pg, b = (double)pb;
        int best = 0;
        double bd = INFINITY;
        for (int k = 0; k < K; ++k) {
            const double t0 = r - cs[3 * k], t1 = g - cs[3 * k + 1], t2 = b - cs[3 * k + 2];
            double d = 0.0;
            d = d + t0 * t0;
            d = d + t1 * t1;
            d = d + t2 * t2;
            if (d < bd) {
                bd = d;
                best = k;
            }
        }
        assign[p] = best;
        atomicAdd(&acc[4 * best], (unsigned)pr);
        atomicAdd(&acc[4 * best + 1], (unsigned)pg);
        atomicAdd(&acc[4 * best + 2], (unsigned)pb);
        atomicAdd(&acc[4 * best + 3], 1u);
    }
    __syncthreads();
    for (int e = tid; e < 4 * K; e += kKmThreads)
        if (acc[e] != 0u) atomicAdd(&S[e], (unsigned long long)acc[e]);
}

// Update from the sums of the last assignment, then clear them for the next.
template <bool RECORDS>
__global__ __launch_bounds__(kKmMax) void km_update(int K, double* __restrict__ C,
                                                    unsigned long long* __restrict__ S, float4* __restrict__ rec) {
    const int k = threadIdx.x;
    double c[3] = {0.0, 0.0, 0.0};
    bool empty = false;
    if (k < K) {
        const unsigned long long n = S[k * 4 + 3];
        empty = n == 0ull;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            c[t] = n > 0ull ? (double)S[k * 4 + t] / (double)n : C[k * 3 + t];
            C[k * 3 + t] = c[t];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) S[k * 4 + t] = 0ull;
    }
    // the later of two equal centroids is empty (two clusters whose means have
    // just become equal are found one pass later)
    if constexpr (RECORDS) km_records(K, __syncthreads_or(empty) != 0, c[0], c[1], c[2], rec);
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

size_t kmeans_record_bytes(int K) { return 16 * (size_t)km_pad(K); }

int launch_kmeans(const uint8_t* px, int64_t P, int K, int iters, double* C, unsigned long long* S, float* records,
                  int32_t* assign, float* pts, float* mass, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (K < 1 || K > kKmMax) return (int)hipErrorInvalidValue;
    const unsigned kb = (unsigned)((K + kKmThreads - 1) / kKmThreads);
    const unsigned kt = (unsigned)((K + 63) & ~63);
    // a workgroup takes up to kKmGroups x 256 pixels, which spreads its staging
    // of the centroids over more of them; fewer while that leaves compute units
    // idle (smooth images, K = 256, always four against this rule: 360 x 360 572
    // and 390 us, 512 x 512 604 and 548, 720 x 720 the same)
    const int64_t pieces = (P + kKmThreads - 1) / kKmThreads;
    const bool direct = K <= kKmDirectMax && pieces < 512;
    float4* rec = reinterpret_cast<float4*>(records);
    const int groups = (int)std::max<int64_t>(1, std::min<int64_t>(kKmGroups, pieces / 512));
    const unsigned pb = (unsigned)((pieces + groups - 1) / groups);
    const size_t lds = kmeans_lds_bytes(K);
    if (lds > 48 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)km_assign, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    if (direct) {
        hipLaunchKernelGGL(km_init<false>, dim3(1), dim3(kt), 0, st, px, P, K, C, S, rec);
        for (int it = 0; it <= iters; ++it) {
            hipLaunchKernelGGL(km_assign_direct, dim3((unsigned)pieces), dim3(kKmThreads), 0, st, px, P, K, C, S, assign);
            if (it < iters) hipLaunchKernelGGL(km_update<false>, dim3(1), dim3(kt), 0, st, K, C, S, rec);
        }
    } else {
        hipLaunchKernelGGL(km_init<true>, dim3(1), dim3(kt), 0, st, px, P, K, C, S, rec);
        for (int it = 0; it <= iters; ++it) {
            hipLaunchKernelGGL(km_assign, dim3(pb), dim3(kKmThreads), lds, st, px, P, K, groups, C, rec, S, assign);
            if (it < iters) hipLaunchKernelGGL(km_update<true>, dim3(1), dim3(kt), 0, st, K, C, S, rec);
        }
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
