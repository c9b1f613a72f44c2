// FP32 nearest-supplier search of one round (the NNS step of Algorithm 1,
// Sec. III-A) for a pair whose active suppliers sit in LDS as search
// records, shared by the one-workgroup pair solver and the single-workgroup
// finish of the multi-workgroup path.  Every pick is the FP64 argmin (ties
// to the smallest slot, and slots are in ascending supplier order); the
// consumers whose two nearest FP32 keys are closer than the rounding bound
// plus the near-tie window are re-scored in FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "internal.hpp"
#include "round_common.hpp"

namespace nnsemd {
namespace ps {

using namespace rc;

// Supplier records in flight per step of the vector search (L1, and fewer than
// kTileConsumers consumers): 8, or 4 in the kernels with one or two points per
// thread, whose lower register use keeps more wavefronts resident (8 there:
// 2048 L1 pairs of 32..256 points 217 -> 226 us, 4096 of 8..64 193 -> 203 us;
// 1024 pairs of 128..1024 points, d = 5, 512 threads 464 -> 615 us).
template <int CSMAX>
constexpr int search_unroll() { return CSMAX <= 2 ? 4 : 8; }

// Exact FP64 key in the definition's operation order (dimension order, no
// fused multiply-add): squared Euclidean, or L1.
template <int D, bool L1>
__device__ inline double key64(const float* __restrict__ x, const float* __restrict__ y) {
#pragma clang fp contract(off)
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        double diff = (double)x[t] - (double)y[t];
        if (L1)
            acc = acc + fabs(diff);
        else
            acc = acc + diff * diff;
    }
    return acc;
}

// Search gap bound (Euclidean metrics).  With x^ = fl(x - c), y^ = fl(y - c)
// (c the FP32 centre of the supplier box), the record (-2 x^, fl(||x^||^2))
// and the FMA chain key = ||x^||^2 + sum_t (-2 x^_t) y^_t, one key differs
// from ||x - y||^2 - ||y^||^2 by at most B = (2D + 2) u e^2 to first order,
// e = ||x^|| + ||y^|| <= rhat + ||y^|| (u = 2^-24): D roundings in the norm
// (<= D u ||x^||^2), D in the chain (<= D u (||x^||^2 + 2 ||x^|| ||y^||)) and
// 2u e^2 from the two centring subtractions.  If the FP32 argmin were not
// the FP64 one, some other key would lie within 2B of the best, so the
// threshold 2 x 2B = 8 (D + 1) u e^2 leaves a factor 2 for second-order
// terms, the FP64 reference's own rounding and the rounding of e.
template <int D>
__device__ inline float search_gap_bound(float rhat, float yn2) {
    const float e = rhat + sqrtf(yn2);
    return 8.f * (float)(D + 1) * kU32 * e * e + 1e-30f;
}

// L1 keys sum D rounded |x_t - y_t| terms (no centring): relative error at
// most D u of the key, so two keys of one consumer can disagree with their
// FP64 order only within 2 D u b1; 4 (D + 1) u b1 leaves a factor 2.
template <int D>
__device__ inline float search_gap_bound_l1(float b1) {
    return 4.f * (float)(D + 1) * kU32 * b1 + 1e-30f;
}

// Fractional bits of a finite FP32 value: the smallest q >= 0 with v a
// multiple of 2^-q (0 for 0; a large value for subnormals, which never
// qualify for the exact-key test below).
__device__ inline int frac_bits(float v) {
    const uint32_t u = __float_as_uint(v) & 0x7fffffffu;
    if (u == 0u) return 0;
    const int e = (int)(u >> 23);
    if (e == 0) return 200;
    const int tz = __builtin_ctz((u & 0x7fffffu) | 0x800000u);
    const int q = 23 - tz - (e - 127);
    return q > 0 ? q : 0;
}

// The same of a centred coordinate xc = fl(x - c), which only counts when the
// subtraction did not round (a point near zero can lose its low bits to a
// larger centre and then look like a lattice point).  x - c can need more bits
// than FP64 has, too (x = 1, c = 2^-53), so the FP64 difference is taken with
// its rounding error (Knuth's two-sum) and has to be free of one.
__device__ inline int centred_bits(float x, float c, float xc) {
    const double xd = (double)x, cd = (double)c;
    const double s = xd - cd, t = s - xd;
    const double err = (xd - (s - t)) - (cd + t);
    return s == (double)xc && err == 0.0 ? frac_bits(xc) : 200;
}

// Exact-key test.  If every centred coordinate is a multiple of 2^-q with
// magnitude <= R, every term of a Euclidean key (x^_t^2, 2 x^_t y^_t) is a
// multiple of 2^-2q and every partial sum is at most 3 D R^2 in magnitude, so
// all of them are FP32 numbers when 3 D R^2 4^q < 2^24: each FMA of the key
// chain is then exact, the FP32 keys equal the exact ones (shifted by the
// exact ||y^||^2), and the FP32 argmin with its smallest-slot tie rule is the
// FP64 definition's.  L1 (uncentred): terms |x_t - y_t| <= 2R, sums <= 2DR,
// exact when 2 D R 2^q < 2^24.  Integer-lattice inputs (pixel grids) pass.
template <int D, bool L1>
__device__ inline bool keys_exact(double q, double R) {
    if (q > 40.0) return false;
    const double s = exp2(q);
    return L1 ? 2.0 * D * R * s < 16777216.0 : 3.0 * D * R * R * s * s < 16777216.0;
}

// Search record of a supplier: its coordinates as given and, for the
// Euclidean metrics, ||x^||^2 in component D (zeros after it).  The centring
// x^ = fl(x - c) is repeated where a key is formed (one subtraction, the same
// value every time), so the record also serves the exact FP64 keys and no
// supplier row is read from memory inside the rounds.
// FP32 key of record `rec`: y holds -2 y^ (Euclidean; scaling by -2 is exact,
// so fma(x^, -2 y^, k) is fma(-2 x^, y^, k)) or y as given (L1).
template <int D, int RS, bool L1>
__device__ inline float key32(const float* __restrict__ rec, const float (&y)[D], const float (&centre)[D]) {
    if (L1) {
        float k = 0.f;
#pragma unroll
        for (int t = 0; t < D; ++t) k += fabsf(rec[t] - y[t]);
        return k;
    } else {
        float k = rec[D];
#pragma unroll
        for (int t = D - 1; t >= 0; --t) k = fmaf(rec[t] - centre[t], y[t], k);
        return k;
    }
}

// Whether a consumer's best two FP32 keys leave its pick open (it is then
// re-scored in FP64).  Exact keys never do: the pick stands, and the two
// nearest distances are b + ||y||^2 exactly (FP64 holds the sum exactly), so
// the near tie is counted here (several: a consumer with two suppliers).
template <int D, bool L1>
__device__ inline bool settle(SharedCore& sh, float b1, float b2, float yn2, float rhat, bool several, bool exact,
                              int metric) {
    if (exact) {
        if (several) {
            const double k1 = L1 ? (double)b1 : (double)b1 + (double)yn2;
            const double k2 = L1 ? (double)b2 : (double)b2 + (double)yn2;
            if (keys_near(k1, k2, metric)) atomicAdd(&sh.tie_nn, 1ull);
        }
        return false;
    }
    // win: the proven search bound (see search_gap_bound) plus the window
    // in which the two nearest suppliers may still be a near tie.
    float win;
    if (L1) {
        const float thr = search_gap_bound_l1<D>(b1);
        win = thr + near_window(b1, true);
    } else {
        const float thr = search_gap_bound<D>(rhat, yn2);
        win = thr + near_window(b1 + yn2 + thr, false);
    }
    return !(b2 - b1 > win);
}

// Queue consumer j for the re-score, or store its pick, the pick's exact FP64
// key (x: the picked record, y: the consumer, both as given) and its claim.
template <int D, bool L1, typename LT>
__device__ inline void store_pick(const LT& L, SharedCore& sh, const float* __restrict__ x,
                                  const float* __restrict__ y, int j, bool flag, int pick) {
    if (flag) {
        const int f = atomicAdd(&sh.nflag, 1);
        L.list[f] = j;
    } else {
        L.cnn[j] = pick;
        L.ckey[j] = key64<D, L1>(x, y);
        cnt_add(L.scnt, pick);
    }
}

// One pass of the search for the consumers q = qa + k*G (k < KC) of this
// lane; S lanes share each consumer and scan every S-th active supplier.
// Per consumer: FP32 best and second-best keys; if they are closer than the
// rounding bound the consumer is queued for the FP64 re-score, otherwise its
// pick and the exact FP64 key of the pick are stored.
template <int D, int RS, bool L1, int KC, int UN, typename LT>
__device__ inline void nns_pass(const LT& L, SharedCore& sh, const float* __restrict__ Y, const float (&centre)[D], float rhat,
                                int mact, int nact, int S, int qa, int G, int r, bool exact, int metric) {
    int jj[KC];
    bool valid[KC];
    float yr[KC][D];  // the consumer as given
    float y[KC][D];   // as key32 takes it
    float yn2[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int q = qa + k * G;
        valid[k] = q < nact;
        jj[k] = L.cact[valid[k] ? q : 0];
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        yn2[k] = 0.f;
#pragma unroll
        for (int t = 0; t < D; ++t) {
            yr[k][t] = Y[(size_t)jj[k] * D + t];
            const float yv = L1 ? yr[k][t] : yr[k][t] - centre[t];
            y[k][t] = L1 ? yv : -2.f * yv;
            yn2[k] = fmaf(yv, yv, yn2[k]);
        }
    }
    float b1[KC], b2[KC];
    int bs[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        b1[k] = INFINITY;
        b2[k] = INFINITY;
        bs[k] = 0x7fffffff;
    }
    // Full blocks of UN records.  Two keys at a time update the pair
    // (b1, b2): b2 <- min(b2, med3(b1, ka, kb)) and b1 <- min(b1, ka, kb)
    // give the two smallest of {b1, b2, ka, kb} (as a multiset, so equal
    // keys leave b2 = b1).  Only the block in which b1 last fell strictly
    // is remembered; its records are scanned again afterwards for the first
    // slot holding b1, which is the smallest slot with the smallest key.
    const int stride = S * UN;
    const int full = (mact / stride) * stride;
    int blk[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) blk[k] = -1;
    for (int s0 = r; s0 < full; s0 += stride) {
        float rec[UN][RS];
#pragma unroll
        for (int u = 0; u < UN; ++u) load_rec<RS>(L.srec, s0 + u * S, rec[u]);
        float b1o[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) b1o[k] = b1[k];
#pragma unroll
        for (int u = 0; u < UN; u += 2) {
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const float ka = key32<D, RS, L1>(rec[u], y[k], centre);
                const float kb = key32<D, RS, L1>(rec[u + 1], y[k], centre);
                b2[k] = fminf(b2[k], __builtin_amdgcn_fmed3f(b1[k], ka, kb));
                b1[k] = fminf(b1[k], fminf(ka, kb));
            }
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) blk[k] = b1[k] < b1o[k] ? s0 : blk[k];
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        if (blk[k] >= 0) {
            int u = UN - 1;
#pragma unroll
            for (int v = UN - 2; v >= 0; --v) {
                float rv[RS];
                load_rec<RS>(L.srec, blk[k] + v * S, rv);
                u = key32<D, RS, L1>(rv, y[k], centre) == b1[k] ? v : u;
            }
            bs[k] = blk[k] + u * S;
        }
    }
    for (int s = full + r; s < mact; s += S) {
        float rec[RS];
        load_rec<RS>(L.srec, s, rec);
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const float key = key32<D, RS, L1>(rec, y[k], centre);
            const bool lt = key < b1[k];
            bs[k] = lt ? s : bs[k];
            b2[k] = __builtin_amdgcn_fmed3f(b1[k], key, b2[k]);
            b1[k] = fminf(b1[k], key);
        }
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        for (int o = 1; o < S; o <<= 1) {
            const float c1 = __shfl_xor(b1[k], o);
            const float c2 = __shfl_xor(b2[k], o);
            const int cs2 = __shfl_xor(bs[k], o);
            const float n2 = fminf(fmaxf(b1[k], c1), fminf(b2[k], c2));
            const bool take = (c1 < b1[k]) || (c1 == b1[k] && cs2 < bs[k]);
            b1[k] = take ? c1 : b1[k];
            bs[k] = take ? cs2 : bs[k];
            b2[k] = n2;
        }
    }
    if (r != 0) return;
    bool flag[KC];
    int pick[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k)
        flag[k] = settle<D, L1>(sh, b1[k], b2[k], yn2[k], rhat, valid[k] && mact > 1, exact, metric);
#pragma unroll
    for (int k = 0; k < KC; ++k) pick[k] = flag[k] ? 0 : bs[k];
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if (valid[k]) {
            float rv[RS];
            load_rec<RS>(L.srec, pick[k], rv);
            store_pick<D, L1>(L, sh, rv, yr[k], jj[k], flag[k], pick[k]);
        }
}

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2;

// The best two of two lanes' or tiles' (best, second, code): equal bests go
// to the smaller code.
struct Top2 {
    float b1, b2;
    int code;
};
__device__ inline Top2 merge_top2(const Top2& x, const Top2& y) {
    Top2 o;
    o.b2 = fminf(fmaxf(x.b1, y.b1), fminf(x.b2, y.b2));
    const bool take = y.b1 < x.b1 || (y.b1 == x.b1 && y.code < x.code);
    o.b1 = take ? y.b1 : x.b1;
    o.code = take ? y.code : x.code;
    return o;
}
// Swap the upper half of x with the lower half of y (W = 32), or the odd
// 16-lane rows of x with the even rows of y (W = 16).
template <int W>
__device__ inline void lane_swap(unsigned& x, unsigned& y) {
    const u32x2 v = W == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                            : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = v[0];
    y = v[1];
}
template <int W>
__device__ inline Top2 swap_merge(Top2 x, Top2 y) {
    unsigned a, b;
    a = __float_as_uint(x.b1); b = __float_as_uint(y.b1); lane_swap<W>(a, b);
    x.b1 = __uint_as_float(a); y.b1 = __uint_as_float(b);
    a = __float_as_uint(x.b2); b = __float_as_uint(y.b2); lane_swap<W>(a, b);
    x.b2 = __uint_as_float(a); y.b2 = __uint_as_float(b);
    a = (unsigned)x.code; b = (unsigned)y.code; lane_swap<W>(a, b);
    x.code = (int)a; y.code = (int)b;
    return merge_top2(x, y);
}

// The search of up to KT * 16 consumers of one wavefront on the matrix cores
// (Euclidean metrics).  A 16 x 16 block of keys is the product of 16 supplier
// records (x^, ||x^||^2) with 16 columns (-2 y^, 1): v_mfma_f32_16x16x4_f32
// for d <= 3, two of them for d = 4..7.  The instruction adds its four
// products to the accumulator one after the other, each a fused multiply-add
// rounded to nearest (checked on gfx950 against fmaf, bit for bit, with
// subnormals), so with the record's components fed last to first the keys are
// exactly key32's: nothing downstream can tell the two searches apart.  (The
// slot of the best is found by that equality; a key that no record gives again
// would send its consumer to the FP64 re-score.)
// Lane l holds the keys of suppliers 4 (l / 16) + 0..3 of a block against
// consumer l % 16; four keys update (best, second) with two med3 and three
// min3 and the block is remembered when the best falls strictly.  At the end
// the four 16-lane rows exchange tiles (lane_swap) while merging, which leaves
// lane l with consumer l of the 64, and the four records of the winning
// (block, row) are read once more for the first slot that holds the best.
// Bound: a block takes 32 cycles of the FP32 matrix pipe (one tile, d <= 3) and
// 28 of vector issue, which overlap little, where the vector form needs 75
// (d = 3; the grid-wide search of one large pair, which issues nothing else,
// gained nothing from it and stays on the vector form); what is left of
// the search in a launch is the latency of its first and last reads.  With the
// coordinates in the records (no supplier row read from memory for the exact
// key): 4096 pairs of 128..1024 points 1159 -> 1083 us, 2048 pixel grids
// 3272 -> 2950 us, one 256 x 256 pair 52 -> 49 us (bucket-major rounds on both
// sides).
template <int D, int RS, int KT, typename LT>
__device__ inline void nns_tiles(const LT& L, SharedCore& sh, const float* __restrict__ Y, const float (&centre)[D], float rhat, int mact, int qend, int q0, bool exact,
                                 int metric) {
    const int lane = threadIdx.x & (kWave - 1);
    const int col = lane & 15, row = lane >> 4;
    constexpr int KM = RS / 4;  // matrix instructions per block
    // this lane's component of a record, RS - 1 - (4 h + row), and its centre
    // (0 for the norm and the zeros: subtracting it changes nothing)
    float cen[KM];
#pragma unroll
    for (int h = 0; h < KM; ++h) {
        cen[h] = 0.f;
#pragma unroll
        for (int k = 0; k < D; ++k) cen[h] = RS - 1 - (4 * h + row) == k ? centre[k] : cen[h];
    }
    float bv[KT][KM];
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const int q = q0 + 16 * t + col;
        const float* yp = Y + (size_t)L.cact[q < qend ? q : 0] * D;
#pragma unroll
        for (int h = 0; h < KM; ++h) {
            const int comp = RS - 1 - (4 * h + row);
            const float yv = yp[comp < D ? comp : 0];
            bv[t][h] = comp < D ? -2.f * (yv - cen[h]) : (comp == D ? 1.f : 0.f);
        }
    }
    // lane l finishes consumer q0 + l
    const int q = q0 + lane;
    const bool valid = lane < 16 * KT && q < qend;
    const int j = L.cact[valid ? q : 0];
    float yr[D];
#pragma unroll
    for (int k = 0; k < D; ++k) yr[k] = Y[(size_t)j * D + k];
    Top2 best[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        best[t].b1 = INFINITY;
        best[t].b2 = INFINITY;
        best[t].code = 0x7fffffff;
    }
    auto block = [&](const float (&av)[KM], int s0) {
        f32x4 acc[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 0; h < KM; ++h)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[h], bv[t][h], acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            const float o = best[t].b1;
            const float m = __builtin_amdgcn_fmed3f(o, acc[t][0], acc[t][1]);
            const float n = fminf(o, fminf(acc[t][0], acc[t][1]));
            const float p = __builtin_amdgcn_fmed3f(n, acc[t][2], acc[t][3]);
            best[t].b2 = fminf(best[t].b2, fminf(m, p));
            best[t].b1 = fminf(n, fminf(acc[t][2], acc[t][3]));
            best[t].code = best[t].b1 < o ? s0 : best[t].code;
        }
    };
    const float* ap = L.srec + (size_t)col * RS + (RS - 1 - row);
    constexpr int UB = 4;  // blocks whose records are in flight together
    int s0 = 0;
    for (; s0 + 16 * UB <= mact; s0 += 16 * UB) {
        float av[UB][KM];
#pragma unroll
        for (int i = 0; i < UB; ++i)
#pragma unroll
            for (int h = 0; h < KM; ++h) av[i][h] = ap[(size_t)(s0 + 16 * i) * RS - 4 * h] - cen[h];
#pragma unroll
        for (int i = 0; i < UB; ++i) block(av[i], s0 + 16 * i);
    }
    if (s0 < mact) {  // fewer than UB blocks; slots past the end give the key +inf
        float av[UB][KM];
#pragma unroll
        for (int i = 0; i < UB; ++i)
#pragma unroll
            for (int h = 0; h < KM; ++h) {
                const int s = s0 + 16 * i + col;
                const float v = L.srec[(size_t)min(s, mact - 1) * RS + RS - 1 - row - 4 * h] - cen[h];
                av[i][h] = s < mact ? v : (RS - 1 - (4 * h + row) == D ? INFINITY : 0.f);
            }
#pragma unroll
        for (int i = 0; i < UB; ++i)
            if (i == 0 || s0 + 16 * i < mact) block(av[i], s0 + 16 * i);
    }
#pragma unroll
    for (int t = 0; t < KT; ++t)
        if (best[t].code != 0x7fffffff) best[t].code += 4 * row;  // first slot of the lane's four
    const Top2 w = swap_merge<16>(swap_merge<32>(best[0], best[2]), swap_merge<32>(best[1], best[3]));
    float y[D], yn2 = 0.f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const float yc = yr[k] - centre[k];
        yn2 = fmaf(yc, yc, yn2);
        y[k] = -2.f * yc;
    }
    bool flag = settle<D, false>(sh, w.b1, w.b2, yn2, rhat, valid && mact > 1, exact, metric);
    // the first of the four slots that holds the best; should none of them give
    // the best again, the pick is not known and the consumer is flagged (exact
    // keys, whose near ties are counted by now, are the same in any form)
    const int c0 = min(w.code, mact - 1);
    int pick = -1;
    float px[D];
#pragma unroll
    for (int k = 0; k < D; ++k) px[k] = 0.f;
#pragma unroll
    for (int v = 3; v >= 0; --v) {
        float rv[RS];
        const int s = min(c0 + v, mact - 1);
        load_rec<RS>(L.srec, s, rv);
        const bool take = key32<D, RS, false>(rv, y, centre) == w.b1;
        pick = take ? s : pick;
#pragma unroll
        for (int k = 0; k < D; ++k) px[k] = take ? rv[k] : px[k];
    }
    flag |= pick < 0;
    if (valid) store_pick<D, false>(L, sh, px, yr, j, flag, pick);
}


// One round's search: every active consumer's pick (active slot in cnn[j],
// exact FP64 key in ckey[j]) counted into scnt; returns the number of
// consumers re-scored in FP64.  Ends with a workgroup barrier.
// S lanes share one consumer (each scans every S-th supplier) when there
// are too few consumers to fill the workgroup.  Otherwise the active
// consumers are cut into 64-consumer slots and the slots dealt to the
// wavefronts as evenly as possible; a wavefront with k slots scans the
// records once with k consumers per lane (one record load feeds k key
// chains), so only the last slot has idle lanes.  S is the largest power of
// two (at most 64 and at most mact) with nact * S * split <= T, so every
// active consumer gets its S lanes.
// Consumers from which the search runs on the matrix cores.  Fewer: several
// lanes of the vector form share a consumer, which fills the workgroup where
// 16-consumer tiles would leave wavefronts idle.  Two tiles on two wavefronts
// are level with the vector form at d <= 3 and ahead of it at d >= 4, whose
// centring costs d subtractions a key: 64 against 32 as the line, 64 pairs of
// 64..512 points, d = 7, 273 and 265 us, one pair of 1000 x 64 points, d = 6, 265
// and 235, 1024 pairs of 128..1024, d = 3, 525 and 521.  At 16, one tile, small
// pairs lose (200 x 30 points, d = 3, 76.7 and 78.4).
constexpr int kTileConsumers = 32;
template <int D, int T, int CSMAX, bool L1, typename LT>
__device__ inline int search_round(const LT& L, SharedCore& sh, const float* __restrict__ Y,
                                   const float (&centre)[D], float rhat, int mact, int nact, int split, bool exact, int metric) {
    constexpr int RS = record_stride(D);
    constexpr int NW = T / kWave;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    int near = 0;
    constexpr int UN = search_unroll<CSMAX>();
    // log2 of S: floor(log2(T)) - ceil(log2(nact * split)), capped by log2(64) and floor(log2(mact))
    const int lt = 31 - __builtin_clz(T), ln = nact * split > 1 ? 32 - __builtin_clz(nact * split - 1) : 0;
    const int S = 1 << max(0, min(min(6, 31 - __builtin_clz(mact)), lt - ln));
    if (!L1 && (S == 1 || nact >= kTileConsumers)) {
        const int nt = (nact + 15) / 16;
        const int lo = wave * nt / NW, hi = (wave + 1) * nt / NW;
        // most tiles of a pass: the 512-thread variants held to 80 VGPRs take two,
        // which spill 20 to 26 registers where four spill 27 to 32 (4096 pairs of
        // 128..1024 points, d = 3, 1215 -> 1160 us, of 62..500 points 801 -> 711)
        constexpr int KT = T == 512 && CSMAX == 2 && D <= 3 ? 2 : 4;
        for (int t0 = lo; t0 < hi; t0 += KT) {
            const int k = hi - t0;  // wavefront-uniform
            const int qend = min(nact, 16 * hi);  // three tiles of a pass of four run as four, the last one idle
            if (KT == 4 && k >= 3)
                nns_tiles<D, RS, KT>(L, sh, Y, centre, rhat, mact, qend, 16 * t0, exact, metric);
            else if (k >= 2)
                nns_tiles<D, RS, 2>(L, sh, Y, centre, rhat, mact, qend, 16 * t0, exact, metric);
            else
                nns_tiles<D, RS, 1>(L, sh, Y, centre, rhat, mact, qend, 16 * t0, exact, metric);
        }
    } else if (S > 1) {
        nns_pass<D, RS, L1, 1, UN>(L, sh, Y, centre, rhat, mact, nact, S, tid / S, T / S, tid & (S - 1), exact, metric);
    } else if constexpr (L1) {
        const int nslots = (nact + kWave - 1) / kWave;
        const int lo = wave * nslots / NW, hi = (wave + 1) * nslots / NW;
        // a wavefront holds at most CSMAX slots (nact <= CSMAX * T)
        constexpr int KMAX = CSMAX < 4 ? CSMAX : 4;
        for (int u0 = lo; u0 < hi; u0 += KMAX) {
            const int k = min(KMAX, hi - u0);  // wavefront-uniform
            const int qa = u0 * kWave + lane;
            if (KMAX >= 4 && k == 4)
                nns_pass<D, RS, L1, KMAX, UN>(L, sh, Y, centre, rhat, mact, nact, 1, qa, kWave, 0, exact, metric);
            else if (KMAX >= 3 && k == 3)
                nns_pass<D, RS, L1, KMAX >= 3 ? 3 : 1, UN>(L, sh, Y, centre, rhat, mact, nact, 1, qa, kWave, 0, exact, metric);
            else if (KMAX >= 2 && k == 2)
                nns_pass<D, RS, L1, KMAX >= 2 ? 2 : 1, UN>(L, sh, Y, centre, rhat, mact, nact, 1, qa, kWave, 0, exact, metric);
            else
                nns_pass<D, RS, L1, 1, UN>(L, sh, Y, centre, rhat, mact, nact, 1, qa, kWave, 0, exact, metric);
        }
    }
    __syncthreads();
    const int nf = sh.nflag;
    if (nf > 0) {
        // FP64 re-score of the flagged consumers, one wavefront per
        // consumer: the argmin (ties to the smallest slot) and the
        // second-smallest key decide the pick and the near-tie count.
        for (int f = wave; f < nf; f += NW) {
            const int j = L.list[f];
            const float* yp = Y + (size_t)j * D;
            double best = INFINITY, sec = INFINITY;
            int bsl = 0x7fffffff;
            for (int s = lane; s < mact; s += kWave) {
                float rv[RS];
                load_rec<RS>(L.srec, s, rv);
                const double k = key64<D, L1>(rv, yp);
                if (k < best) {
                    sec = best;
                    best = k;
                    bsl = s;
                } else if (k < sec) {
                    sec = k;
                }
            }
#pragma unroll
            for (int o = kWave / 2; o > 0; o >>= 1) {
                const double cb = __shfl_xor(best, o);
                const double c2 = __shfl_xor(sec, o);
                const int cs2 = __shfl_xor(bsl, o);
                sec = fmin(fmax(best, cb), fmin(sec, c2));
                if (cb < best || (cb == best && cs2 < bsl)) {
                    best = cb;
                    bsl = cs2;
                }
            }
            if (lane == 0) {
                L.cnn[j] = bsl;
                L.ckey[j] = best;
                cnt_add(L.scnt, bsl);
                if (mact > 1 && near_tie_dist(dist_of_key(best, metric), dist_of_key(sec, metric)))
                    atomicAdd(&sh.tie_nn, 1ull);
            }
        }
        near += nf;
        __syncthreads();
    }
    return near;
}

}  // namespace ps
}  // namespace nnsemd
