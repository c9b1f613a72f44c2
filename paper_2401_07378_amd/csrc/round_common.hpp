// Pieces shared by the one-workgroup-per-pair solvers (point path and the
// BF16 document path): LDS layout of a pair, workgroup scans and reductions,
// and the generic phases of one round of Algorithm 1 (Sec. III-A) that run
// after the search has stored every active consumer's pick (active supplier
// slot in cnn[j], exact FP64 key in ckey[j]) and counted it into scnt[slot]:
//   round_buckets  claimant sets a_i: scan of the counts, scatter
//   round_rank     each claimant's place in its bucket
//   round_walk     one lane per claimed supplier serves in that order (FP64)
//   round_compact  plan append + surviving suppliers / consumers
// in two forms: consumer-major (document path, whose greedy order works on
// FP32 keys with exact ones filled in where needed) and bucket-major (*_pos:
// point path, given-D path, single-workgroup finish).
// Every function ends with a workgroup barrier; all of them must be called
// by every thread of the workgroup with block-uniform arguments.
#pragma once

#include <stdint.h>

#include "internal.hpp"

// Optional per-phase cycle accounting for profiling builds only
// (-DNNSEMD_PHASE_TIMING).  Every thread reads the clock (no divergent code);
// thread 0 adds its totals to the phase buffer once, at the end of the pair.
#ifdef NNSEMD_PHASE_TIMING
#define NNSEMD_PH_DECL uint64_t ph[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}; uint64_t ph_t = clock64();
#define NNSEMD_PH(k) { const uint64_t ph_n = clock64(); ph[k] += ph_n - ph_t; ph_t = ph_n; }
#define NNSEMD_PH_FLUSH(buf)                                                              \
    if (threadIdx.x == 0 && (buf) != nullptr)                                             \
        for (int k = 0; k < 9; ++k) atomicAdd(&(buf)[k], (unsigned long long)ph[k]);
#else
#define NNSEMD_PH_DECL
#define NNSEMD_PH(k)
#define NNSEMD_PH_FLUSH(buf)
#endif

namespace nnsemd {
namespace rc {

constexpr int kWave = 64;

// LDS arrays of one pair; I is the index type (int32_t, or uint16_t in the
// compact layout).  In the bucket-major phases ckey, cnn and list go by bucket
// position once the buckets are formed.
template <typename I>
struct LdsT {
    double* smass;  // [M] supplier mass (by local index while loading, then by active slot)
    double* cmass;  // [N] consumer mass by local index
    double* ckey;   // [N] FP64 key of (pick, j); consumer-major after the serve: flow (0 = unserved)
    float* srec;    // [M * RS] active supplier records, compacted
    I* sidx;        // [M] local index of active supplier slot
    I* scnt;        // [M] claimant count by active slot
    I* soff;        // [M] bucket start, then bucket end, by active slot
    I* cact;        // [N] active consumers, compacted, ascending
    I* cnn;         // [N] pick (active slot) by consumer; consumer-major after the serve: supplier local index
    I* list;        // [N] near-tie consumers during the search; claimant buckets after
    I* sorted;      // [N] claimant buckets in serve order (the list's storage when shared)
    float* yl;      // [N * cd] consumer coordinates by local index (coordinate variant only)
    const int32_t* jmap;  // [N] caller's consumer index of each local one (null: the same)
};
using Lds = LdsT<int32_t>;
using Lds16 = LdsT<uint16_t>;

constexpr int kMaxWaves = 8;    // workgroups of up to 512 threads
constexpr int kMaxReduce = 17;  // values per block reduction (3 + 2d, d <= 7)
static_assert(sizeof(double) * kMaxWaves * kMaxReduce == kPairRedBytes, "reduction scratch size");

// Static LDS of a workgroup: scan scratch and counters.  The block
// reductions' scratch (kMaxWaves x kMaxReduce doubles) is passed separately:
// Shared carries one, the compact point path lends its FP64 key array.
struct SharedCore {
    unsigned long long scan[kMaxWaves];
    unsigned btot[kWave];  // per (chunk, wavefront) totals: claimants (round_buckets_pos), later in the
                           // round the three streams of round_compact_pos, 8 bits each
    unsigned long long tie_nn;     // near-tie counters of the pair (LDS atomics: hits are rare,
    unsigned long long tie_order;  // and no register is held across the rounds for them)
    int32_t nflag;  // near-tie consumers of the search
    int32_t namb;   // claimants whose serve order needs exact keys (high-dimensional path)
};
struct Shared : SharedCore {
    double red[kMaxWaves][kMaxReduce];
};

template <typename I>
__device__ inline LdsT<I> carve_t(char* base, const PairLdsLayout& L) {
    LdsT<I> s;
    s.smass = reinterpret_cast<double*>(base + L.smass);
    s.cmass = reinterpret_cast<double*>(base + L.cmass);
    s.ckey = reinterpret_cast<double*>(base + L.ckey);
    s.srec = reinterpret_cast<float*>(base + L.srec);
    s.sidx = reinterpret_cast<I*>(base + L.sidx);
    s.scnt = reinterpret_cast<I*>(base + L.scnt);
    s.soff = reinterpret_cast<I*>(base + L.soff);
    s.cact = reinterpret_cast<I*>(base + L.cact);
    s.cnn = reinterpret_cast<I*>(base + L.cnn);
    s.list = reinterpret_cast<I*>(base + L.list);
    s.sorted = reinterpret_cast<I*>(base + L.sorted);
    s.yl = reinterpret_cast<float*>(base + L.yl);
    s.jmap = nullptr;
    return s;
}

__device__ inline Lds carve(char* base, int M, int N, int rs, int cd = 0) {
    return carve_t<int32_t>(base, pair_lds_layout(M, N, rs, cd));
}

__device__ inline Lds16 carve16(char* base, int M, int N, int rs, int cd, bool share) {
    return carve_t<uint16_t>(base, pair_lds_layout(M, N, rs, cd, true, share));
}

// Claimant counter increment; returns the count before it.  16-bit counters
// take a 32-bit atomic on their word (counts stay below 2^16, so nothing
// carries into the neighbouring counter).
__device__ inline int cnt_add(int32_t* a, int s) { return atomicAdd(&a[s], 1); }
__device__ inline int cnt_add(uint16_t* a, int s) {
    unsigned* w = reinterpret_cast<unsigned*>(a) + (s >> 1);
    const int sh = (s & 1) * 16;
    return (int)((atomicAdd(w, 1u << sh) >> sh) & 0xffffu);
}

__device__ inline double dist_of_key(double key, int metric) {
    return metric == NNSEMD_L2 ? sqrt(key) : key;
}

// Near tie of two distances d1 <= d2 (FP64): a gap of at most 1e-6 relative,
// or at most 1e-12 when d1 is 0.
__device__ inline bool near_tie_dist(double d1, double d2) {
    const double gap = d2 - d1;
    return d1 == 0.0 ? gap <= 1e-12 : gap <= 1e-6 * d1;
}

// Near tie of two keys k1 <= k2 (L2: of their square roots).  For L2 the
// key-space test first rejects every pair whose distances are more than
// (2e-6 + 1e-12) apart relative, so square roots are taken only for the few
// candidates; the decision itself is always the one on distances.
__device__ inline bool keys_near(double k1, double k2, int metric) {
    if (metric == NNSEMD_L2 && k2 - k1 > 2.1e-6 * k1 + 1e-24) return false;
    if (k1 == k2) return true;  // equal keys (exact ties are common on lattices): no square roots
    return near_tie_dist(dist_of_key(k1, metric), dist_of_key(k2, metric));
}

// Width, in FP32 key units, of the window past the proven search bound in
// which two keys may still be a near tie.  Squared keys: the distances'
// relative gap 1e-6 is a key gap of at most (2e-6 + 1e-12) of the smaller
// squared distance (2.2e-6 bounds it with room for the FP32 roundings); L1
// keys are distances (1.1e-6).  kmax bounds the larger true key; the 1e-12
// covers the absolute rule at zero distance.
__device__ inline float near_window(float kmax, bool l1) {
    return (l1 ? 1.1e-6f : 2.2e-6f) * fmaxf(kmax, 0.f) + 1e-12f;
}

// SplitMix64 output function of the counter (seed, round, consumer): the
// random protocol's serve order key.
__device__ inline uint64_t rp_key(uint64_t seed, int64_t round, int32_t j) {
    uint64_t ctr = ((uint64_t)round << 32) ^ (uint64_t)(uint32_t)j;
    uint64_t z = seed + (ctr + 1u) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// One DPP move of a 64-bit value (both halves); lanes without a source, or
// in rows the row mask leaves out, read 0.
template <int CTRL, int ROWS>
__device__ inline unsigned long long dpp_u64(unsigned long long x) {
    const int lo = (int)(unsigned)(x & 0xffffffffull), hi = (int)(unsigned)(x >> 32);
    const unsigned rlo = (unsigned)__builtin_amdgcn_update_dpp(0, lo, CTRL, ROWS, 0xf, false);
    const unsigned rhi = (unsigned)__builtin_amdgcn_update_dpp(0, hi, CTRL, ROWS, 0xf, false);
    return ((unsigned long long)rhi << 32) | rlo;
}

// Inclusive scan over the 64 lanes of a wavefront with DPP moves: shifts by
// 1, 2, 4, 8 within 16-lane rows, then lane 15's total added to rows 1 and
// 3 and lane 31's to rows 2 and 3.  No LDS traffic (a shuffle is an LDS
// permute).  Every lane of the wavefront must be active.
__device__ inline unsigned long long wave_incl_scan_u64(unsigned long long x) {
    x += dpp_u64<0x111, 0xf>(x);  // row_shr:1
    x += dpp_u64<0x112, 0xf>(x);  // row_shr:2
    x += dpp_u64<0x114, 0xf>(x);  // row_shr:4
    x += dpp_u64<0x118, 0xf>(x);  // row_shr:8
    x += dpp_u64<0x142, 0xa>(x);  // row_bcast:15
    x += dpp_u64<0x143, 0xc>(x);  // row_bcast:31
    return x;
}

// The same scan of 32-bit values: one DPP add per step.
__device__ inline unsigned wave_incl_scan_u32(unsigned x) {
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
    return x;
}

// Number of set bits of a wavefront mask below this lane.
__device__ inline unsigned mask_rank(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Exclusive block scan of one 64-bit value per thread; *total = block sum.
template <int T>
__device__ inline unsigned long long block_scan_u64(unsigned long long v, unsigned long long* total,
                                                    SharedCore& sh) {
    static_assert(T / kWave <= kMaxWaves, "workgroup too large for the scan scratch");
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    unsigned long long x = wave_incl_scan_u64(v);
    if (lane == kWave - 1) sh.scan[w] = x;
    __syncthreads();
    unsigned long long off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < T / kWave; ++k) {
        unsigned long long s = sh.scan[k];
        off += (k < w) ? s : 0ull;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + x - v;
}

// Block-wide reduction of K values per thread (op 0 = sum, 1 = min, 2 = max),
// deterministic (fixed butterfly + fixed wave order).  Results in out[].
template <int T, int K>
__device__ inline void block_reduce(double (&v)[K], const int (&op)[K], double* scratch) {
    double(*red)[kMaxReduce] = reinterpret_cast<double(*)[kMaxReduce]>(scratch);
    static_assert(T / kWave <= kMaxWaves && K <= kMaxReduce, "reduction scratch too small");
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            double y = __shfl_xor(v[k], o);
            v[k] = op[k] == 0 ? v[k] + y : (op[k] == 1 ? fmin(v[k], y) : fmax(v[k], y));
        }
        if (lane == 0) red[w][k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double r = red[0][k];
#pragma unroll
        for (int q = 1; q < T / kWave; ++q) {
            double y = red[q][k];
            r = op[k] == 0 ? r + y : (op[k] == 1 ? fmin(r, y) : fmax(r, y));
        }
        v[k] = r;
    }
    __syncthreads();
}

// FP32 search key of record `rec` for consumer y (see file comment).
template <int RS>
__device__ inline void load_rec(const float* __restrict__ base, int s, float (&r)[RS]) {
    const float4* p = reinterpret_cast<const float4*>(base + (size_t)s * RS);
#pragma unroll
    for (int q = 0; q < RS / 4; ++q) {
        float4 v = p[q];
        r[4 * q + 0] = v.x;
        r[4 * q + 1] = v.y;
        r[4 * q + 2] = v.z;
        r[4 * q + 3] = v.w;
    }
}

template <int RS>
__device__ inline void store_rec(float* __restrict__ base, int s, const float (&r)[RS]) {
    float4* p = reinterpret_cast<float4*>(base + (size_t)s * RS);
#pragma unroll
    for (int q = 0; q < RS / 4; ++q)
        p[q] = make_float4(r[4 * q + 0], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]);
}


// ---- claimant sets a_i: scan the counts, scatter the claimants
template <int T, typename LT>
__device__ inline void round_buckets(const LT& L, SharedCore& sh, int mact, int nact) {
    const int tid = threadIdx.x;
    {
        const int cs = (mact + T - 1) / T;
        const int lo = min(tid * cs, mact), hi = min(lo + cs, mact);
        int sum = 0;
        for (int s = lo; s < hi; ++s) sum += L.scnt[s];
        unsigned long long tot;
        int run = (int)block_scan_u64<T>((unsigned long long)sum, &tot, sh);
        for (int s = lo; s < hi; ++s) {
            L.soff[s] = run;
            run += L.scnt[s];
        }
    }
    __syncthreads();
    for (int q = tid; q < nact; q += T) {
        const int j = L.cact[q];
        const int pos = cnt_add(L.soff, L.cnn[j]);
        L.list[pos] = j;
    }
    __syncthreads();
}

// ---- claimant order of the random protocol: each claimant counts the bucket
// members with a smaller (random key, j) and writes itself to that rank in the
// separate serve-order array.
template <int T, typename LT>
__device__ inline void round_rank(const LT& L, int nact, uint64_t seed, int rounds) {
    for (int q = threadIdx.x; q < nact; q += T) {
        const int j = L.cact[q];
        const int sl = L.cnn[j];
        const int c = L.scnt[sl];
        const int end = L.soff[sl];
        int rank = 0;
        if (c > 1) {
            const uint64_t k = rp_key(seed, rounds, j);
#pragma unroll 4
            for (int e = end - c; e < end; ++e) {
                const int j2 = L.list[e];
                const uint64_t k2 = rp_key(seed, rounds, j2);
                rank += (k2 < k) || (k2 == k && j2 < j);
            }
        }
        L.sorted[end - c + rank] = j;
    }
    __syncthreads();
}

// ---- flow & cost: one lane per claimed supplier walks its ordered
// claimants while it still holds mass.  A served claimant records the local
// index of its supplier (for the plan) and its flow in place of its key; an
// unserved one gets flow 0.  With COST (the keys are the exact FP64 keys),
// `cost` accumulates this thread's part of R; without it, R is left to the
// caller.
template <int T, bool COST = true, typename LT>
__device__ inline void round_walk(const LT& L, int mact, int metric, double& cost) {
    for (int s = threadIdx.x; s < mact; s += T) {
        const int c = L.scnt[s];
        if (c == 0) continue;
        const int end = L.soff[s];
        const int start = end - c;
        const int isup = L.sidx[s];
        int pos = start;
        double sm = L.smass[s];
        while (pos < end && sm > 0.0) {
            const int j = L.sorted[pos];
            const double cm = L.cmass[j];
            const double f = sm < cm ? sm : cm;
            sm = sm - f;
            L.cmass[j] = cm - f;
            if constexpr (COST) cost = cost + f * dist_of_key(L.ckey[j], metric);
            L.ckey[j] = f;
            L.cnn[j] = isup;
            ++pos;
        }
        for (int e = pos; e < end; ++e) L.ckey[L.sorted[e]] = 0.0;
        L.smass[s] = sm;
    }
    __syncthreads();
}

// ---- weights update: plan append + compaction of the active sets (and of
// the RS-float search records when RS > 0), one scan for all three streams.
template <int T, int CSMAX, int RS, typename LT>
__device__ inline void round_compact(const LT& L, SharedCore& sh, int& mact, int& nact, int64_t& nnz,
                                     int32_t* plan_src, int32_t* plan_dst, double* plan_flow, int64_t plan_base) {
    constexpr int RSA = RS > 0 ? RS : 4;
    const int tid = threadIdx.x;
    const int pc = (nact + T - 1) / T;
    const int plo = min(tid * pc, nact), phi = min(plo + pc, nact);
    // this thread's claimants in serve order and their flows (pc <= CSMAX),
    // read once for the count and the plan append (kept in registers for up
    // to four per thread)
    constexpr int PK = CSMAX <= 4 ? CSMAX : 1;
    int pj[PK];
    double pf[PK];
    int kp = 0;
    if constexpr (CSMAX <= 4) {
#pragma unroll
        for (int u = 0; u < CSMAX; ++u) {
            const int k = plo + u;
            pj[u] = k < phi ? (int)L.sorted[k] : 0;
            pf[u] = k < phi ? L.ckey[pj[u]] : 0.0;
            kp += pf[u] > 0.0;
        }
    } else {
        for (int k = plo; k < phi; ++k) kp += L.ckey[L.sorted[k]] > 0.0;
    }
    const int cs = (mact + T - 1) / T;
    const int slo = min(tid * cs, mact);
    float rec[CSMAX][RSA];
    double smv[CSMAX];
    int sid[CSMAX], cid[CSMAX];
    int ks = 0, kc2 = 0;
#pragma unroll
    for (int u = 0; u < CSMAX; ++u) {
        const int s = slo + u;
        sid[u] = -1;
        smv[u] = 0.0;
        if (u < cs && s < mact) {
            smv[u] = L.smass[s];
            if (smv[u] > 0.0) {
                sid[u] = L.sidx[s];
                if constexpr (RS > 0) load_rec<RS>(L.srec, s, rec[u]);
                ++ks;
            }
        }
        const int q = plo + u;
        cid[u] = -1;
        if (u < pc && q < nact) {
            const int j = L.cact[q];
            if (L.cmass[j] > 0.0) {
                cid[u] = j;
                ++kc2;
            }
        }
    }
    unsigned long long tot;
    const unsigned long long pre = block_scan_u64<T>(
        (unsigned long long)kp | ((unsigned long long)ks << 21) | ((unsigned long long)kc2 << 42), &tot, sh);
    const unsigned long long mask = (1ull << 21) - 1;
    int wp = (int)(pre & mask), ws = (int)((pre >> 21) & mask), wc = (int)(pre >> 42);
    if (plan_src != nullptr) {
        if constexpr (CSMAX <= 4) {
#pragma unroll
            for (int u = 0; u < CSMAX; ++u) {
                if (pf[u] > 0.0) {
                    const int j = pj[u];
                    const int64_t e = plan_base + nnz + wp;
                    plan_src[e] = L.cnn[j];
                    plan_dst[e] = L.jmap != nullptr ? L.jmap[j] : j;
                    plan_flow[e] = pf[u];
                    ++wp;
                }
            }
        } else {
            for (int k = plo; k < phi; ++k) {
                const int j = L.sorted[k];
                const double f = L.ckey[j];
                if (f > 0.0) {
                    const int64_t e = plan_base + nnz + wp;
                    plan_src[e] = L.cnn[j];
                    plan_dst[e] = L.jmap != nullptr ? L.jmap[j] : j;
                    plan_flow[e] = f;
                    ++wp;
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < CSMAX; ++u) {
        if (sid[u] >= 0) {
            if constexpr (RS > 0) store_rec<RS>(L.srec, ws, rec[u]);
            L.sidx[ws] = sid[u];
            L.smass[ws] = smv[u];
            L.scnt[ws] = 0;
            ++ws;
        }
        if (cid[u] >= 0) L.cact[wc++] = cid[u];
    }
    nnz += (int64_t)(tot & mask);
    mact = (int)((tot >> 21) & mask);
    nact = (int)(tot >> 42);
    if (tid == 0) sh.nflag = 0;
    __syncthreads();
}

// =====================================================================
// Bucket-major form of the phases after the search (point path, given-D path
// and the single-workgroup finish).  After the search has stored each active
// consumer's pick and exact key, the claimants are moved into bucket order
// together with their keys and slots, so that the order, the walk and the
// plan append read consecutive LDS words instead of chasing consumer indices:
//   round_buckets_pos  list[p] = consumer, ckey[p] = key, cnn[p] = slot
//   round_rank_pos     the same arrays in serve order
//   round_walk_pos     flows, left in the mass arrays (see there)
//   round_compact_pos  cost, near ties, plan append, surviving sets
// Work is dealt in chunks of T consecutive slots (thread t: slots t, t + T,
// ...), so every LDS access of a wavefront is unit-stride, a wavefront skips
// the chunks past the active count, and the block prefixes are one ballot or
// one 32-bit DPP scan per chunk plus one scan over the at most 64
// (chunk, wavefront) totals that every wavefront takes from LDS by itself.
// What bounds these phases is issued instructions in batches and the
// barrier-to-barrier latency for a single pair.  Against the consumer-major
// form before it (each claimant walked its bucket through two dependent LDS
// reads per member, all chunks of the largest pair always unrolled, 64-bit
// packed scans), thousands of cycles per pair, rank phase (whole pair):
//   256-point clouds, 1000 pairs      137 (396) ->  55 (295), 0.43 -> 0.29 ms
//   128..1024-point pairs, 4096       84 (440) ->  40 (421), 1.185 -> 1.159 ms
//   32 x 32 pixel grids, 2048       1245 (2701) -> 451 (2040), 4.28 -> 3.27 ms
constexpr int kPartialServe = 0x8000;  // cnn[p] flag: served in part, its supplier is exhausted

// Order keys with the consumer index in the low bits of the mantissa: when
// every key of a launch has at least 12 trailing zero mantissa bits (FP32
// entries, exact lattice keys), (key, j) order is one FP64 comparison and no
// two keys are equal.  j < 4096.
constexpr unsigned long long kPackMask = 0xfffull;
__device__ inline double pack_key(double k, int j) {
    return __longlong_as_double(__double_as_longlong(k + 0.0) | (long long)j);  // + 0.0: no negative zero
}
__device__ inline double unpack_key(double k) {
    return __longlong_as_double(__double_as_longlong(k) & ~(long long)kPackMask);
}

// ---- claimant sets a_i in bucket order.  pack (greedy protocol): see pack_key;
// the keys of buckets with two or more members are left packed for
// round_rank_pos.
template <int T, int CS, typename LT>
__device__ inline void round_buckets_pos(const LT& L, SharedCore& sh, int mact, int nact, bool pack) {
    constexpr int NW = T / kWave;
    static_assert(CS * NW <= kWave, "one total per lane");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    unsigned cnt[CS], inc[CS];
    int jv[CS], sv[CS];
    double kv[CS];
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        const int s = u * T + tid;
        cnt[u] = 0u;
        if (u * T + wave * kWave < mact) cnt[u] = s < mact ? (unsigned)L.scnt[s] : 0u;
    }
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        const int q = u * T + tid;
        jv[u] = 0;
        sv[u] = 0;
        kv[u] = 0.0;
        if (q < nact) {
            jv[u] = L.cact[q];
            sv[u] = L.cnn[jv[u]];
            kv[u] = L.ckey[jv[u]];
        }
    }
    // two chunks per 32-bit scan: a wavefront's counts sum to at most 4096
#pragma unroll
    for (int u = 0; u < CS; u += 2) {
        const unsigned hi = u + 1 < CS ? cnt[u + 1 < CS ? u + 1 : u] : 0u;
        unsigned x = 0u;
        if (u * T + wave * kWave < mact) x = wave_incl_scan_u32(cnt[u] | (hi << 16));
        inc[u] = x & 0xffffu;
        if (u + 1 < CS) inc[u + 1 < CS ? u + 1 : u] = x >> 16;
    }
    if (lane == kWave - 1) {
#pragma unroll
        for (int u = 0; u < CS; ++u) sh.btot[u * NW + wave] = inc[u];
    }
    __syncthreads();
    {
        const unsigned v = lane < CS * NW ? sh.btot[lane] : 0u;
        const unsigned ex = wave_incl_scan_u32(v) - v;
#pragma unroll
        for (int u = 0; u < CS; ++u) {
            const int s = u * T + tid;
            const unsigned base = (unsigned)__builtin_amdgcn_readlane((int)ex, u * NW + wave);
            if (s < mact) L.soff[s] = (int)(base + inc[u] - cnt[u]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        if (u * T + tid < nact) {
            const int pos = cnt_add(L.soff, sv[u]);
            L.list[pos] = jv[u];
            L.cnn[pos] = sv[u];
            L.ckey[pos] = pack && L.scnt[sv[u]] > 1 ? pack_key(kv[u], jv[u]) : kv[u];
        }
    }
    __syncthreads();
}

// ---- serve order inside each bucket: a claimant's rank is the number of
// members below it, counted over consecutive keys that all members of the
// bucket read together.  Random protocol: each claimant's random key is drawn
// once and takes the place of its distance key (held in a register meanwhile)
// for the count, instead of being drawn again by every member of the bucket.
template <int T, int CS, typename LT>
__device__ inline void round_rank_pos(const LT& L, int nact, int protocol, uint64_t seed, int rounds, bool pack) {
    const int tid = threadIdx.x;
    int np[CS], jv[CS];
    double kv[CS];
    if (protocol != NNSEMD_GREEDY) {
#pragma unroll
        for (int u = 0; u < CS; ++u) {
            const int p = u * T + tid;
            kv[u] = 0.0;
            if (p < nact && L.scnt[L.cnn[p]] > 1) {
                const int j = L.list[p];
                kv[u] = L.ckey[p];
                // the random order is drawn for the caller's consumer indices
                L.ckey[p] = __longlong_as_double((long long)rp_key(seed, rounds, L.jmap != nullptr ? L.jmap[j] : j));
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        const int p = u * T + tid;
        np[u] = -1;
        jv[u] = 0;
        if (p >= nact) continue;
        const int sl = L.cnn[p];
        const int c = L.scnt[sl];
        if (c < 2) continue;
        const int end = L.soff[sl], start = end - c;
        const int j = L.list[p];
        const double k = L.ckey[p];
        int rank = 0, le = 0;
        if (protocol == NNSEMD_GREEDY) {
#pragma unroll 4
            for (int e = start; e < end; ++e) {
                const double k2 = L.ckey[e];
                rank += k2 < k;
                le += k2 <= k;
            }
            kv[u] = pack ? unpack_key(k) : k;
        } else {
            const uint64_t r = (uint64_t)__double_as_longlong(k);
#pragma unroll 4
            for (int e = start; e < end; ++e) {
                const uint64_t r2 = (uint64_t)__double_as_longlong(L.ckey[e]);
                rank += r2 < r;
                le += r2 <= r;
            }
        }
        if (le - rank > 1) {  // equal keys: by consumer index
            const long long kb = __double_as_longlong(k);
            for (int e = start; e < end; ++e) {
                const double k2 = L.ckey[e];
                rank += (protocol == NNSEMD_GREEDY ? k2 == k : __double_as_longlong(k2) == kb) && L.list[e] < j;
            }
        }
        np[u] = start + rank;
        jv[u] = j;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        if (np[u] >= 0) {
            L.list[np[u]] = jv[u];
            L.ckey[np[u]] = kv[u];
        }
    }
    __syncthreads();
}

// ---- flows: one lane per claimed supplier serves its claimants in order
// while it holds mass.  The chain holds only the masses; flows stay where
// the masses were: a consumer served in full keeps -f (its mass is gone), and
// the one served in part (the supplier's last) is flagged in cnn[p] with the
// supplier's slot keeping -f.  Both read as "not active any more", and the
// keys stay untouched for the near-tie count and the cost.  `serve` is
// called for every serve (position, consumer, flow) in order.
template <int T, typename LT, typename F>
__device__ inline void walk_supplier(const LT& L, int s, F&& serve) {
    const int c = L.scnt[s];
    if (c == 0) return;
    const int end = L.soff[s];
    int pos = end - c;
    double sm = L.smass[s];
    while (pos < end && sm > 0.0) {
        const int j = L.list[pos];
        const double cm = L.cmass[j];
        const double f = sm < cm ? sm : cm;
        serve(pos, j, f);
        if (sm < cm) {
            L.cmass[j] = cm - f;
            L.cnn[pos] = s | kPartialServe;
            sm = -f;
        } else {
            L.cmass[j] = -f;
            sm = sm - f;
        }
        ++pos;
    }
    L.smass[s] = sm;
}
template <int T, typename LT>
__device__ inline void round_walk_pos(const LT& L, int mact) {
    for (int s = threadIdx.x; s < mact; s += T) walk_supplier<T>(L, s, [](int, int, double) {});
    __syncthreads();
}

// ---- cost and near ties of the round, plan append, compaction of the
// active sets.  COST: this thread's part of R from the keys.
template <int T, int CS, int RS, bool COST, typename LT>
__device__ inline void round_compact_pos(const LT& L, SharedCore& sh, int& mact, int& nact, int64_t& nnz,
                                         int32_t* plan_src, int32_t* plan_dst, double* plan_flow, int64_t plan_base,
                                         int metric, bool greedy, double& cost) {
    constexpr int RSA = RS > 0 ? RS : 4;
    constexpr int NW = T / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    double pf[CS], smv[CS];
    int pj[CS], psu[CS], sid[CS], cid[CS];
    float rec[CS][RSA];
    unsigned pre[CS];
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        const int p = u * T + tid;
        unsigned tot = 0u;
        pre[u] = 0u;
        pf[u] = 0.0;
        pj[u] = psu[u] = 0;
        sid[u] = cid[u] = -1;
        smv[u] = 0.0;
        if (u * T + wave * kWave < nact) {
            // every first-level read is issued before any is used, then the
            // reads behind them: two LDS latencies per chunk, no branches
            const int pc = min(p, nact - 1);
            const int pp = max(pc - 1, 0);
            const int raw = L.cnn[pc], rawp = L.cnn[pp];
            const int j = L.list[pc], jq = L.cact[pc];
            const double k = L.ckey[pc], kp = L.ckey[pp];
            const int slot = raw & (kPartialServe - 1);
            const double cm = L.cmass[j], cq = L.cmass[jq], sm = L.smass[slot];
            psu[u] = L.sidx[slot];
            pj[u] = j;
            const bool in = p < nact;
            const double f = cm < 0.0 ? -cm : ((raw & kPartialServe) != 0 ? -sm : 0.0);
            pf[u] = in ? f : 0.0;
            const bool alive = in && cq > 0.0;
            if (alive) cid[u] = jq;
            const bool nb1 = greedy && in && p > 0 && (rawp & (kPartialServe - 1)) == slot;
            bool near = false;
            if (__ballot(nb1) != 0ull) near = nb1 && keys_near(kp, k, metric);
            const unsigned long long bp = __ballot(pf[u] > 0.0), bc = __ballot(alive), nb = __ballot(near);
            if constexpr (COST)
                if (bp != 0ull) cost = cost + pf[u] * dist_of_key(k, metric);
            if (nb != 0ull && lane == 0) atomicAdd(&sh.tie_order, (unsigned long long)__popcll(nb));
            pre[u] = mask_rank(bp) | (mask_rank(bc) << 16);
            tot = (unsigned)__popcll(bp) | ((unsigned)__popcll(bc) << 16);
        }
        if (u * T + wave * kWave < mact) {
            bool alive = false;
            if (p < mact) {
                smv[u] = L.smass[p];
                alive = smv[u] > 0.0;
                if (alive) {
                    sid[u] = L.sidx[p];
                    if constexpr (RS > 0) load_rec<RS>(L.srec, p, rec[u]);
                }
            }
            const unsigned long long bs = __ballot(alive);
            pre[u] |= mask_rank(bs) << 8;
            tot |= (unsigned)__popcll(bs) << 8;
        }
        if (lane == 0) sh.btot[u * NW + wave] = tot;
    }
    __syncthreads();
    int32_t* const psrc = plan_src != nullptr ? plan_src + plan_base + nnz : nullptr;  // uniform
    int32_t* const pdst = plan_dst + plan_base + nnz;
    double* const pflw = plan_flow + plan_base + nnz;
    const unsigned v = lane < CS * NW ? sh.btot[lane] : 0u;
    const unsigned va = (v & 0xffu) | ((v & 0xff00u) << 8), vc = v >> 16;
    const unsigned ia = wave_incl_scan_u32(va), ic = wave_incl_scan_u32(vc);
#pragma unroll
    for (int u = 0; u < CS; ++u) {
        const unsigned ba = (unsigned)__builtin_amdgcn_readlane((int)(ia - va), u * NW + wave);
        const unsigned bc = (unsigned)__builtin_amdgcn_readlane((int)(ic - vc), u * NW + wave);
        if (psrc != nullptr && pf[u] > 0.0) {
            const unsigned e = (ba & 0xffffu) + (pre[u] & 0xffu);
            psrc[e] = psu[u];
            pdst[e] = L.jmap != nullptr ? L.jmap[pj[u]] : pj[u];
            pflw[e] = pf[u];
        }
        if (sid[u] >= 0) {
            const int ws = (int)((ba >> 16) + ((pre[u] >> 8) & 0xffu));
            if constexpr (RS > 0) store_rec<RS>(L.srec, ws, rec[u]);
            L.sidx[ws] = sid[u];
            L.smass[ws] = smv[u];
            L.scnt[ws] = 0;
        }
        if (cid[u] >= 0) L.cact[bc + (pre[u] >> 16)] = cid[u];
    }
    const unsigned ta = (unsigned)__builtin_amdgcn_readlane((int)ia, kWave - 1);
    nnz += (int64_t)(ta & 0xffffu);
    mact = (int)(ta >> 16);
    nact = __builtin_amdgcn_readlane((int)ic, kWave - 1);
    if (tid == 0) sh.nflag = 0;
    __syncthreads();
}

}  // namespace rc
}  // namespace nnsemd
