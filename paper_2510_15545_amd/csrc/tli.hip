// Token-Level Intersection proposal rows (App. D Alg. 3) on gfx950.
//
// For each draft distribution q over V_d, q' over V_t is q(x) / S at y = d2t[x] for draft ids
// x in the vocabulary intersection and 0 elsewhere; S is the mass q puts on the intersection.
// Standard speculative sampling (App. D Alg. 4, tt_verify_dense) then runs with p and q'.
//
// Numerics: q is clamped to [0, 1] (NaN -> 0).  S is formed as the sampler forms its masses:
// every intersected q(x) is truncated to Q62 fixed point and the integers are summed exactly
// (128 bits per lane, so any row length and any order give the same sum), then the sum is
// rounded once to the nearest fp32 (ties to even).  q'(y) is the IEEE fp32 quotient
// q(x) / S; a row with S = 0 is written as zeros.
//
// Two kernels: tli_mass forms S (coalesced 16-byte reads of q and d2t, Q62 sums in registers, a
// wave and then a workgroup reduction of the 128-bit sums), tli_fill writes q' by slices of
// 2,048 target ids with q(x) gathered through t2d.  The gathers bound the call: each takes
// a cache line of the row for 4 bytes, so the rows being gathered from have to stay in
// the XCD's L2.  A row's slices run together on one XCD (3 to 4 rows of 512 KB in flight there);
// with one workgroup per row 32 rows (16 MB) were, and nearly every gather went to the Infinity
// Cache.  1,024 rows of 128,256 -> 151,936 ids with 60% shared: 1,215 us with one workgroup per
// row, 499 so (tli_fill about 200 G gathers/s).  Short rows keep the one kernel
// (tli_rows).  The maps are shared by every row and stay in cache.
#include "verify_core.h"

TT_STAMPS_TABLE(tli)

namespace tt {
namespace {

using vcore::clamp01;
using vcore::q62;

constexpr int kThreads = 1024;
constexpr int kWave = 64;
constexpr int kUnroll = 4;  // 16-byte loads of each array a thread keeps in flight
constexpr int kSlice = 2048;  // target ids of a workgroup of tli_fill
constexpr int kFillThreads = 256;
constexpr int kXcds = 8;
constexpr int kCus = 256;
// When the proposal rows take two kernels.  Few rows: once they are long enough to be worth spreading
// (16 rows of 78,456 -> 14,532 ids 9.9 us against 15.7 in one kernel, of 128,256 -> 151,936 17.4
// against 87; of 30,000 -> 4,000 10.6 against 7.9).  Many rows: when the draft rows in flight in one
// kernel (one per CU, 32 per XCD) overflow the XCD's 4 MB L2 and there are target ids enough to
// gather for (300 rows of 32,000 -> 50,257: 34.5 us against 36.3 with few shared
// tokens, 49.6 against 65.8 with 70%; 256 rows of 40,000 -> 22,000: 23.7 against 17.2, 32.8 against
// 35.3; 256 of 12,000 -> 50,000: 18.8 against 16.0, 23.0 against 20.7).  The share is not known here: with 5% of
// the tokens shared and v_t about v_d or less two kernels take up to 1.15 times as long (600 rows of 60,000 -> 40,000 85 us
// against 80), with 60% 0.7 of the time (120 against 180).
constexpr int kFewRows = 64, kFewRowsVocab = 65536;
constexpr int kManyRowsDraft = 16384, kManyRowsTarget = 32768;
// Rows that take between half and all of the compute units are in flight all at once, one on each, so one kernel has no
// last wave of rows to wait for: there two kernels only from longer draft rows on, or with target rows long enough that
// the spread writes pay.  Three sets of buffers in turn, two kernels against one, few shared tokens and most: 256 rows of
// 17,000 -> 33,000 ids 16.4 us against 13.8 and 22.5 against 21.9, of 28,000 -> 33,000 18.7 against 16.3 and 31.3 against
// 34.3, of 17,000 -> 75,296 24.5 against 20.9 and 30.4 against 29.8, of 24,000 -> 88,001 30.0 against 27.4 and 37.2
// against 47.3; but 130 of 17,000 -> 60,000 15.3 against 16.0 and 18.4 against 22.4, 257 of 17,000 -> 33,000 20.2 against
// 21.0 and 25.8 against 31.0, 1,024 52.2 against 56.0 and 73.0 against 80.4 (475, the worst seen, 26.8 against 25.2 and
// 37.2 against 37.1).
constexpr int kHalfFull = 128, kFullDraft = 28672, kFullTarget = 81920;
// Draft bytes, and draft and target bytes, of a part of the rows.  tli_fill gathers from the draft rows that tli_mass has
// read: they stay in the 256 MB Infinity Cache only if the part's own writes, which go through it as well, leave room;
// up to kPartSmall of draft bytes a part is not worth dividing.  Three sets of buffers in turn, against parts of 256 MB of
// draft bytes alone, 5% of the tokens shared and 60%: 1,024 rows of 40,000 -> 50,257 ids 113 us against 134 and 163 against
// 186 (one kernel 106 and 210), of 40,000 -> 151,936 180 against 243 and 267 against 302 (180 and 326), of 128,256 ->
// 151,936 330 against 350 and 492 against 507 (370 and 1,180); 2,048 of 24,000 -> 75,296 206 against 273 (197).  By all
// bytes alone 768 rows of 17,000 -> 151,936 took 98 us, 89 so; with 112 MB of draft bytes 400 rows of 60,000 -> 40,000 went in two parts, 55, 48 so.
constexpr int64_t kPartDraft = int64_t(128) << 20, kPartBytes = int64_t(340) << 20, kPartSmall = int64_t(80) << 20;
constexpr int64_t kMaxItems = int64_t(1) << 21;      // workgroups of one grid
// Verification with the proposal formed on the fly: a row is spread over workgroups from this many
// chunks on and up to this many streams, more for long rows.  128,256 -> 151,936 ids with the
// drafter's masses: one stream 11.8 us against 35 to 66 on one compute unit (few to many shared
// tokens), 32 streams 24-32 against 46-105, 128 streams 44-80 against 50-157, but 256 streams
// 69 against 64 with few; 32 streams of 50,257 14.4-15.9 against 21.9-31.0, 128 24.6-33.1 against
// 25.2-36.2 (without masses 37.5 against 35.7); 32 of 12,000 14.1 against 11.1.
constexpr int kTliSplitChunks = 32, kTliLongChunks = 128;
constexpr int kTliSplitStreams = 64, kTliLongStreams = 128;
constexpr int kMaxSplits = 16;  // workgroups a row's mass is split over at most

struct U128 {
    uint64_t lo, hi;
};

__device__ __forceinline__ U128 add128(U128 a, U128 b) {
    U128 r;
    r.lo = a.lo + b.lo;
    r.hi = a.hi + b.hi + (r.lo < a.lo ? 1u : 0u);
    return r;
}

__device__ __forceinline__ U128 shfl_xor128(U128 v, int m) {
    U128 r;
    r.lo = __shfl_xor(v.lo, m);
    r.hi = __shfl_xor(v.hi, m);
    return r;
}

// N * 2^-62 rounded to the nearest fp32, ties to even (N < 2^128).
__device__ inline float q62_to_f32(U128 n) {
    if (n.hi == 0 && n.lo == 0) return 0.0f;
    const int bl = n.hi ? 128 - __clzll(n.hi) : 64 - __clzll(n.lo);  // bit length
    if (bl <= 24) return ldexpf((float)n.lo, -62);                   // exact
    const int sh = bl - 24;                                           // bits dropped, >= 1
    const uint64_t mant = sh >= 64 ? (n.hi >> (sh - 64)) : ((n.lo >> sh) | (n.hi << (64 - sh)));
    const int rb = sh - 1;  // the highest dropped bit
    const uint32_t round = (uint32_t)((rb >= 64 ? (n.hi >> (rb - 64)) : (n.lo >> rb)) & 1u);
    bool sticky;  // any dropped bit below the round bit
    if (rb == 0) sticky = false;
    else if (rb <= 64) sticky = (rb == 64 ? n.lo : (n.lo & ((1ull << rb) - 1))) != 0;
    else sticky = n.lo != 0 || (n.hi & ((1ull << (rb - 64)) - 1)) != 0;
    const uint64_t m = mant + ((round && (sticky || (mant & 1u))) ? 1u : 0u);  // may reach 2^24: still exact
    return ldexpf((float)m, sh - 62);
}

// The Q62 sum of the intersected q(x) (clamped to [0, 1], truncated) over x0 <= x < x1, exact, by the
// whole workgroup (barriers inside; sh_part holds a partial sum per wave); the total is valid in
// thread 0.
__device__ U128 mass_sum(const float *q, const int32_t *d2t, int x0, int x1, U128 *sh_part) {
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    U128 acc{0, 0};
    auto add = [&](float x, int32_t m) {  // branch-free: the loads stay batched
        const uint64_t keep = 0ull - (uint64_t)(m >= 0);
        acc = add128(acc, U128{q62(clamp01(x)) & keep, 0});
    };
    const int n4 = (x1 - x0) / 4;
    int k = tid;
    for (; k + (kUnroll - 1) * kThreads < n4; k += kUnroll * kThreads) {  // kUnroll loads of each in flight
        float4 v[kUnroll];
        int4 m[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            v[u] = vcore::load4(q + x0 + 4 * (k + u * kThreads));
            m[u] = vcore::load4(d2t + x0 + 4 * (k + u * kThreads));
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            add(v[u].x, m[u].x);
            add(v[u].y, m[u].y);
            add(v[u].z, m[u].z);
            add(v[u].w, m[u].w);
        }
    }
    for (; k < n4; k += kThreads) {
        const float4 v = vcore::load4(q + x0 + 4 * k);
        const int4 m = vcore::load4(d2t + x0 + 4 * k);
        add(v.x, m.x);
        add(v.y, m.y);
        add(v.z, m.z);
        add(v.w, m.w);
    }
    for (int x = x0 + 4 * n4 + tid; x < x1; x += kThreads) add(q[x], d2t[x]);
    for (int m = kWave / 2; m > 0; m >>= 1) acc = add128(acc, shfl_xor128(acc, m));
    if (lane == 0) sh_part[wave] = acc;
    __syncthreads();
    U128 tot{0, 0};
    if (tid == 0)
        for (int w = 0; w < kThreads / kWave; ++w) tot = add128(tot, sh_part[w]);
    return tot;
}

// S, the mass row q puts on the intersection: the exact sum rounded once to fp32, in every thread.
__device__ float row_mass(const float *q, const int32_t *d2t, int v_d, U128 *sh_part, float *sh_S) {
    const U128 tot = mass_sum(q, d2t, 0, v_d, sh_part);
    if (threadIdx.x == 0) *sh_S = q62_to_f32(tot);
    __syncthreads();
    return *sh_S;
}

// q'(y) for the draft id x = t2d[y] whose mass g = q(x) was gathered (g = 0 when x lies
// outside [0, v_d): the entry is 0 either way); 0 when S is not positive.
__device__ __forceinline__ float qprime(float g, float S) { return S > 0.0f ? clamp01(g) / S : 0.0f; }

// Short rows: one 1024-thread workgroup per row, the mass and then the row.
__global__ void __launch_bounds__(kThreads) tli_rows(TliArgs a) {
    const int r = blockIdx.x;
    const int tid = threadIdx.x;
    const float *q = a.draft_probs + (int64_t)r * a.draft_ld;
    float *out = a.q_out + (int64_t)r * a.q_ld;
    __shared__ U128 sh_part[kThreads / kWave];
    __shared__ float sh_S;

    // 1. exact Q62 sum of the intersected mass
    const float S = row_mass(q, a.d2t, a.v_d, sh_part, &sh_S);

    // 2. q' over the target vocabulary
    // every lane loads (q[0] outside the intersection) so the gathers of a batch stay in flight together
    auto gather = [&](int32_t x) -> float { return q[(x >= 0 && x < a.v_d) ? x : 0]; };
    auto value = [&](int32_t x, float g) -> float {
        return (x >= 0 && x < a.v_d && S > 0.0f) ? clamp01(g) / S : 0.0f;
    };
    int y0 = 0;
    auto store4 = [&](int k, vcore::f4u v) { *reinterpret_cast<vcore::f4u *>(out + 4 * k) = v; };
    {
        const int n4 = a.v_t / 4;
        int k = tid;
        for (; k + (kUnroll - 1) * kThreads < n4; k += kUnroll * kThreads) {
            int4 m[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) m[u] = vcore::load4(a.t2d + 4 * (k + u * kThreads));
            float4 g[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                g[u] = make_float4(gather(m[u].x), gather(m[u].y), gather(m[u].z), gather(m[u].w));
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                store4(k + u * kThreads, vcore::f4u{value(m[u].x, g[u].x), value(m[u].y, g[u].y),
                                                    value(m[u].z, g[u].z), value(m[u].w, g[u].w)});
        }
        for (; k < n4; k += kThreads) {
            const int4 m = vcore::load4(a.t2d + 4 * k);
            const float4 g = make_float4(gather(m.x), gather(m.y), gather(m.z), gather(m.w));
            store4(k, vcore::f4u{value(m.x, g.x), value(m.y, g.y), value(m.z, g.z), value(m.w, g.w)});
        }
        y0 = 4 * n4;
    }
    for (int y = y0 + tid; y < a.v_t; y += kThreads) {
        const int32_t x = a.t2d[y];
        out[y] = value(x, gather(x));
    }
}

// tli_mass: the masses, for rows [row0, ...).  A row is split over `splits` workgroups (1 once the rows fill the chip);
// they hand their sums to tli_fill in the output row itself, once per slice of tli_fill: S in the
// slice's first entry (one split), or the splits' 128-bit sums in its first 4 * splits entries.
__global__ void __launch_bounds__(kThreads) tli_mass(TliArgs a, int row0, int splits, int slices) {
    const int r = row0 + blockIdx.x / splits, sp = blockIdx.x % splits;
    const int tid = threadIdx.x;
    const float *q = a.draft_probs + (int64_t)r * a.draft_ld;
    uint32_t *out = reinterpret_cast<uint32_t *>(a.q_out + (int64_t)r * a.q_ld);
    __shared__ U128 sh_part[kThreads / kWave];
    __shared__ U128 sh_tot;
    const int per = ((a.v_d + splits - 1) / splits + 3) & ~3;
    const int x0 = sp * per < a.v_d ? sp * per : a.v_d;
    const int x1 = a.v_d - x0 < per ? a.v_d : x0 + per;
    const U128 tot = mass_sum(q, a.d2t, x0, x1, sh_part);
    if (tid == 0) sh_tot = tot;
    __syncthreads();
    if (splits == 1) {
        const uint32_t S = __float_as_uint(q62_to_f32(sh_tot));
        for (int s = tid; s < slices; s += kThreads) out[(int64_t)s * kSlice] = S;
    } else {
        const uint64_t w = (tid & 2) ? sh_tot.hi : sh_tot.lo;
        const uint32_t word = (tid & 1) ? (uint32_t)(w >> 32) : (uint32_t)w;
        for (int s = tid / 4; s < slices; s += kThreads / 4) out[(int64_t)s * kSlice + 4 * sp + (tid & 3)] = word;
    }
}

// tli_fill: q' of one slice of kSlice target ids of a row.
__global__ void __launch_bounds__(kFillThreads) tli_fill(TliArgs a, int row0, int splits, int slices, int items) {
    const int G = gridDim.x, g = blockIdx.x;
    const int work = (g % kXcds) * (G / kXcds) + g / kXcds;
    if (work >= items) return;
    const int r = row0 + work / slices, sl = work % slices;
    const int tid = threadIdx.x;
    const float *q = a.draft_probs + (int64_t)r * a.draft_ld;
    float *out = a.q_out + (int64_t)r * a.q_ld;
    const int y0 = sl * kSlice;
    const int y1 = sl == slices - 1 ? a.v_t : y0 + kSlice;  // the last slice takes the remainder

    constexpr int kVec = kSlice / (4 * kFillThreads);
    // every lane loads (q[0] outside the intersection) so the gathers of a batch stay in flight together
    auto gather = [&](int32_t x) -> float { return q[(x >= 0 && x < a.v_d) ? x : 0]; };
    int4 m[kVec];
    float4 gv[kVec];
    const bool full = y1 - y0 >= kSlice;
    if (full) {
#pragma unroll
        for (int u = 0; u < kVec; ++u) m[u] = vcore::load4(a.t2d + y0 + 4 * (tid + u * kFillThreads));
#pragma unroll
        for (int u = 0; u < kVec; ++u) gv[u] = make_float4(gather(m[u].x), gather(m[u].y), gather(m[u].z), gather(m[u].w));
    }
    float S;
    if (splits == 1) {
        S = out[y0];
    } else {
        U128 tot{0, 0};
        const uint32_t *w = reinterpret_cast<const uint32_t *>(out + y0);
        for (int k = 0; k < splits; ++k)
            tot = add128(tot, U128{((uint64_t)w[4 * k + 1] << 32) | w[4 * k], ((uint64_t)w[4 * k + 3] << 32) | w[4 * k + 2]});
        S = q62_to_f32(tot);
    }
    __syncthreads();  // every thread has read the slice's masses: its entries may be written
    auto value = [&](int32_t x, float g) -> float { return x >= 0 && x < a.v_d ? qprime(g, S) : 0.0f; };
    int y = y0 + tid;
    if (full) {
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
            const vcore::f4u o{value(m[u].x, gv[u].x), value(m[u].y, gv[u].y), value(m[u].z, gv[u].z),
                               value(m[u].w, gv[u].w)};
            __builtin_nontemporal_store(o, reinterpret_cast<vcore::f4u *>(out + y0 + 4 * (tid + u * kFillThreads)));
        }
        y += kSlice;
    }
    for (; y < y1; y += kFillThreads) {
        const int32_t x = a.t2d[y];
        out[y] = value(x, gather(x));
    }
}

// ------------------------------------------------------------------ fused verification
// Standard speculative sampling (App. D Alg. 4) with the TLI proposal of each drafted
// position formed where it is used, so q' rows are never written: one 1024-thread workgroup
// per stream.
//   acceptance: q'_j(t_j) = q_j(t2d[t_j]) / S_j, one gathered draft mass per position; S_j
//     from draft_mass (wave 0 tests 64 positions per ballot) or, without it, by a pass over
//     draft row j (the whole workgroup, row after row until the first rejection);
//   residual: the chunk sums of max(0, p - q') over target row gamma, q' gathered through t2d
//     from draft row gamma (the bonus row as is after full acceptance), the row read in
//     vcore::load_chunk's element order (a 16-byte load instruction covers 1 KB; a chunk's sum
//     does not depend on the order), then the exact inverse-CDF sample by wave 0, which reads
//     the crossing chunk again in position order -- the arithmetic of tt_verify_dense element
//     for element.
constexpr int kWaves = kThreads / kWave;

struct TliRec {
    int r;    // gamma (-1: a sentinel stream)
    float S;  // the rejected row's mass
};

struct TliVerifyParams {
    TliVerifyArgs a;
    int32_t nc, splits, cps;  // chunks of a row, workgroups per stream, chunks of one
    TliRec *rec;              // [n_streams]
    uint64_t *sums;           // [n_streams][nc] Q62 chunk sums
};

// The 16 draft ids t2d of a lane's elements x0 .. x0+15 (x0 = c*1024 + lane*16; -1 past v_t).
__device__ __forceinline__ void load_x(const TliVerifyArgs &a, int x0, int32_t (&xs)[16]) {
    if (x0 + 16 <= a.v_t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int4 t = vcore::load4(a.t2d + x0 + 4 * q);
            xs[4 * q] = t.x;
            xs[4 * q + 1] = t.y;
            xs[4 * q + 2] = t.z;
            xs[4 * q + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) xs[k] = vcore::entry_or(a.t2d, x0 + k, a.v_t, -1);
    }
}

// Their target probabilities (0 past v_t) and ids (the sampler's crossing chunk, in position order).
__device__ __forceinline__ void load_px(const TliVerifyArgs &a, const float *prow, int x0, float (&pv)[16],
                                        int32_t (&xs)[16]) {
    vcore::read16(prow, x0, a.v_t, pv);
    load_x(a, x0, xs);
}

// The draft masses q(x) at the 16 ids (0 for an id outside [0, v_d), or without a draft row).
// Only the lanes that keep an id load (the intersection is often a small part of V_t).
__device__ __forceinline__ void gather16(const TliVerifyArgs &a, const float *drow, const int32_t (&xs)[16],
                                         float (&gv)[16]) {
#pragma unroll
    for (int k = 0; k < 16; ++k) gv[k] = (drow != nullptr && xs[k] >= 0 && xs[k] < a.v_d) ? drow[xs[k]] : 0.0f;
}

// Q62 residual entries q62(clamp01(p - q')) of the 16 elements (q' = qprime(g, S); 0 past v_t,
// where p = g = 0).
__device__ __forceinline__ uint64_t residual16(const float (&pv)[16], const float (&gv)[16], float S, int x0, int vt,
                                               uint64_t (&qv)[16]) {
    uint64_t sum = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        qv[k] = x0 + k < vt ? q62(clamp01(pv[k] - qprime(gv[k], S))) : 0ull;
        sum += qv[k];
    }
    return sum;
}

// The row pass in vcore::load_chunk's element order (lane l holds elements 256 u + 4 l + j of a
// chunk, so each 16-byte load instruction covers 1 KB of the row): the target probabilities
// with the non-temporal hint, the 16 ids t2d in the same order (-1 past v_t).
__device__ __forceinline__ void load_px_strided(const TliVerifyArgs &a, const float *prow, int c, float4 (&pv)[4], int32_t (&xs)[16]) {
    const int lane = threadIdx.x % kWave;
    const int xb = c * vcore::kChunk;
    vcore::load_chunk(prow, xb, lane, a.v_t, pv);
    if (xb + vcore::kChunk <= a.v_t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int4 t = vcore::load4(a.t2d + xb + u * 256 + lane * 4);
            xs[4 * u] = t.x;
            xs[4 * u + 1] = t.y;
            xs[4 * u + 2] = t.z;
            xs[4 * u + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int y = xb + (k >> 2) * 256 + lane * 4 + (k & 3);
            xs[k] = vcore::entry_or(a.t2d, y, a.v_t, -1);
        }
    }
}

// q' of a row's masses by its reciprocal: with r = RN(1 / S), a quotient estimate within one unit in
// the last place and the exact remainder (fused multiply-adds), one more step gives the correctly
// rounded quotient (Markstein 1990), so q' is the IEEE quotient in 5 instructions instead of the 10 of
// a division.  The first step takes g * r (within two units) to within one.  Exact while nothing
// underflows: S in [2^-30, 2^10] and g = 0 or g >= 2^-60; else the division.  256 streams of
// 151,936 ids: 61.6 us, 63.6 with divisions.  S = 0, as for a bonus row, needs none (every quotient is
// defined as 0): 64 streams of 16,384 ids that accept every proposal 9.1 us, 9.4 with divisions.
struct RowMass {
    float S, r;
    bool fast;
};

__device__ __forceinline__ RowMass row_reciprocal(float S) {
    RowMass m;
    m.S = S;
    m.r = S == 0.0f ? 0.0f : 1.0f / S;
    m.fast = S == 0.0f || (S >= 0x1p-30f && S <= 0x1p10f);
    return m;
}

__device__ __forceinline__ float quotient(float g, const RowMass &m) {
    const float q0 = g * m.r;
    const float q1 = fmaf(fmaf(-q0, m.S, g), m.r, q0);
    return fmaf(fmaf(-q1, m.S, g), m.r, q1);
}

// Q62 sum of the 16 residual entries in that order (p = g = 0 past v_t gives 0).
__device__ __forceinline__ uint64_t residual_sum_strided(const float4 (&pv)[4], float (&gv)[16], const RowMass &m) {
    uint64_t sum = 0;
    uint32_t least = 0xFFFFFFFFu;  // the least positive mass, as bits less one (0 wraps to the top)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        gv[k] = clamp01(gv[k]);
        const uint32_t bits = __float_as_uint(gv[k]) - 1u;
        least = bits < least ? bits : least;
    }
    if (__all(m.fast && least >= 0x21800000u - 1u)) {  // 2^-60
#pragma unroll
        for (int k = 0; k < 16; ++k) gv[k] = quotient(gv[k], m);
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) gv[k] = qprime(gv[k], m.S);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        sum += q62(clamp01(pv[u].x - gv[4 * u])) + q62(clamp01(pv[u].y - gv[4 * u + 1])) +
               q62(clamp01(pv[u].z - gv[4 * u + 2])) + q62(clamp01(pv[u].w - gv[4 * u + 3]));
    }
    return sum;
}

// Whether every proposal's id lies inside the target vocabulary (one wave).
__device__ __forceinline__ bool ids_ok(const TliVerifyArgs &a, int t0, int M, int lane) {
    bool ok = true;
    for (int base = 0; ok && base < M; base += kWave) {
        const int j = base + lane;
        ok = !__any(j < M && (a.target_ids[t0 + j] < 0 || a.target_ids[t0 + j] >= a.v_t));
    }
    return ok;
}

// gamma and S_gamma with the drafter's masses (one wave, 64 positions a ballot).
__device__ __forceinline__ void mass_scan(const TliVerifyArgs &a, int b, int t0, int M, int lane, int &gamma, float &S_r) {
    gamma = M;
    S_r = 0.0f;
    for (int base = 0; base < M && gamma == M; base += kWave) {
        const int j = base + lane;
        bool rej = false;
        float Sj = 0.0f;
        if (j < M) {
            const int tok = a.target_ids[t0 + j];
            const float uj = a.u_accept[t0 + j];
            Sj = a.draft_mass[t0 + j];
            if (tok >= 0 && tok < a.v_t) {
                const float pt = a.target_probs[(int64_t)(t0 + b + j) * a.target_ld + tok];
                const int32_t x = a.t2d[tok];
                const float g = (x >= 0 && x < a.v_d) ? a.draft_probs[(int64_t)(t0 + j) * a.draft_ld + x] : 0.0f;
                const float qj = qprime(g, Sj);
                rej = !((qj <= 0.0f) || (uj < pt / qj));
            }
        }
        const unsigned long long rm = __ballot(rej);
        if (rm != 0ull) {
            const int l = __ffsll(rm) - 1;
            gamma = base + l;
            S_r = __shfl(Sj, l);
        }
    }
}

// gamma and S_gamma without masses (the whole workgroup of kThreads): S_j of each tested row, formed as
// tt_tli_proposal forms it, row after row.
__device__ void row_scan(const TliVerifyArgs &a, int b, int t0, int M, U128 *sh_red, float *sh_S, int *sh_rej, int &gamma,
                         float &S_r) {
    gamma = M;
    S_r = 0.0f;
    for (int j = 0; j < M; ++j) {
        const float *drow = a.draft_probs + (int64_t)(t0 + j) * a.draft_ld;
        const float Sj = row_mass(drow, a.d2t, a.v_d, sh_red, sh_S);
        if (threadIdx.x == 0) {
            const int tok = a.target_ids[t0 + j];
            const float pt = a.target_probs[(int64_t)(t0 + b + j) * a.target_ld + tok];
            const int32_t x = a.t2d[tok];
            const float g = (x >= 0 && x < a.v_d) ? drow[x] : 0.0f;
            const float qj = qprime(g, Sj);
            *sh_rej = !((qj <= 0.0f) || (a.u_accept[t0 + j] < pt / qj)) ? 1 : 0;
        }
        __syncthreads();
        if (*sh_rej) {
            gamma = j;
            S_r = Sj;
            return;
        }
    }
}

// The token of the residual (or bonus, drow null) row from its chunk sums part(c), by one wave.
template <class Part>
__device__ __forceinline__ int sample_residual(const TliVerifyArgs &a, const float *prow, const float *drow, float S_r, int nc,
                                               float u, Part part) {
    const int lane = threadIdx.x % kWave;
    uint64_t Z, T, base;
    int cs;
    const int st = vcore::find_crossing(nc, part, u, Z, T, cs, base);
    if (st == 1) return vcore::wave_first_argmax(prow, a.v_t);
    if (st == 2) return a.v_t - 1;
    const int x0 = cs * vcore::kChunk + lane * 16;
    float pv[16], gv[16];
    int32_t xs[16];
    load_px(a, prow, x0, pv, xs);
    gather16(a, drow, xs, gv);
    uint64_t qv[16];
    const uint64_t sum = residual16(pv, gv, S_r, x0, a.v_t, qv);
    const uint64_t lincl = vcore::wave_inclusive_scan(sum) + base;
    const uint64_t lexcl = lincl - sum;
    const unsigned long long lhit = __ballot(lexcl <= T && T < lincl);
    if (lhit == 0ull) return a.v_t - 1;
    const int tl = __ffsll(lhit) - 1;
    uint64_t run = lexcl;
    int k_at = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        run += qv[k];
        k_at += run <= T ? 1 : 0;
    }
    return __builtin_amdgcn_readlane(x0 + k_at, tl);
}

__global__ void __launch_bounds__(kThreads) verify_tli_row(TliVerifyParams p) {
    const TliVerifyArgs &a = p.a;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    extern __shared__ uint64_t sh_part[];  // nc chunk sums (Q62)
    __shared__ U128 sh_red[kWaves];
    __shared__ float sh_S, sh_Sr;
    __shared__ int sh_ok, sh_gamma, sh_ctr, sh_rej;

    TT_STAMP(0);
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    if (!(M >= 0 && M <= a.max_m)) {
        if (tid == 0) {
            a.n_accepted[b] = -1;
            a.out_token[b] = -1;
        }
        return;
    }
    if (wave == kWaves - 1) {
        const bool ok = ids_ok(a, t0, M, lane);
        if (lane == 0) {
            sh_ok = ok ? 1 : 0;
            sh_ctr = kWaves;
        }
    }
    if (a.draft_mass != nullptr && wave == 0) {
        int g;
        float S;
        mass_scan(a, b, t0, M, lane, g, S);
        if (lane == 0) {
            sh_gamma = g;
            sh_Sr = S;
        }
    }
    __syncthreads();
    if (!sh_ok) {
        if (tid == 0) {
            a.n_accepted[b] = -1;
            a.out_token[b] = -1;
        }
        return;
    }
    int gamma;
    float S_r;
    if (a.draft_mass != nullptr) {
        gamma = sh_gamma;
        S_r = sh_Sr;
    } else {
        row_scan(a, b, t0, M, sh_red, &sh_S, &sh_rej, gamma, S_r);
    }
    TT_STAMP(1);
    // residual (or bonus) row: Q62 chunk sums of max(0, p - q') into LDS
    const float *prow = a.target_probs + (int64_t)(t0 + b + gamma) * a.target_ld;
    const float *drow = gamma < M ? a.draft_probs + (int64_t)(t0 + gamma) * a.draft_ld : nullptr;
    const int nc = p.nc;
    {
        // each wave: chunk c's probabilities and draft masses, chunk cn's probabilities and ids
        // in flight behind them (a chunk's gathers wait for its ids only)
        float4 pv[4], pn[4];
        float gv[16];
        int32_t xs[16];
        int c = wave, cn = nc;
        const RowMass mass = row_reciprocal(S_r);
        if (c < nc) {
            load_px_strided(a, prow, c, pv, xs);
            gather16(a, drow, xs, gv);
            cn = vcore::next_chunk(&sh_ctr, c, kWaves);
            if (cn < nc) load_px_strided(a, prow, cn, pn, xs);
        }
        while (c < nc) {
            uint64_t acc = residual_sum_strided(pv, gv, mass);
            acc = vcore::wave_total(acc);
            if (lane == kWave - 1) sh_part[c] = acc;
            c = cn;
            if (c < nc) {
#pragma unroll
                for (int u = 0; u < 4; ++u) pv[u] = pn[u];
                gather16(a, drow, xs, gv);
                cn = vcore::next_chunk(&sh_ctr, c, kWaves);
                if (cn < nc) load_px_strided(a, prow, cn, pn, xs);
            }
        }
    }
    if (wave < 12) TT_STAMP_WAVE(4 + wave);
    __syncthreads();
    TT_STAMP(2);
    if (wave != 0) return;
    const int token = sample_residual(a, prow, drow, S_r, nc, a.u_sample[b], [&](int c) { return sh_part[c]; });
    if (lane == 0) {
        a.n_accepted[b] = gamma;
        a.out_token[b] = token;
    }
    TT_STAMP(3);
}

// The same in three kernels for batches that leave compute units idle (one workgroup per stream reads
// its whole row, and gathers for it, on one): the acceptance (tli_gamma), the residual row's chunk
// sums by `splits` workgroups a stream, a stream's together on one XCD (tli_stream), and the sample
// (tli_sample).  A few streams' draft rows stay in L2 while they are gathered from, as in tli_fill.
template <int THREADS>
__global__ void __launch_bounds__(THREADS) tli_gamma(TliVerifyParams p) {
    const TliVerifyArgs &a = p.a;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave;
    __shared__ U128 sh_red[kWaves];
    __shared__ float sh_S;
    __shared__ int sh_rej;
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    // (every wave checks the ids: the result is the same in all)
    const bool ok = M >= 0 && M <= a.max_m && ids_ok(a, t0, M, lane);
    int gamma = -1;
    float S_r = 0.0f;
    if (ok) {
        if constexpr (THREADS == kWave) mass_scan(a, b, t0, M, lane, gamma, S_r);
        else row_scan(a, b, t0, M, sh_red, &sh_S, &sh_rej, gamma, S_r);
    }
    if (tid == 0) {
        p.rec[b] = TliRec{gamma, S_r};
        if (!ok) {
            a.n_accepted[b] = -1;
            a.out_token[b] = -1;
        }
    }
}

__global__ void __launch_bounds__(kFillThreads) tli_stream(TliVerifyParams p) {
    const TliVerifyArgs &a = p.a;
    const int G = gridDim.x, g = blockIdx.x;
    const int work = (g % kXcds) * (G / kXcds) + g / kXcds;
    if (work >= a.n_streams * p.splits) return;
    const int b = work / p.splits, sp = work % p.splits;
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    constexpr int kW = kFillThreads / kWave;
    const TliRec rec = p.rec[b];
    if (rec.r < 0) return;
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    const float *prow = a.target_probs + (int64_t)(t0 + b + rec.r) * a.target_ld;
    const float *drow = rec.r < M ? a.draft_probs + (int64_t)(t0 + rec.r) * a.draft_ld : nullptr;
    const int c1 = (sp + 1) * p.cps < p.nc ? (sp + 1) * p.cps : p.nc;
    const RowMass mass = row_reciprocal(rec.S);
    for (int c = sp * p.cps + wave; c < c1; c += kW) {
        float4 pv[4];
        float gv[16];
        int32_t xs[16];
        load_px_strided(a, prow, c, pv, xs);
        gather16(a, drow, xs, gv);
        const uint64_t acc = vcore::wave_total(residual_sum_strided(pv, gv, mass));
        if (lane == kWave - 1) p.sums[(int64_t)b * p.nc + c] = acc;
    }
}

__global__ void __launch_bounds__(kWave) tli_sample(TliVerifyParams p) {
    const TliVerifyArgs &a = p.a;
    const int b = blockIdx.x;
    const TliRec rec = p.rec[b];
    if (rec.r < 0) return;  // sentinel stream, outputs already written
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    const float *prow = a.target_probs + (int64_t)(t0 + b + rec.r) * a.target_ld;
    const float *drow = rec.r < M ? a.draft_probs + (int64_t)(t0 + rec.r) * a.draft_ld : nullptr;
    const uint64_t *sums = p.sums + (int64_t)b * p.nc;
    const int token = sample_residual(a, prow, drow, rec.S, p.nc, a.u_sample[b], [&](int c) { return sums[c]; });
    if (threadIdx.x == 0) {
        a.n_accepted[b] = rec.r;
        a.out_token[b] = token;
    }
}

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

int launch_tli_proposal(const TliArgs &a, hipStream_t stream) {
    if (a.n_rows == 0) return TT_OK;
    const bool full = a.n_rows > kHalfFull && a.n_rows <= kCus;  // one kernel: every row at once, on most of the chip
    const bool two = a.n_rows <= kFewRows ? (int64_t)a.v_d + a.v_t >= kFewRowsVocab
                                          : a.v_t > kManyRowsTarget && a.v_d > (full && a.v_t <= kFullTarget ? kFullDraft : kManyRowsDraft);
    if (!two) {
        hipLaunchKernelGGL(tli_rows, dim3(a.n_rows), dim3(kThreads), 0, stream, a);
        return hipGetLastError() == hipSuccess ? TT_OK : TT_ELAUNCH;
    }
    const int slices = a.v_t >= kSlice ? a.v_t / kSlice : 1;
    // the rows go through both kernels in equal parts, multiples of the compute units (a mass workgroup takes one),
    // a short rest with the part before it, each part few enough for one grid
    const int64_t draft_row = 4 * (int64_t)a.v_d, row = draft_row + 4 * (int64_t)a.v_t;
    int64_t chunk = kPartDraft / draft_row < kPartBytes / row ? kPartDraft / draft_row : kPartBytes / row;
    if (chunk < kPartSmall / draft_row) chunk = kPartSmall / draft_row;
    chunk = chunk < kCus ? kCus : chunk / kCus * kCus;
    const int64_t parts = (a.n_rows + chunk - 1) / chunk;
    chunk = a.n_rows <= chunk + kCus / 4 ? a.n_rows : ((a.n_rows + parts - 1) / parts + kCus - 1) / kCus * kCus;
    if (chunk > kMaxItems / slices) chunk = kMaxItems / slices;
    int splits = (int)(kCus / chunk);
    if (splits > kMaxSplits) splits = kMaxSplits;
    while (splits > 1 && (splits * 4 > a.v_t || a.v_d / splits < 4096)) --splits;
    if (splits < 1) splits = 1;
    for (int64_t r0 = 0; r0 < a.n_rows; r0 += chunk) {
        const int rows = (int)(a.n_rows - r0 < chunk ? a.n_rows - r0 : chunk);
        hipLaunchKernelGGL(tli_mass, dim3(rows * splits), dim3(kThreads), 0, stream, a, (int)r0, splits, slices);
        if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
        const int items = rows * slices;
        hipLaunchKernelGGL(tli_fill, dim3((items + kXcds - 1) / kXcds * kXcds), dim3(kFillThreads), 0, stream, a, (int)r0,
                           splits, slices, items);
        if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
    }
    return hipGetLastError() == hipSuccess ? TT_OK : TT_ELAUNCH;
}

size_t tli_workspace_bytes(int32_t n_streams, int32_t v_t) {
    const int64_t nc = ((int64_t)v_t + vcore::kChunk - 1) / vcore::kChunk;
    if (n_streams == 0 || nc < kTliSplitChunks || n_streams > (nc >= kTliLongChunks ? kTliLongStreams : kTliSplitStreams))
        return 0;
    return align256(sizeof(TliRec) * (size_t)n_streams) + 8 * (size_t)n_streams * (size_t)nc;
}

int launch_verify_tli(const TliVerifyArgs &a, void *workspace, size_t workspace_bytes, hipStream_t stream) {
    if (a.n_streams == 0) return TT_OK;
    TliVerifyParams p{};
    p.a = a;
    p.nc = (a.v_t + vcore::kChunk - 1) / vcore::kChunk;
    const size_t need = tli_workspace_bytes(a.n_streams, a.v_t);
    if (workspace == nullptr || need == 0) {
        hipLaunchKernelGGL(verify_tli_row, dim3(a.n_streams), dim3(kThreads), 8 * (size_t)p.nc, stream, p);
        return hipGetLastError() == hipSuccess ? TT_OK : TT_ELAUNCH;
    }
    if (workspace_bytes < need) return TT_EWORKSPACE;
    p.rec = static_cast<TliRec *>(workspace);
    p.sums = reinterpret_cast<uint64_t *>(static_cast<uint8_t *>(workspace) + align256(sizeof(TliRec) * (size_t)a.n_streams));
    p.cps = kFillThreads / kWave;  // a chunk a wave
    p.splits = (p.nc + p.cps - 1) / p.cps;
    if (a.draft_mass != nullptr) hipLaunchKernelGGL(tli_gamma<kWave>, dim3(a.n_streams), dim3(kWave), 0, stream, p);
    else hipLaunchKernelGGL(tli_gamma<kThreads>, dim3(a.n_streams), dim3(kThreads), 0, stream, p);
    if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
    const int items = a.n_streams * p.splits;
    hipLaunchKernelGGL(tli_stream, dim3((items + kXcds - 1) / kXcds * kXcds), dim3(kFillThreads), 0, stream, p);
    if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
    hipLaunchKernelGGL(tli_sample, dim3(a.n_streams), dim3(kWave), 0, stream, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_ELAUNCH;
}

}  // namespace tt
