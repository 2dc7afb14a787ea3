// Verification from bf16 target logits with a temperature on gfx950: the target softmax of
// Sec. 3's acceptance rule and App. D Alg. 4's residual is formed inside the verification
// (App. F lists the sampling temperatures), so the caller never materialises fp32
// probability rows.
//
// Arithmetic (every step specified, so any summation order gives the same token), in base 2:
//   c      = inv_temp * log2(e) (fp32, once per stream); y = fp32(bf16 logit) * c, NaN counts
//            as minus infinity (no mass, never the max)
//   mu     = max y over the row, or L * log2(e) for a caller's log-sum-exp L (natural units)
//   z      = fma(logit, c, 31 - mu) held in [-1, 31]: the logit's scaled base-2 exponent
//   2^z    = p * 2^k, k = rint(z), p the degree-5 Taylor polynomial of 2^(z - k) (Horner, FMAs)
//   e31    = floor(p * 2^k), the weight in Q31, summed exactly in 64 bits (rows <= 2^23 entries)
//   E      = p * 2^(k - 31) (0 for z < 0); S = sum * 2^-31 rounded once to fp32 (ties to even)
//   P(t_j) = E(t_j) / S (E(t_j) with L); accept while q_j <= 0 or u_j < P(t_j) / q_j
//   after a rejection at r the entry t_r of the residual is
//            floor(clamp(E(t_r) - q_r S, 0, 1) * 2^31), proportional to max(0, P - q_r e_t);
//            after full acceptance the bonus row's e31 is sampled as is
//   token  = first index whose prefix exceeds floor(u * Z); first largest y when Z = 0.
//
// verify_logits_row: one 1024-thread workgroup per stream.  Without normalisers it walks its rows 0, 1, ...
// until the first rejection (each row: a max pass, then a pass of chunk sums into LDS -- the
// second read mostly from the caches).  With per-row log-sum-exp values L from the caller
// (an LM head can emit them with its logits) it uses m = L and S = 1: the acceptance test
// needs one gathered logit per position and only the residual (or bonus) row is read, once.
// Wave 0 samples: the chunk sums lane-blocked, the crossing chunk's e31 recomputed from its
// 1024 logits.  In the row passes a lane reads 16 bf16 with two 16-byte loads, each load
// instruction covering 1 KB of the row; the sampler reads 16 consecutive bf16 a lane.
// With a workspace, rows are spread over the GPU: without normalisers they are screened many at once
// and the walk starts where the screen stopped; with them, and after the screen, few streams form the
// selected row's sums with several workgroups each (the sections below).
#include "verify_core.h"

TT_STAMPS_TABLE(logits)

namespace tt {
namespace {

using vcore::entry_or;
using vcore::exact_threshold;
using vcore::lane_value;
using vcore::wave_inclusive_scan;

constexpr int kThreads = 1024;
constexpr int kWave = 64;
constexpr int kWaves = kThreads / kWave;
constexpr int kChunk = 1024;  // logits per chunk: one wave, 16 per lane

__device__ __forceinline__ float bf16_value(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

constexpr float kLog2e = 0x1.715476p+0f;  // log2(e) rounded to fp32

// 2^z = p * 2^k for z held in [-1, 31] (NaN gives p * 2^k < 1, a zero weight): k = rint(z),
// f = z - k in [-1/2, 1/2] (exact), p = 1 + f ln2 + ... + (f ln2)^5 / 5! by Horner's rule.
__device__ __forceinline__ float exp2_parts(float z, int &k) {
    z = fminf(fmaxf(z, -1.0f), 31.0f);
    const float kf = rintf(z);
    const float f = z - kf;
    float p = 0x1.5d87fep-10f;
    p = fmaf(p, f, 0x1.3b2ab6p-7f);
    p = fmaf(p, f, 0x1.c6b08ep-5f);
    p = fmaf(p, f, 0x1.ebfbe0p-3f);
    p = fmaf(p, f, 0x1.62e430p-1f);
    p = fmaf(p, f, 1.0f);
    k = (int)kf;
    return p;
}

// floor(2^z): the weight in Q31 of a logit whose scaled exponent is z (p * 2^k < 2^32)
__device__ __forceinline__ uint32_t e31_at(float z) {
    int k;
    const float p = exp2_parts(z, k);
    return (uint32_t)ldexpf(p, k);
}

// E = 2^(z - 31) as fp32, 0 when z < 0 or NaN (where the Q31 weight is 0)
__device__ __forceinline__ float weight_at(float z) {
    if (!(z >= 0.0f)) return 0.0f;
    int k;
    const float p = exp2_parts(z, k);
    return ldexpf(p, k - 31);
}

// floor(r * 2^31) for r in [0, 1]
__device__ __forceinline__ uint32_t q31(float r) { return (uint32_t)ldexpf(r, 31); }

// n * 2^-31 rounded to the nearest fp32, ties to even
__device__ inline float q31_to_f32(uint64_t n) {
    if (n == 0) return 0.0f;
    const int bl = 64 - __clzll(n);
    if (bl <= 24) return ldexpf((float)n, -31);
    const int sh = bl - 24;
    uint64_t mant = n >> sh;
    const uint64_t rem = n & ((1ull << sh) - 1), half = 1ull << (sh - 1);
    if (rem > half || (rem == half && (mant & 1u))) ++mant;
    return ldexpf((float)mant, sh - 31);
}

// y = logit * c.  A NaN y is left as is: fmaxf ignores it in the max pass and it never
// compares greater in the first-argmax fallback; its scaled exponent gives a zero weight.
__device__ __forceinline__ float scaled(uint32_t bits16, float c) { return bf16_value(bits16) * c; }

// the scaled exponent z of a logit: fma(logit, c, b31) with b31 = 31 - mu
__device__ __forceinline__ float expo(uint32_t bits16, float c, float b31) { return fmaf(bf16_value(bits16), c, b31); }

// Eight bf16 at an address aligned to 2 bytes only: rows of an odd stride start anywhere, and
// gfx950's 16-byte global loads take any address, so every row takes the wide path.
typedef unsigned int u4u __attribute__((ext_vector_type(4), aligned(2)));

// 16 consecutive logits x0 .. x0 + 15 of a lane (the sampler's crossing chunk; zero bits past v).
__device__ __forceinline__ void load16(const uint16_t *row, int x0, int v, uint32_t (&w)[8]) {
    if (x0 + 16 <= v) {
        const u4u a = *reinterpret_cast<const u4u *>(row + x0);
        const u4u b = *reinterpret_cast<const u4u *>(row + x0 + 8);
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
        w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t lo = x0 + 2 * k < v ? row[x0 + 2 * k] : 0u;
            const uint32_t hi = x0 + 2 * k + 1 < v ? row[x0 + 2 * k + 1] : 0u;
            w[k] = lo | (hi << 16);
        }
    }
}

// The 16 bf16 a lane takes of chunk c in the row passes: elements 512 u + 8 lane + j (u < 2,
// j < 8), so that each of the two 16-byte load instructions covers 1 KB of the row (16
// consecutive logits a lane would make each span 2 KB); 0 past v.  NT: the non-temporal hint
// (the row's last read).  A chunk's sums and maximum do not depend on the order.
template <bool NT>
__device__ __forceinline__ void load16s(const uint16_t *row, int c, int lane, int v, uint32_t (&w)[8]) {
    const int xb = c * kChunk;
    if (xb + kChunk <= v) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const u4u *src = reinterpret_cast<const u4u *>(row + xb + u * 512 + lane * 8);
            u4u t;
            if constexpr (NT) t = __builtin_nontemporal_load(src);
            else t = *src;
            w[4 * u] = t.x;
            w[4 * u + 1] = t.y;
            w[4 * u + 2] = t.z;
            w[4 * u + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int x = xb + (k >> 2) * 512 + lane * 8 + 2 * (k & 3);
            const uint32_t lo = entry_or(row, x, v, uint16_t(0));
            const uint32_t hi = entry_or(row, x + 1, v, uint16_t(0));
            w[k] = lo | (hi << 16);
        }
    }
}

// Index of element k (0..15) of a lane's 16 in chunk c, in load16s's order.
__device__ __forceinline__ int elem_index_s(int c, int lane, int k) {
    return c * kChunk + (k >> 3) * 512 + lane * 8 + (k & 7);
}

// bf16 element k (0..15) of a lane's 16
__device__ __forceinline__ uint32_t elem(const uint32_t (&w)[8], int k) {
    return (k & 1) ? (w[k >> 1] >> 16) : (w[k >> 1] & 0xFFFFu);
}

// Per-row table of the Q31 weights.  For a fixed scale and offset the weight of a logit is a
// function of its 16 bits, so the row pass looks it up instead of evaluating the exponential:
// the table holds e31_at(expo(bits)) for every pattern whose magnitude lies in [2^-20, 2^8)
// (exponent fields 107 .. 134, 3,584 patterns a sign), as 64-bit entries that add straight into
// the 64-bit sums.  Each sign owns a half of 4,096 slots (32 KiB, so the pattern's sign bit,
// left in place, is the byte offset of its half); slot 0 and slot 3,585 of a half are sentinels,
// 2^40 (a weight is at most 2^31: z <= 31), onto which magnitudes outside the domain clamp
// (tiny values, |x| >= 256, infinities, NaNs).  A lane group whose sum reaches 2^40 met one and
// is summed again from the formula.
constexpr uint32_t kMagLo = 107u << 7;  // bf16 magnitude bits of 2^-20
constexpr uint32_t kTabMags = 28u << 7;
constexpr int kTabHalf = 4096;
constexpr int kTabSlots = 2 * kTabHalf;
constexpr uint64_t kSentinel = 1ull << 40;

__device__ __forceinline__ void build_table(uint64_t *tab, float sc, float b31) {
    for (int i = threadIdx.x; i < kTabSlots; i += kThreads) {
        const uint32_t s = (uint32_t)i / kTabHalf, j = (uint32_t)i % kTabHalf;
        if (j > kTabMags + 1) continue;  // never addressed
        uint64_t e = kSentinel;
        if (j > 0 && j <= kTabMags) e = e31_at(expo((s << 15) | (kMagLo + j - 1), sc, b31));
        tab[i] = e;
    }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// The LDS byte offsets of the two bf16 in a 32-bit word (low half first), both formed at once
// with packed 16-bit operations: the magnitude clamped to the domain's frame, rebased and
// scaled to a byte offset, and the pattern's sign bit kept as the half's offset.
__device__ __forceinline__ uint32_t tab_offsets(uint32_t w) {
    u16x2 t = __builtin_bit_cast(u16x2, w & 0x7FFF7FFFu);
    t = __builtin_elementwise_max(t, (u16x2)(unsigned short)(kMagLo - 1));
    t = __builtin_elementwise_min(t, (u16x2)(unsigned short)(kMagLo + kTabMags));
    // (t - (kMagLo - 1)) * 8, modulo 2^16 (the true value is below 2^15)
    t = t * (u16x2)(unsigned short)8 - (u16x2)(unsigned short)((kMagLo - 1) * 8);
    return __builtin_bit_cast(uint32_t, t) | (w & 0x80008000u);
}

__device__ __forceinline__ uint64_t tab_at(const uint64_t *tab, uint32_t byte_off) {
    return *reinterpret_cast<const uint64_t *>(reinterpret_cast<const char *>(tab) + byte_off);
}

// The 16 weights of a lane's logits x0 .. x0+15 (0 past v) into e; a sentinel for a logit
// outside the table's domain is replaced by the formula's weight.  Without a table (tab null)
// all by the formula.
__device__ __forceinline__ void lane_weights(const uint64_t *tab, const uint32_t (&w)[8], int x0, int v, float sc,
                                             float b31, uint64_t (&e)[16]) {
    uint64_t any = tab == nullptr ? kSentinel : 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (tab == nullptr) break;
        const uint32_t o = tab_offsets(w[k]);
        e[2 * k] = x0 + 2 * k < v ? tab_at(tab, o & 0xFFFFu) : 0u;
        e[2 * k + 1] = x0 + 2 * k + 1 < v ? tab_at(tab, o >> 16) : 0u;
        any |= e[2 * k] | e[2 * k + 1];
    }
    if (any >= kSentinel) {
#pragma unroll
        for (int k = 0; k < 16; ++k) e[k] = x0 + k < v ? e31_at(expo(elem(w, k), sc, b31)) : 0u;
    }
}

// As lane_weights for a lane's 16 logits of chunk c in load16s's order.
__device__ __forceinline__ void lane_weights_s(const uint64_t *tab, const uint32_t (&w)[8], int c, int v, float sc,
                                               float b31, uint64_t (&e)[16]) {
    const int lane = threadIdx.x % kWave;
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t o = tab_offsets(w[k]);
        e[2 * k] = elem_index_s(c, lane, 2 * k) < v ? tab_at(tab, o & 0xFFFFu) : 0u;
        e[2 * k + 1] = elem_index_s(c, lane, 2 * k + 1) < v ? tab_at(tab, o >> 16) : 0u;
        any |= e[2 * k] | e[2 * k + 1];
    }
    if (any >= kSentinel) {
#pragma unroll
        for (int k = 0; k < 16; ++k) e[k] = elem_index_s(c, lane, k) < v ? e31_at(expo(elem(w, k), sc, b31)) : 0u;
    }
}

// The wave's total of per-lane sums of 16 weights (each at most 2^35), in lane 63: the low 20
// and the high 15 bits are summed as 32-bit values (64 of them stay below 2^26 and 2^21).
__device__ __forceinline__ uint64_t chunk_total(uint64_t a) {
    const uint32_t lo = vcore::wave_scan32((uint32_t)a & 0xFFFFFu);
    const uint32_t hi = vcore::wave_scan32((uint32_t)(a >> 20));
    return ((uint64_t)hi << 20) + lo;
}

// The row's weight table, then its chunk sums of e31 into sh_part.  Every wave first issues the
// loads of its first two chunks, so that their latency passes while the table is built; waves
// take chunks from the LDS counter *next (which the caller sets to kWaves before a barrier that
// precedes the call; wave w starts at chunk w), one chunk in flight ahead of the one summed.
__device__ __forceinline__ void chunk_sums(const uint16_t *row, int v, int nc, float sc, float b31,
                                           uint64_t *tab, uint64_t *sh_part, int *next) {
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t w[8] = {}, nx[8] = {};
    int c = wave, cn = nc, cnn = nc;  // chunk summed, chunk in flight, the one after it
    if (c < nc) {
        load16s<true>(row, c, lane, v, w);
        cn = vcore::next_chunk(next, c, kWaves);
        if (cn < nc) {
            load16s<true>(row, cn, lane, v, nx);
            cnn = vcore::next_chunk(next, cn, kWaves);
        }
    }
    build_table(tab, sc, b31);
    __syncthreads();
    while (c < nc) {
        uint64_t acc = 0;
        if ((c + 1) * kChunk <= v) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t o = tab_offsets(w[k]);
                acc += tab_at(tab, o & 0xFFFFu) + tab_at(tab, o >> 16);
            }
            if (acc >= kSentinel) {  // a logit outside the table's domain: the lane group by the formula
                acc = 0;
#pragma unroll
                for (int k = 0; k < 16; ++k) acc += e31_at(expo(elem(w, k), sc, b31));
            }
        } else {  // the row's ragged end
            uint64_t e[16];
            lane_weights_s(tab, w, c, v, sc, b31, e);
#pragma unroll
            for (int k = 0; k < 16; ++k) acc += e[k];
        }
        acc = chunk_total(acc);
        if (lane == kWave - 1) sh_part[c] = acc;
        c = cn;
        if (c < nc) {
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = nx[k];
            cn = cnn;
            if (cn < nc) {
                load16s<true>(row, cn, lane, v, nx);
                cnn = vcore::next_chunk(next, cn, kWaves);
            }
        }
    }
}

// Inverse-CDF sample of a row from its chunk sums (one wave).  When t >= 0 the entry at t
// counts adj instead of the before its chunk sum holds (the residual's entry); Z is the row's
// total so adjusted.  The first largest x when Z = 0.
__device__ inline int sample_row(const uint16_t *row, int v, int nc, float sc, float b31,
                                 const uint64_t *tab, int t, uint64_t adj, uint64_t before, float u,
                                 const uint64_t *sh_part) {
    const int lane = threadIdx.x % kWave;
    // chunk sums lane-blocked: lane l holds chunks [l*per, (l+1)*per)
    const int per = (nc + kWave - 1) / kWave;
    const int ca = lane * per < nc ? lane * per : nc;
    const int cb = ca + per < nc ? ca + per : nc;
    const int ct = t >= 0 ? t / kChunk : -1;
    uint64_t local = 0;
    for (int c = ca; c < cb; ++c) local += sh_part[c];
    if (ct >= ca && ct < cb) local = local - before + adj;
    const uint64_t incl = wave_inclusive_scan(local);
    const uint64_t Z = lane_value(incl, kWave - 1);
    if (Z == 0) {
        float bv = -INFINITY;
        int bi = INT_MAX;
        for (int x = lane; x < v; x += kWave) {
            const float xv = scaled(row[x], sc);
            if (xv > bv) {
                bv = xv;
                bi = x;
            }
        }
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const float ov = __shfl_xor(bv, off);
            const int oi = __shfl_xor(bi, off);
            if (ov > bv || (ov == bv && oi < bi)) {
                bv = ov;
                bi = oi;
            }
        }
        return bi == INT_MAX ? 0 : bi;
    }
    const uint64_t T = exact_threshold(u, Z);
    const uint64_t excl = incl - local;
    const unsigned long long hit = __ballot(excl <= T && T < incl);
    if (hit == 0ull) return v - 1;  // only if the sums wrapped (rows longer than allowed)
    const int owner = __ffsll(hit) - 1;
    int cs = ca;
    uint64_t base_sum = excl;
    if (lane == owner) {
        uint64_t run = excl;
        for (int c = ca; c < cb; ++c) {
            const uint64_t nx = run + (c == ct ? sh_part[c] - before + adj : sh_part[c]);
            if (nx > T) break;
            cs = c + 1;
            base_sum = nx;
            run = nx;
        }
    }
    cs = __builtin_amdgcn_readlane(cs, owner);
    base_sum = lane_value(base_sum, owner);
    // the crossing chunk: lane holds elements cs*1024 + lane*16 + [0, 16)
    const int x0 = cs * kChunk + lane * 16;
    uint32_t w[8];
    load16(row, x0, v, w);
    uint64_t qv[16];
    lane_weights(tab, w, x0, v, sc, b31, qv);
    uint64_t sum = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (x0 + k == t) qv[k] = adj;
        sum += qv[k];
    }
    const uint64_t lincl = wave_inclusive_scan(sum) + base_sum;
    const uint64_t lexcl = lincl - sum;
    const unsigned long long lhit = __ballot(lexcl <= T && T < lincl);
    if (lhit == 0ull) return v - 1;
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

// The acceptance scan with normalisers, by one wave: the first rejected position (M after full
// acceptance) and its L, t, q, P and logit (the bonus row's L), one gathered logit per position.
struct LseScan {
    int r, t, x;
    float L, q, P;
};

__device__ __forceinline__ LseScan lse_scan(const LogitsArgs &a, int b, int t0, int M, float cb, int lane) {
    const int v = a.v_t;
    const float L_bonus = a.lse[t0 + b + M];
    int gamma = M, t_r = -1, x_r = 0;
    float L_r = L_bonus, q_r = 0.0f, P_r = 0.0f;
    for (int base = 0; base < M && gamma == M; base += kWave) {
        const int j = base + lane;
        bool rej = false;
        int tj = 0, xj = 0;
        float Lj = 0.0f, qj = 0.0f, P = 0.0f;
        if (j < M) {
            const int64_t r = t0 + b + j;
            tj = a.target_ids[t0 + j];
            Lj = a.lse[r];
            qj = a.q[t0 + j];
            if (tj >= 0 && tj < v) {
                xj = a.logits[r * a.ld + tj];
                P = fminf(fmaxf(weight_at(expo(xj, cb, 31.0f - Lj * kLog2e)), 0.0f), 1.0f);
                rej = !(qj <= 0.0f || a.u_accept[t0 + j] < P / qj);
            }
        }
        const unsigned long long rm = __ballot(rej);
        if (rm != 0ull) {
            const int src = __ffsll(rm) - 1;
            gamma = base + src;
            t_r = __builtin_amdgcn_readlane(tj, src);
            x_r = __builtin_amdgcn_readlane(xj, src);
            L_r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Lj), src));
            q_r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(qj), src));
            P_r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(P), src));
        }
    }
    return LseScan{gamma, t_r, x_r, L_r, q_r, P_r};
}

// the residual entry at the rejected proposal: it loses q of its mass, clamped
__device__ __forceinline__ uint64_t lse_residual(const LseScan &rec) {
    return q31(fminf(fmaxf(rec.P - rec.q, 0.0f), 1.0f));
}

// ------------------------------------------------------------------ screening (no normalisers)
// Without normalisers a row's S needs the row's mu first (two passes) and row j + 1 matters only
// once row j accepted, so one workgroup per stream spends (gamma + 1) row walks of about 20 us
// in series while the streams that stopped leave their compute units idle: 256 streams of
// 151,936 logits, mean gamma about 1.1, 180-230 us.  Instead the rows are screened first, many
// at once: one pass over a row gives its exact largest logit and an fp32 sum of 2^(y - max);
// wherever the acceptance test holds with a relative margin kMargin the position is
// accepted for certain, and the exact walk starts at the first position that is not (about one
// row per stream).  Rows go in rounds: round r screens a window of positions of the streams
// that every earlier window accepted whole, each window three times as long as the one before, so a
// few launches cover any number of positions and little is read that no test needs.  The same
// batch takes 84 us (rounds of 18, 22 and 11 us, 5 between, the walk 22).  Where half of the tests accept, 4 to 16
// positions a stream, against one workgroup per stream: 64 streams 44 against 118, 8 streams 22 against 51; of 32,000
// logits 64 streams 26 against 59, 512 70 against 89; of 4,000 logits 256 streams 24 against 47.
//
// The margin: P = E / S and its estimate e / s differ (relative, |mu| < 512, q < 2^60) by
//   3.2e-5  exponents of the exact weights held at 31 (mu rounded by at most 2^-16, 31 - mu by
//           2^-15; a shift common to a row's weights cancels in E / S)
//   5.4e-6  the polynomial of the exact weights, in E and in S (below 2.7e-6 each)
//   2.7e-6  roundings of the exponents of both sides (2^-20 each where a weight counts)
//   6.2e-5  a lane's running sum: up to 256 chunks (2^23 logits in at least 8 splits of four waves), each
//           may raise the largest y and rescale the sum (hardware exponential 2^-23, product and
//           sum 2^-24 each), and the sum of its 16 terms
//   3.8e-6  lanes, waves and up to 32 splits combined
//   0.5e-6  S, the quotients and the products of the test
// below 1.1e-4 in all; the truncation of the exact weights only lowers S (a larger P), and weights too
// small for these figures only raise s (a smaller estimate).
constexpr int kScreenThreads = 256;
constexpr int kScreenWaves = kScreenThreads / kWave;
constexpr float kMargin = 2e-4f;
constexpr float kLowest = -3e38f;  // below every scaled logit that counts
constexpr int kScreenRows = 64;    // positions screened at most; the exact walk goes on from there
// Streams of a screened batch at most: 1,024 streams of 32,000 to 64,000 logits gain nothing (0.8 to 1.06 times the
// speed of the one kernel at any acceptance), 512 gain 1.1 to 1.3 times.
constexpr int kScreenStreams = 512;
// The first round's window: the positions whose rows make kWindowBytes, from about a row per compute
// unit to kWindowRows.  A round costs about 8 us with its tests, which is what 40 MB take, so short rows go
// in one round (256 streams of 4,000 logits, up to 8 positions: 25 us at any acceptance, 33 in three);
// past 2,048 rows a batch that stops at once pays for rows that none of it needs.  Each later window is three
// times as long; the fourth takes all that is left (few streams get there).
constexpr int64_t kWindowBytes = int64_t(20) << 20;
constexpr int kWindowRows = 2048;
constexpr int kMaxRounds = 4;

struct Window {
    int a, b;  // positions [a, b)
};

struct ScreenParams {
    LogitsArgs a;
    int32_t nc, rows, splits, cps;  // rows: positions with partials; cps: chunks of a split
    int32_t sum_splits, sum_cps;    // the exact sums' split (logits_sums)
    int32_t n_rounds;
    Window win[kMaxRounds];
    int32_t *from;     // [n] position the exact walk starts at (after logits_advance; the last window's
                       // start while undecided)
    int32_t *alive;    // [kMaxRounds][1 + n] count and streams of each round from the second on
    float2 *part;      // [n][rows][splits] largest y and sum of 2^(y - largest)
    uint64_t *sums;    // [n][nc] chunk sums of the selected row
    LseScan *rec;      // [n] the scan's result (normalisers)
};

struct Screened {
    int j;      // position the exact walk starts at
    int known;  // its mu is known
    float mu;
};

// The largest y and the sum of 2^(y - largest) of row j of stream b, from its splits.
__device__ __forceinline__ float2 screen_combine(const ScreenParams &p, int b, int j) {
    const float2 *q = p.part + ((int64_t)b * p.rows + j) * p.splits;
    float m = kLowest, s = 0.0f;
    for (int k0 = 0; k0 < p.splits; k0 += 8) {  // eight loads in flight
        float2 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = q[k0 + k < p.splits ? k0 + k : k0];
        float mn = m;
#pragma unroll
        for (int k = 0; k < 8; ++k) mn = fmaxf(mn, v[k].x);
        s *= __builtin_amdgcn_exp2f(m - mn);
#pragma unroll
        for (int k = 0; k < 8; ++k) s += k0 + k < p.splits ? v[k].y * __builtin_amdgcn_exp2f(v[k].x - mn) : 0.0f;
        m = mn;
    }
    return make_float2(m, s);
}

// Whether position j of stream b is accepted for certain.
__device__ __forceinline__ bool screen_accepts(const ScreenParams &p, int b, int j) {
    const LogitsArgs &a = p.a;
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    if (M > a.max_m || j >= M) return false;
    const int t = a.target_ids[t0 + j];
    const float q = a.q[t0 + j], u = a.u_accept[t0 + j];
    if (t < 0 || t >= a.v_t) return false;
    const uint32_t x = a.logits[(int64_t)(t0 + b + j) * a.ld + t];
    const float2 ms = screen_combine(p, b, j);
    if (q <= 0.0f) return true;
    const float e = __builtin_amdgcn_exp2f(fmaf(bf16_value(x), a.inv_temp[b] * kLog2e, -ms.x));
    // (the exact weight is 0 below 2^-31; NaN, overlarge logits and overlarge q are left to the
    // exact test: here P >= 2^-31 / 2^23, so P / q is a normal number while q < 2^60)
    return e >= 0x1.01p-31f && fabsf(ms.x) < 512.0f && q < 0x1p60f && u * q < e / ms.y * (1.0f - kMargin);
}

// Where the exact walk of stream b starts, by one wave: the last round's window is tested here.
__device__ __forceinline__ Screened screen_result(const ScreenParams &p, int b, int lane) {
    const Window w = p.win[p.n_rounds - 1];
    int j = p.n_rounds > 1 ? p.from[b] : w.a;
    if (j == w.a) {  // every earlier window accepted (a stream that stopped before has j < w.a)
        bool go = true;
        while (go && j < w.b) {
            const bool acc = j + lane < w.b && screen_accepts(p, b, j + lane);
            const uint64_t no = ~__ballot(acc);
            const int f = no != 0 ? __ffsll((unsigned long long)no) - 1 : kWave;
            j += f;
            go = f == kWave;
        }
    }
    Screened r{j, 0, 0.0f};
    if (j < p.rows) {
        r.mu = screen_combine(p, b, j).x;
        r.known = r.mu > kLowest && r.mu < INFINITY && p.a.inv_temp[b] < 1e30f ? 1 : 0;
    }
    return r;
}

// Between rounds: the streams whose window was accepted whole go on (the list of round `round`, in any
// order), the others' positions are final; a wave per stream.  A kernel of its own: done by every workgroup
// of the next round instead, the tests' scattered loads took more than the rows (256 streams, second
// round: 40 us for 270 rows, 17 us without them).
__global__ void __launch_bounds__(kScreenThreads) logits_advance(ScreenParams p, int round) {
    const int lane = threadIdx.x % kWave;
    const int i = blockIdx.x * kScreenWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = p.a.n_streams;
    const Window pw = p.win[round - 1];
    const int32_t *list = p.alive + (int64_t)(round - 1) * (n + 1);
    int32_t *out = p.alive + (int64_t)round * (n + 1);
    if (i >= (round > 1 ? list[0] : n)) return;
    const int b = round > 1 ? list[1 + i] : i;
    const int rows = pw.b - pw.a;  // at most kScreenRows = kWave
    const uint64_t no = ~__ballot(lane < rows && screen_accepts(p, b, pw.a + lane));
    const int f = no != 0 ? __ffsll((unsigned long long)no) - 1 : kWave;
    if (lane == 0) {
        p.from[b] = pw.a + (f < rows ? f : rows);
        if (f >= rows) out[1 + atomicAdd(out, 1)] = b;
    }
}

// One round: the splits of the window's rows of the streams still undecided, a workgroup each.
__global__ void __launch_bounds__(kScreenThreads) logits_screen(ScreenParams p, int round) {
    const LogitsArgs &a = p.a;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    __shared__ float2 sh_ms[kScreenWaves];
    const Window w = p.win[round];
    const int rows = w.b - w.a;
    const int32_t *list = p.alive + (int64_t)round * (a.n_streams + 1);
    const int n_alive = round > 0 ? list[0] : a.n_streams;
    const int items = n_alive * rows * p.splits;
    if (round + 1 < p.n_rounds && blockIdx.x == 0 && tid == 0) p.alive[(int64_t)(round + 1) * (a.n_streams + 1)] = 0;
    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        const int sp = item % p.splits, row_item = item / p.splits;
        const int i = row_item / rows, j = w.a + row_item % rows;
        const int b = round > 0 ? list[1 + i] : i;
        const int t0 = a.target_off[b];
        const int M = a.target_off[b + 1] - t0;
        if (M > a.max_m || j > M) continue;  // (M < 0: j > M)
        const float c = a.inv_temp[b] * kLog2e;
        const uint16_t *row = a.logits + (int64_t)(t0 + b + j) * a.ld;
        const int c1 = (sp + 1) * p.cps < p.nc ? (sp + 1) * p.cps : p.nc;
        float m = kLowest, s = 0.0f;
        int ck = sp * p.cps + wave;
        uint32_t wd[8] = {}, nx[8] = {};
        if (ck < c1) load16s<false>(row, ck, lane, a.v_t, wd);
        for (; ck < c1; ck += kScreenWaves) {
            if (ck + kScreenWaves < c1) load16s<false>(row, ck + kScreenWaves, lane, a.v_t, nx);
            float x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = bf16_value(elem(wd, k));
            if ((ck + 1) * kChunk > a.v_t) {  // the row's ragged end
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (elem_index_s(ck, lane, k) >= a.v_t) x[k] = -INFINITY;
            }
            float mx = x[0];
#pragma unroll
            for (int k = 1; k < 16; ++k) mx = fmaxf(mx, x[k]);
            const float mn = fmaxf(m, mx * c);  // scaling by c > 0 keeps the order: the largest y
            float t = 0.0f;
#pragma unroll
            for (int k = 0; k < 16; ++k) t += __builtin_amdgcn_exp2f(fmaf(x[k], c, -mn));
            s = s * __builtin_amdgcn_exp2f(m - mn) + t;
            m = mn;
#pragma unroll
            for (int k = 0; k < 8; ++k) wd[k] = nx[k];
        }
        float wm = m;
        for (int off = kWave / 2; off > 0; off >>= 1) wm = fmaxf(wm, __shfl_xor(wm, off));
        float ws = s * __builtin_amdgcn_exp2f(m - wm);
        for (int off = kWave / 2; off > 0; off >>= 1) ws += __shfl_xor(ws, off);
        if (lane == 0) sh_ms[wave] = make_float2(wm, ws);
        __syncthreads();
        if (tid == 0) {
            float bm = sh_ms[0].x, bs = 0.0f;
            for (int k = 1; k < kScreenWaves; ++k) bm = fmaxf(bm, sh_ms[k].x);
            for (int k = 0; k < kScreenWaves; ++k) bs += sh_ms[k].y * __builtin_amdgcn_exp2f(sh_ms[k].x - bm);
            p.part[((int64_t)b * p.rows + j) * p.splits + sp] = make_float2(bm, bs);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ exact sums over many workgroups
// Fewer streams than compute units: the chunk sums of every stream's selected row by sum_splits
// workgroups each (with normalisers after the acceptance scan, else of the position the screen
// stopped at), the sampling in a second kernel.  A workgroup takes a few chunks, so the
// weights come from the formula: a table would cost more than it saves.
template <bool LSE>
__global__ void __launch_bounds__(kScreenThreads) logits_sums(ScreenParams p) {
    const LogitsArgs &a = p.a;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int b = blockIdx.x / p.sum_splits, sp = blockIdx.x % p.sum_splits;
    __shared__ LseScan sh_rec;
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    const float it = a.inv_temp[b];
    const float cb = it * kLog2e;
    if (!(M >= 0 && M <= a.max_m && it > 0.0f)) return;  // the sampling kernel writes the sentinels
    if (wave == 0) {
        LseScan rec;
        if (LSE) {
            rec = lse_scan(a, b, t0, M, cb, lane);
            if (sp == 0 && lane == 0) p.rec[b] = rec;
        } else {
            const Screened scr = screen_result(p, b, lane);
            rec.r = scr.known ? scr.j : -1;
            rec.L = scr.mu;
        }
        if (lane == 0) sh_rec = rec;
    }
    __syncthreads();
    const int r = sh_rec.r;
    if (r < 0) return;  // left to the walk
    const float b31 = 31.0f - (LSE ? sh_rec.L * kLog2e : sh_rec.L);
    const uint16_t *row = a.logits + (int64_t)(t0 + b + r) * a.ld;
    const int c1 = (sp + 1) * p.sum_cps < p.nc ? (sp + 1) * p.sum_cps : p.nc;
    for (int c = sp * p.sum_cps + wave; c < c1; c += kScreenWaves) {
        uint32_t w[8];
        load16s<true>(row, c, lane, a.v_t, w);
        uint64_t acc = 0;
        if ((c + 1) * kChunk <= a.v_t) {
#pragma unroll
            for (int k = 0; k < 16; ++k) acc += e31_at(expo(elem(w, k), cb, b31));
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (elem_index_s(c, lane, k) < a.v_t) acc += e31_at(expo(elem(w, k), cb, b31));
        }
        acc = chunk_total(acc);
        if (lane == kWave - 1) p.sums[(int64_t)b * p.nc + c] = acc;
    }
}

// With normalisers: one wave per stream samples from logits_sums' chunk sums.
__global__ void __launch_bounds__(kWave) logits_sample(ScreenParams p) {
    const LogitsArgs &a = p.a;
    const int b = blockIdx.x, lane = threadIdx.x;
    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    const float it = a.inv_temp[b];
    const float cb = it * kLog2e;
    bool ok = M >= 0 && M <= a.max_m && it > 0.0f;
    for (int base = 0; ok && base < M; base += kWave) {
        const int j = base + lane;
        ok = !__any(j < M && (a.target_ids[t0 + j] < 0 || a.target_ids[t0 + j] >= a.v_t));
    }
    int r = -1, token = -1;
    if (ok) {
        const LseScan rec = p.rec[b];
        const float b31 = 31.0f - rec.L * kLog2e;
        const uint16_t *row = a.logits + (int64_t)(t0 + b + rec.r) * a.ld;
        uint64_t adj = 0, before = 0;
        if (rec.r < M) {
            adj = lse_residual(rec);
            before = e31_at(expo((uint32_t)rec.x, cb, b31));
        }
        r = rec.r;
        token = sample_row(row, a.v_t, p.nc, cb, b31, nullptr, rec.t, adj, before, a.u_sample[b], p.sums + (int64_t)b * p.nc);
    }
    if (lane == 0) {
        a.n_accepted[b] = r;
        a.out_token[b] = token;
    }
}

// ------------------------------------------------------------------ one workgroup per stream
// kWalk: all rows here.  kFrom: without normalisers, the walk starts where the screen stopped.
// kSums: as kFrom, and that position's chunk sums are in p.sums.
enum { kWalk, kFrom, kSums };

template <int MODE>
__global__ void __launch_bounds__(kThreads) verify_logits_row(ScreenParams p) {
    const LogitsArgs &a = p.a;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    extern __shared__ uint64_t sh_part[];  // nc chunk sums of e31
    __shared__ float sh_red[kWaves];
    __shared__ int sh_ok;
    __shared__ float sh_m;
    __shared__ LseScan sh_rec;
    __shared__ Screened sh_scr;
    __shared__ int sh_next;  // 1: accepted, go to the next row
    __shared__ uint64_t sh_before, sh_adj;
    __shared__ int sh_t;
    __shared__ int sh_ctr;  // the row pass's chunk counter
    __shared__ uint64_t sh_tab[kTabSlots];  // the row's weight table

    const int t0 = a.target_off[b];
    const int M = a.target_off[b + 1] - t0;
    const float it = a.inv_temp[b];
    const float cb = it * kLog2e;  // the stream's base-2 scale
    const int v = a.v_t, nc = p.nc;
    TT_STAMP(0);
    if (!(M >= 0 && M <= a.max_m && it > 0.0f)) {
        if (tid == 0) {
            a.n_accepted[b] = -1;
            a.out_token[b] = -1;
        }
        return;
    }
    if (wave == kWaves - 1) {  // every proposal's id inside the vocabulary (beside wave 0's scan)
        bool ok = true;
        for (int base = 0; ok && base < M; base += kWave) {
            const int j = base + lane;
            const bool bad = j < M && (a.target_ids[t0 + j] < 0 || a.target_ids[t0 + j] >= v);
            ok = !__any(bad);
        }
        if (lane == 0) sh_ok = ok ? 1 : 0;
    }
    if (MODE != kWalk && wave == 0) {
        const Screened scr = screen_result(p, b, lane);
        if (lane == 0) sh_scr = scr;
    }
    if (MODE == kWalk && a.lse != nullptr) {
        // normalisers given: the acceptance test from one gathered logit per position, then
        // one pass over the residual (or bonus) row
        // (the rejecting lane's L, t, q, P and logit, or the bonus row's L, go to LDS with
        // gamma, so the row pass and the residual entry need no further dependent load; an id
        // outside the vocabulary is not gathered, and the stream then ends as a sentinel)
        if (wave == 0) {
            const LseScan rec = lse_scan(a, b, t0, M, cb, lane);
            if (lane == 0) {
                sh_ctr = kWaves;
                sh_rec = rec;
            }
        }
        __syncthreads();
        TT_STAMP(1);
        if (!sh_ok) {
            if (tid == 0) {
                a.n_accepted[b] = -1;
                a.out_token[b] = -1;
            }
            return;
        }
        const LseScan rec = sh_rec;
        const int r = rec.r;
        const uint16_t *row = a.logits + (int64_t)(t0 + b + r) * a.ld;
        const float b31 = 31.0f - rec.L * kLog2e;
        chunk_sums(row, v, nc, cb, b31, sh_tab, sh_part, &sh_ctr);
        if (wave < 12) TT_STAMP_WAVE(4 + wave);
        __syncthreads();
        TT_STAMP(2);
        if (wave != 0) return;
        int t = -1;
        uint64_t adj = 0, before = 0;
        if (r < M) {  // the rejected proposal loses q_r of its mass: its entry is E(t) - q_r, clamped
            t = rec.t;
            adj = lse_residual(rec);
            before = e31_at(expo((uint32_t)rec.x, cb, b31));  // the weight the chunk sums counted at t
        }
        const int token = sample_row(row, v, nc, cb, b31, sh_tab, t, adj, before, a.u_sample[b], sh_part);
        if (lane == 0) {
            a.n_accepted[b] = r;
            a.out_token[b] = token;
        }
        TT_STAMP(3);
        return;
    }
    __syncthreads();
    if (!sh_ok) {
        if (tid == 0) {
            a.n_accepted[b] = -1;
            a.out_token[b] = -1;
        }
        return;
    }
    int j = 0;
    bool known = false;  // this row's mu (kSums: and chunk sums) are there already
    if (MODE != kWalk) {
        j = sh_scr.j;
        known = sh_scr.known != 0;
    }
    for (; j <= M; ++j, known = false) {
        const uint16_t *row = a.logits + (int64_t)(t0 + b + j) * a.ld;
        const uint64_t *tab = sh_tab;
        // pass 1: the row's largest y
        float m = -INFINITY;
        if (known) {
            m = sh_scr.mu;
            if (tid == 0) sh_ctr = kWaves;
            if (MODE == kSums) {
                for (int c = tid; c < nc; c += kThreads) sh_part[c] = p.sums[(int64_t)b * nc + c];
                tab = nullptr;
            }
            __syncthreads();
        } else {
            uint32_t w[8] = {}, nx[8] = {};
            if (wave < nc) load16s<false>(row, wave, lane, v, w);
            for (int c = wave; c < nc; c += kWaves) {
                if (c + kWaves < nc) load16s<false>(row, c + kWaves, lane, v, nx);
                if ((c + 1) * kChunk <= v) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) m = fmaxf(m, scaled(elem(w, k), cb));
                } else {
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        if (elem_index_s(c, lane, k) < v) m = fmaxf(m, scaled(elem(w, k), cb));
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) w[k] = nx[k];
            }
            for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
            if (lane == 0) sh_red[wave] = m;
            __syncthreads();
            if (tid == 0) {
                float mm = -INFINITY;
                for (int k = 0; k < kWaves; ++k) mm = fmaxf(mm, sh_red[k]);
                sh_m = mm;
                sh_ctr = kWaves;
            }
            __syncthreads();
            m = sh_m;
        }
        // pass 2: chunk sums of e31
        const float b31 = 31.0f - m;
        if (MODE != kSums || !known) chunk_sums(row, v, nc, cb, b31, sh_tab, sh_part, &sh_ctr);
        __syncthreads();
        // S, the acceptance test of position j, and the residual's entry at t_j
        if (wave == 0) {
            uint64_t local = 0;
            for (int c = lane; c < nc; c += kWave) local += sh_part[c];
            const uint64_t Sq = lane_value(wave_inclusive_scan(local), kWave - 1);
            if (lane == 0) {
                const float S = q31_to_f32(Sq);
                int next = 0;
                uint64_t before = 0, adj = 0;
                int t = -1;
                if (j < M) {
                    t = a.target_ids[t0 + j];
                    const float qj = a.q[t0 + j];
                    const float et = weight_at(expo(row[t], cb, b31));
                    const float P = et / S;
                    if (qj <= 0.0f || a.u_accept[t0 + j] < P / qj) {
                        next = 1;
                    } else {
                        const float rt = fminf(fmaxf(et - qj * S, 0.0f), 1.0f);  // NaN -> 0
                        before = e31_at(expo(row[t], cb, b31));
                        adj = q31(rt);
                    }
                }
                sh_next = next;
                sh_before = before;
                sh_t = next ? -1 : t;
                sh_adj = adj;
            }
        }
        __syncthreads();
        if (sh_next) continue;
        if (wave == 0) {
            const int token = sample_row(row, v, nc, cb, b31, tab, sh_t, sh_adj, sh_before, a.u_sample[b], sh_part);
            if (lane == 0) {
                a.n_accepted[b] = j;
                a.out_token[b] = token;
            }
        }
        return;
    }
}

}  // namespace

namespace {

constexpr int kCus = 256;
constexpr int kSumGrid = 1024;     // workgroups of logits_sums to aim for
constexpr int kScreenGrid = 2048;  // workgroups of a screening round
// With normalisers, the row split over workgroups and sampled by a second kernel: for rows long enough
// to pay for that launch, longer the more streams there are to fill the chip without it.  Three sets of buffers in
// turn: 32 streams of 151,936 logits 11.5 us against 18.1 in one kernel, of 32,768 8.9 against 9.4; 64 of 28,672 9.4
// against 9.4, of 64,000 10.3 against 12.3; 100 of 57,344 11.5 against 11.2, of 64,000 11.9 against 12.4; 128 of 40,960
// 11.5 against 10.3, of 81,920 13.6 against 13.4, of 100,000 15.1 against 15.1, of 151,936 17.8 against 19.0; 200 of
// 151,936 22.9 against 20.9.  32 of 16,000 10.2 against 9.6.
constexpr int kLseSplitStreams = 128;
constexpr int kLseSplitChunks = 28;
constexpr int kLseSplitPerStream = 36;  // chunks and this at least the number of streams

// Which kernels a call takes (with a workspace).
enum Route { kRowRoute, kLseSplit, kScreenRow, kScreenSplit };

Route route(const LogitsArgs &a, int nc) {
    if (a.lse != nullptr)
        return a.n_streams <= kLseSplitStreams && nc >= kLseSplitChunks && nc + kLseSplitPerStream >= a.n_streams ? kLseSplit
                                                                                                                  : kRowRoute;
    // Speed against the one kernel where half of the tests accept.  One test a stream: two kernels more cost what
    // the second row's walk takes, so only few streams of long rows gain (64 streams of 32,000 logits 1.17 times; of
    // 4,000 below 0.95, 200 of 32,000 0.73).  Two tests: not while rows of middling length fill the chip (200 streams of
    // 32,000 to 64,000 logits 0.84 to 0.95; of 4,000 1.09, of 151,936 1.05).  From three on 1.0 to 4 times, but
    // few streams gain or lose by their luck (one stream 0.64 to 3.6).  A batch that rejects every first proposal loses with any
    // number (0.4 to 0.75 times; 8 streams of 151,936 logits 1.0): a caller that knows gives no workspace.
    const bool screened = a.n_streams <= kScreenStreams &&
                          (a.max_m >= 3 || (a.max_m == 2 && (a.n_streams <= 128 || nc <= 8 || nc >= 128)) ||
                           (a.max_m == 1 && a.n_streams <= 64 && nc >= 16));
    if (!screened) return kRowRoute;
    return a.n_streams < kCus ? kScreenSplit : kScreenRow;
}

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// The parameters and workspace layout of a call; returns the bytes.
size_t layout(ScreenParams &p, Route rt, uint8_t *ws) {
    const LogitsArgs &a = p.a;
    const size_t n = a.n_streams > 0 ? (size_t)a.n_streams : 0;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const uintptr_t at = reinterpret_cast<uintptr_t>(ws) + off;  // (ws is null in a size query)
        off = align256(off + bytes);
        return at;
    };
    p.nc = (a.v_t + kChunk - 1) / kChunk;
    p.n_rounds = 0;
    if (rt == kRowRoute) return 0;
    if (rt == kScreenRow || rt == kScreenSplit) {
        const int last = a.max_m + 1 < kScreenRows ? a.max_m + 1 : kScreenRows;  // rows 0 .. M, the bonus row among them
        int64_t rows = kWindowBytes / (2 * (int64_t)a.v_t);
        rows = rows < kCus ? kCus : rows > kWindowRows ? kWindowRows : rows;
        int len = rows < a.n_streams ? 1 : (int)(rows / a.n_streams);
        for (int at = 0; at < last;) {
            int b = at + len;
            if (last - b <= len / 2 || p.n_rounds == kMaxRounds - 1) b = last;  // (half a window or less goes along)
            p.win[p.n_rounds++] = Window{at, b};
            at = b;
            len *= 3;
        }
        p.rows = last;
        int splits = kScreenGrid / (a.n_streams * (p.win[0].b - p.win[0].a));
        splits = splits < 8 ? 8 : splits > 32 ? 32 : splits;
        const int most = (p.nc + kScreenWaves - 1) / kScreenWaves;
        if (splits > most) splits = most;
        p.cps = (p.nc + splits - 1) / splits;
        p.splits = (p.nc + p.cps - 1) / p.cps;
        p.from = reinterpret_cast<int32_t *>(take(4 * n));
        p.alive = reinterpret_cast<int32_t *>(take(4 * (n + 1) * kMaxRounds));
        p.part = reinterpret_cast<float2 *>(take(8 * n * p.rows * p.splits));
    }
    if (rt == kLseSplit || rt == kScreenSplit) {
        int splits = (kSumGrid + a.n_streams - 1) / (a.n_streams > 0 ? a.n_streams : 1);
        const int most = (p.nc + kScreenWaves - 1) / kScreenWaves;
        if (splits > most) splits = most;
        p.sum_cps = (p.nc + splits - 1) / splits;
        p.sum_splits = (p.nc + p.sum_cps - 1) / p.sum_cps;
        p.sums = reinterpret_cast<uint64_t *>(take(8 * n * p.nc));
        p.rec = reinterpret_cast<LseScan *>(take(sizeof(LseScan) * n));
    }
    return off;
}

template <int MODE>
int launch_row(const ScreenParams &p, hipStream_t stream) {
    // the chunk sums (up to 64 KiB at the longest rows) sit beside the 64 KiB weight table in LDS
    const size_t lds = 8 * (size_t)p.nc;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&verify_logits_row<MODE>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return TT_ELAUNCH;
    hipLaunchKernelGGL(verify_logits_row<MODE>, dim3(p.a.n_streams), dim3(kThreads), lds, stream, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_ELAUNCH;
}

}  // namespace

size_t logits_workspace_bytes(const LogitsArgs &a) {
    if (a.n_streams == 0) return 0;
    ScreenParams p{};
    p.a = a;
    return layout(p, route(a, (a.v_t + kChunk - 1) / kChunk), nullptr);
}

int launch_verify_logits(const LogitsArgs &a, void *workspace, size_t workspace_bytes, hipStream_t stream) {
    if (a.n_streams == 0) return TT_OK;
    ScreenParams p{};
    p.a = a;
    Route rt = workspace == nullptr ? kRowRoute : route(a, (a.v_t + kChunk - 1) / kChunk);
    if (layout(p, rt, static_cast<uint8_t *>(workspace)) > workspace_bytes) return TT_EWORKSPACE;
    for (int r = 0; r < p.n_rounds; ++r) {
        const int items = a.n_streams * (p.win[r].b - p.win[r].a) * p.splits;
        if (r > 0)
            hipLaunchKernelGGL(logits_advance, dim3((a.n_streams + kScreenWaves - 1) / kScreenWaves), dim3(kScreenThreads), 0,
                               stream, p, r);
        hipLaunchKernelGGL(logits_screen, dim3(items < kScreenGrid ? items : kScreenGrid), dim3(kScreenThreads), 0, stream, p, r);
        if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
    }
    if (rt == kScreenRow) return launch_row<kFrom>(p, stream);
    if (rt == kRowRoute) return launch_row<kWalk>(p, stream);
    const dim3 grid(a.n_streams * p.sum_splits);
    if (rt == kScreenSplit) {
        hipLaunchKernelGGL(logits_sums<false>, grid, dim3(kScreenThreads), 0, stream, p);
        if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
        return launch_row<kSums>(p, stream);
    }
    hipLaunchKernelGGL(logits_sums<true>, grid, dim3(kScreenThreads), 0, stream, p);
    if (hipGetLastError() != hipSuccess) return TT_ELAUNCH;
    hipLaunchKernelGGL(logits_sample, dim3(a.n_streams), dim3(kWave), 0, stream, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_ELAUNCH;
}

}  // namespace tt
