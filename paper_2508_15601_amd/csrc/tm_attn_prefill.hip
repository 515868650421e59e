// Prompt attention over the quantised KV cache: a chunk of query tokens, causal (paper Sec. 3.3: the attention pipeline's
// prefill side; Sec. 4.3 conversion between the matrix instructions, Sec. 4.4 loading pipeline).
//
// A prompt multiplies every cached key and value with hundreds of query rows, so unlike at a decoding step the matrix cores
// and the softmax arithmetic bound the kernel, not the cache's bytes.  The split of the work follows from that:
//   - A CTA is eight waves over up to 256 query rows of one KV head.  A row is a (token, query head) pair and rows are
//     numbered token by token, so that any group size fills the tiles; a wave owns 32 rows.
//   - The codes are converted ONCE per CTA: all waves turn a stage of 64 tokens into fp16 values q - z (exact) in LDS, in
//     the order in which the 32x32x16 matrix instruction takes its operands (fragment by fragment, lane by lane: reads and
//     writes are conflict-free without padding), one stage ahead of the multiplication.  The 16-column kernel of the decoding
//     step converts per 16 rows and spends more instructions on that than on the softmax.
//   - Scores are computed transposed (S^T = K Q^T).  The rows of the K operand are the stage's tokens in the order
//     0-7, 16-23, 8-15, 24-31, so that the result layout hands a lane the probabilities of exactly the tokens whose values it
//     multiplies as the k-index of O^T = V^T P^T: P never leaves its registers.
//   - Per score the vector ALU does: one multiply-add (the key's scale, minus the running reference), half a maximum, one
//     exponential, one addition (denominator), one multiply-and-round (the value's scale).  The reference moves only when a
//     score exceeds it by 2^kSlack, which makes the rescaling of the 64 output registers rare; probabilities up to 2^kSlack
//     times a scale still fit fp16.
//   - The scores of the next 32 tokens are computed while the exponentials of the current ones are, the products with V while
//     the next scores are scaled: each half of a step has matrix work and independent vector work.
// With fewer rows two groups of four waves (RW = 4, 128 rows) split the context instead: each takes every second run of 32
// tokens, and they meet in LDS at the end.
//
// Measured (32 query / 8 KV heads, 4000 tokens, 8-bit / 4-bit codes; the 16-column kernel ran this before): 345 -> 152-162 us /
// 289 -> 150 us; 64 / 8 heads, 2048 tokens after 6000, 4-bit: 880 -> 465 us = 1.0 PFLOP/s, half of what an MFMA-only loop sustains
// on this chip.  What bounds it is vector and matrix issue together, and the uneven end of a causal launch: a 32-token run is 16
// MFMAs of 32 clocks and 140-150 vector instructions (conversion included), two waves per SIMD; over the whole launch of 4000 tokens
// the matrix pipe is busy 35-37 % of the clocks, the vector pipes issue in 27 % of the waves' time.  Forced interleaving of the two
// (scheduling groups of one MFMA, seven vector instructions, one LDS read) is 6-9 % slower than the compiler's own order, wave
// priorities change nothing.
#include "tm_w4_host.h"

namespace tmw4 {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kHeadDim = 128;
constexpr float kNegBig = -1.0e30f;     // a masked score: "minus infinity" that stays finite under subtraction
constexpr float kMaskFloor = -1.0e20f;  // lowest reference: exp2(kNegBig - kMaskFloor) is 0

__device__ __forceinline__ f32x16 mfma32x32x16(f16x8 a, f16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32); }

__device__ __forceinline__ f16x8 add_pairs(f16x8 v, f16x2 a, f16x2 b, f16x2 c, f16x2 d)
{
    const f16x2 r0 = f16x2{v[0], v[1]} + a, r1 = f16x2{v[2], v[3]} + b, r2 = f16x2{v[4], v[5]} + c, r3 = f16x2{v[6], v[7]} + d;
    return f16x8{r0.x, r0.y, r1.x, r1.y, r2.x, r2.y, r3.x, r3.y};
}

constexpr int ST = 64;                           // tokens per stage
constexpr int kStageBytes = ST * kHeadDim * 2;   // one stage of keys (or values) in fp16
constexpr int kStagePairs = ST * 10;             // one stage of scales and zero-points
// Keys are read one stage ahead of the barrier that ends it, values after it: two key buffers, three value buffers, and
// four sets of pairs (read from the conversion of a stage to its last product).
constexpr int kLdsBytes = 5 * kStageBytes + 4 * kStagePairs;

template <int BITS, int RW>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_prefill_kernel(
    AttnCache kv, const uint16_t* __restrict__ Q, const int32_t* __restrict__ positions, const int32_t* __restrict__ counts,
    int count, uint16_t* __restrict__ O, int q_heads, float scale_log2e)
{
    constexpr int KS = 8 / RW;                             // wave groups along the context
    constexpr int NB = 2 / KS;                             // 32-token runs per wave and stage
    constexpr int ROWS = 32 * RW;
    constexpr float kSlack = BITS == 8 ? 6.0f : 2.0f;      // 2^6 * (2 * 65504 / 255), 2^2 * (2 * 65504 / 15) < 65504
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* const kbase = smem;
    unsigned char* const vbase = smem + 2 * kStageBytes;
    unsigned char* const pbase = vbase + 3 * kStageBytes;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave % RW, ksg = wave / RW;
    const int hl = lane >> 5;
    const int hk = blockIdx.x, b = blockIdx.y;
    const int tile = (int)gridDim.z - 1 - (int)blockIdx.z;  // the longest rows first
    const int G = q_heads / kv.heads;
    const size_t bh = (size_t)b * kv.heads + hk;

    const int cnt = counts ? min(max(counts[b], 0), count) : count;
    const long pos0 = positions[b];
    const int row0 = tile * ROWS;
    const int tok_first = row0 / G;
    if (tok_first >= cnt || pos0 + tok_first >= kv.cap) return;                     // (uniform) no row to write
    const int len_all = (int)min(max(pos0 + min(cnt, (row0 + ROWS - 1) / G + 1), 0L), (long)kv.cap);
    if (len_all == 0) return;
    const int nst = (len_all + ST - 1) / ST;

    // this wave's rows, and this lane's
    const int w0 = row0 + rg * 32;
    const int wtok = w0 / G;
    int wlen = (int)min(max(pos0 + min(cnt, (w0 + 31) / G + 1), 0L), (long)kv.cap);   // tokens its longest row attends over
    if (wtok >= cnt) wlen = 0;
    const long wmin = pos0 + wtok + 1;                                              // and its shortest
    const int row = w0 + (lane & 31);
    int tok = row / G;
    const int head = row - tok * G;
    const long pos = pos0 + tok;
    const bool real = tok < cnt && pos >= 0 && pos < kv.cap;
    const int len = real ? (int)pos + 1 : 0;
    if (!real) tok = tok_first;                                                     // an address that exists
    const size_t qrow = (((size_t)b * count + tok) * q_heads + (size_t)hk * G + head) * kHeadDim;

    f16x8 qf[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) qf[t] = *(const f16x8*)(Q + qrow + 16 * t + 8 * hl);

    // ---- staging: codes in registers one stage ahead of their conversion, scale/zero pairs two
    constexpr int kCodeBytes = kHeadDim * BITS / 8;                                 // of one token
    const uint32_t code_end = (uint32_t)(len_all + 31) / 32 * 32 * kCodeBytes;
    const __amdgpu_buffer_rsrc_t krs = make_rsrc(kv.k + bh * kv.cap * kCodeBytes, code_end);
    const __amdgpu_buffer_rsrc_t vrs = make_rsrc(kv.v + bh * kv.cap * kCodeBytes, code_end);
    const __amdgpu_buffer_rsrc_t zrs = make_rsrc(kv.sz + bh * kv.cap * 2, (uint32_t)len_all * 8u);   // zeros past the context
    u32x4 codes[BITS == 8 ? 2 : 1];                                                 // 16-byte chunks of a thread and stage
    u32x2 pairs = {0u, 0u};
    auto load_codes = [&](int st) {
        if constexpr (BITS == 8) {
            codes[0] = __builtin_amdgcn_raw_buffer_load_b128(krs, st * (ST * 128) + tid * 16, 0, 0);
            codes[1] = __builtin_amdgcn_raw_buffer_load_b128(vrs, st * (ST * 128) + tid * 16, 0, 0);
        } else {                                           // half the waves take the keys, half the values
            codes[0] = wave < 4 ? __builtin_amdgcn_raw_buffer_load_b128(krs, st * (ST * 64) + tid * 16, 0, 0)
                                : __builtin_amdgcn_raw_buffer_load_b128(vrs, st * (ST * 64) + (tid - 256) * 16, 0, 0);
        }
    };
    auto load_pairs = [&](int st) {
        if (tid < ST) pairs = __builtin_amdgcn_raw_buffer_load_b64(zrs, (st * ST + tid) * 8, 0, 0);
    };
    // LDS image of a stage's pairs: [ST] K scales times scale * log2(e) in fp32 (in the query's fp16 values the factor's rounding
    // would be a fifth of the result's error), then [ST] V scales, [ST] K zero-points, [ST] V zero-points (fp16).
    // A token that was never stored may hold anything; its scores are masked, and with finite numbers here its values
    // cannot reach a sum (0 * q).
    auto store_pairs = [&](int st) {
        if (tid < ST) {
            unsigned char* const p = pbase + (st & 3) * kStagePairs;
            const f16x2 k = as_f16x2(pairs.x), v = as_f16x2(pairs.y);
            const _Float16 top = BITS == 8 ? (_Float16)255.0f : (_Float16)15.0f, nul = (_Float16)0.0f;
            const _Float16 vs = v.x < (_Float16)65504.0f && v.x > (_Float16)-65504.0f ? v.x : nul;
            const _Float16 kz = __builtin_fminf16(__builtin_fmaxf16(k.y, nul), top);
            const _Float16 vz = __builtin_fminf16(__builtin_fmaxf16(v.y, nul), top);
            ((float*)p)[tid] = (float)k.x * scale_log2e;
            ((_Float16*)(p + ST * 4))[tid] = vs;
            ((_Float16*)(p + ST * 6))[tid] = kz;
            ((_Float16*)(p + ST * 8))[tid] = vz;
        }
    };
    const Magic mg = make_magic();
    // one 16-byte chunk of the cache -> fp16 fragments (32 bytes of 8-bit codes, 64 of 4-bit ones)
    auto convert_k = [&](int id, const u32x4& w, unsigned char* kb, const unsigned char* zk) {
        constexpr int CPB = BITS == 8 ? 256 : 128;                                  // chunks per 32 tokens
        const int blk = id / CPB, chunk = id % CPB;
        const int c = chunk & 15, hh = (chunk >> 4) & 3, j = BITS == 8 ? chunk >> 7 : chunk >> 6;
        const int r = 16 * (c >> 3) + 8 * j + (c & 7);                              // operand row of token 16j + c
        const _Float16 z = ((const _Float16*)zk)[blk * 32 + 16 * j + c];
        const _Float16 a = (_Float16)-1024.0f - z;
        const f16x2 hi = {a, a};
        unsigned char* const dst = kb + blk * 8192 + r * 16;
        if constexpr (BITS == 8) {
            const int t = 2 * hh + ((chunk >> 6) & 1);
            *(f16x8*)(dst + t * 1024) = add_pairs(biased8_w8(w.x, w.y), hi, hi, hi, hi);
            *(f16x8*)(dst + t * 1024 + 512) = add_pairs(biased8_w8(w.z, w.w), hi, hi, hi, hi);
        } else {
            const _Float16 e = (_Float16)-64.0f - z;
            const f16x2 lo = {e, e};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(f16x8*)(dst + (2 * hh + (i >> 1)) * 1024 + (i & 1) * 512) = add_pairs(biased8(w[i], mg), hi, lo, hi, lo);
        }
    };
    auto convert_v = [&](int id, const u32x4& w, unsigned char* vb, const unsigned char* zv) {
        constexpr int CPB = BITS == 8 ? 256 : 128;
        const int blk = id / CPB, chunk = id % CPB;
        const int c = chunk & 15, hh = (chunk >> 4) & 3, ii = chunk >> 6;
        // the chunk's tokens: 4hh .. 4hh + 3 and 16 + 4hh .. 16 + 4hh + 3
        const u32x2 z0 = *(const u32x2*)(zv + (blk * 32 + 4 * hh) * 2), z1 = *(const u32x2*)(zv + (blk * 32 + 16 + 4 * hh) * 2);
        const f16x2 b1024 = {(_Float16)-1024.0f, (_Float16)-1024.0f};
        const f16x2 blo = BITS == 8 ? b1024 : f16x2{(_Float16)-64.0f, (_Float16)-64.0f};
        const f16x2 p0 = b1024 - as_f16x2(z0.x), p1 = blo - as_f16x2(z0.y), p2 = b1024 - as_f16x2(z1.x), p3 = blo - as_f16x2(z1.y);
        unsigned char* const dst = vb + blk * 8192 + (hh >> 1) * 1024 + (hh & 1) * 512 + c * 16;
        if constexpr (BITS == 8) {
            *(f16x8*)(dst + ii * 2048) = add_pairs(biased8_w8(w.x, w.y), p0, p1, p2, p3);
            *(f16x8*)(dst + ii * 2048 + 256) = add_pairs(biased8_w8(w.z, w.w), p0, p1, p2, p3);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(f16x8*)(dst + (2 * ii + (i >> 1)) * 2048 + (i & 1) * 256) = add_pairs(biased8(w[i], mg), p0, p1, p2, p3);
        }
    };
    auto convert_stage = [&](int st) {
        unsigned char* const kb = kbase + (st & 1) * kStageBytes;
        unsigned char* const vb = vbase + (st % 3) * kStageBytes;
        const unsigned char* const zk = pbase + (st & 3) * kStagePairs + ST * 6;
        const unsigned char* const zv = zk + ST * 2;
        if constexpr (BITS == 8) {
            convert_k(tid, codes[0], kb, zk);
            convert_v(tid, codes[1], vb, zv);
        } else if (wave < 4) {
            convert_k(tid, codes[0], kb, zk);
        } else {
            convert_v(tid - 256, codes[0], vb, zv);
        }
    };
    auto barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                          // LDS only: loads stay in flight
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    load_codes(0);
    load_pairs(0);
    store_pairs(0);
    load_pairs(1);
    store_pairs(1);
    load_pairs(2);
    barrier();
    convert_stage(0);
    load_codes(1);

#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[t][e] = real ? qf[t][e] : (_Float16)0.0f;
    barrier();

    f32x16 o[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[d][e] = 0.f;
    float m_run = kMaskFloor, l_run = 0.f;
    f32x16 x;                                              // the current 32 tokens' scores, less the reference
    f32x4 ks[4];                                           // their keys' scales
    u32x2 vs[4];                                           // and their values' (fp16)
    float mx;

    // raw scores of the 32 tokens whose keys start at kb
    auto multiply_k = [&](const unsigned char* kb) -> f32x16 {
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) s = mfma32x32x16(*(const f16x8*)(kb + t * 1024 + lane * 16), qf[t], s);
        return s;
    };
    // scales of the lane's tokens: element i of register g is token {0, 16, 8, 24}[g] + 4 * hl + i of the run
    auto read_scales = [&](const unsigned char* p, int run) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int token = run * 32 + (g & 1) * 16 + (g >> 1) * 8 + 4 * hl;
            ks[g] = *(const f32x4*)(p + token * 4);
            vs[g] = *(const u32x2*)(p + ST * 4 + token * 2);
        }
    };
    // x = s * scale - ref; masked: tokens from the row's length on get kNegBig.  t0: first of the 32 tokens
    auto scale_scores = [&](const f32x16& s, float ref, auto MASKED, int t0) {
        const int rem = len - t0 - 4 * hl;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float v = __builtin_fmaf(s[e], ks[e >> 2][e & 3], -ref);
            x[e] = !decltype(MASKED)::value || ((e >> 2) & 1) * 16 + (e >> 3) * 8 + (e & 3) < rem ? v : kNegBig;
        }
        mx = x[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, x[e]);
    };
    auto first_token = [&](int st, int sub) { return st * ST + (KS > 1 ? ksg : sub) * 32; };

    {
        const int t0 = first_token(0, 0);
        const f32x16 s = multiply_k(kbase + (KS > 1 ? ksg : 0) * 8192);
        read_scales(pbase, KS > 1 ? ksg : 0);
        scale_scores(s, 0.f, std::true_type{}, t0);
        m_run = fmaxf(fmaxf(mx, other_half(mx)), kMaskFloor);
        scale_scores(s, m_run, std::true_type{}, t0);
    }

    for (int st = 0; st < nst; ++st) {
        convert_stage(st + 1);
        store_pairs(st + 2);
        load_codes(st + 2);
        load_pairs(st + 3);
#pragma unroll
        for (int sub = 0; sub < NB; ++sub) {
            const int t0 = first_token(st, sub);
            const int st_n = sub + 1 < NB ? st : st + 1, sub_n = sub + 1 < NB ? sub + 1 : 0;
            if (sub + 1 == NB) barrier();                  // the next stage is in LDS
            if (t0 < wlen) {                               // wave-uniform
                if (__any(mx > kSlack)) {
                    const float up = fmaxf(fmaxf(mx, other_half(mx)), 0.f);
                    const float alpha = __builtin_amdgcn_exp2f(-up);
                    m_run += up;
                    l_run *= alpha;
#pragma unroll
                    for (int e = 0; e < 16; ++e) x[e] -= up;
#pragma unroll
                    for (int d = 0; d < 4; ++d) o[d] *= alpha;
                }
                // the next scores next to the exponentials of these
                const int run_n = KS > 1 ? ksg : sub_n;
                const f32x16 s = multiply_k(kbase + (st_n & 1) * kStageBytes + run_n * 8192);
                f16x8 p[2];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float pe = __builtin_amdgcn_exp2f(x[e]);
                    l_run += pe;
                    const f16x2 two = as_f16x2((e & 2) ? vs[e >> 2].y : vs[e >> 2].x);
                    p[e >> 3][e & 7] = (_Float16)__builtin_fmaf((float)((e & 1) ? two.y : two.x), pe, 0.0f);
                }
                // the products with V next to the scaling of the next scores
                const unsigned char* const vb = vbase + (st % 3) * kStageBytes + (KS > 1 ? ksg : sub) * 8192 + lane * 16;
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int d = 0; d < 4; ++d) o[d] = mfma32x32x16(*(const f16x8*)(vb + (2 * d + k) * 1024), p[k], o[d]);
                read_scales(pbase + (st_n & 3) * kStagePairs, run_n);
                const int t_n = first_token(st_n, sub_n);
                if (t_n + 32 > wmin) scale_scores(s, m_run, std::true_type{}, t_n);
                else scale_scores(s, m_run, std::false_type{}, t_n);
            }
        }
    }

    float l = l_run + other_half(l_run);
    if constexpr (KS > 1) {
        // the second group hands its reference, denominator and rows to the first: [row wave][66][64 lanes]
        float* const part = (float*)smem;
        barrier();
        float* const slot = part + rg * (66 * 64) + lane;
        if (ksg > 0) {
            slot[0] = m_run;
            slot[64] = l;
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e) slot[(2 + 16 * d + e) * 64] = o[d][e];
        }
        barrier();
        if (ksg > 0) return;
        const float M = fmaxf(m_run, slot[0]);
        const float f0 = __builtin_amdgcn_exp2f(m_run - M), f1 = __builtin_amdgcn_exp2f(slot[0] - M);
        l = l * f0 + slot[64] * f1;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[d][e] = o[d][e] * f0 + slot[(2 + 16 * d + e) * 64] * f1;
    }
    if (!real) return;
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    uint16_t* const out = O + qrow + 4 * hl;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            u32x2 w;
            w.x = (uint32_t)f32_to_f16_bits(o[d][4 * g] * inv) | ((uint32_t)f32_to_f16_bits(o[d][4 * g + 1] * inv) << 16);
            w.y = (uint32_t)f32_to_f16_bits(o[d][4 * g + 2] * inv) | ((uint32_t)f32_to_f16_bits(o[d][4 * g + 3] * inv) << 16);
            *(u32x2*)(out + 32 * d + 8 * g) = w;
        }
}

static_assert(4 * 66 * 64 * sizeof(float) <= kLdsBytes, "the merge of the wave groups reuses the stages' LDS");

template <int BITS, int RW>
hipError_t launch(const AttnCache& kv, const uint16_t* Q, const int32_t* positions, const int32_t* counts, int count, uint16_t* O,
                  int q_heads, float scale, hipStream_t stream)
{
    const long rows = (long)count * (q_heads / kv.heads);
    const long tiles = (rows + 32 * RW - 1) / (32 * RW);
    if (kv.heads > 65535 || kv.batch > 65535 || tiles > 65535 || tiles < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((attn_prefill_kernel<BITS, RW>), dim3(kv.heads, kv.batch, (unsigned)tiles), dim3(512), kLdsBytes, stream, kv, Q,
                       positions, counts, count, O, q_heads, scale * 1.4426950408889634f);
    return hipGetLastError();
}

template <int BITS, int RW>
hipError_t allow_lds()
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill_kernel<BITS, RW>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kLdsBytes);
}

}  // namespace

hipError_t attn_prefill_setup()
{
    hipError_t e = allow_lds<8, 8>();
    if (e == hipSuccess) e = allow_lds<8, 4>();
    if (e == hipSuccess) e = allow_lds<4, 8>();
    if (e == hipSuccess) e = allow_lds<4, 4>();
    return e;
}

// Rows per CTA for a chunk of `count` tokens: 256 or 128 here, 0 = the 16-column kernel.  The context is known on the device
// only, so the rule compares what one token of it costs in each form: rounds of CTAs (512 of the 16-column form fit the
// chip, 256 of these) times the time of a round relative to a round of 16-column CTAs.  What the host does know is the
// capacity.  Where that is little more than the chunk, the CTAs of a launch attend over anything between nothing and all of it:
// further rounds fill up evenly, but a launch of one round lasts as long as its longest CTA, up to twice the average (less in
// short chunks, where fixed costs count).  Where the capacity is much larger the CTAs are taken to be alike and rounds to be whole.
// With 2.4 and 3.85 none of 110 random launches (16 ... 8192 tokens, 0 ... 16384 before them, 1 ... 32 KV heads, batch 1 ... 8, capacity
// one, two or eight times the context) that leave the 16-column form is slower for it; all of them average 1.32 times its speed and that
// of the fastest form of each, the worst is 26 % behind it (profiles/attn_prefill_rule__random_launches.txt).
int attn_prefill_rows(const AttnCache& kv, int count, int q_heads, int num_cu)
{
    const long bh = (long)kv.batch * kv.heads;
    const int group = q_heads / kv.heads, gw = group < 16 ? group : 16;
    const long rows = (long)count * group, groups = (count + 16 / gw - 1) / (16 / gw) * ((group + 15) / 16);
    const double longest = count < kv.cap ? kv.cap / (kv.cap - 0.5 * count) : 2.0;      // over the average, if the cache fills up
    auto rounds = [&](long ctas) {
        if (ctas <= num_cu) return 1.0 + (longest - 1.0) * (count < 1024 ? count / 1024.0 : 1.0);
        const double r = (double)ctas / num_cu, whole = (double)((ctas + num_cu - 1) / num_cu);
        return r + (whole - r) * (2.0 - longest);
    };
    const double t16 = bh * groups > 2 * num_cu ? (double)(bh * groups) / (2 * num_cu) : 1.0;
    const double t128 = 2.4 * rounds(bh * ((rows + 127) / 128));
    const double t256 = 3.85 * rounds(bh * ((rows + 255) / 256));
    if (t16 <= t128 && t16 <= t256) return 0;
    return t128 < t256 ? 128 : 256;
}

hipError_t launch_attn_prefill_rows(int rows, const AttnCache& kv, const uint16_t* Q, const int32_t* positions, const int32_t* counts,
                                    int count, uint16_t* O, int q_heads, float scale, hipStream_t stream)
{
    if (kv.bits == 8)
        return rows == 256 ? launch<8, 8>(kv, Q, positions, counts, count, O, q_heads, scale, stream)
                           : launch<8, 4>(kv, Q, positions, counts, count, O, q_heads, scale, stream);
    return rows == 256 ? launch<4, 8>(kv, Q, positions, counts, count, O, q_heads, scale, stream)
                       : launch<4, 4>(kv, Q, positions, counts, count, O, q_heads, scale, stream);
}

}  // namespace tmw4
