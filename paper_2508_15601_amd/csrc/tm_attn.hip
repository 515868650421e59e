// Decode attention over an 8-bit or 4-bit KV cache (paper Sec. 3.3 attention pipeline; Sec. 4.2, 4.3, 4.4), and the kernel that
// quantises new keys / values into the cache.
//
// What differs from the paper's design, which rearranges Q in shared memory so that a 32-lane fragment load of the
// low-bit K tile lines up with it, and stages K/V tiles through shared memory:
//   - The matrix-core operand layout of gfx950 is an explicit index map, and a dot product does not care in which
//     order its 128 dimensions are visited.  Lane (c, h) of a wave therefore simply takes the 32 consecutive key bytes
//     32h .. 32h+31 of "its" token as the k-values of the four MFMA steps, and the query operand is loaded once in that
//     same order.  That is the whole of the head alignment: no LDS, no shuffle, for any code width.
//   - Scores are computed transposed (S^T = K Q^T, tokens as rows).  The MFMA result layout then hands every lane the
//     probabilities of exactly the tokens whose value bytes it needs as the k-values of O^T = V^T P^T, so P never
//     leaves its registers either; the cache stores V in blocks of 32 tokens in that operand order.
//   - Scale and zero-point are per token, i.e. per row of S^T and per k-index of the second product: they are applied
//     to four scores and eight probabilities per lane and block instead of to 2 x 128 code values per token.  The codes
//     enter the matrix cores as 1024 + q (one byte permute per two codes); the bias of the keys and the zero-points leave
//     through fp32 terms per query head, the bias of the values block by block.
//   - The cache itself is stored in operand order (blocks of 32 tokens x 128 dimensions), the hardware-aware packing of
//     the weights applied to K and V: every load instruction of a wave reads 1 KiB of consecutive bytes (row-major keys
//     had every instruction touch half of sixteen 128-byte rows: 4.1 instead of 5.7 TB/s).
//   - The codes of the next two 32-token blocks are in flight in registers while the current block is multiplied; the
//     blocks' scale/zero words go through a small per-wave LDS ring (direct-to-LDS loads); a CTA's waves take blocks
//     round-robin and meet in LDS at the end; long contexts are split across CTAs and merged by the CTA that arrives last, or,
//     above sixteen pieces, by a second, tiny kernel.
#include "tm_w4_host.h"

namespace tmw4 {

namespace {


constexpr int kHeadDim = 128;
constexpr float kNegBig = -1.0e30f;     // "minus infinity" that stays finite under subtraction
constexpr float kMaskFloor = -1.0e20f;  // far below any score, far above kNegBig: exp2(kNegBig - kMaskFloor) is 0
constexpr int kNonTemporal = 2;         // cache-policy bit of a buffer load: streamed once, do not keep

// 2^x by the hardware instruction alone: arguments here are at most kSlack (a score less a reference that may lag behind the largest
// score by that much; the product with a value's scale still fits fp16, see SoftmaxState), and a result below the smallest
// normal number may flush to zero (the library function spends four more instructions per call on that range).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float xor_max(float v, int mask) { return fmaxf(v, __shfl_xor(v, mask)); }
__device__ __forceinline__ float xor_add(float v, int mask) { return v + __shfl_xor(v, mask); }

// ------------------------------------------------------------------------------------------------ quantise + store
// Minimum and maximum over every row of sixteen lanes, in each of its lanes.
__device__ __forceinline__ void row_min_max(float& mn, float& mx)
{
    auto fold = [&](auto CTRL) {
        constexpr int ctrl = decltype(CTRL)::value;        // row_ror by 8, 4, 2, 1
        const float a = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, mn), ctrl, 0xf, 0xf, true));
        const float b = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, mx), ctrl, 0xf, 0xf, true));
        mn = fminf(mn, a);
        mx = fmaxf(mx, b);
    };
    fold(std::integral_constant<int, 0x128>{});
    fold(std::integral_constant<int, 0x124>{});
    fold(std::integral_constant<int, 0x122>{});
    fold(std::integral_constant<int, 0x121>{});
}

// The same over the wave: rows first, then swaps between rows.
__device__ __forceinline__ void wave_min_max(float& mn, float& mx)
{
    row_min_max(mn, mx);
#if defined(__HIP_DEVICE_COMPILE__)
    auto pair = [](auto r, auto f) { return f(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1])); };
    auto lo = [](float x, float y) { return fminf(x, y); };
    auto hi = [](float x, float y) { return fmaxf(x, y); };
    uint32_t a = __builtin_bit_cast(uint32_t, mn), b = __builtin_bit_cast(uint32_t, mx);
    mn = pair(__builtin_amdgcn_permlane16_swap(a, a, false, false), lo);
    mx = pair(__builtin_amdgcn_permlane16_swap(b, b, false, false), hi);
    a = __builtin_bit_cast(uint32_t, mn), b = __builtin_bit_cast(uint32_t, mx);
    mn = pair(__builtin_amdgcn_permlane32_swap(a, a, false, false), lo);
    mx = pair(__builtin_amdgcn_permlane32_swap(b, b, false, false), hi);
#endif
}

// a / b rounded to nearest, exactly as the division gives it, from the correctly rounded reciprocal of b: a product and one
// correction (Markstein), three instructions where a division is ten.  The tests check it against the division for every mantissa of an
// fp16 value over every one of an fp16 scale, and for every fp32 mantissa over 15 and 255.
__device__ __forceinline__ float quotient(float a, float b, float inv)
{
    const float q = a * inv;
    return __builtin_fmaf(__builtin_fmaf(-q, b, a), inv, q);
}

// Scale and zero-point of a vector from its extremes, and the codes of its values: scale = range / levels rounded to fp16 (1 where
// that is zero or not finite), code = round(x / scale) + zero-point, within the levels.
template <int BITS>
struct Quantiser {
    static constexpr float top = BITS == 8 ? 255.0f : 15.0f;
    _Float16 s16;
    float s, inv, zero;
    bool odd;                              // the scale was replaced by 1 (only then can a value be infinite)

    __device__ __forceinline__ Quantiser(float mn, float mx)
    {
        s16 = (_Float16)quotient(mx - mn, top, 1.0f / top);
        s = (float)s16;
        odd = !(s > 0.0f) || __builtin_isinf(s);
        if (odd) {
            s = 1.0f;
            s16 = (_Float16)1.0f;
        }
        const float r = __builtin_amdgcn_rcpf(s);            // within an ulp; one step makes it the nearest number
        inv = __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);
        zero = fminf(fmaxf(rintf(over_scale(-mn)), 0.0f), top);
    }
    __device__ __forceinline__ float over_scale(float x) const { return odd ? x : quotient(x, s, inv); }
    __device__ __forceinline__ uint32_t code(float x) const { return (uint32_t)fminf(fmaxf(rintf(over_scale(x)) + zero, 0.0f), top); }
    __device__ __forceinline__ uint32_t pair() const
    {
        return (uint32_t)__builtin_bit_cast(unsigned short, s16) | ((uint32_t)__builtin_bit_cast(unsigned short, (_Float16)zero) << 16);
    }
};

// The codes of the lane's two values and the vector's scale / zero word.
template <int BITS>
__device__ __forceinline__ uint32_t quantise_pair(float x0, float x1, uint32_t& q0, uint32_t& q1)
{
    float mn = fminf(x0, x1), mx = fmaxf(x0, x1);
    wave_min_max(mn, mx);
    const Quantiser<BITS> z(mn, mx);
    q0 = z.code(x0);
    q1 = z.code(x1);
    return z.pair();
}

// The block-wise appends: sixteen lanes hold a vector, eight dimensions each.  A thread's four vectors (two tokens, keys then
// values; `it` of vector it) are all requested before the first is used: one round trip to memory instead of four in a row.
// What bounds these kernels is the arithmetic of the codes beside that round trip; with four requests in a row and a division per
// value, 4000 tokens x 8 heads took 10.8 us (8-bit) and 10.2 (4-bit), now 8.0 and 7.2; 100 tokens 5.1, now 3.7.
struct AppendSlot {
    int u;                                 // token of the 32-token block
    bool live;
};
__device__ __forceinline__ AppendSlot append_slot(int it, int u0, int u1)
{
    const int u = (int)(threadIdx.x >> 6) * 8 + (it & 1) * 4 + (int)((threadIdx.x & 63) >> 4);
    return AppendSlot{u, u >= u0 && u < u1};
}
__device__ __forceinline__ void append_request(u32x4 (&raw)[4], const uint16_t* Kn, const uint16_t* Vn, int heads, int h, int b,
                                               int count, long first_token, int u0, int u1)
{
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const AppendSlot a = append_slot(it, u0, u1);
        raw[it] = u32x4{0u, 0u, 0u, 0u};
        if (a.live) {
            const size_t src = (((size_t)b * count + (size_t)(first_token + a.u)) * heads + h) * kHeadDim + 8 * (threadIdx.x & 15);
            raw[it] = *reinterpret_cast<const u32x4*>((it >> 1 ? Vn : Kn) + src);
        }
    }
}
// The codes of the lane's eight values and the vector's scale / zero word.
template <int BITS>
__device__ __forceinline__ uint32_t quantise_row8(const u32x4& raw, uint32_t (&q)[8])
{
    float x[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const f16x2 two = as_f16x2(raw[k]);
        x[2 * k] = (float)two.x;
        x[2 * k + 1] = (float)two.y;
    }
    float mn = x[0], mx = x[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) {
        mn = fminf(mn, x[k]);
        mx = fmaxf(mx, x[k]);
    }
    row_min_max(mn, mx);
    const Quantiser<BITS> z(mn, mx);
#pragma unroll
    for (int k = 0; k < 8; ++k) q[k] = z.code(x[k]);
    return z.pair();
}

// The append of a decoding step (few tokens).  A CTA of two waves per (sequence, new token, KV head): one quantises the
// key, one the value; lane l owns dimensions l and l + 64.  Such a launch is one chain of dependent latencies, so the vector
// is requested together with the sequence's position, not after it.
__global__ __launch_bounds__(128) void kv_append_kernel(AttnCache kv, const uint16_t* __restrict__ Kn,
                                                        const uint16_t* __restrict__ Vn,
                                                        const int32_t* __restrict__ positions, int count)
{
    const int lane = threadIdx.x & 63, which = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = blockIdx.x % kv.heads;
    const int j = (blockIdx.x / kv.heads) % count;
    const int b = blockIdx.x / (kv.heads * count);
    const uint16_t* const x = (which ? Vn : Kn) + (((size_t)b * count + j) * kv.heads + h) * kHeadDim;
    const uint16_t r0 = x[lane], r1 = x[lane + 64];
    const int t = positions[b] + j;
    if (t < 0 || t >= kv.cap) return;                       // CTA-uniform
    const size_t bh = (size_t)b * kv.heads + h;
    uint32_t q0, q1;
    const uint32_t pair = quantise_pair<8>((float)__builtin_bit_cast(_Float16, r0), (float)__builtin_bit_cast(_Float16, r1), q0, q1);
    const int u = t & 31;
    uint8_t* const blk = (which ? kv.v : kv.k) + (bh * (kv.cap / 32) + (t >> 5)) * 4096;
    if (which == 0) {
        // dimension d -> byte ((i*2 + half)*64 + 16*hh + c)*16 + x, i = u/16, c = u%16, hh = d/32, half = (d%32)/16
        const int i = u >> 4, c = u & 15;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int d = lane + 64 * k;
            blk[((i * 2 + ((d & 31) >> 4)) * 64 + 16 * (d >> 5) + c) * 16 + (d & 15)] = (uint8_t)(k ? q1 : q0);
        }
    } else {
        // dimension d = 16*i + c -> byte ((i/2)*64 + 16*hh + c)*16 + (i%2)*8 + e, hh = (u%16)/4, e = u%4 + 4*(u/16)
        const int hh = (u & 15) >> 2, e = (u & 3) + 4 * (u >> 4);
        const int c = lane & 15;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = (lane >> 4) + 4 * k;
            blk[((i >> 1) * 64 + 16 * hh + c) * 16 + (i & 1) * 8 + e] = (uint8_t)(k ? q1 : q0);
        }
    }
    if (lane == 0) kv.sz[(bh * kv.cap + t) * 2 + which] = pair;
}

// Prompt-sized appends: one CTA of 256 threads per (KV head, 32-token block touched, sequence).  Sixteen lanes share a
// token (eight dimensions = one 16-byte load each), so a wave quantises four tokens at a time; codes are assembled in
// LDS in cache order and leave as 16-byte stores: a fully covered block is written as 2 x 4 KiB of consecutive bytes.
// A partly covered block keeps its other tokens: key chunks belong to one token each (stored or skipped), value chunks
// hold eight tokens and are merged bytewise with what the cache holds (calls on one cache are ordered on one stream).
// Same arithmetic, operation for operation, as kv_append_kernel.
__global__ __launch_bounds__(256) void kv_append_block_kernel(AttnCache kv, const uint16_t* __restrict__ Kn,
                                                              const uint16_t* __restrict__ Vn,
                                                              const int32_t* __restrict__ positions, int count)
{
    __shared__ __align__(16) uint8_t lds[2][4096];
    const int h = blockIdx.x, b = blockIdx.z;
    const int pos = positions[b];
    long first = pos < 0 ? 0 : pos, last = (long)pos + count;         // tokens [first, last) of the cache are new
    if (last > kv.cap) last = kv.cap;
    if (first >= last) return;
    const int tb = (int)(first >> 5) + (int)blockIdx.y;                // this CTA's block of 32 tokens
    const long t0 = first > (long)tb * 32 ? first : (long)tb * 32;
    const long t1 = last < (long)(tb + 1) * 32 ? last : (long)(tb + 1) * 32;
    if (t0 >= t1) return;                                              // CTA-uniform
    const int u0 = (int)(t0 - (long)tb * 32), u1 = (int)(t1 - (long)tb * 32);
    const int sub = threadIdx.x & 15;                                  // dimensions 8*sub .. 8*sub + 7
    const size_t bh = (size_t)b * kv.heads + h;
    u32x4 raw[4];
    append_request(raw, Kn, Vn, kv.heads, h, b, count, (long)tb * 32 - pos, u0, u1);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int which = it >> 1;                                     // 0: keys, 1: values
        const AppendSlot a = append_slot(it, u0, u1);
        const int u = a.u;                                             // token of the block
        uint32_t q[8];
        const uint32_t pair = quantise_row8<8>(raw[it], q);
        if (which == 0) {
            // dimensions 8*sub .. +7 of token u: eight consecutive bytes of chunk (j*2 + half)*64 + 16*hh + c
            const int d = 8 * sub;
            const int chunk = ((u >> 4) * 2 + ((d & 31) >> 4)) * 64 + 16 * (d >> 5) + (u & 15);
            u32x2 w;
            w[0] = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
            w[1] = q[4] | (q[5] << 8) | (q[6] << 16) | (q[7] << 24);
            *reinterpret_cast<u32x2*>(&lds[0][chunk * 16 + (d & 15)]) = w;
        } else {
            const int hh = (u & 15) >> 2, e = (u & 3) + 4 * (u >> 4);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int d = 8 * sub + k, i = d >> 4;
                lds[1][((i >> 1) * 64 + 16 * hh + (d & 15)) * 16 + (i & 1) * 8 + e] = (uint8_t)q[k];
            }
        }
        if (a.live && sub == 0) kv.sz[(bh * kv.cap + (size_t)tb * 32 + u) * 2 + which] = pair;
    }
    __syncthreads();
    const size_t blk = (bh * (kv.cap / 32) + tb) * 4096;
    const int chunk = threadIdx.x;                                     // 256 chunks of 16 bytes per block
    const u32x4 kc = *reinterpret_cast<const u32x4*>(&lds[0][chunk * 16]);
    u32x4 vc = *reinterpret_cast<const u32x4*>(&lds[1][chunk * 16]);
    u32x4* kdst = reinterpret_cast<u32x4*>(kv.k + blk) + chunk;
    u32x4* vdst = reinterpret_cast<u32x4*>(kv.v + blk) + chunk;
    if (u0 == 0 && u1 == 32) {
        *kdst = kc;
        *vdst = vc;
        return;
    }
    const int ku = (chunk >> 7) * 16 + (chunk & 15);                   // the token of this key chunk
    if (ku >= u0 && ku < u1) *kdst = kc;
    // value chunk: byte e of either half belongs to token (e % 4) + 4*hh + 16*(e / 4), hh = (chunk % 64) / 16
    const int hh = (chunk & 63) >> 4;
    uint32_t keep_lo = 0, keep_hi = 0;                                 // byte masks of tokens e = 0..3 and e = 4..7
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ua = e + 4 * hh, ub = ua + 16;
        if (ua >= u0 && ua < u1) keep_lo |= 0xffu << (8 * e);
        if (ub >= u0 && ub < u1) keep_hi |= 0xffu << (8 * e);
    }
    const u32x4 old = *vdst;
    vc[0] = (vc[0] & keep_lo) | (old[0] & ~keep_lo);
    vc[1] = (vc[1] & keep_hi) | (old[1] & ~keep_hi);
    vc[2] = (vc[2] & keep_lo) | (old[2] & ~keep_lo);
    vc[3] = (vc[3] & keep_hi) | (old[3] & ~keep_hi);
    *vdst = vc;
}

// 4-bit codes: one CTA of 256 threads per (KV head, 32-token half block touched, sequence), for runs of any length (two
// tokens share bytes of the value block, so tokens are never written by independent waves).  Quantisation as above
// with 15 levels; key codes leave a lane as one whole operand word, value codes are staged as bytes in LDS and gathered
// into operand words (eight tokens per word).  A partly covered half block is merged with what the cache holds: key
// chunks belong to one token each, value words are merged nibble by nibble.
__global__ __launch_bounds__(256) void kv4_append_block_kernel(AttnCache kv, const uint16_t* __restrict__ Kn,
                                                               const uint16_t* __restrict__ Vn,
                                                               const int32_t* __restrict__ positions, int count)
{
    __shared__ __align__(16) uint32_t kwords[512];                     // the key half block in cache order
    __shared__ __align__(8) uint8_t vcodes[32][136];                   // value codes [token][dimension], padded rows
    const int h = blockIdx.x, b = blockIdx.z;
    const int pos = positions[b];
    long first = pos < 0 ? 0 : pos, last = (long)pos + count;
    if (last > kv.cap) last = kv.cap;
    if (first >= last) return;
    const int tb = (int)(first >> 5) + (int)blockIdx.y;
    const long t0 = first > (long)tb * 32 ? first : (long)tb * 32;
    const long t1 = last < (long)(tb + 1) * 32 ? last : (long)(tb + 1) * 32;
    if (t0 >= t1) return;                                              // CTA-uniform
    const int u0 = (int)(t0 - (long)tb * 32), u1 = (int)(t1 - (long)tb * 32);
    const int sub = threadIdx.x & 15;                                  // dimensions 8*sub .. 8*sub + 7
    const size_t bh = (size_t)b * kv.heads + h;
    u32x4 raw[4];
    append_request(raw, Kn, Vn, kv.heads, h, b, count, (long)tb * 32 - pos, u0, u1);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int which = it >> 1;
        const AppendSlot a = append_slot(it, u0, u1);
        const int u = a.u;
        uint32_t q[8];
        const uint32_t pair = quantise_row8<4>(raw[it], q);
        if (which == 0) {
            // dimensions 32*hh + 8*tt + e, e = 0..7: word tt of chunk (u/16)*64 + 16*hh + u%16; element e at nibble
            // e/2 + 4*(e % 2)
            const int chunk = (u >> 4) * 64 + 16 * (sub >> 2) + (u & 15);
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) w |= q[e] << (4 * ((e >> 1) + 4 * (e & 1)));
            kwords[chunk * 4 + (sub & 3)] = w;
        } else {
            u32x2 w;
            w[0] = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
            w[1] = q[4] | (q[5] << 8) | (q[6] << 16) | (q[7] << 24);
            *reinterpret_cast<u32x2*>(&vcodes[u][8 * sub]) = w;
        }
        if (a.live && sub == 0) kv.sz[(bh * kv.cap + (size_t)tb * 32 + u) * 2 + which] = pair;
    }
    __syncthreads();
    const size_t blk = (bh * (kv.cap / 32) + tb) * 2048;
    const bool whole = u0 == 0 && u1 == 32;
    const int chunk = threadIdx.x & 127;                               // 128 chunks of 16 bytes per half block
    if (threadIdx.x < 128) {
        const int ku = (chunk >> 6) * 16 + (chunk & 15);               // the token of this key chunk
        if (whole || (ku >= u0 && ku < u1))
            reinterpret_cast<u32x4*>(kv.k + blk)[chunk] = *reinterpret_cast<const u32x4*>(&kwords[chunk * 4]);
        return;
    }
    // value chunk (i/4)*64 + 16*hh + c: word i % 4 holds dimension 16*i + c of the tokens (e % 4) + 4*hh + 16*(e / 4)
    const int ii = chunk >> 6, hh = (chunk & 63) >> 4, c = chunk & 15;
    u32x4 vc = {0u, 0u, 0u, 0u};
    uint32_t keep = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int u = (e & 3) + 4 * hh + 16 * (e >> 2);
        const int sh = 4 * ((e >> 1) + 4 * (e & 1));
        if (u >= u0 && u < u1) keep |= 0xfu << sh;
#pragma unroll
        for (int w = 0; w < 4; ++w) vc[w] |= (uint32_t)vcodes[u][16 * (4 * ii + w) + c] << sh;
    }
    u32x4* vdst = reinterpret_cast<u32x4*>(kv.v + blk) + chunk;
    if (!whole) {
        const u32x4 old = *vdst;
#pragma unroll
        for (int w = 0; w < 4; ++w) vc[w] = (vc[w] & keep) | (old[w] & ~keep);
    }
    *vdst = vc;
}

// 4-bit codes, one new token per sequence (the append of a decoding step): one wave for the key and one for the value of a
// (sequence, KV head); lane l owns dimensions l and l + 64.  Key codes: the eight lanes of an operand word OR their nibbles
// together and one of them stores the word.  Value codes: every dimension has its own word, shared with seven other tokens,
// so each lane replaces one nibble in each of its two words (no other wave of the launch touches this sequence and head's).
__global__ __launch_bounds__(128) void kv4_append_token_kernel(AttnCache kv, const uint16_t* __restrict__ Kn,
                                                               const uint16_t* __restrict__ Vn,
                                                               const int32_t* __restrict__ positions)
{
    const int lane = threadIdx.x & 63, which = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = blockIdx.x % kv.heads, b = blockIdx.x / kv.heads;
    const size_t bh = (size_t)b * kv.heads + h;
    const uint16_t* const x = (which ? Vn : Kn) + bh * kHeadDim;
    const uint16_t r0 = x[lane], r1 = x[lane + 64];
    const int t = positions[b];
    if (t < 0 || t >= kv.cap) return;                       // CTA-uniform
    const int u = t & 31;
    const size_t blk = (bh * (kv.cap / 32) + (t >> 5)) * 512;      // in words
    // dimension d = 16*i + c: word ((i/4)*64 + 16*hh + c)*4 + i%4, hh = (u%16)/4; this token is operand element
    // e = u%4 + 4*(u/16) of the word.  The words are requested before the arithmetic.
    const int ve = (u & 3) + 4 * (u >> 4), vsh = 4 * ((ve >> 1) + 4 * (ve & 1));
    uint32_t* vp[2];
    uint32_t old[2] = {0u, 0u};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int d = lane + 64 * k, i = d >> 4;
        vp[k] = reinterpret_cast<uint32_t*>(kv.v) + blk + ((i >> 2) * 64 + 16 * ((u & 15) >> 2) + (d & 15)) * 4 + (i & 3);
        if (which) old[k] = *vp[k];
    }
    uint32_t q0, q1;
    const uint32_t pair = quantise_pair<4>((float)__builtin_bit_cast(_Float16, r0), (float)__builtin_bit_cast(_Float16, r1), q0, q1);
    if (which == 0) {
        // dimension d = 32*hh + 8*tt + e: word ((u/16)*64 + 16*hh + u%16)*4 + tt, nibble e/2 + 4*(e % 2)
        const int e = lane & 7;
        const int sh = 4 * ((e >> 1) + 4 * (e & 1));
        uint32_t w0 = q0 << sh, w1 = q1 << sh;
#pragma unroll
        for (int m = 1; m < 8; m <<= 1) {
            w0 |= (uint32_t)__shfl_xor((int)w0, m);
            w1 |= (uint32_t)__shfl_xor((int)w1, m);
        }
        if (e == 0) {
            uint32_t* kw = reinterpret_cast<uint32_t*>(kv.k) + blk;
            const int d = lane;                              // and d + 64: two more 32-dimension groups up
            const int word = ((u >> 4) * 64 + 16 * (d >> 5) + (u & 15)) * 4 + ((d & 31) >> 3);
            kw[word] = w0;
            kw[word + 2 * 16 * 4] = w1;
        }
    } else {
        *vp[0] = (old[0] & ~(0xfu << vsh)) | (q0 << vsh);
        *vp[1] = (old[1] & ~(0xfu << vsh)) | (q1 << vsh);
    }
    if (lane == 0) kv.sz[(bh * kv.cap + t) * 2 + which] = pair;
}

// ------------------------------------------------------------------------------------------------ decode attention
// The codes of a block travel in registers (they are the in-flight memory of the pipeline: two blocks ahead).  The 64
// scale/zero words of a block would cost as many registers per lane as its 8 KiB of codes, so they go through LDS
// instead: one direct-to-LDS load per block and wave (lane l fetches word l) into a slot private to the wave.
struct BlockRegs {
    u32x4 k[2][2];      // two 16-token tiles: 32 key bytes of the lane's token (dimensions 32h .. 32h+31)
    u32x4 v[4];         // 64 value bytes: eight 16-row tiles x the lane's eight tokens
};

// Descriptors of one (sequence, head): its K blocks, V blocks and scale/zero words, each cut off after the last block
// of the context.  A load past that end returns zeros without touching memory, which lets the pipeline issue its loads
// unconditionally (the surplus ones at the end of a wave's range cost nothing).
struct HeadRsrc {
    __amdgpu_buffer_rsrc_t k, v, sz;
};

// A block is 4096 bytes of key codes and as many of value codes: 32 tokens of 8-bit codes, or 64 tokens of 4-bit codes
// (two 32-token halves of 2048 bytes each, r.k[half][tile], r.v[2*half + i/4]); the load instructions are the same.
template <int BITS>
__device__ __forceinline__ void load_block(BlockRegs& r, uint32_t* sz_slot, const HeadRsrc& rs, int blk, int lane)
{
    // (the host pass of the compiler only needs the kernel's signature; it cannot express the LDS pointer)
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (BITS == 8) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs.sz, (__attribute__((address_space(3))) void*)sz_slot, 4,
                                                 lane * 4 + blk * 256, 0, 0, 0);
    } else {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs.sz, (__attribute__((address_space(3))) void*)sz_slot, 4,
                                                 lane * 4 + blk * 512, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs.sz, (__attribute__((address_space(3))) void*)(sz_slot + 64), 4,
                                                 lane * 4 + blk * 512 + 256, 0, 0, 0);
    }
#else
    (void)sz_slot;
#endif
    // every load instruction of the wave reads 1 KiB of consecutive bytes: the blocks are stored in operand order.
    // The block offset sits in the per-lane offset, which the descriptor's range check covers.
    const int off = lane * 16 + blk * 4096;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        r.k[j][0] = __builtin_amdgcn_raw_buffer_load_b128(rs.k, off + (j * 2 + 0) * 1024, 0, kNonTemporal);
        r.k[j][1] = __builtin_amdgcn_raw_buffer_load_b128(rs.k, off + (j * 2 + 1) * 1024, 0, kNonTemporal);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs.v, off + i * 1024, 0, kNonTemporal);
}

// Running state of one wave (per query head m = lane % 16; m_run is equal in the four lanes that share an m, l_run and
// corr are per-lane partial sums over the lane's own tokens).  m_run is the reference the exponents are taken against: the
// largest score up to a factor of 2^kSlack.  It moves only when a score exceeds it by more than that, so a block normally
// needs no exchange between lanes and no rescaling: the shuffles of a running maximum were the longest part of the chain of
// dependent instructions that two waves per SIMD cannot hide.  Probabilities of at most 2^kSlack times a scale fit fp16.
struct SoftmaxState {
    float m_run, l_run, corr;
    f32x4 bias;                            // 8-bit codes: minus the value bias that acc carries at the moment
};
template <int BITS>
constexpr float kSlack = BITS == 8 ? 6.0f : 2.0f;      // 2^6 * (2 * 65504 / 255), 2^2 * (2 * 65504 / 15) < 65504

__device__ __forceinline__ uint32_t swap_half_rows(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);      // row_ror:8 = lane c <-> c ^ 8
}

// Moves the reference to the largest score of every query head so far (mx: the lane's largest new score, not reduced).
template <int BITS, bool PACK>
__device__ __forceinline__ void move_reference(float mx, SoftmaxState& st, f32x4 (&acc)[8])
{
    if constexpr (PACK) mx = fmaxf(mx, __builtin_bit_cast(float, swap_half_rows(__builtin_bit_cast(uint32_t, mx))));
    mx = xor_max(xor_max(mx, 16), 32);
    const float m_new = fmaxf(st.m_run, mx);
    const float alpha = fast_exp2(st.m_run - m_new);
    st.m_run = m_new;
    st.l_run *= alpha;
    st.corr *= alpha;
    if constexpr (BITS == 8) st.bias *= alpha;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= alpha;
}

// Runs N0 .. N0 + NH - 1 of thirty-two tokens of a block (8-bit codes: one run, 4-bit codes: two).  qsum =
// sum of the query's 128 values; neg_qbias = minus the sum of the conversion bias of each code position times the query
// value it meets.  len: tokens the lane's query column attends over (the same in every lane at a decoding step; at prefill
// every column has its own causal limit).
//
// PACK: at most eight query heads share the KV head.  The query operand then carries every head twice
// (column c and c + 8 both hold head c % 8), so both score tiles of a run come out with all 16 columns live, and a lane keeps
// tile c / 8 only - four scores instead of eight, half the softmax arithmetic.  The probabilities of the other tile's
// tokens reach the lane through one exchange with lane c ^ 8 before the second product; running sums are per lane over
// its own tokens and meet at the end (xor 8, 16, 32).
template <int BITS, bool PACK, int N0, int NH>
__device__ __forceinline__ void process_runs(const BlockRegs& r, const uint32_t* sz_slot, const f16x8 (&qf)[4],
                                              float scale_log2e, float qsum, const f32x4& neg_qbias, const Magic& mg, int blk, int len,
                                              int lane, SoftmaxState& st, f32x4 (&acc)[8])
{
    constexpr int NS = PACK ? 1 : 2;                         // score tiles a lane keeps of a run
    const int h = lane >> 4, jl = PACK ? (lane >> 3) & 1 : 0;      // jl: the 16-token tile this lane keeps
    const int rem = len - blk * (256 / BITS) - 32 * N0 - 4 * h - 16 * jl;      // slot (n, j, rr) is a live token iff 32*n + 16*j + rr < rem
    float t[NH][NS][4];                                      // scores before the key's scale
    f16x2 kp[NH][NS][4];                                     // (scale, zero-point) of the slot's key
    uint32_t vw[NH][NS][4];                                  // and of its value; 0 for a dead token
#pragma unroll
    for (int n = 0; n < NH; ++n) {
        // S^T for the two 16-token tiles: rows = tokens, columns = query heads.  The accumulator starts at minus the bias
        // term: sum_d (bias_d + q_d) Q_d - sum_d bias_d Q_d = sum_d q_d Q_d
        f32x4 d[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (BITS == 8) {
                d[j] = mfma16x16x32(biased8_w8(r.k[j][0].x, r.k[j][0].y), qf[0], neg_qbias);
                d[j] = mfma16x16x32(biased8_w8(r.k[j][0].z, r.k[j][0].w), qf[1], d[j]);
                d[j] = mfma16x16x32(biased8_w8(r.k[j][1].x, r.k[j][1].y), qf[2], d[j]);
                d[j] = mfma16x16x32(biased8_w8(r.k[j][1].z, r.k[j][1].w), qf[3], d[j]);
            } else {
                const u32x4 w = r.k[N0 + n][j];
                d[j] = mfma16x16x32(biased8(w.x, mg), qf[0], neg_qbias);
                d[j] = mfma16x16x32(biased8(w.y, mg), qf[1], d[j]);
                d[j] = mfma16x16x32(biased8(w.z, mg), qf[2], d[j]);
                d[j] = mfma16x16x32(biased8(w.w, mg), qf[3], d[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            // (K pair, V pair) of the lane's four tokens 16*(j or jl) + 4h .. +3: eight consecutive words of the slot
            const uint32_t* const z = sz_slot + 64 * (N0 + n) + 32 * (PACK ? jl : j) + 8 * h;
            const u32x4 p0 = *(const u32x4*)z, p1 = *(const u32x4*)(z + 4);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                // a dead token contributes nothing, whatever its pair holds: scale 0 and zero-point 0 for its values
                const bool live = 32 * n + 16 * j + rr < rem;
                kp[n][j][rr] = as_f16x2(rr < 2 ? p0[2 * rr] : p1[2 * (rr - 2)]);
                vw[n][j][rr] = live ? (rr < 2 ? p0[2 * rr + 1] : p1[2 * (rr - 2) + 1]) : 0u;
                // sum_d q_d Q_d  -  z sum_d Q_d  =  sum_d (q_d - z) Q_d, times scale * log2(e).  (The pair enters a multiply-add,
                // which takes fp16 directly.  The scale goes here, in fp32, and not into the query's fp16 values, where its rounding
                // would be a fifth of the result's error.)
                const float dm = PACK ? (jl ? d[1][rr] : d[0][rr]) : d[j][rr];
                t[n][j][rr] = scale_log2e * __builtin_fmaf(-(float)kp[n][j][rr].y, qsum, dm);
            }
        }
    }
    // scores in base 2 less the reference
    float x[NH][NS][4], mx = kNegBig;
    auto scores = [&](float ref) {
        mx = kNegBig;
#pragma unroll
        for (int n = 0; n < NH; ++n)
#pragma unroll
            for (int j = 0; j < NS; ++j)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const float v = __builtin_fmaf((float)kp[n][j][rr].x, t[n][j][rr], -ref);
                    x[n][j][rr] = 32 * n + 16 * j + rr < rem ? v : kNegBig;
                    mx = fmaxf(mx, x[n][j][rr]);
                }
    };
    scores(st.m_run);
    if (__any(mx > kSlack<BITS>)) {
        scores(0.0f);
        move_reference<BITS, PACK>(mx, st, acc);
        scores(st.m_run);
    }
    // probability times the value scale of that token, rounded to fp16: the operand of the second product.  The zero-point
    // term must be built from the very fp16 values the matrix core multiplies: a zero-point is as large as the codes and the
    // two sums cancel, so a disagreement of one fp16 ulp per probability would stay in the result at full size.  Left to itself
    // the compiler rounds p * vs once for the operand (fused multiply-and-convert) and once more, through fp32, for the sum
    // below; the two differ when the fp32 product lands on an fp16 tie.  Pinning the packed operand makes it the only copy.
    float psum = 0.f, zsum = 0.f;
    f16x8 pb[NH];
#pragma unroll
    for (int n = 0; n < NH; ++n) {
        uint32_t own[NS][2];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            _Float16 q[4];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const float p = fast_exp2(x[n][j][rr]);      // 0 for masked tokens
                psum += p;
                q[rr] = (_Float16)__builtin_fmaf((float)as_f16x2(vw[n][j][rr]).x, p, 0.0f);
            }
            own[j][0] = (uint32_t)__builtin_bit_cast(uint16_t, q[0]) | ((uint32_t)__builtin_bit_cast(uint16_t, q[1]) << 16);
            own[j][1] = (uint32_t)__builtin_bit_cast(uint16_t, q[2]) | ((uint32_t)__builtin_bit_cast(uint16_t, q[3]) << 16);
            asm volatile("" : "+v"(own[j][0]), "+v"(own[j][1]));
            // sum over the lane's tokens of z * p'
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const f16x2 two = as_f16x2(own[j][rr >> 1]);
                const float pv = (float)(rr & 1 ? two.y : two.x);
                zsum = __builtin_fmaf((float)as_f16x2(vw[n][j][rr]).y, pv, zsum);
            }
        }
        u32x4 bits;                                          // k-values 0..3: tile 0, 4..7: tile 1
        if constexpr (PACK) {
            const uint32_t x0 = swap_half_rows(own[0][0]), x1 = swap_half_rows(own[0][1]);
            bits.x = jl ? x0 : own[0][0];
            bits.y = jl ? x1 : own[0][1];
            bits.z = jl ? own[0][0] : x0;
            bits.w = jl ? own[0][1] : x1;
        } else {
            bits = u32x4{own[0][0], own[0][1], own[NS - 1][0], own[NS - 1][1]};
        }
        pb[n] = __builtin_bit_cast(f16x8, bits);
    }
    st.l_run += psum;
    st.corr += zsum;
    // The bias of a value code is several times the payload (4-bit codes: up to a hundred times): carried along to the end of
    // a long context it would cost the sums their low bits, in proportion to the context.  Products with the constant operand -bias
    // (1024; 64 at the k-values 2, 3, 6 and 7 of a 4-bit word) sum up what has to leave.  4-bit codes: per block, before the codes
    // that carry it go in.  8-bit codes: every fourth block (128 tokens times 1151 are a seventh of the 8192 times 127 that the codes
    // themselves sum up to over 32768 tokens; taken out of every code before the product it cost the 16-column prompt form up to 8 %:
    // 64 tokens after 12000, 8 heads: 65.2 us, like this 60.9).
    const _Float16 bias_a = (_Float16)-1024.0f, bias_b = BITS == 8 ? bias_a : (_Float16)-64.0f;
    const f16x8 minus_bias = {bias_a, bias_a, bias_b, bias_b, bias_a, bias_a, bias_b, bias_b};
    if constexpr (BITS == 4) {
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < NH; ++n) bias = mfma16x16x32(minus_bias, pb[n], bias);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += bias;
    } else {
        st.bias = mfma16x16x32(minus_bias, pb[0], st.bias);
    }
    // O^T += V^T P'^T : rows = dimensions (eight 16-row tiles), k = the 32 tokens of a run
#pragma unroll
    for (int n = 0; n < NH; ++n)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            f16x8 a;
            if constexpr (BITS == 8) {
                const u32x4 w = r.v[i >> 1];
                a = (i & 1) ? biased8_w8(w.z, w.w) : biased8_w8(w.x, w.y);
            } else {
                a = biased8(r.v[2 * (N0 + n) + (i >> 2)][i & 3], mg);
            }
            acc[i] = mfma16x16x32(a, pb[n], acc[i]);
        }
    if constexpr (BITS == 8) {
        if ((blk >> 2 & 3) == 3) {                           // (wave-uniform) a wave takes every fourth block
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += st.bias;
            st.bias = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
}

// A whole block.  The two runs of a 4-bit block go through together, which gives each wave two independent chains of
// instructions; with two score tiles a lane that takes more registers than there are, so there they go one after the other.
template <int BITS, bool PACK>
__device__ __forceinline__ void process_block(const BlockRegs& r, const uint32_t* sz_slot, const f16x8 (&qf)[4],
                                              float scale_log2e, float qsum, const f32x4& neg_qbias, const Magic& mg, int blk, int len, int len_all,
                                              int lane, SoftmaxState& st, f32x4 (&acc)[8])
{
    if constexpr (BITS == 8 || PACK) {
        process_runs<BITS, PACK, 0, BITS == 8 ? 1 : 2>(r, sz_slot, qf, scale_log2e, qsum, neg_qbias, mg, blk, len, lane, st, acc);
    } else {
        process_runs<BITS, PACK, 0, 1>(r, sz_slot, qf, scale_log2e, qsum, neg_qbias, mg, blk, len, lane, st, acc);
        if (blk * 64 + 32 < len_all)                         // (wave-uniform) the second run may lie wholly behind the context
            process_runs<BITS, PACK, 1, 1>(r, sz_slot, qf, scale_log2e, qsum, neg_qbias, mg, blk, len, lane, st, acc);
    }
}

// Four consecutive dimensions d0 .. d0+3 of query head `head` of sequence b, rounded to fp16.
__device__ __forceinline__ void store_out4(uint16_t* O, int b, int q_heads, int head, int d0, const float (&o)[4])
{
    u32x2 out;
    out.x = (uint32_t)f32_to_f16_bits(o[0]) | ((uint32_t)f32_to_f16_bits(o[1]) << 16);
    out.y = (uint32_t)f32_to_f16_bits(o[2]) | ((uint32_t)f32_to_f16_bits(o[3]) << 16);
    *(u32x2*)(O + ((size_t)b * q_heads + head) * kHeadDim + d0) = out;
}

// grid (kv heads, batch, splits); 256 threads.  Partial layout per (b, h, split): m[16], l[16], out[128][16] floats.
constexpr int kPartialFloats = 32 + kHeadDim * 16;
constexpr int kMergeBatch = 8;           // splits the last-arriving CTA loads at a time (all in flight at once)

// PREFILL: the same kernel over a short chunk of prompt tokens, or one of few heads (paper Sec. 3.3: one attention pipeline for
// both phases; chunks that fill the chip with 128- or 256-row CTAs run on tm_attn_prefill.hip).  The 16
// query columns of a CTA are then 16 / G consecutive tokens x the G query heads of the KV head (column c = token c / G,
// head c % G), blockIdx.z counts such token groups instead of context splits, `lens` holds the cache position of every
// sequence's first query token, and each column attends causally over the cache up to its own token: the length that
// masks scores becomes a per-lane value, everything else - loading pipeline, head alignment, biased codes - is shared.
template <int BITS, bool PACK, bool PREFILL = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_decode_kernel(AttnCache kv, const uint16_t* __restrict__ Q,
                                                          const int32_t* __restrict__ lens, uint16_t* __restrict__ O,
                                                          int q_heads, float scale_log2e, int blocks_per_split,
                                                          int splits, int merge_here, int head0, int gw,
                                                          const int32_t* __restrict__ counts = nullptr, int count = 1)
{
    static_assert(!(PREFILL && PACK), "prompt chunks use all 16 query columns");
    __shared__ float sm_ml[4][2][16];
    __shared__ float sm_out[4][8][4][64];
    // scale/zero words of the blocks in flight: [wave][64 words]; one array per ring slot so that the compiler can tell
    // which direct-to-LDS load a read depends on
    constexpr int TOK = 256 / BITS;                 // tokens per block
    __shared__ __attribute__((aligned(16))) uint32_t sz_ring0[4][2 * TOK];
    __shared__ __attribute__((aligned(16))) uint32_t sz_ring1[4][2 * TOK];
    __shared__ __attribute__((aligned(16))) uint32_t sz_ring2[4][2 * TOK];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, h = lane >> 4;
    const int hk = blockIdx.x, b = blockIdx.y, split = blockIdx.z;
    // A launch covers query heads head0 .. head0 + gw - 1 (gw <= 16) of every KV head's group of q_heads / kv.heads:
    // larger groups take one launch per sixteen heads.  G is the width the columns are laid out for, hq the first query
    // head of this CTA.
    const int G = gw;
    const int hq = hk * (q_heads / kv.heads) + head0;
    const size_t bh = (size_t)b * kv.heads + hk;
    int len, len_all;                                        // this lane's column; the CTA's longest column
    int tok = 0, head = c;                                   // query token (within the chunk) and head (within G) of column c
    bool real;
    if constexpr (PREFILL) {
        const int tpg = 16 / G;                              // tokens per CTA
        const int tq = c / G;
        head = c - tq * G;
        tok = split * tpg + tq;
        const int cnt = counts ? min(max(counts[b], 0), count) : count;
        const int first = split * tpg;                    // first token of this group
        if (first >= cnt) return;                            // (uniform) nothing to do for this sequence
        const int pos0 = lens[b];
        const int pos = pos0 + tok;
        real = tq < tpg && tok < cnt && pos >= 0 && pos < kv.cap;
        len = real ? pos + 1 : 0;
        len_all = min(max(pos0 + min(cnt, first + tpg), 0), kv.cap);
        if (!real) tok = first;                              // an address that exists
    } else {
        // the splits cover blocks_per_split * splits blocks (the host's max_len): a longer sequence is cut there
        len = len_all = min(min(max(lens[b], 0), kv.cap), blocks_per_split * splits * TOK);
        real = (PACK ? (c & 7) : c) < G;
    }
    // Nothing is requested before the length is known: two blocks per wave ahead of it are 64 KiB per CTA that a short sequence
    // does not use (64 sequences x 8 heads of 1 / 100 tokens under a capacity of 32768: 7.3 / 7.7 us, with the length first
    // 5.3 / 6.8), and save nothing where the context is used whole (0.2 % over 60 launches of 7-85 us).
    const int nblk = (len_all + TOK - 1) / TOK;
    const int blk0 = PREFILL ? 0 : split * blocks_per_split;
    const int blk1 = PREFILL ? nblk : min(nblk, blk0 + blocks_per_split);

    // Order of the prologue: the query's raw loads, then at once the first two blocks of the KV memory loading pipeline,
    // and only then the arithmetic on the query, which so runs under the blocks' latency (loads return in order, so the
    // query must be requested first).
    const int qc = PREFILL ? head : (PACK ? (c & 7) : c);    // the query head of operand column c
    f16x8 qraw[4];
    {
        const size_t qrow = PREFILL ? (size_t)b * count + tok : (size_t)b;
        const uint16_t* qp = Q + (qrow * q_heads + (size_t)hq + (real ? qc : 0)) * kHeadDim + 32 * h;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) qraw[tt] = *(const f16x8*)(qp + 8 * tt);
    }

    // KV memory loading pipeline: the next two blocks of this wave are in flight while the current one is multiplied
    // (three register sets and three LDS slots, rotated by unrolling; with one block ahead the waves spent half their
    // time waiting for memory).  Loads are unconditional - past the end of the wave's range they point behind the
    // descriptors' ranges and return zeros without memory traffic - so that the loop body is straight-line code with a
    // known number of loads in flight.
    HeadRsrc rs;
    rs.k = make_rsrc(kv.k + bh * (kv.cap / TOK) * 4096, (uint32_t)nblk * 4096u);
    rs.v = make_rsrc(kv.v + bh * (kv.cap / TOK) * 4096, (uint32_t)nblk * 4096u);
    rs.sz = make_rsrc(kv.sz + bh * kv.cap * 2, (uint32_t)nblk * (8u * TOK));
    uint32_t* const z0 = sz_ring0[wave];
    uint32_t* const z1 = sz_ring1[wave];
    uint32_t* const z2 = sz_ring2[wave];
    BlockRegs r0, r1, r2;
    int blk = blk0 + wave;
    load_block<BITS>(r0, z0, rs, blk < blk1 ? blk : nblk, lane);
    load_block<BITS>(r1, z1, rs, blk + 4 < blk1 ? blk + 4 : nblk, lane);

    // Query operand (adaptive head alignment): column m = c, k-values of step tt = dimensions 32h + 8tt .. +7, the
    // order in which the lane's key bytes arrive.
    f16x8 qf[4];
    float qsum = 0.f, qbias = 0.f;
    const Magic mg = make_magic();
    {
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                qf[tt][e] = real ? qraw[tt][e] : (_Float16)0.0f;
            }
            // (an ordering point only: it holds this arithmetic behind the requests above; without it launches of 10-15 us take 3 % longer)
            u32x4 bits = __builtin_bit_cast(u32x4, qf[tt]);
            asm volatile("" : "+v"(bits.x), "+v"(bits.y), "+v"(bits.z), "+v"(bits.w));
            qf[tt] = __builtin_bit_cast(f16x8, bits);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                qsum += (float)qf[tt][e];
                qbias += ((e & 2) ? 64.0f : 1024.0f) * (float)qf[tt][e];     // bias of a 4-bit code at operand position e
            }
        }
        qsum = xor_add(xor_add(qsum, 16), 32);
        qbias = BITS == 8 ? 1024.0f * qsum : xor_add(xor_add(qbias, 16), 32);   // every 8-bit code carries the bias 1024
    }
    const f32x4 neg_qbias = {-qbias, -qbias, -qbias, -qbias};

    // The first block of a decoding step exceeds the reference kNegBig by more than kSlack in every column, which moves it to that
    // block's largest score.  (At prefill a wave may meet blocks in which some column has no live token yet: the reference then
    // starts above the mask value, so that masked scores still turn into zero probabilities.)
    SoftmaxState st{PREFILL ? kMaskFloor : kNegBig, 0.f, 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
    f32x4 acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (blk < blk1) {
        while (true) {
            load_block<BITS>(r2, z2, rs, blk + 8 < blk1 ? blk + 8 : nblk, lane);
            process_block<BITS, PACK>(r0, z0, qf, scale_log2e, qsum, neg_qbias, mg, blk, len, len_all, lane, st, acc);
            blk += 4;
            if (blk >= blk1) break;
            load_block<BITS>(r0, z0, rs, blk + 8 < blk1 ? blk + 8 : nblk, lane);
            process_block<BITS, PACK>(r1, z1, qf, scale_log2e, qsum, neg_qbias, mg, blk, len, len_all, lane, st, acc);
            blk += 4;
            if (blk >= blk1) break;
            load_block<BITS>(r1, z1, rs, blk + 8 < blk1 ? blk + 8 : nblk, lane);
            process_block<BITS, PACK>(r2, z2, qf, scale_log2e, qsum, neg_qbias, mg, blk, len, len_all, lane, st, acc);
            blk += 4;
            if (blk >= blk1) break;
        }
    }

    // the four lanes of a query head add their partial sums; the waves meet in LDS
    float l_w = xor_add(xor_add(st.l_run, 16), 32);
    float corr_w = xor_add(xor_add(st.corr, 16), 32);
    if constexpr (PACK) {                                    // the two tiles' lanes of a query head
        l_w = xor_add(l_w, 8);
        corr_w = xor_add(corr_w, 8);
    }
    if (h == 0) {
        sm_ml[wave][0][c] = st.m_run;
        sm_ml[wave][1][c] = l_w;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)                       // the zero-points leave here
            sm_out[wave][i][rr][lane] = (BITS == 8 ? acc[i][rr] + st.bias[rr] : acc[i][rr]) - corr_w;
    __syncthreads();
    // thread (wave w, lane) finalises row tiles 2w and 2w+1 of its column
    float M = kNegBig;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, sm_ml[w][0][c]);
    float L = 0.f, f[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        f[w] = exp2f(sm_ml[w][0][c] - M);
        L += sm_ml[w][1][c] * f[w];
    }
    if (splits == 1) {
        const float inv = L > 0.f ? 1.0f / L : 0.f;
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
            const int i = 2 * wave + ii;
            float o[4];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) v += sm_out[w][i][rr][lane] * f[w];
                o[rr] = v * inv;
            }
            if constexpr (PREFILL) {
                if (real) store_out4(O, b * count + tok, q_heads, hq + head, 16 * i + 4 * h, o);
            } else {
                if (c < G) store_out4(O, b, q_heads, hq + c, 16 * i + 4 * h, o);
            }
        }
        return;
    }
    if constexpr (PREFILL) return;                           // prompt chunks are never split along the context

    // Split context: this CTA's maximum, denominator and unnormalised rows go to the workspace - values of row tile i,
    // register rr at float 32 + (4*i + rr)*64 + lane, so that writer and reader touch whole 256-byte lines - as
    // write-through stores that CTAs on other XCDs can read back without a device-wide fence.
    float* part = kv.partial + (((size_t)bh * splits) + split) * kPartialFloats;
    if (wave == 0 && h == 0) {
        st_partial(part + c, M);
        st_partial(part + 16 + c, L);
    }
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
        const int i = 2 * wave + ii;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) v += sm_out[w][i][rr][lane] * f[w];
            st_partial(part + 32 + (4 * i + rr) * 64 + lane, v);
        }
    }
    if (!merge_here) return;                                  // many splits: the merge kernel follows

    // The CTA that arrives last at this (sequence, head)'s counter merges the splits, in their order.
    __shared__ uint32_t s_last;
    wait_stores_done();
    __syncthreads();
    if (tid == 0) {
        const uint32_t prev = atomicAdd(&kv.counters[bh], 1u);
        s_last = (prev == (uint32_t)splits - 1u) ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    // kMergeBatch splits at a time: all their loads are issued before the first use (the loop is unrolled and a missing
    // split reads split 0 again with a factor of zero)
    const float* base = kv.partial + (size_t)bh * splits * kPartialFloats;
    float Mg = kNegBig, Lg = 0.f;
    float o[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int s0 = 0; s0 < splits; s0 += kMergeBatch) {
        float ms[kMergeBatch], ls[kMergeBatch], vals[kMergeBatch][2][4];
#pragma unroll
        for (int sp = 0; sp < kMergeBatch; ++sp) {
            const float* ps = base + (size_t)(s0 + sp < splits ? s0 + sp : 0) * kPartialFloats;
            ms[sp] = ld_partial(ps + c);
            ls[sp] = ld_partial(ps + 16 + c);
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) vals[sp][ii][rr] = ld_partial(ps + 32 + (4 * (2 * wave + ii) + rr) * 64 + lane);
        }
        float Mn = Mg;
#pragma unroll
        for (int sp = 0; sp < kMergeBatch; ++sp) Mn = fmaxf(Mn, s0 + sp < splits ? ms[sp] : kNegBig);
        const float fg = exp2f(Mg - Mn);
        Mg = Mn;
        Lg *= fg;
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) o[ii][rr] *= fg;
#pragma unroll
        for (int sp = 0; sp < kMergeBatch; ++sp) {
            const float fs = s0 + sp < splits ? exp2f(ms[sp] - Mg) : 0.f;
            Lg += ls[sp] * fs;
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) o[ii][rr] += vals[sp][ii][rr] * fs;
        }
    }
    const float invg = Lg > 0.f ? 1.0f / Lg : 0.f;
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) o[ii][rr] *= invg;
        if (c < G) store_out4(O, b, q_heads, hq + c, 16 * (2 * wave + ii) + 4 * h, o[ii]);
    }
    if (tid == 0) __hip_atomic_store(&kv.counters[bh], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Merge of the context splits: grid (kv heads, batch, 8 chunks of 16 dimensions), 256 threads = 16 query heads x 16.
// Phase 1 (every CTA, all threads): running maximum and denominator over the splits, four splits per thread, reduced
// through LDS; the per-split factors exp2(m_s - M) / L stay in LDS.  Phase 2: thread (m, dd) sums dimension
// 16*chunk + dd of query head m over the splits.
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnCache kv, uint16_t* __restrict__ O, int q_heads, int splits,
                                                         int head0, int gw)
{
    __shared__ float red[16][16];
    __shared__ float fac[64][16];                  // splits <= 64
    const int hk = blockIdx.x, b = blockIdx.y, chunk = blockIdx.z;
    const int G = gw;
    const int hq = hk * (q_heads / kv.heads) + head0;
    const size_t bh = (size_t)b * kv.heads + hk;
    const float* base = kv.partial + (size_t)bh * splits * kPartialFloats;
    const int m = threadIdx.x & 15, g = threadIdx.x >> 4;
    float ms[4], ls[4];
    float mx = kNegBig;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int s = g + 16 * i;
        ms[i] = s < splits ? ld_partial(base + (size_t)s * kPartialFloats + m) : kNegBig;
        ls[i] = s < splits ? ld_partial(base + (size_t)s * kPartialFloats + 16 + m) : 0.f;
        mx = fmaxf(mx, ms[i]);
    }
    red[g][m] = mx;
    __syncthreads();
    float M = kNegBig;
#pragma unroll
    for (int i = 0; i < 16; ++i) M = fmaxf(M, red[i][m]);
    __syncthreads();
    float part = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float f = exp2f(ms[i] - M);
        part += ls[i] * f;
        if (g + 16 * i < splits) fac[g + 16 * i][m] = f;
    }
    red[g][m] = part;
    __syncthreads();
    float L = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) L += red[i][m];
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    if (m >= G) return;
    const int d = 16 * chunk + g;
    // dimension d = 16*chunk + 4*hh + rr of query head m sits at float 32 + (4*chunk + rr)*64 + 16*hh + m
    const int at = 32 + (4 * chunk + (g & 3)) * 64 + 16 * (g >> 2) + m;
    float v = 0.f;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) v += ld_partial(base + (size_t)s * kPartialFloats + at) * fac[s][m];
    O[((size_t)b * q_heads + (size_t)hq + m) * kHeadDim + d] = f32_to_f16_bits(v * inv);
}

}  // namespace

hipError_t launch_kv_append(const AttnCache& kv, const uint16_t* Kn, const uint16_t* Vn, const int32_t* positions,
                            int count, hipStream_t stream)
{
    const long tokens = (long)kv.batch * count * kv.heads;
    if (tokens <= 0 || tokens > 0x7fffffffL) return hipErrorInvalidValue;
    if (kv.bits == 4) {
        if (kv.heads > 65535 || kv.batch > 65535 || ((((uintptr_t)Kn | (uintptr_t)Vn) & 15))) return hipErrorInvalidValue;
        if (count == 1) {
            hipLaunchKernelGGL(kv4_append_token_kernel, dim3((unsigned)tokens), dim3(128), 0, stream, kv, Kn, Vn, positions);
            return hipGetLastError();
        }
        const unsigned blocks = (unsigned)((count + 31) / 32 + 1);
        hipLaunchKernelGGL(kv4_append_block_kernel, dim3(kv.heads, blocks, kv.batch), dim3(256), 0, stream, kv, Kn, Vn,
                           positions, count);
        return hipGetLastError();
    }
    if (count >= 16 && kv.heads <= 65535 && kv.batch <= 65535 && !(((uintptr_t)Kn | (uintptr_t)Vn) & 15)) {
        // blocks a run of `count` tokens can touch: one more than it fills when it starts inside a block
        const unsigned blocks = (unsigned)((count + 31) / 32 + 1);
        hipLaunchKernelGGL(kv_append_block_kernel, dim3(kv.heads, blocks, kv.batch), dim3(256), 0, stream, kv, Kn, Vn,
                           positions, count);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(kv_append_kernel, dim3((unsigned)tokens), dim3(128), 0, stream, kv, Kn, Vn, positions, count);
    return hipGetLastError();
}

// Pieces the context of every (sequence, KV head) is cut into at a decoding step; max_len <= 0: the capacity.
int attn_decode_splits(const AttnCache& kv, int max_len, int num_cu, int* blocks_per_split)
{
    const int tok = 256 / kv.bits;                                   // tokens per 4 KiB block
    if (max_len <= 0 || max_len > kv.cap) max_len = kv.cap;
    const int nblk = (max_len + tok - 1) / tok;
    // One CTA per CU.  A CU streams its share as fast with one CTA as with two, and what a launch waits for is the CU with
    // the most: a second, partial round of CTAs (or lengths that leave two long ones on one CU) costs more than idle CUs do.  4-bit cache, 32
    // sequences of 4096-8192 tokens, 8 heads: 44.7 us in two splits, 39.5 unsplit; 8-bit, 27 x 4 heads, 10-20 thousand tokens:
    // 85 us in five, 72 in two; 109 x 4 heads, 500-1000 tokens: 21.8 in two, 14.3 unsplit.  About 170 CTAs are enough for
    // the memory rate that 256 reach (4-bit, 16384 tokens: 176 pairs 66 us, 256 pairs 90).
    const int segs = kv.batch * kv.heads;
    int splits = segs >= num_cu ? 1 : num_cu / segs;
    // Two CTAs per CU (rounded up) over long contexts where one per CU leaves the most to a few of them (kv4/8 = bits of the codes,
    // equal lengths / lengths between half and all, us; more in profiles/attn_decode_splits__sweep.txt):
    //   just over half the CUs                  1 split        3              4              5
    //     136 pairs x 8192, kv4              35.2 / 33.2      31.8 / 30.8      36.1 / 26.8      31.8 / 28.5
    //     144 pairs x 8192, kv8              54.3 / 48.2      51.9 / 48.8      57.7 / 43.7      53.4 / 50.7
    //     144 pairs x 4096, kv8              29.5 / 27.9      28.6 / 26.7      32.7 / 27.0      29.0 / 29.6
    //     160 pairs x 8192, kv8              55.6 / 48.7      56.8 / 52.8      61.3 / 54.4      64.0 / 51.9
    //   a few pairs more than CUs               1 split        2
    //     272 pairs x 8192, kv4              70.8 / 51.8      63.1 / 45.6
    //     320 pairs x 8192, kv8             120.7 / 100.5    113.8 / 92.0
    //     352 pairs x 8192, kv4              72.3 / 62.7      69.0 / 62.7
    //     288 pairs x 2048, kv8              32.6 / 25.3      32.6 / 25.1
    const bool half = segs * 2 > num_cu && segs * 16 <= num_cu * 9 && max_len >= 8192;
    const bool few_over = segs > num_cu && segs * 4 <= num_cu * 5 && nblk >= 128;
    if (half || few_over) splits = (2 * num_cu + segs - 1) / segs;
    // (Cutting more finely where max_len is only the capacity does not pay: 4 x 8 heads, capacity 32768, in 8 / 16 splits:
    // 1000 tokens 11.3 / 12.2 us, 4000 tokens 24.7 / 17.9, all 32768 26 / 29.)
    // at least four blocks per wave and split (short contexts: up to eight splits of at least two - a 2048-token context
    // is cut in four or eight instead of two or four pieces, which shortens each CTA's serial chain more than the merge
    // costs; none below 24 blocks, where it costs more: 17 blocks 6.0 us unsplit, 7.1 in two), and no more partial results
    // than the cache's workspace holds
    const int few = nblk < 24 ? 1 : nblk / 8 < 8 ? nblk / 8 : 8;
    const int by_work = nblk / 16 > few ? nblk / 16 : few;
    if (splits > by_work) splits = by_work;
    if (splits > kv.max_splits) splits = kv.max_splits;
    const int bps = (nblk + splits - 1) / splits;
    *blocks_per_split = bps;
    return (nblk + bps - 1) / bps;
}

hipError_t launch_attn_decode(const AttnCache& kv, const uint16_t* Q, const int32_t* lens, uint16_t* O, int q_heads,
                              float scale, int max_len, int num_cu, hipStream_t stream)
{
    int bps;
    const int splits = attn_decode_splits(kv, max_len, num_cu, &bps);
    if (kv.heads > 65535 || kv.batch > 65535) return hipErrorInvalidValue;
    const float scale_log2e = scale * 1.4426950408889634f;
    // up to sixteen splits are merged by the CTA that finishes last, eight loads in flight at once (two splits:
    // 27.6 instead of 29.7 us at batch 32 x 2048; a loop over the splits, one load chain after the other, cost 11.5
    // instead of 8.5 us at batch 1 x 2048); more splits go to the merge kernel, which spreads a (sequence, head) over
    // eight CTAs
    const int merge_here = splits > 1 && splits <= 2 * kMergeBatch;
    const dim3 grid(kv.heads, kv.batch, splits);
    // one pass per sixteen query heads of a KV head's group (the sixteen columns of an MFMA tile); the passes follow
    // each other on the stream and share the cache's split workspace
    const int group = q_heads / kv.heads;
    for (int head0 = 0; head0 < group; head0 += 16) {
        const int gw = group - head0 < 16 ? group - head0 : 16;
        const bool pack = gw <= 8;                           // both score tiles share one softmax pass
        if (kv.bits == 8 && pack)
            hipLaunchKernelGGL((attn_decode_kernel<8, true>), grid, dim3(256), 0, stream, kv, Q, lens, O, q_heads, scale_log2e,
                               bps, splits, merge_here, head0, gw);
        else if (kv.bits == 8)
            hipLaunchKernelGGL((attn_decode_kernel<8, false>), grid, dim3(256), 0, stream, kv, Q, lens, O, q_heads, scale_log2e,
                               bps, splits, merge_here, head0, gw);
        else if (pack)
            hipLaunchKernelGGL((attn_decode_kernel<4, true>), grid, dim3(256), 0, stream, kv, Q, lens, O, q_heads, scale_log2e,
                               bps, splits, merge_here, head0, gw);
        else
            hipLaunchKernelGGL((attn_decode_kernel<4, false>), grid, dim3(256), 0, stream, kv, Q, lens, O, q_heads, scale_log2e,
                               bps, splits, merge_here, head0, gw);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (splits > 1 && !merge_here) {
            hipLaunchKernelGGL(attn_merge_kernel, dim3(kv.heads, kv.batch, 8), dim3(256), 0, stream, kv, O, q_heads, splits, head0, gw);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t launch_attn_prefill(const AttnCache& kv, const uint16_t* Q, const int32_t* positions, const int32_t* counts,
                               int count, uint16_t* O, int q_heads, float scale, int num_cu, hipStream_t stream)
{
    const int rows = attn_prefill_rows(kv, count, q_heads, num_cu);
    if (rows) return launch_attn_prefill_rows(rows, kv, Q, positions, counts, count, O, q_heads, scale, stream);
    const int group = q_heads / kv.heads;
    const float scale_log2e = scale * 1.4426950408889634f;
    for (int head0 = 0; head0 < group; head0 += 16) {        // one pass per sixteen query heads of a group, as at decode
        const int gw = group - head0 < 16 ? group - head0 : 16;
        const int tpg = 16 / gw;                             // query tokens per CTA
        const int groups = (count + tpg - 1) / tpg;
        if (kv.heads > 65535 || kv.batch > 65535 || groups > 65535 || groups < 1) return hipErrorInvalidValue;
        const dim3 grid(kv.heads, kv.batch, groups);
        if (kv.bits == 8)
            hipLaunchKernelGGL((attn_decode_kernel<8, false, true>), grid, dim3(256), 0, stream, kv, Q, positions, O, q_heads,
                               scale_log2e, 0, 1, 0, head0, gw, counts, count);
        else
            hipLaunchKernelGGL((attn_decode_kernel<4, false, true>), grid, dim3(256), 0, stream, kv, Q, positions, O, q_heads,
                               scale_log2e, 0, 1, 0, head0, gw, counts, count);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tmw4
