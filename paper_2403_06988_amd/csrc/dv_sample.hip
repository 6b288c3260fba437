// Masked sampling on CDNA4 (gfx950): the sampled decode of Algorithm 1 (the
// paper samples at temperature 1.0, Sec. 4) as a Gumbel-max draw over each
// row's admissible tokens:
//     token = argmax over allowed i of  fma(x_i, 1/T, G_i),  G_i = -ln(-ln U_i),
// with U_i from Philox4x32-10 (Salmon et al., SC 2011) keyed by the seed and
// counted by (i / 4, row, offset), and ln in binary32 by fixed steps that
// round alike on every IEEE implementation (no library log, no division), so
// the draw is reproducible bit for bit.
//
// The cost is arithmetic, not memory: a Philox call (ten rounds of two
// 32x32->64 multiplies) per 4 tokens and two logarithms per token.  Only
// admissible tokens need noise, so each wave compacts its 4-token groups
// that hold at least one allowed token into an LDS queue (one allow word of
// 32 tokens per lane, or half of one when few blocks are resident; one
// prefix sum over the lanes for the queue offsets), then every
// lane takes one queued group: one Philox call per group, and a logarithm pair
// only for the tokens whose key could still be the row's best.  A token's noise
// has an upper bound that costs two conversions and one multiply-add
// (gumbel_bound_of_word); a token whose logit and bound stay below the best key
// that the block has found cannot win nor tie, so its logarithms are left out.
// Of a dense wave's tokens that leaves one or two passes in its first trips
// and hardly any later: us per step with a pair for every token and now, three
// fifths of the tokens allowed: 256 x 128,256 59.4 and 35.7, 64 x 32,000 10.7
// and 9.3, 1,024 x 16,000 36.9 and 23.1, 8 x 128,256 10.7 and 9.1; rows that
// start at any alignment, 100 x 50,257, 20.6 and 13.0.  Where a wave's allowed
// tokens are hardly more than its groups (sparse masks) it queues single
// tokens instead, so that no lane waits on a neighbour's second logarithm
// pair; dense masks keep the groups and so one Philox call per 4 tokens.
// Lanes combine exact (order-preserving fp32 key << 32 | ~index) maxima, so
// ties go to the lowest index and the result does not depend on the order of
// the work.
#include "dv_sample.h"

namespace dv {
namespace {

constexpr int kThreads = 256;       // split rows: several blocks per row, meeting in the workspace
constexpr int kRowThreads = 1024;   // one block per row once B >= kOneBlockRows
                                    // (below that, split rows keep more waves per CU, which this
                                    // latency-laden arithmetic needs more than it saves a launch)
constexpr int kOneBlockRows = 1024;  // four or more rows per CU keep enough waves resident
// A wave queues single tokens instead of 4-token groups when its allowed
// tokens number at most kTokenRatio4 / 4 times its allowed groups: a lane then
// pays one Philox call and one logarithm pair per trip and nothing else.  Such
// a sparse wave makes three or four trips in all, too few for bounds to rule
// much out, while a group trip pays four bounds and the choice among them.  Us
// per step with lines at 0, 5 and 8 (a twentieth of the tokens allowed): 256 x
// 128,256 21.4, 21.3, 20.1; 64 x 32,000 7.9, 7.6, 7.2; 8 x 32,000 6.2, 6.3,
// 5.4; masks of runs and of three fifths take groups at all three.
constexpr int kTokenRatio4 = 8;
// order key of -2^22, below which a binary32 key holds little or nothing of its
// token's noise
constexpr uint32_t kTieKey = 0x357FFFFFu;
constexpr int kTargetBlocks = 2048;
constexpr int kHalfSpanBlocks = 512;
constexpr int kMaxChunks = 64;

struct SampleGeometry {
    int threads;
    int chunk_tok;  // a multiple of threads * span tokens (span tokens per lane per iteration)
    int nchunks;
    int span;  // tokens per lane per iteration: 32 (a whole allow word) or 16
};

SampleGeometry sample_geometry(int B, int V)
{
    if (B >= kOneBlockRows) {
        // Rows that fill at most half of the 1,024 lanes with allow words take
        // 256 of them (half a word each up to 4,096 tokens): every wave that
        // finds no word still costs its start, the block's barriers and a
        // place on its compute unit.  us per step in 1,024 lanes and now, a
        // twentieth and all of the tokens allowed: 1,024 x 1,000 8.5 and 6.7,
        // 16.9 and 7.9; 2,048 x 4,096 15.6 and 8.1, 48.5 and 15.4; 2,048 x
        // 16,384 20.2 and 14.3, 45.8 and 36.6; 1,024 x 20,000 12.9 and 11.2,
        // 27.8 and 28.7; 1,024 x 32,000 15.5 and 14.6, 33.8 and 40.2.
        if (V <= kRowThreads * 16) {
            const int span = V <= kThreads * 16 ? 16 : 32;
            const int iter = kThreads * span;
            return {kThreads, (V + iter - 1) / iter * iter, 1, span};
        }
        const int per_iter = kRowThreads * 32;
        return {kRowThreads, (V + per_iter - 1) / per_iter * per_iter, 1, 32};
    }
    const int b = B > 0 ? B : 1;
    // Below two blocks per compute unit (a row of whole allow words per lane
    // giving fewer than kHalfSpanBlocks blocks), lanes take half a word each:
    // twice the waves for the same tokens, which this issue-bound kernel
    // needs when so few are resident (B = 64 x V = 32,000: 11-12 against
    // 15.5-16.5 us per step).  Above that the extra blocks only add their
    // start-up and their meeting in the workspace (B = 64 x V = 128,256:
    // 17.3 against 11.2 us).
    int span = 32;
    if ((int64_t)b * ((V + kThreads * 32 - 1) / (kThreads * 32)) < kHalfSpanBlocks)
        span = 16;
    const int per_iter = kThreads * span;
    const int iters = (V + per_iter - 1) / per_iter;
    int want = (kTargetBlocks + b - 1) / b;
    want = want > iters ? iters : want;
    want = want > kMaxChunks ? kMaxChunks : want;
    want = want < 1 ? 1 : want;
    const int per = (iters + want - 1) / want;
    return {kThreads, per * per_iter, (iters + per - 1) / per, span};
}

// a ^ b ^ c in one v_bitop3_b32 (truth table 0x96); the compiler leaves
// the Philox rounds' three-way XORs as two instructions otherwise.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    return make_uint4(c0, c1, c2, c3);
}

// Word e (0 .. 3) of philox4x32_10's output, for a lane that needs only
// that word: the same ten rounds, the last of which computes only the
// product the word comes from (words 0 and 1 from the multiple of c2,
// words 2 and 3 from the multiple of c0) -- one 32 x 32 -> 64-bit
// multiply fewer per call.
__device__ __forceinline__ uint32_t philox4x32_10_word(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                       uint32_t k0, uint32_t k1, int e)
{
#pragma unroll
    for (int round = 0; round < 9; ++round) {
        if (round > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    const bool from_c2 = e < 2;
    const uint64_t p = (uint64_t)(from_c2 ? 0xCD9E8D57u : 0xD2511F53u) * (from_c2 ? c2 : c0);
    const uint32_t high = xor3((uint32_t)(p >> 32), from_c2 ? c1 : c3, from_c2 ? k0 : k1);
    return (e & 1) ? (uint32_t)p : high;
}

// ln of a positive normal binary32: x = m 2^e, m in [sqrt(1/2), sqrt(2));
// z = (m - 1) / (m + 1) with the reciprocal by four Newton steps from 1/2;
// ln m = 2 (z + z^3 (1/3 + w (1/5 + w (1/7 + w / 9)))), w = z^2;
// ln x = fma(e, ln 2, ln m).  Every operation is a rounded IEEE add,
// multiply or fused multiply-add, written out (no contraction).
__device__ __forceinline__ float ln_f32(float x)
{
#pragma clang fp contract(off)
    const uint32_t bits = __float_as_uint(x);
    int e = (int)(bits >> 23) - 127;
    uint32_t mb = (bits & 0x007FFFFFu) | 0x3F800000u;
    if (mb > 0x3FB504F3u) {
        mb -= 0x00800000u;
        e += 1;
    }
    const float f = __uint_as_float(mb) - 1.0f;
    const float d = f + 2.0f;
    float r = 0.5f;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const float t = __builtin_fmaf(-d, r, 1.0f);
        r = __builtin_fmaf(r, t, r);
    }
    const float z = f * r;
    const float w = z * z;
    float p = __builtin_fmaf(w, 0x1.c71c72p-4f, 0x1.24924ap-3f);
    p = __builtin_fmaf(w, p, 0x1.99999ap-3f);
    p = __builtin_fmaf(w, p, 0x1.555556p-2f);
    const float zw = z * w;
    const float half = __builtin_fmaf(zw, p, z);
    const float lnm = half + half;
    return __builtin_fmaf((float)e, 0x1.62e430p-1f, lnm);
}

__device__ __forceinline__ float gumbel_of_word(uint32_t w)
{
#pragma clang fp contract(off)
    const float u = (float)(2u * (w >> 9) + 1u) * 0x1p-24f;  // exact, strictly inside (0, 1)
    return -ln_f32(-ln_f32(u));
}

// An upper bound of gumbel_of_word(w) in one conversion each way and one
// fused multiply-add.  -ln u >= 1 - u, so G <= -ln(1 - u); 1 - u is at least
// 2^-32 f with f the word's complement without its low byte (exact in
// binary32; where it is zero, 1 - u is 2^-24), and log2 f is at least its
// linear interpolation between powers of two, which is f's bit pattern / 2^23
// - 127.  2^-10 covers the rounding of both sides (below 2^-15 together).
__device__ __forceinline__ float gumbel_bound_of_word(uint32_t w)
{
    const float f = (float)~(w | 0xFFu);
    return __builtin_fmaf((float)__float_as_uint(f), -0x1.62e430p-24f, 0x1.b8d874p+6f);
}

// Order-preserving key of a binary32 value: NaN ranks as -inf, -0.0 as
// +0.0; every value's key is > 0, so 0 stands for "nothing yet".  Adding
// +0.0 turns -0.0 into +0.0 and leaves every other value as it is (round to
// nearest); then negatives have all their bits flipped, the rest their sign.
__device__ __forceinline__ uint32_t order_key(float x)
{
#pragma clang fp contract(off)
    float c = x + 0.0f;
    c = c != c ? -__builtin_inff() : c;
    const uint32_t u = __float_as_uint(c);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// The value of an order key; NaN (nothing is below it) of 0, "nothing yet".
__device__ __forceinline__ float key_value(uint32_t k)
{
    return __uint_as_float(k & 0x80000000u ? k ^ 0x80000000u : ~k);
}

__device__ __forceinline__ uint64_t max_u64(uint64_t a, uint64_t b) { return a > b ? a : b; }

template <int DT>
__device__ __forceinline__ float logit_at(const char *row, int i)
{
    if constexpr (DT == 0)
        return reinterpret_cast<const float *>(row)[i];
    else
        return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(row)[i] << 16);
}

// The 4 logits of group g (tokens 4g .. 4g+3) as they lie in memory: one load
// at the row's own alignment (an element at a time, rows off 8 or 16 bytes took
// 16.8 us instead of 13.0 at 100 x 50,257).  The last group may run past V: its load ends at
// V instead, and group_value takes that into account.  Rows of fewer than 4
// tokens are read token by token.
template <int DT>
struct GroupWords;
template <>
struct GroupWords<0> {
    uint32_t w[4];
};
template <>
struct GroupWords<1> {
    uint64_t w;
};

template <int DT>
__device__ __forceinline__ GroupWords<DT> load_group(const char *row, uint32_t g, int V)
{
    constexpr int kElt = DT == 0 ? 4 : 2;
    GroupWords<DT> v;
    if (V >= 4) {
        const int i0 = min((int)(g * 4u), V - 4);
        __builtin_memcpy(&v, row + (size_t)i0 * kElt, 4 * kElt);
    } else {
        char *dst = reinterpret_cast<char *>(&v);
        for (int e = 0; e < 4; ++e)
            __builtin_memcpy(dst + e * kElt, row + (size_t)min(e, V - 1) * kElt, kElt);
    }
    return v;
}

// the logit of token 4g + e in group g's words, as a binary32 bit pattern
template <int DT>
__device__ __forceinline__ void group_values(GroupWords<DT> v, uint32_t g, int V, uint32_t (&x)[4])
{
    const int past = V >= 4 ? max((int)(g * 4u) + 4 - V, 0) : 0;  // 0 .. 3 tokens past V
    if constexpr (DT == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            x[e] = v.w[e];
        for (int k = 0; k < past; ++k) {
            x[0] = x[1];
            x[1] = x[2];
            x[2] = x[3];
        }
    } else {
        const uint64_t w = v.w >> (16 * past);
        x[0] = (uint32_t)w << 16;
        x[1] = (uint32_t)w & 0xFFFF0000u;
        x[2] = (uint32_t)(w >> 32) << 16;
        x[3] = (uint32_t)(w >> 32) & 0xFFFF0000u;
    }
}

// Inclusive prefix sum over the wave: within each row of 16 lanes by shifts of
// 1, 2, 4 and 8 lanes, then lane 15 of rows 0 and 2 into the row above and
// lane 31 into the upper two rows.  Two small counts share a word, so one scan
// serves both: six adds and no scalar registers, where the ballots of the
// counts' bits took about fifty instructions and twenty scalar registers (us
// per step with those and now, timed in turn: a twentieth of the tokens allowed
// 256 x 128,256 17.8 and 17.1, 8 x 32,000 5.7 and 5.5, 1,024 x 32,000 17.2 and
// 16.6; one in 500 256 x 128,256 12.1 and 11.2).
// Every lane of the wave must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}

__device__ __forceinline__ uint32_t wave_prefix(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xF>(v);  // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    v += dpp_or_zero<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// At most 80 scalar registers: with more a SIMD unit holds seven waves, not
// eight, and a launch that just fills the chip (2,048 blocks of 256 lanes, 512
// of 1,024) waits for a second round.  81 to 90 of them took 22.8 to 23.3 us
// instead of 20.6 at 256 x 128,256 and 26.7 instead of 22.3 at 1,024 x 32,000
// (about a twentieth of the tokens allowed).
template <int DT, int THREADS, int SPAN>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_num_sgpr(80))) void masked_sample_kernel(
    const int32_t *__restrict__ next_state, const uint32_t *__restrict__ allow, int S, int V, int W,
    const int32_t *__restrict__ states, const void *__restrict__ logits, int64_t ld, float inv_t, uint32_t seed_lo,
    uint32_t seed_hi, uint32_t off_lo, uint32_t off_hi, int chunk_tok, int nchunks, RowMeet meet,
    int32_t *__restrict__ token, int32_t *__restrict__ new_state)
{
#pragma clang fp contract(off)
    constexpr int kWaves = THREADS / kWave;
    static_assert(SPAN == 32 || SPAN == 16, "a whole allow word or one half of it per lane");
    constexpr int kTokPerIter = THREADS * SPAN;
    __shared__ uint32_t queue[kWaves][kWave * 8];  // up to 8 groups per lane per iteration, or 512 tokens
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int b = blockIdx.x / nchunks;
    const int c = blockIdx.x - b * nchunks;
    const int s = states[b];
    const bool live = (uint32_t)s < (uint32_t)S;  // block-uniform
    uint64_t best = 0;
    uint32_t wave_key = 0;          // wave-uniform order key of the best key this wave knows of
    __shared__ uint32_t block_key;  // and of the block's, over its waves
    if (tid == 0)
        block_key = 0;
    __syncthreads();
    if (live) {
        const char *row = static_cast<const char *>(logits) + (size_t)b * (size_t)ld * (DT == 0 ? 4 : 2);
        const uint32_t *arow = allow + (size_t)s * W;
        const int t0 = c * chunk_tok;
        const int t1 = min(V, t0 + chunk_tok);
        for (int base = t0; base < t1; base += kTokPerIter) {  // block-uniform trip count
            const int tok0 = base + tid * SPAN;  // a multiple of SPAN: the word's low or high half
            uint32_t word = tok0 < t1 ? arow[tok0 >> 5] : 0u;
            if constexpr (SPAN == 16)
                word = (word >> (tok0 & 16)) & 0xFFFFu;
            if (tok0 < t1 && t1 - tok0 < SPAN)
                word &= (1u << (t1 - tok0)) - 1u;  // a chunk ends inside this span only at V
            // groups (4 tokens) holding an allowed token: bit 4k of `nz`
            uint32_t nz = (word | (word >> 1) | (word >> 2) | (word >> 3)) & 0x11111111u;
            // token and group counts (at most 32 and 8 per lane), one per half
            const uint32_t counts = (uint32_t)__popc(word) | (uint32_t)__popc(nz) << 16;
            const uint32_t upto = wave_prefix(counts);
            const uint32_t all = lane_value(upto, kWave - 1);
            const int toks = (int)(all & 0xFFFFu), groups = (int)(all >> 16);
            const uint32_t before = upto - counts;
            const int tpos = (int)(before & 0xFFFFu), gpos = (int)(before >> 16);
            // wave-uniform: single tokens when they fit the queue and are few per group
            const bool by_token = toks <= kWave * 8 && 4 * toks <= kTokenRatio4 * groups;
            if (by_token) {
                int pos = tpos;
                uint32_t w = word;
                while (w) {
                    queue[wave][pos++] = (uint32_t)(tok0 + __builtin_ctz(w));
                    w &= w - 1u;
                }
            } else {
                int pos = gpos;
                while (nz) {
                    const int k = __builtin_ctz(nz) >> 2;
                    nz &= nz - 1u;
                    // token group index (token / 4) and its 4 mask bits
                    queue[wave][pos++] = ((uint32_t)((tok0 >> 2) + k) << 4) | ((word >> (4 * k)) & 0xFu);
                }
            }
            wave_lds_sync();
            if (by_token) {
                for (int q = lane; q < toks; q += kWave) {
                    const uint32_t i = queue[wave][q];
                    const float x = logit_at<DT>(row, (int)i);  // in flight during the Philox rounds
                    const uint32_t word =
                        philox4x32_10_word(i >> 2, (uint32_t)b, off_lo, off_hi, seed_lo, seed_hi, (int)(i & 3u));
                    const float key = __builtin_fmaf(x, inv_t, gumbel_of_word(word));
                    const uint64_t packed =
                        ((uint64_t)order_key(key) << 32) | (uint64_t)(0xFFFFFFFFu - i);
                    best = max_u64(best, packed);
                }
            } else {
                // Only a token whose bound (logit and gumbel_bound_of_word)
                // reaches the best key known needs its logarithm pair: one or
                // two passes in a wave's first trips, then hardly any.  Where
                // the best key is so low that it has swallowed the noise, a
                // lane that holds it passes over tokens of higher index that
                // could only tie: in rows that a filter left at -inf, or at a
                // large negative number, nearly all tokens do, and every trip
                // drew all four of a group.  us per step, all but 50 logits of
                // a row at -inf, 95 % of the tokens allowed, before and now:
                // bf16 128 x 128,256 42.6 and 26.4, fp32 64 x 32,000 13.5 and
                // 10.3 (other values 22.8 and 10.3).  Asked once a trip has
                // drawn a token, it costs other rows nothing; asked ahead of
                // that too, the first falls to 23.2 and they take 1 % longer.
                for (int q0 = 0; q0 < groups; q0 += kWave) {  // wave-uniform trip count
                    const uint32_t entry = q0 + lane < groups ? queue[wave][q0 + lane] : 0u;
                    const uint32_t g = entry >> 4;
                    uint32_t left = entry & 0xFu;
                    // the logits first: their load is in flight during the
                    // Philox rounds (a lane without a group reads group 0)
                    const GroupWords<DT> raw = load_group<DT>(row, g, V);
                    const uint32_t seen = __hip_atomic_load(&block_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const uint4 rnd = philox4x32_10(g, (uint32_t)b, off_lo, off_hi, seed_lo, seed_hi);
                    const uint32_t noise[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
                    uint32_t x[4];
                    group_values<DT>(raw, g, V, x);
                    const uint32_t others = __builtin_amdgcn_readfirstlane(seen);
                    wave_key = others > wave_key ? others : wave_key;
                    float floor = key_value(wave_key);
                    float bound[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        bound[e] = __builtin_fmaf(__uint_as_float(x[e]), inv_t, gumbel_bound_of_word(noise[e]));
                        left &= bound[e] < floor ? ~(1u << e) : ~0u;
                    }
                    if (__ballot(left != 0)) {
                        do {
                            // each lane's highest bound first (the lowest index
                            // of equals): the others seldom need their noise then
                            uint32_t pick = 0, px = 0, pw = 0;
                            float pb = -__builtin_inff();
#pragma unroll
                            for (int e = 3; e >= 0; --e)
                                if ((left & (1u << e)) && !(bound[e] < pb)) {
                                    pick = (uint32_t)e;
                                    px = x[e];
                                    pw = noise[e];
                                    pb = bound[e];
                                }
                            if (left) {
                                const float key = __builtin_fmaf(__uint_as_float(px), inv_t, gumbel_of_word(pw));
                                const uint32_t i = g * 4u + pick;
                                best = max_u64(best, (uint64_t)order_key(key) << 32 | (uint64_t)(0xFFFFFFFFu - i));
                                left &= ~(1u << pick);
                            }
                            const uint32_t k = wave_reduce<true>((uint32_t)(best >> 32));
                            wave_key = k > wave_key ? k : wave_key;
                            floor = key_value(wave_key);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                left &= bound[e] < floor ? ~(1u << e) : ~0u;
                            if (__builtin_expect(wave_key - 1u < kTieKey, 0) && (uint32_t)(best >> 32) == wave_key) {
                                const int own = (int)(0xFFFFFFFFu - (uint32_t)best - g * 4u);  // its place in the group
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    left &= e > own && bound[e] <= floor ? ~(1u << e) : ~0u;
                            }
                        } while (__ballot(left != 0));
                        if (lane == 0 && wave_key > others)
                            (void)__hip_atomic_fetch_max(&block_key, wave_key, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
            wave_lds_sync();  // every lane has read its entries before the next iteration writes
        }
    }
    // block-wide maximum
    __shared__ uint64_t red[THREADS / kWave];
    best = wave_reduce<true>(best);
    if (lane == 0)
        red[wave] = best;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w)
            best = max_u64(best, red[w]);
        if (nchunks == 1 || meet_row(meet, b, c, nchunks, best, best)) {  // else another block finishes the row
            const int tok = best ? (int)(0xFFFFFFFFu - (uint32_t)best) : -1;
            const bool found = live && tok >= 0 && tok < V;  // guards the read
            token[b] = found ? tok : -1;
            new_state[b] = found ? next_state[(size_t)s * V + tok] : -1;
        }
    }
}


}  // namespace

size_t sample_workspace_bytes(int B, int V)
{
    return row_meet_bytes_upto(B, sample_geometry(B, V).nchunks, kOneBlockRows);
}

hipError_t launch_masked_sample(const int32_t *next_state, const uint32_t *allow, int S, int V,
                                const int32_t *states, const void *logits, int dtype, int B, int64_t ld,
                                float inv_temperature, uint64_t seed, uint64_t offset, int32_t *token,
                                int32_t *new_state, void *workspace, hipStream_t stream)
{
    const int W = (V + 31) / 32;
    const SampleGeometry g = sample_geometry(B, V);
    const RowMeet meet = row_meet(workspace, B);
    const unsigned grid = (unsigned)B * (unsigned)g.nchunks;
    const uint32_t s_lo = (uint32_t)seed, s_hi = (uint32_t)(seed >> 32);
    const uint32_t o_lo = (uint32_t)offset, o_hi = (uint32_t)(offset >> 32);
#define DV_SAMPLE_LAUNCH(DT, T, SP)                                                                              \
    masked_sample_kernel<DT, T, SP><<<grid, T, 0, stream>>>(next_state, allow, S, V, W, states, logits, ld,      \
                                                            inv_temperature, s_lo, s_hi, o_lo, o_hi,             \
                                                            g.chunk_tok, g.nchunks, meet, token, new_state)
    if (g.threads == kRowThreads) {
        if (dtype == 0)
            DV_SAMPLE_LAUNCH(0, kRowThreads, 32);
        else
            DV_SAMPLE_LAUNCH(1, kRowThreads, 32);
    } else if (g.span == 32) {
        if (dtype == 0)
            DV_SAMPLE_LAUNCH(0, kThreads, 32);
        else
            DV_SAMPLE_LAUNCH(1, kThreads, 32);
    } else {
        if (dtype == 0)
            DV_SAMPLE_LAUNCH(0, kThreads, 16);
        else
            DV_SAMPLE_LAUNCH(1, kThreads, 16);
    }
#undef DV_SAMPLE_LAUNCH
    return hipGetLastError();
}

}  // namespace dv
