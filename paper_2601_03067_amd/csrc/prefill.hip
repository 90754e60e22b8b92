// Chunked-prefill attention over a fused cache with reuse of the work on fused blocks (motivation section: with
// chunked prefill, any softmax-attention computation that involves a fused block can be reused for the later
// instances of that block, and the result is the merge, with rescaling, of the fused part and the unique part).
//
// One request (Chunks Fast-Fusion is per request).  The queries are a run of tokens [q_begin, q_end) of one chunk
// that starts at token chunk_begin; the query at position pos sees the tokens 0 .. pos of the request through the
// block table: logical block x is scale_k[x] * K[bt[x]], scale_v[x] * V[bt[x]].
//
// What is reused.  Every logical block that ends before the chunk is visible to every query of the chunk.  Among
// those, the logical blocks that point at the same stored block p differ only by their two scale factors, so
//     logits of instance i   = scale_k[x_i] * (Q K_p^T)          -- one matrix product Q K_p^T for all instances
//     their weighted values  = (sum_i scale_v[x_i] P_i) V_p      -- one matrix product with V_p
// The host plan lists, per group, the distinct stored blocks of that part of the context with their instances'
// scale pairs; only the exponentials are taken per instance.  The blocks of the chunk itself (the unique part:
// blocks of one leaf never fuse with each other, and they need the causal mask) are walked one by one from the
// table.  With reuse switched off the plan lists every logical block as its own entry, which gives the baseline
// the reuse is measured against.
//
// Kernel: a workgroup of 4 wavefronts takes 4 x (32 / rep) consecutive query positions of one KV head; a wavefront
// owns (32 / rep) positions x rep query heads = 32 query rows.  The context is walked in tiles of 32 tokens (two
// 16-token pieces, each from one stored block with its own instance list) that the workgroup stages in LDS, double
// buffered, so every K and V byte is fetched once per workgroup.
//   logits^T = K Q^T with v_mfma_f32_32x32x16_bf16: K rows are the A operand as they lie in LDS, the query fragments
//   (B operand) stay in registers.  In the accumulator layout a lane then owns ONE query and 16 of the 32 tokens, so
//   the online softmax (per instance: exponentials of the scaled logits, weights summed with the value scales) is
//   lane-local up to one exchange with lane ^ 32, and so is every rescaling of the output.
//   out^T += V^T P^T: the weights of a lane are already a B operand (the order of the tokens inside the summation
//   index is free as long as both operands agree); V^T fragments come from the row-major V tile through the LDS
//   transpose read ds_read_b64_tr_b16 (16 lanes x 4 values: lane i receives element i & 3 of the rows that lanes
//   i >> 2, 4 + (i >> 2), 8 + (i >> 2), 12 + (i >> 2) point at -- so when source lane s points at 4 consecutive head
//   elements 4 (s & 3) .. of token (s >> 2), lane i ends up with head element i of 4 consecutive tokens).
//   Weights are split into a bfloat16 head and remainder (two MFMAs).
// bfloat16 pools only.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <new>
#include <type_traits>
#include <vector>

namespace kvfuse {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A distinct stored block of the part before the chunk.  Its first two scale pairs stand beside it, so that most tiles need
// one read of the table; the others are at inst_off + 2 ...
struct PEntry {          // 48 bytes; what a tile's weights need is one load of its first 32
    float2 first, second;
    float sk_max, sk_min;            // over the instances
    int32_t inst_off, inst_cnt;
    int32_t phys, pad[3];
};
static_assert(sizeof(PEntry) == 48, "read word by word");

struct PrefillArgs {
    const void *kpool, *vpool;
    const int32_t *bt;
    const float *scale_k, *scale_v;
    const void *q;
    const PEntry *entries;
    const float2 *inst;              // (scale_k, scale_v) of every instance
    const int32_t *entry_begin;      // [groups of the plan + 1]
    float *out;                      // [n_layers][Nq][Hq][D]
    int32_t P, n, t, kv_heads, layer_begin, Hq, rep, rep_pad, npw;
    int32_t req_start, q_begin, q_end, chunk_begin;
    uint64_t ppb_inv;                // 2^40 / pieces per block, rounded up
    float sm_scale;                  // its size; a negative one is turned into the sign of the queries
    uint32_t q_sign;                 // 0, or the sign bits of two bfloat16
    GroupsByXcd groups;              // (layer, KV head)
    Divisor heads;
};

// What this workgroup works on: all that read the keys and values of one (layer, KV head) are put on one XCD (us, by rows of the grid,
// which scatter them over all eight / like this: 2048 queries of a 32768-token prompt, 4 layers of 8 KV heads, 4541 / 4320; 31 of 7177
// tokens, 16 layers of 4, 96.7 / 64.0; 10 of 2012 tokens, 31 layers of 4, 31.6 / 25.0).  Fewer than eight groups, which share the XCDs in
// turn, gain too, three of them and five to seven among them (2048 queries of 32768 tokens, one to seven groups: 235 / 231, 467 / 449, 698 / 671,
// 1025 / 777, 1321 / 1030, 1326 / 1034, 1326 / 1087; 200 of 4296 tokens all 1 to 2 % faster, 1000 of 2000 in one and two groups 0.8 % slower,
// in the others 4 to 17 % faster).
struct PrefillPlace {
    int x, kvh, li;
};
__device__ static __forceinline__ PrefillPlace prefill_place(const PrefillArgs &A)
{
    uint32_t group, x;
    A.groups.place(blockIdx.x + A.groups.per_group.d * (blockIdx.y + (uint32_t)A.kv_heads * blockIdx.z), group, x);
    const uint32_t li = A.heads.of(group);
    return {(int)x, (int)(group - li * (uint32_t)A.kv_heads), (int)li};
}

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// The tables of a call: nothing writes them while it runs, so that a uniform word of theirs is a scalar load, also behind
// statements that the compiler takes for writes to memory.
#define KVF_TABLE __attribute__((address_space(4)))

// One 16-token piece of the context: the words that tables hold of it, as they come from memory.  Nothing is computed from
// them until they are used, a tile later, so that no wait stands between their loads; where they come from is a choice of
// addresses and not a branch.
struct PRows {              // where its rows are
    int32_t phys, sub;      // stored block, piece of that block
    int32_t tok_base;       // position of its first token for the causal test (very negative = visible to every query)
};
struct PScales {            // whose scale pairs apply
    int32_t inst_cnt, inst_off;
    float2 first, second;
    float sk_max, sk_min;   // of a stored block before the chunk
    int32_t tok_base;       // as above; kNowhere past the end of the walk
};
constexpr int32_t kBefore = -(1 << 30), kNowhere = 1 << 30;

// The context of a run of queries, piece by piece: the part before the chunk (distinct stored blocks with their instances),
// then the chunk's own blocks up to pos_last.  The piece's index is uniform over the wavefront, so its words are scalar loads.
template <int D>
struct PWalk {
    const bf16_t *kg, *vg;
    const KVF_TABLE int32_t *btg;
    const KVF_TABLE float *skg, *svg;
    const KVF_TABLE PEntry *eg;
    int ppb, last_block, n_pre, n_pieces;
    uint32_t inv_hi, inv_lo;                                     // 2^40 / ppb, rounded up

    __device__ __forceinline__ PWalk(const PrefillArgs &A, int kvh, int li, int pos_last)
    {
        const int gi = li * A.kv_heads + kvh;                    // group index within the plan
        const int g = (A.layer_begin + li) * A.kv_heads + kvh;
        const int64_t r = (int64_t)A.t * D;
        const int64_t x = (int64_t)g * A.n + A.req_start + A.chunk_begin / A.t;
        kg = (const bf16_t *)A.kpool + (int64_t)g * A.P * r;
        vg = (const bf16_t *)A.vpool + (int64_t)g * A.P * r;
        btg = (const KVF_TABLE int32_t *)(A.bt + x);             // the chunk's first block
        skg = (const KVF_TABLE float *)(A.scale_k + x);
        svg = (const KVF_TABLE float *)(A.scale_v + x);
        ppb = A.t / 16;                                          // pieces per block
        inv_hi = (uint32_t)(A.ppb_inv >> 32);
        inv_lo = (uint32_t)A.ppb_inv;
        eg = (const KVF_TABLE PEntry *)(A.entries + A.entry_begin[gi]);
        last_block = A.entry_begin[gi + 1] - A.entry_begin[gi] - 1;
        n_pre = (last_block + 1) * ppb;
        n_pieces = n_pre + (pos_last - A.chunk_begin) / 16 + 1;
    }

    // p / ppb, exact for p * ppb < 2^40
    __device__ __forceinline__ int block_of(int p) const
    {
        return (int)(((uint64_t)(uint32_t)p * inv_hi + __umulhi((uint32_t)p, inv_lo)) >> 8);
    }

    // past the end of the walk: the rows of the last piece (its values are not used, but they are there to be read)
    __device__ __forceinline__ PRows rows(const PrefillArgs &A, int p) const
    {
        p = min(p, n_pieces - 1);
        const bool pre = p < n_pre;
        const int q = pre ? p : p - n_pre, b = block_of(q);
        PRows rw;
        rw.phys = *(pre ? &eg[b].phys : &btg[b]);
        rw.sub = q - b * ppb;
        rw.tok_base = pre ? kBefore : A.chunk_begin + q * 16;
        return rw;
    }
    // first element of a piece's rows in the group's pool; a bad id in the table must not leave the pool
    __device__ __forceinline__ int64_t first_row(const PrefillArgs &A, const PRows &rw) const
    {
        return ((int64_t)min(max(rw.phys, 0), A.P - 1) * ppb + rw.sub) * (16 * D);
    }

    __device__ __forceinline__ PScales scales(const PrefillArgs &A, int p) const
    {
        const bool pre = p < n_pre;
        const int q = max(min(p, n_pieces - 1) - n_pre, 0);
        // no entries at all: unused words of the plan's own memory
        const KVF_TABLE PEntry *en = &eg[max(min(block_of(p), last_block), 0)];
        PScales sc;
        sc.inst_cnt = en->inst_cnt; sc.inst_off = en->inst_off;
        sc.first.x = *(pre ? &en->first.x : &skg[block_of(q)]);
        sc.first.y = *(pre ? &en->first.y : &svg[block_of(q)]);
        sc.second.x = en->second.x; sc.second.y = en->second.y;
        sc.sk_max = en->sk_max; sc.sk_min = en->sk_min;
        sc.tok_base = pre ? kBefore : p < n_pieces ? A.chunk_begin + q * 16 : kNowhere;
        return sc;
    }

    // the same of a piece before the chunk
    __device__ __forceinline__ PRows rows_before(int p) const
    {
        const int b = block_of(p);
        return PRows{eg[b].phys, p - b * ppb, kBefore};
    }
    __device__ __forceinline__ PScales scales_before(int p) const
    {
        typedef uint32_t words_t __attribute__((ext_vector_type(8), aligned(16)));
        const words_t w = *(const KVF_TABLE words_t *)&eg[block_of(p)];
        return PScales{(int32_t)w[7], (int32_t)w[6], make_float2(__uint_as_float(w[0]), __uint_as_float(w[1])),
                       make_float2(__uint_as_float(w[2]), __uint_as_float(w[3])), __uint_as_float(w[4]), __uint_as_float(w[5]), kBefore};
    }
};

// A uniform factor of vector instructions, in a vector register: gfx950 issues an fp32 multiplication, addition or fused one (and
// and, xor) whose operands are all vector registers at twice the rate of one with a scalar register among them (measured 1.05
// against 1.97 ns a wavefront and SIMD; so are shifts, maxima, v_perm and conversions, an exponential 3.4).
__device__ static __forceinline__ float vector_register(float x)
{
    asm("" : "+v"(x));
    return x;
}
__device__ static __forceinline__ uint32_t vector_register(uint32_t x)
{
    asm("" : "+v"(x));
    return x;
}

// The running maximum is taken before the softmax scale is applied, which must not turn it round: logits of a negative scale
// are those of its size and the queries' opposites.  (In the split kernel once the context's first table words are asked for, so
// that they do not wait for the queries: 46.7 -> 45.7 us for 200 queries of 4296 tokens.)
template <int KS>
__device__ static __forceinline__ void sign_queries(uint4 (&qf)[KS], uint32_t sign)
{
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        qf[ks] = make_uint4(qf[ks].x ^ sign, qf[ks].y ^ sign, qf[ks].z ^ sign, qf[ks].w ^ sign);
}

// max or sum over the two lanes that share a query row (lane, lane ^ 32)
__device__ static __forceinline__ float halves_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ static __forceinline__ float halves_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Online softmax of one tile for this lane's query row: z = the logits of 16 of the tile's 32 tokens (the other 16 are with
// lane ^ 32): accumulator i is token 8 (i / 4) + 4 h2 + i % 4 of the tile, i.e. piece i / 8.  pw = their weights summed over
// the instances of each piece, times the value scales; l_run sums the weights of this lane's tokens only.  Everything works
// in base 2: exp(x) = exp2(x * log2(e)), and v_exp_f32 is an exp2.
// Returns the factor that the sums so far are rescaled by.  (Letting the maximum lag by up to 2^8 would save most rescalings,
// but a row that sees a single token then loses the exact weight of one: error 1.9e-6 -> 2.4e-6 on short contexts.)
template <bool MASKED>
__device__ static __forceinline__ float tile_weights_as(const PrefillArgs &A, const PScales &s0, const PScales &s1, const floatx16 &z,
                                                        int h2, int my_pos, float &m_run, float &l_run, float (&pw)[16])
{
    const float base = A.sm_scale * 1.4426950408889634f;
    // tokens of a piece that this row sees: those whose offset from the lane's first one (i % 4, + 8) is at most `last`
    const int last0 = my_pos - s0.tok_base - 4 * h2, last1 = my_pos - s1.tok_base - 4 * h2;
    auto seen = [&](int i) __attribute__((always_inline)) {
        return !MASKED || 8 * ((i >> 2) & 1) + (i & 3) <= (i < 8 ? last0 : last1);
    };
    // ---- the largest scaled logit of each piece: a product's extremes lie at the extremes of its factors
    float bmax = -INFINITY;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const PScales &sc = half ? s1 : s0;
        const bool own = MASKED && sc.tok_base >= 0;
        const float big = own ? sc.first.x : sc.sk_max, small = own ? sc.first.x : sc.sk_min;
        float hi = -INFINITY, lo = INFINITY;
#pragma unroll
        for (int i = 8 * half; i < 8 * half + 8; ++i)
            hi = fmaxf(hi, seen(i) ? z[i] : -INFINITY);
        if (hi > -INFINITY)
            bmax = fmaxf(bmax, fmaxf(hi * big, hi * small));
        if (small < 0.0f) {
#pragma unroll
            for (int i = 8 * half; i < 8 * half + 8; ++i)
                lo = fminf(lo, seen(i) ? z[i] : INFINITY);
            if (lo < INFINITY)
                bmax = fmaxf(bmax, fmaxf(lo * big, lo * small));
        }
    }
    const float m_new = fmaxf(m_run, halves_max(bmax) * base);
    const float corr = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);      // 0 on the first visible tile
    m_run = m_new;
    float psum = 0.0f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const PScales &sc = half ? s1 : s0;
        const float zs = base * sc.first.x, sv = vector_register(sc.first.y);
#pragma unroll
        for (int i = 8 * half; i < 8 * half + 8; ++i) {
            const float e = __builtin_amdgcn_exp2f(fmaf(z[i], zs, -m_new));
            const float pr = seen(i) ? e : 0.0f;
            psum += pr;
            pw[i] = pr * sv;
        }
        const int n_inst = MASKED && sc.tok_base >= 0 ? 1 : sc.inst_cnt;
        if (n_inst > 1) {                // before the chunk, and visible to every query
            float2 next = sc.second;
            for (int q = 1; q < n_inst; ++q) {
                const float zq = base * next.x, vq = vector_register(next.y);
                if (q + 1 < n_inst) {
                    const KVF_TABLE float2 *in = (const KVF_TABLE float2 *)A.inst + (sc.inst_off + q + 1);
                    next.x = in->x;
                    next.y = in->y;
                }
#pragma unroll
                for (int i = 8 * half; i < 8 * half + 8; ++i) {
                    const float pr = __builtin_amdgcn_exp2f(fmaf(z[i], zq, -m_new));
                    psum += pr;
                    pw[i] = fmaf(pr, vq, pw[i]);
                }
            }
        }
    }
    l_run = l_run * corr + psum;
    return corr;
}

__device__ static __forceinline__ float tile_weights(const PrefillArgs &A, const PScales &s0, const PScales &s1, const floatx16 &z,
                                                     int h2, int my_pos, float &m_run, float &l_run, float (&pw)[16])
{
    if (s0.tok_base >= 0 || s1.tok_base >= 0)
        return tile_weights_as<true>(A, s0, s1, z, h2, my_pos, m_run, l_run, pw);
    return tile_weights_as<false>(A, s0, s1, z, h2, my_pos, m_run, l_run, pw);
}

// The weights as B operands: the 8 values of MFMA jj are accumulators 8 jj .. 8 jj + 7, as a bfloat16 head (nearest) plus
// the bfloat16 of what is left.  Two values at a time: one conversion each for both heads and both rests.  (Left to itself the
// compiler converts every head twice, once to subtract it.)
__device__ static __forceinline__ void split_weights(const float (&pw)[16], bf16x8 (&p_hi)[2], bf16x8 (&p_lo)[2])
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const uint32_t upper = vector_register(0xFFFF0000u);
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = pw[8 * jj + 2 * e], b = pw[8 * jj + 2 * e + 1];
            hi[e] = vector_register(__builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b}));
            lo[e] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)(a - __uint_as_float(hi[e] << 16)), (__bf16)(b - __uint_as_float(hi[e] & upper))});
        }
        p_hi[jj] = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
        p_lo[jj] = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
    }
}

// N times 1 KB from `base` (uniform), 16 bytes per lane from off[i] + 1024 i, straight into LDS, end to end from `to` (uniform): the
// instruction's offset counts on either side.  In assembly, because the compiler makes every LDS read wait for all such loads of its
// own, whichever buffer they are for; who issues one waits for it by hand.  (No register is loaded.  The pause is for scalar registers that
// a vector instruction has just written, and for m0.)
template <int N>
__device__ static __forceinline__ void load_to_lds(uint64_t base, const uint32_t (&off)[N], uint32_t to)
{
    typedef uint32_t desc_t __attribute__((ext_vector_type(4)));
    const desc_t desc = {(uint32_t)base, (uint32_t)(base >> 32), 0xFFFFFFFFu, 0x00020000u};
    static_assert(N == 2 || N == 4, "16 rows of 128 or 256 bytes");
    if constexpr (N == 4)
        asm volatile("s_mov_b32 m0, %5\n\ts_nop 4\n\t"
                     "buffer_load_dwordx4 %0, %4, 0 offen lds\n\t"
                     "buffer_load_dwordx4 %1, %4, 0 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %2, %4, 0 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %3, %4, 0 offen offset:3072 lds" ::"v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(desc), "s"(to) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 4\n\t"
                     "buffer_load_dwordx4 %0, %2, 0 offen lds\n\t"
                     "buffer_load_dwordx4 %1, %2, 0 offen offset:1024 lds" ::"v"(off[0]), "v"(off[1]), "s"(desc), "s"(to) : "memory", "m0");
}

// WAVES: wavefronts of a SIMD that the registers are for, see roomy_pays.
template <int D, int WAVES>
__global__ __launch_bounds__(256, WAVES) void prefill_attn_kernel(PrefillArgs A)
{
    typedef bf16_t T;
    constexpr int KS = D / 16;                 // MFMA steps along the head dimension for the logits
    constexpr int DT = D / 32;                 // 32-row tiles of out^T
    constexpr int ROW = D * 2;                 // bytes of a token row
    constexpr int RCH = D / 8;                 // 16-byte chunks of a token row
    constexpr int TILE = 32 * ROW;             // bytes of a tile, per tensor
    constexpr int NLD = 16 * ROW / 1024;       // 1 KB loads of a 16-token piece
    constexpr bool ROOMY = WAVES < 3;
    constexpr int BUFS = ROOMY ? 3 : 2;        // tiles in LDS: one in use, the others on their way
    constexpr int KQ = ROOMY ? 0 : KS - 4;     // query fragments that live in LDS

    // K rows, then V rows, of each tile.  The loads write a row's 16-byte chunks end to end, so what padding would do is done by
    // the order of the chunks: chunk c of row r is at c ^ k_swizzle(r) / c ^ v_swizzle(r) (conflict-free 16-byte row reads of 16
    // consecutive rows; conflict-free transpose reads of 64 bytes of 4 consecutive rows).
    __shared__ __attribute__((aligned(1024))) char lds[BUFS][2][TILE];
    __shared__ __attribute__((aligned(16))) uint4 q_lds[4][KQ > 0 ? KQ : 1][64];
    auto k_swizzle = [](int r) __attribute__((always_inline)) { return RCH == 16 ? r & 15 : (r >> 1) & 7; };
    auto v_swizzle = [](int r) __attribute__((always_inline)) { return RCH == 16 ? (r & 3) * 4 : ((r >> 1) & 1) * 4; };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PrefillPlace place = prefill_place(A);
    const int kvh = place.kvh, li = place.li;

    // rows of this wavefront: lane & 31 = query row, lane >> 5 = which half of the tokens / head elements it holds
    const int qrow = lane & 31, h2 = lane >> 5;
    const int wg_first = A.q_begin + place.x * 4 * A.npw;
    const int pos_last_wg = min(A.q_end - 1, wg_first + 4 * A.npw - 1);
    const int pos_first = wg_first + wave * A.npw;                // may lie past the end: such a wavefront only helps loading
    const bool wave_live = pos_first < A.q_end;
    const int pos_last = min(A.q_end - 1, pos_first + A.npw - 1);
    const int rs = qrow / A.rep_pad, hh = qrow - rs * A.rep_pad;
    const bool row_used = wave_live && pos_first + rs <= pos_last && hh < A.rep;
    const int my_pos = wave_live ? min(pos_first + rs, pos_last) : A.q_end - 1;   // unused rows mask like a real one

    // B operand of step ks: head elements 16 ks + 8 h2 .. + 7 of the row.  Where a third wavefront of the SIMD needs the
    // registers, all but four of them live in LDS.
    uint4 qf[KS - KQ], q[KS];
    {
        const int64_t qi = (int64_t)li * (A.q_end - A.q_begin) + (my_pos - A.q_begin);
        const T *qp = (const T *)A.q + (qi * A.Hq + (int64_t)kvh * A.rep + (row_used ? hh : 0)) * D + 8 * h2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            q[ks] = row_used ? *reinterpret_cast<const uint4 *>(qp + 16 * ks) : make_uint4(0, 0, 0, 0);
    }

    auto place_queries = [&]() __attribute__((always_inline)) {
        sign_queries(q, A.q_sign);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            if (ks < KS - KQ)
                qf[ks] = q[ks];
            else
                q_lds[wave][ks - (KS - KQ)][lane] = q[ks];
    };
    if constexpr (!ROOMY)
        place_queries();

    const PWalk<D> walk(A, kvh, li, pos_last_wg);
    const int n_tiles = (walk.n_pieces + 1) / 2;

    // ---- loaders: a wavefront fetches one of a tile's two pieces of one tensor, 16 rows end to end, straight into LDS.  The
    // piece's address is uniform, so it goes into the descriptor.
    const int piece = wave & 1, tensor = wave >> 1;
    const bf16_t *my_pool = tensor ? walk.vg : walk.kg;
    auto address_of = [&](const PRows &rw) __attribute__((always_inline)) { return (uint64_t)(uintptr_t)(my_pool + walk.first_row(A, rw)); };
    // This lane's 16 bytes of each of the piece's 1 KB loads.  The swizzles of a load's rows are those of the first one's, but for bit 2 and
    // up of a K chunk, which is flipped by the load's number: what is to be added is 1024 i, and the load's own offset does that.
    const uint32_t ld_row = lane / RCH, ld_flip = tensor ? 0 : 64;
    const uint32_t ld_off = ld_row * ROW + ((lane % RCH) ^ (tensor ? v_swizzle(ld_row) : k_swizzle(ld_row))) * 16;
    auto load = [&](int buf, uint64_t from) __attribute__((always_inline)) {
        const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)&lds[buf][tensor][piece * 16 * ROW];
        uint32_t off[NLD];
        off[0] = ld_off;
        asm volatile("" : "+v"(off[0]));         // (the others are worked out anew for every tile: kept, they would cost registers)
#pragma unroll
        for (int i = 1; i < NLD; ++i)
            off[i] = off[0] ^ (ld_flip * i);
        load_to_lds(from, off, to);
    };

    float m_run = -INFINITY, l_run = 0.0f;       // running maximum in base-2 units, running sum
    floatx16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            o[dt][i] = 0.0f;

    // this lane's addresses inside a tile: K row for the logits, V patch (8 bytes of a row) for the transpose reads
    const int k_off = qrow * ROW + (h2 ^ k_swizzle(qrow)) * 16;
    const int l16 = lane & 15;
    const int v_row = 4 * h2 + (l16 >> 2);
    const int v_off = v_row * ROW + ((2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1)) ^ v_swizzle(v_row)) * 16 + 8 * (l16 & 1);

    // Bound: the softmax's vector instructions beside the matrix instructions of a SIMD's other wavefronts (per tile some 220 of
    // the former, 24 of the latter; vector ALU busy 75 %, matrix units 51 %), at the clock that the board's power leaves for
    // both (1.7 GHz at 1325 of 1400 W).  2048 queries of a 32768-token prompt, 4 layers of 8 KV heads, a third of the blocks fused:
    // 7.15 -> 5.6 ms since table words and fragments come ahead of their use and the maximum is taken before the scales are
    // applied; -> 5.2 ms since the tiles go straight into LDS and a third wavefront fits a SIMD; -> 4.5 ms since a tile takes 80 vector
    // instructions less (addresses of its loads, the weights' halves, uniform factors in vector registers) and the tiles before the
    // chunk have a loop of their own; -> 4.3 ms since a context's readers share an XCD.
    // Everything of a tile that waits for LDS is asked for at once, a product or a softmax ahead of its use: the K fragments
    // before the first product, the V fragments and the next tiles' table words (which wait on the same counter) before the
    // softmax.  The compiler left to itself reads one fragment, waits, multiplies.
    auto compute = [&](auto before, const PScales &s0, const PScales &s1, int buf, auto &&tables) __attribute__((always_inline)) {
        // (worked out anew for every tile: kept, the sixteen addresses of a tile would cost the registers of a third wavefront)
        int k_at = k_off, v_at = v_off;
        asm volatile("" : "+v"(k_at), "+v"(v_at));
        const char *kt = &lds[buf][0][0], *vtile = &lds[buf][1][0];
        uint4 ka[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            ka[ks] = *reinterpret_cast<const uint4 *>(kt + (k_at ^ (ks * 32)));
        __builtin_amdgcn_sched_barrier(0);
        // ---- logits^T of the tile: 32 tokens x 32 query rows
        floatx16 z;
        uint4 qa[4];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            z[i] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[ks & 3]), __builtin_bit_cast(bf16x8, ks < KS - KQ ? qf[ks < KS - KQ ? ks : 0] : qa[ks & 3]), z, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 4 < KS) {
                ka[ks & 3] = *reinterpret_cast<const uint4 *>(kt + (k_at ^ ((ks + 4) * 32)));
                if constexpr (KQ > 0)
                    qa[ks & 3] = q_lds[wave][ks][lane];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        bf16x4 vt[2][DT][2];
        auto read_v = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const char *vp = vtile + (v_at ^ (dt * 64)) + 16 * jj * ROW;
                    vt[jj][dt][0] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)(vp));
                    vt[jj][dt][1] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4 *)(vp + 8 * ROW));
                }
        };
        if constexpr (ROOMY)
            read_v();
        tables();
        __builtin_amdgcn_sched_barrier(0);
        float pw[16];
        const float corr = before ? tile_weights_as<false>(A, s0, s1, z, h2, my_pos, m_run, l_run, pw)
                                  : tile_weights(A, s0, s1, z, h2, my_pos, m_run, l_run, pw);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!ROOMY)
            read_v();
        if (!before && max(s0.tok_base, s1.tok_base) + 15 > pos_last_wg) {
            // values of tokens that no query of this workgroup may see can be anything (tail of the last block): zero
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if ((jj ? s1 : s0).tok_base + 8 * (e >> 2) + 4 * h2 + (e & 3) > pos_last_wg)
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt)
                            vt[jj][dt][e >> 2][e & 3] = (__bf16)0.0f;
        }
        if (__builtin_amdgcn_ballot_w64(corr != 1.0f)) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    o[dt][i] *= corr;
        }
        bf16x8 p_hi[2], p_lo[2];
        split_weights(pw, p_hi, p_lo);
        // ---- out^T += V^T P^T
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const bf16x8 va = __builtin_shufflevector(vt[jj][dt][0], vt[jj][dt][1], 0, 1, 2, 3, 4, 5, 6, 7);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, p_hi[jj], o[dt], 0, 0, 0);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, p_lo[jj], o[dt], 0, 0, 0);
            }
    };

    // The next BUFS - 1 tiles are on their way while one is multiplied.  Where the registers are for three wavefronts a SIMD, the loads go
    // on past the last tile with the last piece's rows: a look at the tile's number costs long walks more (2048 queries of 32768
    // tokens, 4 layers: 5.27 against 5.13 - 5.21 ms) than such loads do.  The roomier kernel, whose grids are small and walks can be a
    // few tiles, neither waits for two tiles that nobody needs nor, before its first loads, for the queries (65 queries of
    // 109 tokens, 21 layers of 8 KV heads, 2 query heads each: 19.0 -> 17.1 us).
    PRows next = walk.rows(A, 2 * (BUFS - 1) + piece);
    PScales s0 = walk.scales(A, 0), s1 = walk.scales(A, 1), n0, n1;
    uint64_t first[BUFS - 1];
#pragma unroll
    for (int i = 0; i < BUFS - 1; ++i)
        first[i] = address_of(walk.rows(A, 2 * i + piece));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (ROOMY)
        place_queries();
#pragma unroll
    for (int i = 0; i < BUFS - 1; ++i)
        if (!ROOMY || i < n_tiles)
            load(i, first[i]);
    int buf = 0, ahead = BUFS - 1;
    auto tile = [&](auto before, int ti) __attribute__((always_inline)) {
        // Tile ti has landed, for every wavefront behind the barrier; and every wavefront is done with tile ti - 1, whose place
        // the next load takes.
        if (!before && ROOMY && ti + 1 == n_tiles)
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((BUFS - 2) * NLD) : "memory");
        if (before || !ROOMY || ti + BUFS - 1 < n_tiles)
            load(ahead, address_of(next));
        compute(before, s0, s1, buf, [&]() __attribute__((always_inline)) {
            next = before ? walk.rows_before(2 * (ti + BUFS) + piece) : walk.rows(A, 2 * (ti + BUFS) + piece);
            n0 = before ? walk.scales_before(2 * (ti + 1)) : walk.scales(A, 2 * (ti + 1));
            n1 = before ? walk.scales_before(2 * (ti + 1) + 1) : walk.scales(A, 2 * (ti + 1) + 1);
        });
        s0 = n0;
        s1 = n1;
        ahead = buf;
        buf = buf + 1 == BUFS ? 0 : buf + 1;
    };
    // The tiles that lie before the chunk with all that is fetched meanwhile, which is most of a long walk, need no choice between entries
    // and table, and no masks.
    const int n_before = min(walk.n_pre / 2 - BUFS, n_tiles);
    int ti = 0;
    for (; ti < n_before; ++ti)
        tile(std::true_type{}, ti);
    for (; ti < n_tiles; ++ti)
        tile(std::false_type{}, ti);
    if constexpr (!ROOMY)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may leave while loads are on their way into LDS
    l_run = halves_sum(l_run);

    // ---- normalise and store: this lane holds out[row qrow][head element 32 dt + 8 (i / 4) + 4 h2 + i % 4]
    if (row_used) {
        const float inv = l_run > 0.0f ? 1.0f / l_run : 0.0f;
        const int64_t qi = (int64_t)li * (A.q_end - A.q_begin) + (pos_first + rs - A.q_begin);
        float *dst = A.out + (qi * A.Hq + (int64_t)kvh * A.rep + hh) * D + 4 * h2;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<float4 *>(dst + 32 * dt + 8 * g4) =
                    make_float4(o[dt][4 * g4] * inv, o[dt][4 * g4 + 1] * inv, o[dt][4 * g4 + 2] * inv, o[dt][4 * g4 + 3] * inv);
    }
}

// The same attention for few queries: one set of 32 query rows per workgroup, the context dealt out to its 8 wavefronts tile
// by tile.  Every wavefront fetches its own tiles straight into registers and needs no one else until the sums are merged
// through LDS at the end: no barriers, no staging, so eight tiles are in flight per workgroup.  The staged kernel shares
// every tile among 4 x 32 rows instead, which is the better trade once its own grid fills the chip.  Bound: latency of a tile
// (table words, rows, two products, one after the other; some 650 instructions, of which a wavefront issues one in seven
// cycles); 200 queries of 4296 tokens, 8 KV heads: 252 -> 45 us.
//   V^T fragment dt of a lane (m = lane & 31): element dt of the DT consecutive head elements DT m .. that it loads of its 8
//   tokens, one v_perm per two values; the tokens are those whose weights the lane already holds.
constexpr int kSplitWaves = 8;
template <int D>
__global__ __launch_bounds__(64 * kSplitWaves, 2) void prefill_split_kernel(PrefillArgs A)
{
    constexpr int KS = D / 16;                 // MFMA steps along the head dimension for the logits
    constexpr int DT = D / 32;                 // 32-row tiles of out^T = head elements of a V row per lane
    typedef uint32_t vrow_t __attribute__((ext_vector_type(DT / 2)));

    __shared__ __attribute__((aligned(16))) float4 s_o[kSplitWaves / 2][4 * DT][64];
    __shared__ float2 s_ml[kSplitWaves / 2][64];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PrefillPlace place = prefill_place(A);
    const int kvh = place.kvh, li = place.li;
    const int qrow = lane & 31, h2 = lane >> 5;
    const int pos_first = A.q_begin + place.x * A.npw;
    const int pos_last = min(A.q_end - 1, pos_first + A.npw - 1);
    const int rs = qrow / A.rep_pad, hh = qrow - rs * A.rep_pad;
    const bool row_used = pos_first + rs <= pos_last && hh < A.rep;
    const int my_pos = min(pos_first + rs, pos_last);             // unused rows mask like a real one
    const int64_t qi = (int64_t)li * (A.q_end - A.q_begin) + (my_pos - A.q_begin);

    uint4 qf[KS];                                     // B operand of step ks: head elements 16 ks + 8 h2 .. + 7 of the row
    {
        const bf16_t *qp = (const bf16_t *)A.q + (qi * A.Hq + (int64_t)kvh * A.rep + (row_used ? hh : 0)) * D + 8 * h2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qf[ks] = row_used ? *reinterpret_cast<const uint4 *>(qp + 16 * ks) : make_uint4(0, 0, 0, 0);
    }
    const PWalk<D> walk(A, kvh, li, pos_last);
    const int n_tiles = (walk.n_pieces + 1) / 2;

    float m_run = -INFINITY, l_run = 0.0f;
    floatx16 o[DT];                            // o[dt][i]: head element DT (8 (i / 4) + 4 h2 + i % 4) + dt of this lane's row
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            o[dt][i] = 0.0f;

    PRows r0 = walk.rows(A, 2 * wave), r1 = walk.rows(A, 2 * wave + 1);       // a tile ahead of their use
    PScales n0 = walk.scales(A, 2 * wave), n1 = walk.scales(A, 2 * wave + 1);
    __builtin_amdgcn_sched_barrier(0);
    sign_queries(qf, A.q_sign);
    auto tile = [&](auto before, int ti) __attribute__((always_inline)) {
        const int64_t u0 = walk.first_row(A, r0), u1 = walk.first_row(A, r1);
        const PScales s0 = n0, s1 = n1;
        uint4 ka[KS];
        vrow_t vr[2][8];                       // [piece][token slot e]: token 8 (e / 4) + 4 h2 + e % 4 of the piece
        const bf16_t *kp = walk.kg + ((qrow & 16) ? u1 : u0) + (qrow & 15) * D + 8 * h2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            ka[ks] = *reinterpret_cast<const uint4 *>(kp + 16 * ks);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                vr[jj][e] = *reinterpret_cast<const vrow_t *>(walk.vg + (jj ? u1 : u0) + (8 * (e >> 2) + 4 * h2 + (e & 3)) * D + DT * qrow);
        const int p = 2 * (ti + kSplitWaves);
        r0 = before ? walk.rows_before(p) : walk.rows(A, p);
        r1 = before ? walk.rows_before(p + 1) : walk.rows(A, p + 1);
        n0 = before ? walk.scales_before(p) : walk.scales(A, p);
        n1 = before ? walk.scales_before(p + 1) : walk.scales(A, p + 1);
        __builtin_amdgcn_sched_barrier(0);     // all loads of the tile are on their way before the first wait
        floatx16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            z[i] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[ks]), __builtin_bit_cast(bf16x8, qf[ks]), z, 0, 0, 0);
        float pw[16];
        const float corr = before ? tile_weights_as<false>(A, s0, s1, z, h2, my_pos, m_run, l_run, pw)
                                  : tile_weights(A, s0, s1, z, h2, my_pos, m_run, l_run, pw);
        if (!before && (s0.tok_base >= 0 || s1.tok_base >= 0)) {
            // values of tokens that no query of this workgroup may see can be anything (tail of the last block): zero
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const PScales &sc = jj ? s1 : s0;
                    if (sc.tok_base + 8 * (e >> 2) + 4 * h2 + (e & 3) > pos_last)
                        vr[jj][e] = (vrow_t)(0u);
                }
        }
        if (__builtin_amdgcn_ballot_w64(corr != 1.0f)) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    o[dt][i] *= corr;
        }
        bf16x8 p_hi[2], p_lo[2];
        split_weights(pw, p_hi, p_lo);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const uint32_t sel = (dt & 1) ? 0x07060302u : 0x05040100u;
                uint4 va;
                va.x = __builtin_amdgcn_perm(vr[jj][1][dt / 2], vr[jj][0][dt / 2], sel);
                va.y = __builtin_amdgcn_perm(vr[jj][3][dt / 2], vr[jj][2][dt / 2], sel);
                va.z = __builtin_amdgcn_perm(vr[jj][5][dt / 2], vr[jj][4][dt / 2], sel);
                va.w = __builtin_amdgcn_perm(vr[jj][7][dt / 2], vr[jj][6][dt / 2], sel);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va), p_hi[jj], o[dt], 0, 0, 0);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va), p_lo[jj], o[dt], 0, 0, 0);
            }
    };
    // (as in the staged kernel: the tiles that lie before the chunk, with the one whose words are fetched meanwhile, apart)
    int ti = wave;
    for (; ti + kSplitWaves < walk.n_pre / 2; ti += kSplitWaves)
        tile(std::true_type{}, ti);
    for (; ti < n_tiles; ti += kSplitWaves)
        tile(std::false_type{}, ti);

    l_run = halves_sum(l_run);
    // ---- merge: the upper half of the wavefronts hands its state to the lower half, lane by lane, until one is left
    for (int half = kSplitWaves / 2; half > 0; half >>= 1) {
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    s_o[wave - half][4 * dt + v][lane] = make_float4(o[dt][4 * v], o[dt][4 * v + 1], o[dt][4 * v + 2], o[dt][4 * v + 3]);
            s_ml[wave - half][lane] = make_float2(m_run, l_run);
        }
        __syncthreads();
        if (wave < half) {
            const float2 ml = s_ml[wave][lane];
            const float m_new = fmaxf(m_run, ml.x);
            const float fa = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_new);
            const float fb = ml.x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml.x - m_new);
            l_run = l_run * fa + ml.y * fb;
            m_run = m_new;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float4 b = s_o[wave][4 * dt + v][lane];
                    o[dt][4 * v] = o[dt][4 * v] * fa + b.x * fb;
                    o[dt][4 * v + 1] = o[dt][4 * v + 1] * fa + b.y * fb;
                    o[dt][4 * v + 2] = o[dt][4 * v + 2] * fa + b.z * fb;
                    o[dt][4 * v + 3] = o[dt][4 * v + 3] * fa + b.w * fb;
                }
        }
        __syncthreads();
    }
    if (wave == 0 && row_used) {
        const float inv = l_run > 0.0f ? 1.0f / l_run : 0.0f;
        float *dst = A.out + (qi * A.Hq + (int64_t)kvh * A.rep + hh) * D;
        typedef float orow_t __attribute__((ext_vector_type(DT)));
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            orow_t w;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                w[dt] = o[dt][i] * inv;
            *reinterpret_cast<orow_t *>(dst + DT * (8 * (i >> 2) + 4 * h2 + (i & 3))) = w;
        }
    }
}

// Whether the split kernel is the faster one, for a walk of `tiles` tiles: grids of the staged kernel of up to 192 workgroups, and
// among them those for which the rounds of split workgroups that the chip runs, one (head size 128) or two (64) per compute
// unit, cost less than one round of staged ones.  In units of a staged tile (1.7 / 1.4 us): 3.5 + tiles for the staged kernel, 4.2 +
// 0.2 tiles for a round of the other.  Both measured (us, staged / split; 4 query heads per KV head, three in ten blocks before the
// chunk fused away), by workgroups of the staged grid, head size 128:
//   tokens   up to 64      128          192          256       head size 64, 192
//      64    9.4 / 8.9   10.0 / 16.4                               7.9 / 8.2
//     128   12.5 / 9.3   13.0 / 17.0  13.8 / 24.4                 10.9 / 12.0
//     256   17.0 / 10.8  17.9 / 20.1  19.7 / 29.0                 15.0 / 14.2
//     512   28.1 / 14.5  30.1 / 26.7  31.2 / 38.1  34.2 / 51.5    23.9 / 18.1
//    1024   45.2 / 17.7  51.4 / 32.3  52.1 / 47.9  53.3 / 62.9    43.7 / 24.4
//    4096    178 / 46     178 / 87     168 / 120    182 / 165      155 / 62
// (Both kernels have become 2 to 15 % faster since, which leaves the line where it is.)
// (Without the second condition 96 queries over 112 tokens, 16 layers of one KV head, took 23.4 us where the staged kernel
// takes 13.5.)
constexpr int64_t kSplitBelow = 192;

static bool split_pays(int64_t staged_wgs, int64_t split_wgs, int64_t tiles, int d)
{
    const int64_t half_rounds = std::max<int64_t>(2, (split_wgs + 255) / 256 * (d == 64 ? 1 : 2));
    return staged_wgs <= kSplitBelow && half_rounds * (42 + 2 * tiles) < 2 * (35 + 10 * tiles);
}

// Head size 128: whether the staged kernel's registers are for two wavefronts per SIMD (all queries in them, V rows read before the
// softmax, two tiles on their way) or for three.  Grids of at most two workgroups per compute unit never have a third; and where
// most of a walk is the chunk itself, so that workgroups differ in length, up to 640 workgroups go to compute units that get free
// better than three at a time to some of them.  Both measured (us, two / three; 8 KV heads, 4 query heads each, three in ten blocks
// before the chunk fused away), by workgroups: 304 43.5 / 45.9; 416 118.2 / 116.5; 512 147.1 / 148.3; 552, three quarters of the
// context before the chunk 658 / 543; 576, all of it in the chunk 169 / 191; 752, likewise 291 / 223; 2048 6515 / 6105.
static bool roomy_pays(int64_t staged_wgs, int64_t tiles_before, int64_t tiles)
{
    return staged_wgs <= (2 * tiles_before < tiles ? 640 : 512);
}

static int pad_pow2_p(int rep)
{
    int p = 1;
    while (p < rep)
        p <<= 1;
    return p;
}

}  // namespace kvfuse

using namespace kvfuse;

struct kvfuse_prefill_plan {
    int32_t dtype = 0, P = 0, n = 0, t = 0, d = 0, G = 0;
    int32_t kv_heads = 0, layer_begin = 0, n_layers = 0, Hq = 0, rep = 0, rep_pad = 0, npw = 1;
    int32_t req_start = 0, q_begin = 0, q_end = 0, chunk_begin = 0;
    std::vector<PEntry> entries;
    std::vector<float2> inst;
    std::vector<int32_t> entry_begin;
    kvfuse_prefill_plan_info info = {};
    size_t off_entries = 0, off_inst = 0, off_begin = 0, bytes = 0;
    char *dev = nullptr;
};

static size_t up256p(size_t x) { return (x + 255) & ~(size_t)255; }

extern "C" {

int kvfuse_prefill_plan_build(kvfuse_ctx *ctx, const kvfuse_pool *pool, const kvfuse_table *table, int32_t kv_heads,
                              int32_t layer_begin, int32_t n_layers, int32_t req_start, int32_t chunk_begin, int32_t q_begin,
                              int32_t q_end, int32_t Hq, int32_t reuse, kvfuse_prefill_plan **plan,
                              kvfuse_prefill_plan_info *info)
{
    if (!ctx)
        return KVFUSE_EINVAL;
    Ctx *c = &ctx->c;
    if (!plan)
        return fail(c, KVFUSE_EINVAL, "prefill plan: null output");
    *plan = nullptr;
    if (!pool || !table || !table->bt || !table->scale_k || !table->scale_v)
        return fail(c, KVFUSE_EINVAL, "prefill plan: null pointer");
    if (pool->dtype != KVFUSE_BF16)
        return fail(c, KVFUSE_ESHAPE, "prefill: bfloat16 pools only");
    if ((pool->d != 64 && pool->d != 128) || pool->t % 16 != 0 || pool->t <= 0)
        return fail(c, KVFUSE_ESHAPE, "prefill: needs d in {64, 128} and t a multiple of 16");
    if (kv_heads <= 0 || Hq <= 0 || Hq % kv_heads != 0 || Hq / kv_heads > 16 || n_layers < 0 || layer_begin < 0 ||
        (int64_t)(layer_begin + n_layers) * kv_heads > pool->G)
        return fail(c, KVFUSE_EINVAL, "prefill plan: head counts or layer range do not fit the pool");
    const int t = pool->t, n = table->n;
    if (req_start < 0 || chunk_begin < 0 || chunk_begin % t != 0 || q_begin < chunk_begin || q_end < q_begin ||
        (int64_t)req_start + ((int64_t)q_end + t - 1) / t > n)
        return fail(c, KVFUSE_EINVAL, "prefill plan: need 0 <= chunk_begin (a multiple of t) <= q_begin <= q_end and the "
                                      "request's blocks inside the table");
    if (kv_heads > 65535 || n_layers > 65535)
        return fail(c, KVFUSE_ESHAPE, "prefill plan: kv_heads and n_layers must be <= 65535 per call");
    kvfuse_prefill_plan *pl = new (std::nothrow) kvfuse_prefill_plan();
    if (!pl)
        return fail(c, KVFUSE_ENOMEM, "prefill plan: out of host memory");
    pl->dtype = pool->dtype; pl->P = pool->P; pl->n = n; pl->t = t; pl->d = pool->d; pl->G = pool->G;
    pl->kv_heads = kv_heads; pl->layer_begin = layer_begin; pl->n_layers = n_layers; pl->Hq = Hq;
    pl->rep = Hq / kv_heads;
    pl->rep_pad = pad_pow2_p(pl->rep);
    pl->npw = 32 / pl->rep_pad;
    pl->req_start = req_start; pl->q_begin = q_begin; pl->q_end = q_end; pl->chunk_begin = chunk_begin;

    const int Gsel = n_layers * kv_heads;
    const int nb_pre = chunk_begin / t;                 // logical blocks that end before the chunk
    std::vector<int32_t> bt((size_t)Gsel * nb_pre);
    std::vector<float> sk((size_t)Gsel * nb_pre), sv((size_t)Gsel * nb_pre);
    if (!bt.empty()) {
        hipError_t e = hipStreamSynchronize(c->stream);
        const int64_t g0 = (int64_t)layer_begin * kv_heads;
        if (e == hipSuccess)
            e = hipMemcpy2D(bt.data(), (size_t)nb_pre * 4, table->bt + g0 * n + req_start, (size_t)n * 4, (size_t)nb_pre * 4,
                            (size_t)Gsel, hipMemcpyDeviceToHost);
        if (e == hipSuccess)
            e = hipMemcpy2D(sk.data(), (size_t)nb_pre * 4, table->scale_k + g0 * n + req_start, (size_t)n * 4,
                            (size_t)nb_pre * 4, (size_t)Gsel, hipMemcpyDeviceToHost);
        if (e == hipSuccess)
            e = hipMemcpy2D(sv.data(), (size_t)nb_pre * 4, table->scale_v + g0 * n + req_start, (size_t)n * 4,
                            (size_t)nb_pre * 4, (size_t)Gsel, hipMemcpyDeviceToHost);
        if (e != hipSuccess) {
            delete pl;
            return fail(c, KVFUSE_EHIP, std::string("prefill plan: reading the table: ") + hipGetErrorString(e));
        }
    }
    kvfuse_prefill_plan_info &I = pl->info;
    pl->entry_begin.assign((size_t)Gsel + 1, 0);
    std::vector<std::pair<int32_t, int32_t>> order((size_t)nb_pre);      // (stored block, logical index)
    for (int gi = 0; gi < Gsel; ++gi) {
        const int32_t *b = bt.data() + (size_t)gi * nb_pre;
        for (int x = 0; x < nb_pre; ++x) {
            if (b[x] < 0 || b[x] >= pool->P) {
                delete pl;
                return fail(c, KVFUSE_EINVAL, "prefill plan: the table holds a physical id outside the pool");
            }
            order[(size_t)x] = std::make_pair(reuse ? b[x] : x, (int32_t)x);
        }
        std::sort(order.begin(), order.end());
        for (size_t s = 0; s < order.size();) {
            size_t e = s + 1;
            while (e < order.size() && order[e].first == order[s].first)
                ++e;
            PEntry en;
            en.phys = b[order[s].second];
            en.inst_off = (int32_t)pl->inst.size();
            en.inst_cnt = (int32_t)(e - s);
            en.pad[0] = en.pad[1] = en.pad[2] = 0;
            for (size_t k = s; k < e; ++k) {
                const float2 pair = make_float2(sk[(size_t)gi * nb_pre + order[k].second], sv[(size_t)gi * nb_pre + order[k].second]);
                pl->inst.push_back(pair);
                if (k == s) {
                    en.first = en.second = pair;
                    en.sk_max = en.sk_min = pair.x;
                }
                if (k == s + 1)
                    en.second = pair;
                en.sk_max = std::max(en.sk_max, pair.x);
                en.sk_min = std::min(en.sk_min, pair.x);
            }
            pl->entries.push_back(en);
            s = e;
        }
        pl->entry_begin[(size_t)gi + 1] = (int32_t)pl->entries.size();
        I.logical_blocks_before_chunk += nb_pre;
        if (pl->inst.size() > (size_t)0x7FFFFFF0) {
            delete pl;
            return fail(c, KVFUSE_ESHAPE, "prefill plan: more than 2^31 instances; plan fewer layers per call");
        }
    }
    I.stored_blocks_before_chunk = (int64_t)pl->entries.size();
    size_t off = 0;
    pl->off_entries = off;
    off = up256p(off + pl->entries.size() * sizeof(PEntry));
    pl->off_inst = off;
    off = up256p(off + pl->inst.size() * sizeof(float2));
    pl->off_begin = off;
    off = up256p(off + pl->entry_begin.size() * sizeof(int32_t));
    pl->bytes = off + 256;
    I.device_bytes = (int64_t)pl->bytes;
    if (info)
        *info = I;
    *plan = pl;
    return KVFUSE_OK;
}

int kvfuse_prefill_plan_upload(kvfuse_ctx *ctx, kvfuse_prefill_plan *plan, void *workspace, size_t workspace_bytes)
{
    if (!ctx)
        return KVFUSE_EINVAL;
    Ctx *c = &ctx->c;
    if (!plan || !workspace)
        return fail(c, KVFUSE_EINVAL, "prefill plan upload: null pointer");
    if (workspace_bytes < plan->bytes)
        return fail(c, KVFUSE_ENOMEM, "prefill plan upload: workspace smaller than info.device_bytes");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(c, KVFUSE_EINVAL, "prefill plan upload: workspace must be 256-byte aligned");
    char *dev = static_cast<char *>(workspace);
    if (!plan->entries.empty())
        KVF_HIP(c, hipMemcpyAsync(dev + plan->off_entries, plan->entries.data(), plan->entries.size() * sizeof(PEntry),
                                  hipMemcpyHostToDevice, c->stream));
    if (!plan->inst.empty())
        KVF_HIP(c, hipMemcpyAsync(dev + plan->off_inst, plan->inst.data(), plan->inst.size() * sizeof(float2),
                                  hipMemcpyHostToDevice, c->stream));
    KVF_HIP(c, hipMemcpyAsync(dev + plan->off_begin, plan->entry_begin.data(), plan->entry_begin.size() * sizeof(int32_t),
                              hipMemcpyHostToDevice, c->stream));
    KVF_HIP(c, hipStreamSynchronize(c->stream));
    plan->dev = dev;
    return KVFUSE_OK;
}

int kvfuse_prefill_plan_destroy(kvfuse_prefill_plan *plan)
{
    delete plan;
    return KVFUSE_OK;
}

int kvfuse_prefill_attn(kvfuse_ctx *ctx, const kvfuse_pool *pool, const kvfuse_table *table, const kvfuse_prefill_plan *plan,
                        const void *q, float sm_scale, float *out)
{
    if (!ctx)
        return KVFUSE_EINVAL;
    Ctx *c = &ctx->c;
    if (!pool || !pool->k || !pool->v || !table || !table->bt || !table->scale_k || !table->scale_v || !plan || !q || !out)
        return fail(c, KVFUSE_EINVAL, "prefill: null pointer");
    if (!plan->dev)
        return fail(c, KVFUSE_EINVAL, "prefill: the plan has not been uploaded");
    if (pool->dtype != plan->dtype || pool->P != plan->P || pool->t != plan->t || pool->d != plan->d || pool->G != plan->G ||
        table->n != plan->n)
        return fail(c, KVFUSE_EINVAL, "prefill: pool or table shape differs from the one the plan was built for");
    const int nq = plan->q_end - plan->q_begin;
    if (nq <= 0 || plan->n_layers == 0)
        return KVFUSE_OK;
    PrefillArgs A;
    A.kpool = pool->k; A.vpool = pool->v; A.bt = table->bt; A.scale_k = table->scale_k; A.scale_v = table->scale_v; A.q = q;
    A.entries = reinterpret_cast<const PEntry *>(plan->dev + plan->off_entries);
    A.inst = reinterpret_cast<const float2 *>(plan->dev + plan->off_inst);
    A.entry_begin = reinterpret_cast<const int32_t *>(plan->dev + plan->off_begin);
    A.out = out;
    A.P = pool->P; A.n = table->n; A.t = pool->t; A.kv_heads = plan->kv_heads; A.layer_begin = plan->layer_begin;
    A.Hq = plan->Hq; A.rep = plan->rep; A.rep_pad = plan->rep_pad; A.npw = plan->npw;
    A.req_start = plan->req_start; A.q_begin = plan->q_begin; A.q_end = plan->q_end; A.chunk_begin = plan->chunk_begin;
    A.ppb_inv = ((1ull << 40) + (uint64_t)(pool->t / 16) - 1) / (uint64_t)(pool->t / 16);
    A.sm_scale = std::fabs(sm_scale);
    A.q_sign = std::signbit(sm_scale) ? 0x80008000u : 0u;
    const int per_wg = 4 * plan->npw;
    const unsigned heads = (unsigned)plan->kv_heads, layers = (unsigned)plan->n_layers;
    const dim3 grid((unsigned)((nq + per_wg - 1) / per_wg), heads, layers);
    const dim3 sgrid((unsigned)((nq + plan->npw - 1) / plan->npw), heads, layers);
    A.heads = Divisor(heads);
    const int64_t per_layer = heads, stored = (int64_t)plan->entries.size() / (per_layer * layers);
    const int64_t tiles = (stored * (pool->t / 16) + (plan->q_end - 1 - plan->chunk_begin) / 16 + 2) / 2;
    const bool split = split_pays(grid.x * per_layer * layers, sgrid.x * per_layer * layers, tiles, pool->d);
    A.groups = GroupsByXcd(per_layer * layers, split ? sgrid.x : grid.x);
    if (split) {
        if (pool->d == 128)
            prefill_split_kernel<128><<<sgrid, 64 * kSplitWaves, 0, c->stream>>>(A);
        else
            prefill_split_kernel<64><<<sgrid, 64 * kSplitWaves, 0, c->stream>>>(A);
    } else if (pool->d == 64)
        prefill_attn_kernel<64, 3><<<grid, 256, 0, c->stream>>>(A);
    else if (roomy_pays(grid.x * per_layer * layers, stored * (pool->t / 16) / 2, tiles))
        prefill_attn_kernel<128, 2><<<grid, 256, 0, c->stream>>>(A);
    else
        prefill_attn_kernel<128, 3><<<grid, 256, 0, c->stream>>>(A);
    KVF_HIP(c, hipGetLastError());
    return KVFUSE_OK;
}

}  // extern "C"
