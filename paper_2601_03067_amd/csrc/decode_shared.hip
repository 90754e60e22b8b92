// Shared-block decode attention: the attention of the paged decode step (analysis section: logits q . k / sqrt(d),
// softmax, weighted values), organised around the blocks that fusion made common to several requests.
//
// Motivation section: a fused representation lets one matrix-matrix product replace several matrix-vector
// products, and the result for a request is the merge (with rescaling) of the attention over its fused part and
// over its unique part; Algorithm 1 marks shared blocks for this purpose.
//
// Host side (the decode plan).  Per group, full blocks are grouped by physical id; physical blocks referenced by
// exactly the same set of requests (each at most once) form a cluster.  A cluster with enough blocks becomes work
// items (tile of up to NREQ requests) x (chunk of its blocks); the NREQ x rep query heads of a tile fill the rows
// of the 16-row MFMA tile that the per-request kernel leaves mostly empty, so a cluster block is read once per
// tile.  Everything else (unshared blocks, small clusters, partial last blocks) becomes per-request items.  Every
// (item, request) pair owns one slot of partial softmax state; a last kernel merges a request's slots.
//
// Device side.  binary32 pools: one kernel, templated on the number of rows it carries through P.V (ROWS = rep for per-request
// items, NREQ x rep for cluster items): same structure as the per-request decode kernel -- logits on the MFMA units
// from K fragments loaded straight from global memory, online softmax in fp32, P.V on the vector ALU -- except that
// the block list comes from the plan and the scale factors of a block are per row (they belong to the logical
// entry of the row's request).  bfloat16 pools: decode_items_bf16_kernel, all items in one launch.
#include "attend.h"

#include <algorithm>
#include <map>
#include <new>
#include <vector>

namespace kvfuse {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kMaxTileReq = 4;        // requests per cluster tile (entries carry that many logical indices)
constexpr int kClusterChunk = 32;     // blocks per cluster work item, about

struct DItem {            // 64 bytes
    int32_t li, kvh, nreq, entry_off, entry_cnt, pad0, pad1, pad2;
    int32_t req[kMaxTileReq];
    int32_t slot[kMaxTileReq];
};
struct DEntry {           // 32 bytes
    int32_t phys, ntok;
    int32_t x[kMaxTileReq];   // logical entry of the block in each request of the tile (unused ones repeat x[0])
    int32_t pad0, pad1;
};
static_assert(sizeof(DItem) == 64 && sizeof(DEntry) == 32, "plan records are read as 16-byte vectors");

struct SharedArgs {
    const void *kpool, *vpool;
    const float *scale_k, *scale_v;
    const void *q;
    const DItem *items;
    const DEntry *entries;
    const int32_t *slot_begin;   // [tuples + 1]
    float *part;                 // [slots][rep_pad][D + 2] : o, then m, l
    float *out;                  // [n_layers][B][Hq][D]
    int32_t P, n, t, kv_heads, layer_begin, B, Hq, rep, rep_pad;
    float sm_scale;
};

__device__ static __forceinline__ void mma_f32(const uint4 &a, const uint4 &b, floatx4 &c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
}

// binary32 pools: one workgroup per plan item; its 4 wavefronts walk the item's blocks round-robin.  Row `head` (0..15) of the MFMA
// tile belongs to request slot head / rep_pad of the item and query head head % rep_pad of the KV head's group.
// With 16 rows two wavefronts share a block: both compute its logits and softmax state, each carries half of the
// rows through P.V (64 instead of 128 accumulators per lane, so that three workgroups fit a compute unit).
template <int D, int ROWS>
__global__ __launch_bounds__(256) void decode_items_kernel(SharedArgs A, int item_base)
{
    constexpr int RSPLIT = ROWS == 16 ? 2 : 1;     // wavefronts per block
    constexpr int NSTREAM = 4 / RSPLIT;            // blocks in flight per workgroup
    constexpr int RPW = ROWS / RSPLIT;             // rows a wavefront carries through P.V
    constexpr int PER = Elem<float>::PER16;
    constexpr int NF = D / (4 * PER);      // 16-byte K fragments per lane (a lane owns a quarter of a token row)
    constexpr int LPR = D / PER;           // lanes per V row
    constexpr int RPP = 64 / LPR;          // V rows per pass
    constexpr int NPASS = 16 / RPP;

    __shared__ __attribute__((aligned(16))) float p_lds[4][16][16];     // per wave: probability * scale_v, [token][row]
    __shared__ float c_lds[4][16];         // per wave: rescale factor per row
    __shared__ float w_m[4][16], w_l[4][16];
    __shared__ float w_o[4][RPW][D];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int stream = wave / RSPLIT, row0 = (wave % RSPLIT) * RPW;
    const DItem item = A.items[item_base + blockIdx.x];
    const int li = item.li, kvh = item.kvh, nreq = item.nreq;
    const int g = (A.layer_begin + li) * A.kv_heads + kvh;
    const int64_t r = (int64_t)A.t * D;
    const float *kg = (const float *)A.kpool + (int64_t)g * A.P * r;
    const float *vg = (const float *)A.vpool + (int64_t)g * A.P * r;
    const float *skg = A.scale_k + (int64_t)g * A.n;
    const float *svg = A.scale_v + (int64_t)g * A.n;

    // logits roles: lane = (row, token group); K fragment roles: lane = (token, row quarter)
    const int head = lane & 15, tg = lane >> 4;
    const int ktok = lane & 15, kq = lane >> 4;
    // P.V roles: lane = (column slice, row within pass)
    const int dl = lane % LPR, tr = lane / LPR;
    // the request slot and query head of this lane's row; rows beyond the item's requests or the group's heads
    // carry a zero query and the scales of slot 0 (finite everywhere, never stored)
    const int rs_raw = head / A.rep_pad, hh = head - rs_raw * A.rep_pad;
    const bool row_used = rs_raw < nreq && hh < A.rep && head < ROWS;
    const int rs = row_used ? rs_raw : 0;
    const int my_req = rs == 0 ? item.req[0] : (rs == 1 ? item.req[1] : (rs == 2 ? item.req[2] : item.req[3]));

    uint4 qf[NF];
    {
        const float *qrow = (const float *)A.q + (((int64_t)li * A.B + my_req) * A.Hq + (int64_t)kvh * A.rep + (row_used ? hh : 0)) * D + kq * (D / 4);
#pragma unroll
        for (int f = 0; f < NF; ++f)
            qf[f] = row_used ? reinterpret_cast<const uint4 *>(qrow)[f] : make_uint4(0, 0, 0, 0);
    }

    float m_run = -INFINITY, l_run = 0.0f;
    float o[RPW][PER];
#pragma unroll
    for (int h = 0; h < RPW; ++h)
#pragma unroll
        for (int e = 0; e < PER; ++e)
            o[h][e] = 0.0f;

    for (int eb = stream; eb < item.entry_cnt; eb += NSTREAM) {
        const DEntry ent = A.entries[item.entry_off + eb];
        const int phys = ent.phys, ntok = ent.ntok;
        const int x = rs == 0 ? ent.x[0] : (rs == 1 ? ent.x[1] : (rs == 2 ? ent.x[2] : ent.x[3]));
        const float zs = A.sm_scale * skg[x];
        const float sv = svg[x];
        const float *kblk = kg + (int64_t)phys * r;
        const float *vblk = vg + (int64_t)phys * r;
        for (int sub = 0; sub < A.t; sub += 16) {
            if (sub >= ntok)
                break;
            // ---- logits: 16 tokens x 16 rows
            floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
            const uint4 *krow = reinterpret_cast<const uint4 *>(kblk + (int64_t)(sub + ktok) * D + kq * (D / 4));
            uint4 kf[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f)
                kf[f] = krow[f];
            uint4 vf[NPASS];
#pragma unroll
            for (int ps = 0; ps < NPASS; ++ps)
                vf[ps] = reinterpret_cast<const uint4 *>(vblk + (int64_t)(sub + ps * RPP + tr) * D)[dl];
#pragma unroll
            for (int f = 0; f < NF; ++f)
                mma_f32(kf[f], qf[f], z);
            // ---- online softmax for this lane's row over its 4 tokens, then over the 4 token groups
            const int tok0 = sub + tg * 4;
            float zz[4];
            float bmax = -INFINITY;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                zz[v] = (tok0 + v < ntok) ? z[v] * zs : -INFINITY;
                bmax = fmaxf(bmax, zz[v]);
            }
            bmax = fmaxf(bmax, __shfl_xor(bmax, 16, 64));
            bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
            const float m_new = fmaxf(m_run, bmax);
            const float corr = __expf(m_run - m_new);      // 0 on the first block (m_run = -inf)
            float psum = 0.0f;
            float pv[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float pr = __expf(zz[v] - m_new);
                psum += pr;
                pv[v] = pr * sv;
            }
            psum += __shfl_xor(psum, 16, 64);
            psum += __shfl_xor(psum, 32, 64);
            l_run = l_run * corr + psum;
            m_run = m_new;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                p_lds[wave][tg * 4 + v][head] = pv[v];
            if (tg == 0)
                c_lds[wave][head] = corr;
            __builtin_amdgcn_wave_barrier();
            // ---- P.V: this lane's column slice, rows tr, tr + RPP, ...
            float cf[RPW];
#pragma unroll
            for (int h = 0; h < RPW; ++h)
                cf[h] = c_lds[wave][row0 + h];
#pragma unroll
            for (int h = 0; h < RPW; ++h)
#pragma unroll
                for (int e = 0; e < PER; ++e)
                    o[h][e] *= cf[h];
#pragma unroll
            for (int ps = 0; ps < NPASS; ++ps) {
                float vv[PER];
                widen_f32<float>(vf[ps], vv);
                const int tok = ps * RPP + tr;
                if (sub + tok >= ntok) {             // rows past the context may hold anything, even NaN
#pragma unroll
                    for (int e = 0; e < PER; ++e)
                        vv[e] = 0.0f;
                }
                if constexpr (RPW % 4 == 0) {        // four rows' probabilities per LDS read
#pragma unroll
                    for (int h4 = 0; h4 < RPW; h4 += 4) {
                        const float4 pw4 = *reinterpret_cast<const float4 *>(&p_lds[wave][tok][row0 + h4]);
                        const float pw[4] = {pw4.x, pw4.y, pw4.z, pw4.w};
#pragma unroll
                        for (int hq = 0; hq < 4; ++hq)
#pragma unroll
                            for (int e = 0; e < PER; ++e)
                                o[h4 + hq][e] = fmaf(pw[hq], vv[e], o[h4 + hq][e]);
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < RPW; ++h) {
                        const float pw = p_lds[wave][tok][row0 + h];
#pragma unroll
                        for (int e = 0; e < PER; ++e)
                            o[h][e] = fmaf(pw, vv[e], o[h][e]);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }

    // ---- reduce o over the rows of a pass (lanes with the same column slice), publish the wave's state
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
        for (int h = 0; h < RPW; ++h)
#pragma unroll
            for (int e = 0; e < PER; ++e)
                o[h][e] += __shfl_xor(o[h][e], off, 64);
    if (tr == 0) {
#pragma unroll
        for (int h = 0; h < RPW; ++h)
#pragma unroll
            for (int e = 0; e < PER; ++e)
                w_o[wave][h][dl * PER + e] = o[h][e];
    }
    if (tg == 0) {
        w_m[wave][head] = m_run;
        w_l[wave][head] = l_run;
    }
    __syncthreads();

    for (int idx = tid; idx < ROWS * D; idx += 256) {
        const int h = idx / D, e = idx - h * D;
        const int hs = h / A.rep_pad, hq = h - hs * A.rep_pad;
        if (hs >= nreq || hq >= A.rep)
            continue;
        // the wavefronts that carried row h: one per block stream
        const int wsel = h / RPW, hl = h - wsel * RPW;
        float M = -INFINITY;
#pragma unroll
        for (int st = 0; st < NSTREAM; ++st)
            M = fmaxf(M, w_m[st * RSPLIT + wsel][h]);
        float L = 0.0f, O = 0.0f;
#pragma unroll
        for (int st = 0; st < NSTREAM; ++st) {
            const int wv = st * RSPLIT + wsel;
            const float f = w_m[wv][h] == -INFINITY ? 0.0f : __expf(w_m[wv][h] - M);
            L += w_l[wv][h] * f;
            O += w_o[wv][hl][e] * f;
        }
        const int slot = hs == 0 ? item.slot[0] : (hs == 1 ? item.slot[1] : (hs == 2 ? item.slot[2] : item.slot[3]));
        float *pp = A.part + ((int64_t)slot * A.rep_pad + hq) * (D + 2);
        pp[e] = O;
        if (e == 0) {
            pp[D] = M;
            pp[D + 1] = L;
        }
    }
}

// bfloat16 pools: the same work item, 32 tokens per step of a wavefront (attend.h).  Cluster and per-request items share one
// launch: each XCD takes a contiguous range of both kinds, so that the tiles of a cluster, which read the same blocks, meet in
// its L2, and deals them out in proportion, so that its compute units see cluster blocks (from L2) and blocks of single requests
// (from HBM) at the same time.
// NW: wavefronts of a workgroup, as many as the plan's longest item has steps of 32 tokens, up to four (decode_bf16_kernel): 200
// requests of 64 tokens, 64 groups of 4 heads, four / NW wavefronts: 110 / 84 us, and 76 since only the rows and slots that
// there are go through memory.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 3) void decode_items_bf16_kernel(SharedArgs A, int n_cluster, int n_residual, uint64_t cluster_share)
{
    constexpr int NF = Attend32<D>::NF, NC = Attend32<D>::NC;
    typedef typename Attend32<D>::vrow_t vrow_t;

    __shared__ float w_m[NW][16], w_l[NW][16];
    // a wavefront's keys on their way to fragments; at the end its sums, [16][D]
    constexpr int KEYS = Attend32<D>::K_LDS;
    static_assert(KEYS >= 16 * D * (int)sizeof(float), "sums of a wavefront fit where its keys were");
    __shared__ __attribute__((aligned(16))) char keys[NW][KEYS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // cluster_share: cluster items per seat of an XCD, times 2^32 and rounded up
    const int xcd = blockIdx.x & 7, seat = blockIdx.x >> 3;
    const int before = (int)((uint64_t)seat * cluster_share >> 32), after = (int)((uint64_t)(seat + 1) * cluster_share >> 32);
    const int which = after > before ? xcd * ((n_cluster + 7) >> 3) + before : xcd * ((n_residual + 7) >> 3) + seat - before;
    if (which >= (after > before ? n_cluster : n_residual))
        return;
    const DItem item = A.items[after > before ? which : n_cluster + which];
    const int li = item.li, kvh = item.kvh, nreq = item.nreq;
    const int g = (A.layer_begin + li) * A.kv_heads + kvh;
    const int64_t r = (int64_t)A.t * D;
    const bf16_t *kgrp = (const bf16_t *)A.kpool + (int64_t)g * A.P * r;
    const bf16_t *vgrp = (const bf16_t *)A.vpool + (int64_t)g * A.P * r;
    const float *skg = A.scale_k + (int64_t)g * A.n;
    const float *svg = A.scale_v + (int64_t)g * A.n;

    const int head = lane & 15, kg = lane >> 4;      // row and token group;  also: token of a K row, column slice of a V row
    const int rs_raw = head / A.rep_pad, hh = head - rs_raw * A.rep_pad;
    const bool row_used = rs_raw < nreq && hh < A.rep;
    const int rs = row_used ? rs_raw : 0;
    const int my_req = rs == 0 ? item.req[0] : (rs == 1 ? item.req[1] : (rs == 2 ? item.req[2] : item.req[3]));
    const int k_src = Attend32<D>::k_source(lane), v_off = 4 * kg * D + head * NC;

    uint4 qf[NF];
    {
        const bf16_t *qrow = (const bf16_t *)A.q + (((int64_t)li * A.B + my_req) * A.Hq + (int64_t)kvh * A.rep + (row_used ? hh : 0)) * D + kg * (D / 4);
#pragma unroll
        for (int f = 0; f < NF; ++f)
            qf[f] = row_used ? reinterpret_cast<const uint4 *>(qrow)[f] : make_uint4(0, 0, 0, 0);
    }

    // 16-token piece p of the item: piece p % ppb of entry p / ppb; the table's words are loaded a step ahead
    const int ppb = A.t >> 4, n_pieces = item.entry_cnt * ppb;
    const int pshift = (ppb & (ppb - 1)) == 0 ? __builtin_ctz(ppb) : -1;
    const double base = (double)A.sm_scale * 1.4426950408889634;
    struct Entry {
        int phys, ntok, sub, x0, x1, x2, x3;
    };
    auto entry_at = [&](int p) __attribute__((always_inline)) {
        const int e = pshift >= 0 ? p >> pshift : p / ppb;
        const DEntry &en = A.entries[item.entry_off + e];
        return Entry{en.phys, en.ntok, (p - e * ppb) * 16, en.x[0], en.x[1], en.x[2], en.x[3]};
    };
    Attend32<D> st;
    Entry en0 = {}, en1 = {};
    if (2 * wave < n_pieces) {
        en0 = entry_at(2 * wave);
        en1 = entry_at(min(2 * wave + 1, n_pieces - 1));
    }
    for (int p = 2 * wave; p < n_pieces; p += 2 * NW) {
        const bool two = p + 1 < n_pieces;                          // an odd last piece is paired with itself, masked
        const int xa = rs == 0 ? en0.x0 : (rs == 1 ? en0.x1 : (rs == 2 ? en0.x2 : en0.x3));
        const int xb = rs == 0 ? en1.x0 : (rs == 1 ? en1.x1 : (rs == 2 ? en1.x2 : en1.x3));
        const float ska = skg[xa], sva = svg[xa], skb = skg[xb], svb = svg[xb];
        const int64_t off0 = (int64_t)en0.phys * r + (int64_t)en0.sub * D, off1 = (int64_t)en1.phys * r + (int64_t)en1.sub * D;
        const int left0 = en0.ntok - en0.sub, left1 = two ? en1.ntok - en1.sub : 0;
        uint4 k0[NF], k1[NF];
        vrow_t vr[8];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            k0[f] = *reinterpret_cast<const uint4 *>(kgrp + off0 + k_src + f * Attend32<D>::K_STEP);
            k1[f] = *reinterpret_cast<const uint4 *>(kgrp + off1 + k_src + f * Attend32<D>::K_STEP);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            vr[j] = *reinterpret_cast<const vrow_t *>(vgrp + (j < 4 ? off0 : off1) + v_off + (j & 3) * D);
        if (p + 2 * NW < n_pieces) {
            en0 = entry_at(p + 2 * NW);
            en1 = entry_at(min(p + 2 * NW + 1, n_pieces - 1));
        }
        __builtin_amdgcn_sched_barrier(0);                          // all loads of the step are on their way before the first wait
        const AttendScale s0(base, ska, sva), s1(base, skb, svb);
        Attend32<D>::turn(keys[wave], lane, k0, k1);
        st.step(qf, k0, k1, vr, s0, s1, left0 >= 16 && left1 >= 16, left0 - 4 * kg, left1 - 4 * kg);
    }

    if (row_used)
        st.store(reinterpret_cast<float *>(keys[wave]) + head * D, kg);
    if (kg == 0) {
        w_m[wave][head] = st.m;
        w_l[wave][head] = st.l;
    }
    __syncthreads();

    for (int idx = tid; idx < nreq * A.rep_pad * D; idx += 64 * NW) {
        const int h = idx / D, e = idx - h * D;
        const int hs = h / A.rep_pad, hq = h - hs * A.rep_pad;
        if (hq >= A.rep)
            continue;
        float M = w_m[0][h];
#pragma unroll
        for (int wv = 1; wv < NW; ++wv)
            M = fmaxf(M, w_m[wv][h]);
        float L = 0.0f, O = 0.0f;
#pragma unroll
        for (int wv = 0; wv < NW; ++wv) {
            const float f = w_m[wv][h] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(w_m[wv][h] - M);
            L += w_l[wv][h] * f;
            O += reinterpret_cast<const float *>(keys[wv])[h * D + e] * f;
        }
        const int slot = hs == 0 ? item.slot[0] : (hs == 1 ? item.slot[1] : (hs == 2 ? item.slot[2] : item.slot[3]));
        float *pp = A.part + ((int64_t)slot * A.rep_pad + hq) * (D + 2);
        pp[e] = O;
        if (e == 0) {
            pp[D] = M;
            pp[D + 1] = L;
        }
    }
}

// Merge of a request's partial states: one workgroup per (layer, request, query head), as in decode_combine_kernel: the states
// of up to 64 slots are loaded by the lanes at once, the threads of a head element share the slots out among them.  BASE2: the
// maxima are base-2 logarithms.
template <int D, bool BASE2>
__global__ __launch_bounds__(256) void decode_shared_combine_kernel(SharedArgs A)
{
    constexpr int GROUPS = 256 / D;
    __shared__ float s_o[GROUPS][D];
    const int64_t tuple = blockIdx.x;
    const int h = blockIdx.y;
    const int kvh = (int)(tuple % A.kv_heads);
    const int64_t lb = tuple / A.kv_heads;       // li * B + b
    const int s0 = A.slot_begin[tuple], s1 = A.slot_begin[tuple + 1];
    const int lane = threadIdx.x & 63, e = threadIdx.x % D;
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / D);      // uniform: D is a multiple of 64
    const float *part = A.part + ((int64_t)s0 * A.rep_pad + h) * (D + 2);
    const int64_t stride = (int64_t)A.rep_pad * (D + 2);
    const int n = s1 - s0;
    float M = -INFINITY;
    for (int s = lane; s < n; s += 64)
        M = fmaxf(M, part[s * stride + D]);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
        M = fmaxf(M, __shfl_xor(M, off, 64));
    float L = 0.0f, O = 0.0f;
    for (int c0 = 0; c0 < n; c0 += 64) {
        const int cnt = min(64, n - c0);
        const float m = lane < cnt ? part[(c0 + lane) * stride + D] : -INFINITY;
        const float f = m == -INFINITY ? 0.0f : BASE2 ? __builtin_amdgcn_exp2f(m - M) : __expf(m - M);
        L += lane < cnt ? part[(c0 + lane) * stride + D + 1] * f : 0.0f;
        for (int s = grp; s < cnt; s += 4 * GROUPS) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = part[(c0 + min(s + k * GROUPS, cnt - 1)) * stride + e];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int sk = s + k * GROUPS;
                if (sk < cnt)
                    O += v[k] * __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), sk));
            }
        }
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
        L += __shfl_xor(L, off, 64);
    s_o[grp][e] = O;
    __syncthreads();
    if (grp == 0) {
#pragma unroll
        for (int k = 1; k < GROUPS; ++k)
            O += s_o[k][e];
        A.out[(lb * A.Hq + (int64_t)kvh * A.rep + h) * D + e] = L > 0.0f ? O / L : 0.0f;
    }
}

// The same merge, one wavefront per (layer, request, query head): for calls with enough of them to fill the chip several
// times, where a workgroup each runs in rounds of 2048 (64 requests, 64 groups of 4 heads: 33 us of the call, which went from 274 to 255 us).  The sums of
// the first slots are asked for together with the states.
template <int D, bool BASE2>
__global__ __launch_bounds__(256) void decode_shared_combine_waves_kernel(SharedArgs A, int64_t heads_total)
{
    constexpr int PL = D / 64, BATCH = 8;          // head elements per lane, slots loaded at a time
    typedef float elems_t __attribute__((ext_vector_type(PL)));
    const int lane = threadIdx.x & 63;
    const int64_t id = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (id >= heads_total)
        return;
    const int64_t tuple = id / A.rep;
    const int h = (int)(id - tuple * A.rep);
    const int kvh = (int)(tuple % A.kv_heads);
    const int64_t lb = tuple / A.kv_heads;         // li * B + b
    const int s0 = A.slot_begin[tuple], n = A.slot_begin[tuple + 1] - s0;
    const float *part = A.part + ((int64_t)s0 * A.rep_pad + h) * (D + 2);
    const int64_t stride = (int64_t)A.rep_pad * (D + 2);
    elems_t v[BATCH];
    auto fetch = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
            if (s + k < n)
                v[k] = *reinterpret_cast<const elems_t *>(part + (s + k) * stride + lane * PL);
    };
    elems_t O = (elems_t)(0.0f);
    float L = 0.0f;
    if (n > 0) {
        fetch(0);
        float M = -INFINITY;
        for (int s = lane; s < n; s += 64)
            M = fmaxf(M, part[s * stride + D]);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1)
            M = fmaxf(M, __shfl_xor(M, off, 64));
        for (int c0 = 0; c0 < n; c0 += 64) {
            const int cnt = min(64, n - c0);
            const float m = lane < cnt ? part[(c0 + lane) * stride + D] : -INFINITY;
            const float f = m == -INFINITY ? 0.0f : BASE2 ? __builtin_amdgcn_exp2f(m - M) : __expf(m - M);
            L += lane < cnt ? part[(c0 + lane) * stride + D + 1] * f : 0.0f;
            for (int s = 0; s < cnt; s += BATCH) {
                if (c0 + s > 0)
                    fetch(c0 + s);
#pragma unroll
                for (int k = 0; k < BATCH; ++k)
                    if (s + k < cnt)
                        O += v[k] * __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), s + k));
            }
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1)
            L += __shfl_xor(L, off, 64);
    }
    const elems_t out = L > 0.0f ? O / L : (elems_t)(0.0f);
    *reinterpret_cast<elems_t *>(A.out + (lb * A.Hq + (int64_t)kvh * A.rep + h) * D + lane * PL) = out;
}

// Little more than one slot each: one workgroup for all heads of a (layer, request, KV head), see launch_merge_slots.
template <int D, bool BASE2>
__global__ __launch_bounds__(256) void decode_shared_combine_few_kernel(SharedArgs A)
{
    const int64_t tuple = blockIdx.x;
    const int64_t lb = tuple / A.kv_heads;         // li * B + b
    const int kvh = (int)(tuple - lb * A.kv_heads);
    const int s0 = A.slot_begin[tuple], n = A.slot_begin[tuple + 1] - s0;
    merge_few_states<D, BASE2>(A.part + (int64_t)s0 * A.rep_pad * (D + 2), n, (int64_t)A.rep_pad * (D + 2), A.rep,
                               A.out + (lb * A.Hq + (int64_t)kvh * A.rep) * D);
}

static int pad_pow2(int rep)
{
    int p = 1;
    while (p < rep)
        p <<= 1;
    return p;
}

// The merge of all slots.  Whole calls (us, a workgroup per head / a wavefront per head / a workgroup for all heads of a
// (layer, request, KV head); head size 128 unless said, 4 heads per KV head):
//   slots each   1, 12800 triples  . / 74 / 73, head size 64 . / 47 / 40, of 16 heads . / 108 / 68, binary32 221 / 182 / 180
//                2, 2048 triples   59 / 53 / 53, 12800 triples . / 220 / 232
//                5, 512 triples    28.1 / 27.1 / 30, of 16 heads . / 40 / 56
//               28, 512 triples    275.1 / 274.0 / .
// and by heads, a workgroup / a wavefront for each: 512 13.7 / 13.9 (head size 64 10.3 / 10.5 - 11.4), 4096 36.2 / 33.4, 8192 59.1 /
// 53.2, 32768 272 / 243.
template <int D, bool BASE2>
static void launch_merge_slots(hipStream_t s, const SharedArgs &A, int64_t tuples, int64_t total_slots)
{
    const int64_t heads_total = tuples * A.rep;
    if (4 * total_slots <= 5 * tuples)
        decode_shared_combine_few_kernel<D, BASE2><<<(unsigned)tuples, 256, 0, s>>>(A);
    else if (heads_total >= 4096 && launch_fits((heads_total + 3) / 4, 256))
        decode_shared_combine_waves_kernel<D, BASE2><<<(unsigned)((heads_total + 3) / 4), 256, 0, s>>>(A, heads_total);
    else
        decode_shared_combine_kernel<D, BASE2><<<dim3((unsigned)tuples, (unsigned)A.rep), 256, 0, s>>>(A);
}

template <int D>
static void launch_items(hipStream_t s, const SharedArgs &A, int rows, int item_base, int n_items)
{
    if (n_items <= 0)
        return;
    switch (rows) {
    case 1: decode_items_kernel<D, 1><<<n_items, 256, 0, s>>>(A, item_base); break;
    case 2: decode_items_kernel<D, 2><<<n_items, 256, 0, s>>>(A, item_base); break;
    case 4: decode_items_kernel<D, 4><<<n_items, 256, 0, s>>>(A, item_base); break;
    case 8: decode_items_kernel<D, 8><<<n_items, 256, 0, s>>>(A, item_base); break;
    default: decode_items_kernel<D, 16><<<n_items, 256, 0, s>>>(A, item_base); break;
    }
}

}  // namespace kvfuse

using namespace kvfuse;

struct kvfuse_decode_plan {
    // parameters the plan was built for
    int32_t dtype = 0, P = 0, n = 0, t = 0, d = 0, G = 0;
    int32_t kv_heads = 0, layer_begin = 0, n_layers = 0, B = 0, Hq = 0, rep = 0, rep_pad = 0, nreq_max = 1;
    // host tables
    std::vector<DItem> items_cluster, items_residual;
    std::vector<DEntry> entries;
    std::vector<int32_t> slot_begin;
    int64_t total_slots = 0;
    kvfuse_decode_plan_info info = {};
    // device placement
    size_t off_items = 0, off_entries = 0, off_slots = 0, off_part = 0, bytes = 0;
    int64_t max_pieces = 0;      // 16-token pieces of the longest item
    char *dev = nullptr;
};

static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

namespace {

struct Inst {
    int32_t p, b, x;
};

int residual_splits(int64_t tuples, int blocks)
{
    int64_t ns = tuples > 0 ? (2048 + tuples - 1) / tuples : 1;
    const int cap = (blocks + 7) / 8;
    if (ns > cap)
        ns = cap;
    if (ns > 64)
        ns = 64;
    if (ns < 1)
        ns = 1;
    return (int)ns;
}

}  // namespace

extern "C" {

int kvfuse_shared_decode_plan_build(kvfuse_ctx *ctx, const kvfuse_pool *pool, const kvfuse_table *table, int32_t kv_heads,
                                    int32_t layer_begin, int32_t n_layers, const int32_t *req_start, const int32_t *ctx_len,
                                    int32_t B, int32_t Hq, int32_t min_cluster_blocks, kvfuse_decode_plan **plan,
                                    kvfuse_decode_plan_info *info)
{
    if (!ctx)
        return KVFUSE_EINVAL;
    Ctx *c = &ctx->c;
    if (!plan)
        return fail(c, KVFUSE_EINVAL, "decode plan: null output");
    *plan = nullptr;
    if (!pool || !table || !table->bt || !req_start || !ctx_len)
        return fail(c, KVFUSE_EINVAL, "decode plan: null pointer");
    if (kv_heads <= 0 || Hq <= 0 || Hq % kv_heads != 0 || Hq / kv_heads > 16 || B < 0 || n_layers < 0 || layer_begin < 0 ||
        (int64_t)(layer_begin + n_layers) * kv_heads > pool->G || min_cluster_blocks < 1)
        return fail(c, KVFUSE_EINVAL, "decode plan: head counts, layer range or min_cluster_blocks out of range");
    if (pool->dtype != KVFUSE_BF16 && pool->dtype != KVFUSE_F32)
        return fail(c, KVFUSE_ESHAPE, "decode plan: dtype must be KVFUSE_BF16 or KVFUSE_F32");
    if ((pool->d != 64 && pool->d != 128) || pool->t % 16 != 0 || pool->t <= 0)
        return fail(c, KVFUSE_ESHAPE, "decode plan: needs d in {64, 128} and t a multiple of 16");
    const int n = table->n, t = pool->t;
    int max_blocks = 0;
    for (int b = 0; b < B; ++b) {
        if (ctx_len[b] < 0 || req_start[b] < 0)
            return fail(c, KVFUSE_EINVAL, "decode plan: negative request start or context length");
        const int nb = (ctx_len[b] + t - 1) / t;
        if ((int64_t)req_start[b] + nb > n)
            return fail(c, KVFUSE_EINVAL, "decode plan: a request's blocks run past the table");
        max_blocks = std::max(max_blocks, nb);
    }
    kvfuse_decode_plan *pl = new (std::nothrow) kvfuse_decode_plan();
    if (!pl)
        return fail(c, KVFUSE_ENOMEM, "decode plan: out of host memory");
    pl->dtype = pool->dtype; pl->P = pool->P; pl->n = n; pl->t = t; pl->d = pool->d; pl->G = pool->G;
    pl->kv_heads = kv_heads; pl->layer_begin = layer_begin; pl->n_layers = n_layers; pl->B = B; pl->Hq = Hq;
    pl->rep = Hq / kv_heads;
    pl->rep_pad = pad_pow2(pl->rep);
    pl->nreq_max = std::max(1, std::min(kMaxTileReq, 16 / pl->rep_pad));

    const int Gsel = n_layers * kv_heads;
    const int64_t tuples = (int64_t)n_layers * B * kv_heads;
    std::vector<int32_t> bt((size_t)Gsel * n);
    if (!bt.empty()) {
        hipError_t e = hipStreamSynchronize(c->stream);
        if (e == hipSuccess)
            e = hipMemcpy(bt.data(), table->bt + (int64_t)layer_begin * kv_heads * n, bt.size() * sizeof(int32_t),
                          hipMemcpyDeviceToHost);
        if (e != hipSuccess) {
            delete pl;
            return fail(c, KVFUSE_EHIP, std::string("decode plan: reading the table: ") + hipGetErrorString(e));
        }
    }
    std::vector<int32_t> slot_count((size_t)tuples, 0);
    std::vector<Inst> inst;
    std::vector<uint8_t> covered((size_t)n);
    const int nsplit_res = residual_splits(tuples, max_blocks);
    kvfuse_decode_plan_info &I = pl->info;

    auto take_slot = [&](DItem &it, int rs, int li, int b, int kvh) {
        const int64_t tuple = ((int64_t)li * B + b) * kv_heads + kvh;
        it.slot[rs] = slot_count[(size_t)tuple]++;      // local index for now; made absolute below
    };

    for (int gi = 0; gi < Gsel; ++gi) {
        const int li = gi / kv_heads, kvh = gi % kv_heads;
        const int32_t *btg = bt.data() + (size_t)gi * n;
        inst.clear();
        std::fill(covered.begin(), covered.end(), 0);
        for (int b = 0; b < B; ++b) {
            const int nb = (ctx_len[b] + t - 1) / t;
            for (int j = 0; j < nb; ++j) {
                const int x = req_start[b] + j;
                const int p = btg[x];
                if (p < 0 || p >= pool->P) {
                    delete pl;
                    return fail(c, KVFUSE_EINVAL, "decode plan: the table holds a physical id outside the pool");
                }
                ++I.logical_blocks;
                if ((int64_t)(j + 1) * t <= ctx_len[b])
                    inst.push_back(Inst{p, b, x});
            }
        }
        std::sort(inst.begin(), inst.end(), [](const Inst &a, const Inst &b2) {
            return a.p != b2.p ? a.p < b2.p : (a.b != b2.b ? a.b < b2.b : a.x < b2.x);
        });
        // physical blocks used by >= 2 requests, each once, keyed by the set of requests
        std::map<std::vector<int32_t>, std::vector<int32_t>> by_set;    // request set -> starts of runs in inst
        std::vector<int32_t> key;
        for (size_t s = 0; s < inst.size();) {
            size_t e = s + 1;
            while (e < inst.size() && inst[e].p == inst[s].p)
                ++e;
            if (e - s >= 2) {
                bool distinct = true;
                for (size_t k = s + 1; k < e; ++k)
                    distinct = distinct && inst[k].b != inst[k - 1].b;
                if (distinct) {
                    key.clear();
                    for (size_t k = s; k < e; ++k)
                        key.push_back(inst[k].b);
                    by_set[key].push_back((int32_t)s);
                }
            }
            s = e;
        }
        for (const auto &kv : by_set) {
            const std::vector<int32_t> &reqs = kv.first;
            const std::vector<int32_t> &runs = kv.second;
            const int nb = (int)runs.size(), k = (int)reqs.size();
            if (nb < min_cluster_blocks)
                continue;
            ++I.clusters;
            I.shared_instances += (int64_t)nb * k;
            const int nchunk = std::max(1, (nb + kClusterChunk / 2) / kClusterChunk);
            for (int s0 = 0; s0 < k; s0 += pl->nreq_max) {
                const int nr = std::min(pl->nreq_max, k - s0);
                for (int ch = 0; ch < nchunk; ++ch) {
                    const int lo = (int)((int64_t)nb * ch / nchunk), hi = (int)((int64_t)nb * (ch + 1) / nchunk);
                    if (hi <= lo)
                        continue;
                    DItem it = {};
                    it.li = li; it.kvh = kvh; it.nreq = nr;
                    it.entry_off = (int32_t)pl->entries.size();
                    it.entry_cnt = hi - lo;
                    for (int rs = 0; rs < kMaxTileReq; ++rs)
                        it.req[rs] = reqs[(size_t)(s0 + std::min(rs, nr - 1))];
                    for (int rs = 0; rs < nr; ++rs)
                        take_slot(it, rs, li, reqs[(size_t)(s0 + rs)], kvh);
                    for (int q = lo; q < hi; ++q) {
                        DEntry en = {};
                        const int32_t run = runs[(size_t)q];
                        en.phys = inst[(size_t)run].p;
                        en.ntok = t;
                        for (int rs = 0; rs < kMaxTileReq; ++rs)
                            en.x[rs] = inst[(size_t)(run + s0 + std::min(rs, nr - 1))].x;
                        pl->entries.push_back(en);
                    }
                    I.cluster_block_reads += hi - lo;
                    pl->items_cluster.push_back(it);
                }
            }
            for (int32_t run : runs)
                for (int q = 0; q < k; ++q)
                    covered[(size_t)inst[(size_t)(run + q)].x] = 1;
        }
        // what is left of every request
        for (int b = 0; b < B; ++b) {
            const int nb = (ctx_len[b] + t - 1) / t;
            int nres = 0;
            for (int j = 0; j < nb; ++j)
                nres += covered[(size_t)(req_start[b] + j)] ? 0 : 1;
            if (nres == 0)
                continue;
            const int nsp = std::min(nsplit_res, nres);
            int j = 0;
            for (int sp = 0; sp < nsp; ++sp) {
                const int want = (int)((int64_t)nres * (sp + 1) / nsp) - (int)((int64_t)nres * sp / nsp);
                DItem it = {};
                it.li = li; it.kvh = kvh; it.nreq = 1;
                it.entry_off = (int32_t)pl->entries.size();
                for (int rs = 0; rs < kMaxTileReq; ++rs)
                    it.req[rs] = b;
                take_slot(it, 0, li, b, kvh);
                int got = 0;
                while (got < want && j < nb) {
                    const int x = req_start[b] + j;
                    if (!covered[(size_t)x]) {
                        DEntry en = {};
                        en.phys = btg[x];
                        en.ntok = std::min(t, ctx_len[b] - j * t);
                        for (int rs = 0; rs < kMaxTileReq; ++rs)
                            en.x[rs] = x;
                        pl->entries.push_back(en);
                        ++got;
                    }
                    ++j;
                }
                it.entry_cnt = got;
                I.residual_block_reads += got;
                pl->items_residual.push_back(it);
            }
        }
        if (pl->entries.size() > (size_t)0x7FFFFFF0) {
            delete pl;
            return fail(c, KVFUSE_ESHAPE, "decode plan: more than 2^31 block entries; plan fewer layers per call");
        }
    }
    // absolute slot numbers: a tuple's slots are consecutive
    pl->slot_begin.assign((size_t)tuples + 1, 0);
    for (int64_t tp = 0; tp < tuples; ++tp)
        pl->slot_begin[(size_t)tp + 1] = pl->slot_begin[(size_t)tp] + slot_count[(size_t)tp];
    pl->total_slots = tuples > 0 ? pl->slot_begin[(size_t)tuples] : 0;
    auto make_absolute = [&](std::vector<DItem> &v) {
        for (DItem &it : v)
            for (int rs = 0; rs < it.nreq; ++rs) {
                const int64_t tuple = ((int64_t)it.li * B + it.req[rs]) * kv_heads + it.kvh;
                it.slot[rs] += pl->slot_begin[(size_t)tuple];
            }
    };
    make_absolute(pl->items_cluster);
    make_absolute(pl->items_residual);
    for (const std::vector<DItem> *v : {&pl->items_cluster, &pl->items_residual})
        for (const DItem &it : *v)
            pl->max_pieces = std::max(pl->max_pieces, (int64_t)it.entry_cnt * (t / 16));
    I.items_cluster = (int64_t)pl->items_cluster.size();
    I.items_residual = (int64_t)pl->items_residual.size();
    // device layout
    size_t off = 0;
    pl->off_items = off;
    off = up256(off + (pl->items_cluster.size() + pl->items_residual.size()) * sizeof(DItem));
    pl->off_entries = off;
    off = up256(off + pl->entries.size() * sizeof(DEntry));
    pl->off_slots = off;
    off = up256(off + pl->slot_begin.size() * sizeof(int32_t));
    pl->off_part = off;
    off = up256(off + (size_t)pl->total_slots * pl->rep_pad * (pl->d + 2) * sizeof(float));
    pl->bytes = off + 256;
    I.device_bytes = (int64_t)pl->bytes;
    if (info)
        *info = I;
    *plan = pl;
    return KVFUSE_OK;
}

int kvfuse_shared_decode_plan_upload(kvfuse_ctx *ctx, kvfuse_decode_plan *plan, void *workspace, size_t workspace_bytes)
{
    if (!ctx)
        return KVFUSE_EINVAL;
    Ctx *c = &ctx->c;
    if (!plan || !workspace)
        return fail(c, KVFUSE_EINVAL, "decode plan upload: null pointer");
    if (workspace_bytes < plan->bytes)
        return fail(c, KVFUSE_ENOMEM, "decode plan upload: workspace smaller than info.device_bytes");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(c, KVFUSE_EINVAL, "decode plan upload: workspace must be 256-byte aligned");
    char *dev = static_cast<char *>(workspace);
    const size_t nc = plan->items_cluster.size(), nr = plan->items_residual.size();
    if (nc)
        KVF_HIP(c, hipMemcpyAsync(dev + plan->off_items, plan->items_cluster.data(), nc * sizeof(DItem), hipMemcpyHostToDevice, c->stream));
    if (nr)
        KVF_HIP(c, hipMemcpyAsync(dev + plan->off_items + nc * sizeof(DItem), plan->items_residual.data(), nr * sizeof(DItem),
                                  hipMemcpyHostToDevice, c->stream));
    if (!plan->entries.empty())
        KVF_HIP(c, hipMemcpyAsync(dev + plan->off_entries, plan->entries.data(), plan->entries.size() * sizeof(DEntry),
                                  hipMemcpyHostToDevice, c->stream));
    KVF_HIP(c, hipMemcpyAsync(dev + plan->off_slots, plan->slot_begin.data(), plan->slot_begin.size() * sizeof(int32_t),
                              hipMemcpyHostToDevice, c->stream));
    KVF_HIP(c, hipStreamSynchronize(c->stream));      // the host vectors may go away after this call
    plan->dev = dev;
    return KVFUSE_OK;
}

int kvfuse_shared_decode_plan_destroy(kvfuse_decode_plan *plan)
{
    delete plan;
    return KVFUSE_OK;
}

int kvfuse_paged_decode_attn_shared(kvfuse_ctx *ctx, const kvfuse_pool *pool, const kvfuse_table *table,
                                    const kvfuse_decode_plan *plan, const void *q, float sm_scale, float *out)
{
    if (!ctx)
        return KVFUSE_EINVAL;
    Ctx *c = &ctx->c;
    if (!pool || !pool->k || !pool->v || !table || !table->scale_k || !table->scale_v || !plan || !q || !out)
        return fail(c, KVFUSE_EINVAL, "shared decode: null pointer");
    if (!plan->dev)
        return fail(c, KVFUSE_EINVAL, "shared decode: the plan has not been uploaded");
    if (pool->dtype != plan->dtype || pool->P != plan->P || pool->t != plan->t || pool->d != plan->d || pool->G != plan->G ||
        table->n != plan->n)
        return fail(c, KVFUSE_EINVAL, "shared decode: pool or table shape differs from the one the plan was built for");
    const int64_t tuples = (int64_t)plan->n_layers * plan->B * plan->kv_heads;
    if (tuples == 0)
        return KVFUSE_OK;
    if (tuples > 0x7FFFFFFF)
        return fail(c, KVFUSE_ESHAPE, "shared decode: too many (layer, request, head) tuples for one call");
    SharedArgs A;
    A.kpool = pool->k; A.vpool = pool->v; A.scale_k = table->scale_k; A.scale_v = table->scale_v; A.q = q;
    A.items = reinterpret_cast<const DItem *>(plan->dev + plan->off_items);
    A.entries = reinterpret_cast<const DEntry *>(plan->dev + plan->off_entries);
    A.slot_begin = reinterpret_cast<const int32_t *>(plan->dev + plan->off_slots);
    A.part = reinterpret_cast<float *>(plan->dev + plan->off_part);
    A.out = out;
    A.P = pool->P; A.n = table->n; A.t = pool->t; A.kv_heads = plan->kv_heads; A.layer_begin = plan->layer_begin;
    A.B = plan->B; A.Hq = plan->Hq; A.rep = plan->rep; A.rep_pad = plan->rep_pad;
    A.sm_scale = sm_scale;
    const int nc = (int)plan->items_cluster.size(), nr = (int)plan->items_residual.size();
    const int rows_cluster = plan->nreq_max * plan->rep_pad, rows_residual = plan->rep_pad;
    // binary32 pools: the cluster pass is bound by the vector ALU, the per-request pass by HBM: they run side by side, the
    // cluster pass on the context's second stream, and meet again before the merge.
    const bool fork = pool->dtype == KVFUSE_F32 && nc > 0 && nr > 0;
    if (fork) {
        if (!c->aux) {
            hipStream_t st = nullptr;
            hipEvent_t e0 = nullptr, e1 = nullptr;
            KVF_HIP(c, hipSetDevice(c->device));
            KVF_HIP(c, hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
            hipError_t er = hipEventCreateWithFlags(&e0, hipEventDisableTiming);
            if (er == hipSuccess)
                er = hipEventCreateWithFlags(&e1, hipEventDisableTiming);
            if (er != hipSuccess) {
                if (e0)
                    (void)hipEventDestroy(e0);
                (void)hipStreamDestroy(st);
                KVF_HIP(c, er);
            }
            c->aux = st; c->fork = e0; c->join = e1;
        }
        KVF_HIP(c, hipEventRecord(c->fork, c->stream));
        KVF_HIP(c, hipStreamWaitEvent(c->aux, c->fork, 0));
    }
    hipStream_t cs = fork ? c->aux : c->stream;
#define KVF_SHARED_LAUNCH(D)                                                     \
    do {                                                                         \
        launch_items<D>(cs, A, rows_cluster, 0, nc);                             \
        launch_items<D>(c->stream, A, rows_residual, nc, nr);                    \
        if (fork) {                                                              \
            (void)hipEventRecord(c->join, c->aux);                               \
            (void)hipStreamWaitEvent(c->stream, c->join, 0);                     \
        }                                                                        \
        launch_merge_slots<D, false>(c->stream, A, tuples, plan->total_slots);   \
    } while (0)
    if (pool->dtype == KVFUSE_BF16) {
        auto items = [&](const SharedArgs &part, int n_cluster, int n_residual) {
            // (any split of an XCD's seats between the two kinds is correct as long as the last seat completes both)
            const uint64_t nc8 = ((uint64_t)n_cluster + 7) / 8, seats = nc8 + ((uint64_t)n_residual + 7) / 8;
            const uint64_t share = seats > 0 ? ((nc8 << 32) + seats - 1) / seats : 0;
            if (seats == 0)
                return;
#define KVF_ITEMS(D, NW)                                                                                            \
    decode_items_bf16_kernel<D, NW><<<(unsigned)(8 * seats), 64 * NW, 0, c->stream>>>(part, n_cluster, n_residual, share)
#define KVF_ITEMS_NW(D)                                                                                             \
    do {                                                                                                            \
        if (plan->max_pieces <= 2) KVF_ITEMS(D, 1);                                                                 \
        else if (plan->max_pieces <= 4) KVF_ITEMS(D, 2);                                                            \
        else KVF_ITEMS(D, 4);                                                                                       \
    } while (0)
            if (pool->d == 128) KVF_ITEMS_NW(128);
            else KVF_ITEMS_NW(64);
#undef KVF_ITEMS_NW
#undef KVF_ITEMS
        };
        if (launch_fits((int64_t)nc + nr + 14, 256)) {
            items(A, nc, nr);
        } else {                       // more items than a launch holds: one launch for each kind
            items(A, nc, 0);
            SharedArgs rest = A;
            rest.items += nc;
            items(rest, 0, nr);
        }
        if (pool->d == 128)
            launch_merge_slots<128, true>(c->stream, A, tuples, plan->total_slots);
        else
            launch_merge_slots<64, true>(c->stream, A, tuples, plan->total_slots);
    } else {
        if (pool->d == 128) KVF_SHARED_LAUNCH(128);
        else KVF_SHARED_LAUNCH(64);
    }
#undef KVF_SHARED_LAUNCH
    KVF_HIP(c, hipGetLastError());
    return KVFUSE_OK;
}

}  // extern "C"
