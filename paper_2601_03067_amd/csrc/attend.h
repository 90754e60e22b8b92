// What the paged and the shared-block decode kernels share.  One step of decode attention over bfloat16 blocks: 32 tokens (two
// 16-token pieces) against 16 query rows, both products on the matrix cores.
//   loads   every load of a wavefront covers rows end to end.  The keys' fragments (16 rows, 16 bytes out of each quarter) would take
//           four times as many cache lines per load, and the vector cache's turns over them were what bounded blocks that come out
//           of the caches; a turn through LDS puts them in place (us, without / with: 8 heads per KV head, 256 x 4096 tokens,
//           16 groups 720 / 561; 48 ragged requests, 8 groups 153 / 141; shared blocks, 64 x 2048 tokens, 64 groups 254 / 238).
//   logits  two 16 tokens x 16 rows groups: lane (row = lane & 15, kg = lane >> 4) ends up with the tokens 4 kg .. + 3 of
//           both pieces, which are the 8 summation indices of the same lane in the second product.
//   P.V     out^T (16 head elements x 16 rows) += V^T P^T, once per column c of the lane's slice: lane (n = lane & 15, kg)
//           loads the rows of its own 8 tokens at the head elements NC n .. NC n + NC - 1 (16 lanes read a row end to end)
//           and V^T's fragment c is element c of its 8 rows, one v_perm per two values.  The order of the summation
//           indices is free as long as both operands agree, so the weights never leave their lane.
// The weights are split exactly: three truncated bfloat16 parts hold all 24 bits of a binary32, so every product is exact
// and the sums are binary32, smallest parts first.  The scale of the logits is carried in two words, so that the exponent's
// argument, where the weight is not small, is as good as the logit (AttendScale::weight).
#ifndef KVFUSE_ATTEND_H
#define KVFUSE_ATTEND_H

#include "common.h"

namespace kvfuse {

typedef float attend_f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 attend_bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ void attend_mma(const uint4 &a, const uint4 &b, attend_f32x4 &c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(attend_bf16x8, a), __builtin_bit_cast(attend_bf16x8, b), c, 0, 0, 0);
}

// The scales of a piece's logical block.  Logits are in base 2, exp(x) = exp2(x log2(e)): sk + sk_rest = scale of the keys *
// softmax scale * log2(e).
struct AttendScale {
    float sk, sk_rest, sv;
    // base = softmax scale * log2(e)
    __device__ __forceinline__ AttendScale(double base, float key, float value)
    {
        const double s = base * (double)key;
        sk = (float)s;
        sk_rest = (float)(s - (double)sk);
        sv = value;
    }
    // exp2(z (sk + sk_rest) - m) for z sk above -inf.  A logit of -inf has weight 0, which its callers see to: sk_rest is of
    // either sign or zero, and -inf times it is +inf or NaN.  z sk - m is taken first: it is small where the weight is not, so
    // that the second word survives the rounding of the sum; z sk_rest - m would be rounded to a unit of m.
    __device__ __forceinline__ float weight(float z, float m) const
    {
        return __builtin_amdgcn_exp2f(fmaf(z, sk_rest, fmaf(z, sk, -m)));
    }
};

template <int D>
struct Attend32 {
    static constexpr int NF = D / 32;      // 16-byte K fragments per lane (a lane owns a quarter of a token row)
    static constexpr int NC = D / 16;      // head elements of a V row per lane = 16-row tiles of out^T
    typedef uint32_t vrow_t __attribute__((ext_vector_type(NC / 2)));

    float m = -INFINITY, l = 0.0f;         // running maximum (base 2) and sum of this lane's row
    attend_f32x4 o[NC];                    // o[c][v]: head element NC (4 kg + v) + c of this lane's row

    __device__ __forceinline__ Attend32()
    {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            o[c] = attend_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // A lane's part of a piece of keys, as it is loaded: 16 bytes each of rows 64 / CH apart, CH lanes to a row, end to end.
    static constexpr int CH = D / 8, K_STEP = 512;      // elements from one of its loads to the next
    static __device__ __forceinline__ int k_source(int lane) { return lane * 8; }

    // ... and turned by way of LDS (the wavefront's own K_LDS bytes) into the fragments that the product takes: token lane & 15, the
    // quarter kg of its row.  Rows are 16 bytes further apart than they are long, so that neither side meets in a bank.
    static constexpr int K_PITCH = 2 * D + 16, K_LDS = 32 * K_PITCH;
    static __device__ __forceinline__ void turn(char *mem, int lane, uint4 (&k0)[NF], uint4 (&k1)[NF])
    {
        char *to = mem + lane / CH * K_PITCH + lane % CH * 16;
        const char *from = mem + (lane & 15) * K_PITCH + (lane >> 4) * (D / 2);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            *reinterpret_cast<uint4 *>(to + f * (64 / CH) * K_PITCH) = k0[f];
            *reinterpret_cast<uint4 *>(to + (f * (64 / CH) + 16) * K_PITCH) = k1[f];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            k0[f] = *reinterpret_cast<const uint4 *>(from + f * 16);
            k1[f] = *reinterpret_cast<const uint4 *>(from + 16 * K_PITCH + f * 16);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // k0, k1: K fragments of the two pieces; vr: V rows, [4 piece + i] = token 4 kg + i.  Tokens 4 kg + i with i < left are
    // inside the context; `full`, uniform, says that all are.
    __device__ __forceinline__ void step(const uint4 (&qf)[NF], const uint4 (&k0)[NF], const uint4 (&k1)[NF], vrow_t (&vr)[8],
                                         const AttendScale &s0, const AttendScale &s1, bool full, int left0, int left1)
    {
        attend_f32x4 z0 = {0.0f, 0.0f, 0.0f, 0.0f}, z1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            attend_mma(k0[f], qf[f], z0);
            attend_mma(k1[f], qf[f], z1);
        }
        // ---- online softmax for this lane's row over its 8 tokens, then over the 4 token groups
        float bmax = -INFINITY, zz[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            zz[v] = (v < 4 ? z0[v & 3] : z1[v & 3]) * (v < 4 ? s0.sk : s1.sk);
            if (!full)
                zz[v] = (v & 3) < (v < 4 ? left0 : left1) ? zz[v] : -INFINITY;
            bmax = fmaxf(bmax, zz[v]);
        }
        bmax = fmaxf(bmax, __shfl_xor(bmax, 16, 64));
        bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
        const float m_new = fmaxf(m, bmax);
        // 0 on the first step (m = -inf); a step may hold no visible token at all
        const float corr = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - m_new);
        float psum = 0.0f, w[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const AttendScale &s = v < 4 ? s0 : s1;
            const float z = v < 4 ? z0[v & 3] : z1[v & 3];
            const float pr = zz[v] == -INFINITY ? 0.0f : s.weight(z, m_new);
            psum += pr;
            w[v] = pr * s.sv;
        }
        psum += __shfl_xor(psum, 16, 64);
        psum += __shfl_xor(psum, 32, 64);
        l = l * corr + psum;
        m = m_new;
        if (!full) {                                   // rows past the context may hold anything, even NaN
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if ((j & 3) >= (j < 4 ? left0 : left1))
                    vr[j] = (vrow_t)(0u);
        }
        // ---- the weights as three bfloat16 parts (upper halves of what is left), two values to a word
        uint32_t ph[3][4];
#pragma unroll
        for (int part = 0; part < 3; ++part)
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const uint32_t a = __float_as_uint(w[j]), c = __float_as_uint(w[j + 1]);
                ph[part][j / 2] = __builtin_amdgcn_perm(c, a, 0x07060302u);
                w[j] -= __uint_as_float(a & 0xFFFF0000u);
                w[j + 1] -= __uint_as_float(c & 0xFFFF0000u);
            }
        // ---- out^T += V^T P^T
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
            uint4 va;
            va.x = __builtin_amdgcn_perm(vr[1][c / 2], vr[0][c / 2], sel);
            va.y = __builtin_amdgcn_perm(vr[3][c / 2], vr[2][c / 2], sel);
            va.z = __builtin_amdgcn_perm(vr[5][c / 2], vr[4][c / 2], sel);
            va.w = __builtin_amdgcn_perm(vr[7][c / 2], vr[6][c / 2], sel);
            attend_f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};  // the smallest part first; one rounding against the sums so far
#pragma unroll
            for (int part = 2; part >= 0; --part)
                attend_mma(va, make_uint4(ph[part][0], ph[part][1], ph[part][2], ph[part][3]), s);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                o[c][v] = fmaf(o[c][v], corr, s[v]);
        }
    }

    // This lane's part of the row's sums into row[0 .. D - 1].
    __device__ __forceinline__ void store(float *row, int kg) const
    {
        float *dst = row + 4 * kg * NC;
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int c = 0; c < NC; c += 4)
                *reinterpret_cast<float4 *>(dst + v * NC + c) = make_float4(o[c][v], o[c + 1][v], o[c + 2][v], o[c + 3][v]);
    }
};

// Merge of a few partial states of all query heads of a (layer, request, KV head), by one workgroup of 256 threads: state s of
// head h is at part + s * stride + h * (D + 2): the sums, then maximum and sum of weights; out: the heads end to end.  BASE2: the
// maxima are base-2 logarithms.
template <int D, bool BASE2>
__device__ __forceinline__ void merge_few_states(const float *__restrict__ part, int n, int64_t stride, int rep, float *__restrict__ out)
{
    for (int idx = threadIdx.x; idx < rep * D; idx += 256) {
        const int h = idx / D, e = idx - h * D;
        const float *ph = part + h * (D + 2);
        float M = -INFINITY;
        for (int s = 0; s < n; ++s)
            M = fmaxf(M, ph[s * stride + D]);
        float L = 0.0f, O = 0.0f;
        for (int s = 0; s < n; ++s) {
            const float m = ph[s * stride + D];
            const float f = m == -INFINITY ? 0.0f : BASE2 ? __builtin_amdgcn_exp2f(m - M) : __expf(m - M);
            L += ph[s * stride + D + 1] * f;
            O += ph[s * stride + e] * f;
        }
        out[idx] = L > 0.0f ? O / L : 0.0f;
    }
}

}  // namespace kvfuse

#endif
