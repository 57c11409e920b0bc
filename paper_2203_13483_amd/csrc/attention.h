// What the kernel of attention.hip takes, and how it stores a query's context.  (attention_blocks_kernel of layer.hip stores the
// same way, from arguments of its own.)
#pragma once

#include "gemm_common.h"

#include <type_traits>

namespace mkq {

struct AttentionParams {
    const uint16_t *qkv;        // [tokens, 3 hidden]: q, k, v of all heads
    const int32_t *cu_seqlens;  // null (every sequence has seq rows) or row offsets; seq then bounds the lengths
    int batch, seq, hidden, heads, dk, q_blocks;  // q_blocks: blocks of 128 queries of seq
    uint16_t *ctx;              // [tokens, hidden] or null
    uint8_t *qout;              // codes, rows of q_pitch, or null
    float s_next;
    int q_bits, q_pitch;
};

typedef float v4f __attribute__((ext_vector_type(4)));

// Chunk of 16 bytes c of head dimension d of V^T is kept at c ^ swz_dims(d): the sixteen rows of a fragment differ in bits 0, 1, 3 and 4
__device__ __forceinline__ int swz_dims(int d) { return (d & 3) | ((d >> 1) & 12); }

// Head dimensions d0 .. d0 + 7 of one query (those below d_k; d0 is a multiple of 8).  VEC = 8: d_k % 8 == 0; 2: even.
template <int VEC>
__device__ __forceinline__ void attention_store(const AttentionParams &p, int64_t row, int head, int d0, const float (&o)[8])
{
    const int nvalid = (p.dk - d0) < 8 ? (p.dk - d0) : 8;
    if (p.ctx) {
        const uint32_t h[4] = {pack2_f16(o[0], o[1]), pack2_f16(o[2], o[3]), pack2_f16(o[4], o[5]), pack2_f16(o[6], o[7])};
        uint16_t *dst = p.ctx + row * p.hidden + head * p.dk + d0;
        if constexpr (VEC == 8) *reinterpret_cast<uint4 *>(dst) = make_uint4(h[0], h[1], h[2], h[3]);
        else
            for (int e = 0; e < nvalid / 2; ++e) reinterpret_cast<uint32_t *>(dst)[e] = h[e];
    }
    const int64_t qo = row * p.q_pitch + head * p.dk + d0;  // in codes
    if (p.qout && p.q_bits == 8) {
        const uint2 pk = quantize8<8>(o, quant_step<8>(p.s_next));
        if constexpr (VEC == 8) *reinterpret_cast<uint2 *>(p.qout + qo) = pk;
        else
            for (int e = 0; e < nvalid; ++e) p.qout[qo + e] = (uint8_t)((e < 4 ? pk.x : pk.y) >> (8 * (e & 3)));
    } else if (p.qout) {
        const uint32_t packed = quantize8<4>(o, quant_step<4>(p.s_next)).x;
        if constexpr (VEC == 8) *reinterpret_cast<uint32_t *>(p.qout + (qo >> 1)) = packed;
        else
            for (int e = 0; e < nvalid / 2; ++e) p.qout[(qo >> 1) + e] = (uint8_t)(packed >> (8 * e));
    }
}

// Padding codes of a row with a pitch: zero (hidden and the pitch are multiples of 8 codes).
__device__ __forceinline__ void attention_pad_codes(const AttentionParams &p, int64_t row)
{
    if (!p.qout) return;
    if (p.q_bits == 8) {
        for (int c = p.hidden; c < p.q_pitch; c += 8) *reinterpret_cast<uint2 *>(p.qout + row * p.q_pitch + c) = make_uint2(0u, 0u);
    } else {
        for (int c = p.hidden; c < p.q_pitch; c += 8) *reinterpret_cast<uint32_t *>(p.qout + ((row * p.q_pitch + c) >> 1)) = 0u;
    }
}

// What attention_route sends to the kernel of attention.hip: up to ATTENTION_HELD_KEYS tokens, d_k <= 32 or a multiple of 8
int run_attention_held(const AttentionParams &p, hipStream_t st);
// once-per-device setup of its instantiations (nothing is launched)
int setup_attention();

}  // namespace mkq
