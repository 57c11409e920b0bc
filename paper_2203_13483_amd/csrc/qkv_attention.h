// The q, k, v projection of a 4-bit layer and the attention behind it, in one launch.
#pragma once

#include "attention.h"

namespace mkq {

struct QkvAttentionParams {
    AttentionParams att;      // (its qkv is what is written here; heads of at most 32, codes of 4 bits)
    const uint8_t *c0;        // [tokens, K / 2] codes of the layer's input
    const uint8_t *W;         // [3 hidden, K / 2]
    const float *s_w, *bias;  // [3 hidden]; bias may be null
    float s_x;
    int K;                    // codes per row of both
    uint16_t *qkv;            // [tokens, 3 hidden]
};

// Launches it (small_layer_attention_choice says for which layers).
int run_qkv_attention(const QkvAttentionParams &p, hipStream_t st);
// once-per-device setup of its instantiations (nothing is launched)
int setup_qkv_attention();

}  // namespace mkq
