// Second half of the 4-bit encoder layer, everything behind the attention, in one launch.
#pragma once

#include "gemm_common.h"

namespace mkq {

struct LayerTailParams {
    int M, H, F, Hp, Fp;      // tokens, hidden and FFN size, codes per row of the buffers that feed a linear of each
    const uint8_t *c1;        // [M, Hp / 2] codes of the attention context
    const uint16_t *h_in;     // [M, H] binary16
    const uint8_t *W_ao, *W_up, *W_down;
    const float *sw_ao, *sw_up, *sw_down;
    const float *b_ao, *b_up, *b_down;  // or null
    float sx_ao, sx_up, sx_down;
    const float *g1, *be1, *g2, *be2;   // LayerNorm
    float eps;
    uint16_t *u, *h1, *d, *h_out;
    uint8_t *c2, *c3;
    uint8_t *q_next;          // or null
    float s_next;
    int next_bits, next_pitch;
};

// Launches it.
int run_layer_tail(const LayerTailParams &p, hipStream_t st);
// Launches the attention output with the LayerNorm behind it alone (u, h1, c2): rows of up to 768 codes.
int run_output_norm(const LayerTailParams &p, hipStream_t st);
// once-per-device setup of its instantiations (nothing is launched)
int setup_layer_tail();

}  // namespace mkq
