// What follows the attention of a 4-bit encoder layer, in one launch: attention output + residual, LayerNorm, FFN, residual, LayerNorm
// (section 3.2), each with its re-quantization.  For small hidden sizes, whose five kernels are mostly launches: a layer of hidden
// size 312 has 0.43 MB of weights behind the attention, and its kernels on 4096 tokens take 6, 4.3, 12.3, 8 and 4.3 us for that.
//
// A workgroup of eight waves has 16 tokens and all their columns, so that no token leaves the CU between the linears.  Every wave
// multiplies the 16 tokens by columns of its own (v_mfma_i32_16x16x64_i8, weights as the A operand): 16 GH of the hidden columns, and of the
// FFN's columns, which go by in chunks, 16 GF; a chunk's codes are the other linear's operand right away.
// Weights are read by every workgroup, so what bounds the products is the path from L2 into a CU, 64 bytes a cycle at best: through
// wave-private rings in LDS, filled by pieces of whole 128-byte rows, 54 were measured with one workgroup and 40 to 49 with all CUs
// (loaded straight into the registers that the matrix core takes, 16 rows to 16 neighbouring lanes, it is 15).  Then vector issue: GELU
// and code decisions of 16 x 1280 columns take 6000 of the workgroup's 37000 cycles, LayerNorm 4800 and 3200, widening 7000.
// Widening is two operations per eight codes, not three: 16 * high nibble meets the token's code, low nibble + 8 meets 16 times the code, and
// 128 times the sum of a token's even codes comes off its accumulators (token_operand).
// Layers of hidden size 312 and 4096 tokens 44.6 -> 35.1 us in a graph, of 1024 30.6 -> 29.0 from call to call (small_layer_tail).  Of hidden size 768 (2.65 MB of
// weights, 50000 cycles at that rate and as much again of vector issue) it takes 56 us at 4096 tokens and 41 at 440, the five kernels 52 and 26.
#include "layer_tail.h"

namespace mkq {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// GH, GF: tiles of 16 hidden and FFN columns of a wave; RH, RF: slots of its ring that these phases use
template <int GH_, int RH_, int GF_, int RF_>
struct LayerTailCfg {
    static constexpr int GH = GH_, GF = GF_, RH = RH_, RF = RF_;
    static constexpr int BM = 16, WAVES = 8, THREADS = 64 * WAVES;
    static constexpr int CF = 16 * GF * WAVES;                    // FFN columns of one chunk
    static constexpr int HCAP = 16 * GH * WAVES;                  // largest hidden size
    static constexpr int KH = (HCAP + 255) / 256 * 256;           // codes per token of the operand made from hidden columns
    static constexpr int PITCH = HCAP * 2 + 16;                   // bytes per token of the binary16 tile
    static constexpr int MAXC = (HCAP + 255) / 256;               // 16-byte chunks of a row per lane of a half wave
    static constexpr int SLOTS = RH > RF ? RH : RF;               // of a wave's ring, 2 KiB each
    static constexpr int NSH = (GH + 3) / 4, NSF = (GF + 3) / 4;  // copies of 64 floats that a wave's scales take
    static constexpr int TILE_AT = WAVES * SLOTS * 2048;          // (the rings come first)
    static constexpr int OPH_AT = TILE_AT + BM * PITCH;
    static constexpr int OPF_AT = OPH_AT + BM * KH;
    static constexpr int OPF_BYTES = BM * CF;                     // two of them: a wave can be a chunk ahead
    static constexpr int CORR_AT = OPF_AT + 2 * OPF_BYTES;        // 16 times the even codes' sums: of c1, c2, c3
    static constexpr int AFFINE_AT = CORR_AT + 3 * BM * 4;        // gamma, then beta of a LayerNorm
    static constexpr int SCALE_AT = AFFINE_AT + 2 * HCAP * 4;     // per wave: scales and biases of hidden, then of FFN columns
    static constexpr int LDS_BYTES = SCALE_AT + WAVES * (NSH + NSF) * 512;
    static_assert(LDS_BYTES <= 160 * 1024 && GF % 2 == 0 && GH % RH == 0 && GF % RF == 0 && CF % 256 == 0, "");
};

// One packed word (8 codes of a token) as the matrix core takes it here: .x the odd codes as they are, .y the even
// codes times 16; what 16 times the even codes sum to is added to sum.
__device__ __forceinline__ uint2 token_operand(uint32_t w, int &sum)
{
    const uint32_t x = (w >> 4) & 0x0F0F0F0Fu, s = x & 0x08080808u;
    const uint32_t lo = (w << 4) & 0xF0F0F0F0u;
    sum = __builtin_amdgcn_sdot4((int)lo, 0x01010101, sum, false);
    return make_uint2(x | ((s << 5) - (s << 1)), lo);
}

// Where the operand of codes k .. k + 7 (k % 8 == 0) of token t lies: 1 KiB for every matrix step of 64 codes, in the order of the lanes
// that read it, but for the turn that spreads the writes of one token over the banks
__device__ __forceinline__ int token_operand_at(int t, int k)
{
    const int sj = ((k >> 6) & 2) | ((k >> 4) & 1), qq = (k >> 5) & 3;
    const int s = ((k >> 8) << 2) | sj;
    return s * 1024 + (qq * 16 + (t ^ qq ^ (sj * 4))) * 16 + (k & 8);
}

// FFN: all of it; otherwise the attention output and the LayerNorm behind it
template <class Cfg, bool FFN>
__global__ __launch_bounds__(Cfg::THREADS, 2) void layer_tail_kernel(const LayerTailParams p)
{
    constexpr int GH = Cfg::GH, GF = Cfg::GF, RH = Cfg::RH, RF = Cfg::RF, BM = Cfg::BM, MAXC = Cfg::MAXC, CF = Cfg::CF;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    uint8_t *const tile = lds + Cfg::TILE_AT, *const oph = lds + Cfg::OPH_AT;
    int *const corr = reinterpret_cast<int *>(lds + Cfg::CORR_AT);  // [3][BM]
    float *const affine = reinterpret_cast<float *>(lds + Cfg::AFFINE_AT);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = lane & 15, q = lane >> 4;
    const int64_t row0 = (int64_t)xcd_index(blockIdx.x, gridDim.x) * BM;
    const int rows = p.M - row0 < BM ? (int)(p.M - row0) : BM;
    const int pitch_h = p.Hp / 2, pitch_f = p.Fp / 2;
    const int units_h = (p.Hp + 255) / 256;

    // ---- weights: a ring of the wave's own, 16 channels x 256 codes to a slot, copied by two instructions of 8 rows x 128 bytes ----
    const uint32_t ring_at = lds0 + wave * Cfg::SLOTS * 2048;
    const uint8_t *const ring = lds + wave * Cfg::SLOTS * 2048;
    const int rd0 = t * 128 + ((q ^ ((t >> 1) & 7)) * 16);  // the lane's pieces of a slot: at rd0, and at rd0 ^ 64 of the second half line
    // byte offsets of the lane's pieces of G tiles from channel n0 on.  Row i of tile T is channel 4 G (i / 4) + 4 T + i % 4, which
    // gives lane (t, q) the channels 4 G q .. 4 G q + 4 G - 1 of token t of the results
    auto rows_of = [&](auto gc, int n0, int n, int pitch, uint32_t (&voff)[decltype(gc)::value][2]) __attribute__((always_inline)) {
        constexpr int G = decltype(gc)::value;
#pragma unroll
        for (int T = 0; T < G; ++T)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = 8 * h + (lane >> 3);
                const int r = n0 + 4 * G * (i >> 2) + 4 * T + (i & 3);
                voff[T][h] = (uint32_t)((r < n ? r : n - 1)) * (uint32_t)pitch + 16u * (uint32_t)((lane & 7) ^ ((i >> 1) & 7));
            }
    };
    auto copy = [&](auto slotc, const uint8_t *W, int k, int pitch, const uint32_t (&voff)[2]) __attribute__((always_inline)) {
        constexpr int slot = decltype(slotc)::value;
        if (k + 128 <= pitch) {
            dma_copy16<slot * 2048>(W + k, voff[0], ring_at);
            dma_copy16<slot * 2048 + 1024>(W + k, voff[1], ring_at);
        } else {  // the row ends with the first half line: its second half is read again where the other would be (times zero codes)
            const uint32_t back = (uint32_t)(lane & 4) << 4;
            dma_copy16<slot * 2048>(W + k, voff[0] - back, ring_at);
            dma_copy16<slot * 2048 + 1024>(W + k, voff[1] - (64u - back), ring_at);
        }
    };
    v4u w[2][2];  // this tile's and the next one's
    auto take = [&](auto slotc, int to) __attribute__((always_inline)) {
        constexpr int slot = decltype(slotc)::value;
        w[to][0] = *reinterpret_cast<const v4u *>(ring + slot * 2048 + rd0);
        w[to][1] = *reinterpret_cast<const v4u *>(ring + slot * 2048 + (rd0 ^ 64));
    };
    auto lds_done = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

    // Tokens' operand of 256 codes: four matrix steps of 64
    const int lane_at = (q * 16 + (t ^ q)) * 16;
    v4i b[4];
    auto fetch_b = [&](auto sc, const uint8_t *op) __attribute__((always_inline)) {
        constexpr int s = decltype(sc)::value;
        b[s] = *reinterpret_cast<const v4i *>(op + s * 1024 + (lane_at ^ (s * 64)));
    };
    // 256 codes of G tiles through R slots.  The tile that is multiplied is in registers, and so is the next one before the multiplication
    // starts; what its slot gets then is the tile R further on, of the next unit (refill(T)) or, in the LAST one of a phase, of the next
    // phase (next(n), its first RN tiles).
    auto unit = [&](auto gc, auto rc, auto rnc, auto lastc, auto &acc, const uint8_t *op_next, auto &&refill, auto &&refill_same, auto &&next) __attribute__((always_inline)) {
        constexpr int G = decltype(gc)::value, R = decltype(rc)::value, RN = decltype(rnc)::value;
        constexpr bool LAST = decltype(lastc)::value;
        static_for<G>([&](auto Tc) {
            constexpr int T = decltype(Tc)::value;
            lds_done();
            if constexpr (T + R < G) refill_same(IntC<T + R>{});
            else if constexpr (!LAST) refill(IntC<T + R - G>{});
            else if constexpr (T + R - G < RN) next(IntC<T + R - G>{});
            // copies issued behind those of the tile that is taken now
            constexpr int sent = T + R - G + 1 < 0 ? 0 : T + R - G + 1 < RN ? T + R - G + 1 : RN;  // tiles of the next phase
            constexpr int behind = !LAST ? R - 1 : T + 1 < G ? (T + R < G ? R - 1 : G - 2 - T + sent) : sent - 1;
            if constexpr (!LAST || T + 1 < G || RN > 0) {
                wait_vmcnt<2 * behind>();
                take(IntC<(T + 1 < G ? (T + 1) % R : 0)>{}, (T + 1) & 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<4>([&](auto sc) {
                constexpr int s = decltype(sc)::value;
                const uint32_t w0 = w[T & 1][s / 2][2 * (s % 2)], w1 = w[T & 1][s / 2][2 * (s % 2) + 1];
                const v4i a = {(int)(w0 & 0xF0F0F0F0u), (int)((w0 & 0x0F0F0F0Fu) ^ 0x08080808u),
                               (int)(w1 & 0xF0F0F0F0u), (int)((w1 & 0x0F0F0F0Fu) ^ 0x08080808u)};
                acc[T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b[s], acc[T], 0, 0, 0);
                if constexpr (!LAST && T == G - 1) fetch_b(sc, op_next);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (G & 1) {
            w[0][0] = w[1][0];
            w[0][1] = w[1][1];
        }
        if constexpr (LAST && RN > R) static_for<RN - R>([&](auto nc) { next(IntC<R + decltype(nc)::value>{}); });
    };
    // n (>= 1) units of the operand at op, whose first R tiles are on their way and whose first one is in registers; fetch(T, k) copies what
    // is k codes behind the first unit, last() runs before the last unit
    auto units = [&](auto gc, auto rc, auto rnc, auto &acc, const uint8_t *op, int n, auto &&fetch, auto &&last, auto &&next) __attribute__((always_inline)) {
        static_for<4>([&](auto sc) { fetch_b(sc, op); });
#pragma unroll 1
        for (int u = 1; u < n; ++u) {
            op += 4 * 1024;
            unit(gc, rc, rnc, IntC<0>{}, acc, op, [&](auto Tc) { fetch(Tc, u * 128); }, [&](auto Tc) { fetch(Tc, u * 128 - 128); }, next);
        }
        last();
        unit(gc, rc, rnc, IntC<1>{}, acc, op, [](auto) {}, [&](auto Tc) { fetch(Tc, n * 128 - 128); }, next);
    };

    // n floats from `from` on to LDS, those past the last one in their places
    auto copy_floats = [&](auto nc, const float *from, int limit, uint32_t to) __attribute__((always_inline)) {
        static_for<decltype(nc)::value>([&](auto ic) {
            const int at = 64 * decltype(ic)::value + lane;
            dma_copy4<256 * decltype(ic)::value>(reinterpret_cast<const uint8_t *>(from), 4u * (uint32_t)(at < limit ? at : limit - 1), to);
        });
    };
    auto copy_affine = [&](const float *gamma, const float *beta) __attribute__((always_inline)) {
        for (int i = wave; i < Cfg::HCAP / 64; i += Cfg::WAVES) {
            const int from = i * 64 < p.H ? i * 64 : 0;
            copy_floats(IntC<1>{}, gamma + from, p.H - from, lds0 + Cfg::AFFINE_AT + i * 256);
            copy_floats(IntC<1>{}, beta + from, p.H - from, lds0 + Cfg::AFFINE_AT + Cfg::HCAP * 4 + i * 256);
        }
    };
    // scales and biases of the wave's 16 G channels from n0 on
    constexpr int SCALES_H = 0, SCALES_F = Cfg::NSH * 512, SCALES = SCALES_F + Cfg::NSF * 512;
    const float *const sc_lds = reinterpret_cast<const float *>(lds + Cfg::SCALE_AT + wave * SCALES);
    auto copy_scales = [&](auto nc, int at, int n0, int n, const float *s_w, const float *bias) __attribute__((always_inline)) {
        constexpr int NS = decltype(nc)::value;
        const int from = n0 < n ? n0 : 0;
        copy_floats(nc, s_w + from, n - from, lds0 + Cfg::SCALE_AT + wave * SCALES + at);
        copy_floats(nc, (bias ? bias : s_w) + from, n - from, lds0 + Cfg::SCALE_AT + wave * SCALES + at + NS * 256);
    };

    // LayerNorm of the tile's rows, one to a half wave; out: what the rows become (binary16, to the tile too), codes to the operand.
    // Sums run in the order of the kernel that has these rows at other token counts (layernorm_half_waves): up to 512 values the whole
    // wave's, in which lane l of 64 has chunk l, and l and l + 32 meet first; beyond, the half wave's, one chunk after the other.
    constexpr bool MEET = FFN;
    static_assert(MEET ? Cfg::HCAP <= 512 && MAXC <= 2 : Cfg::HCAP <= 768, "");
    const int hl = lane & 31, hw = wave * 2 + (lane >> 5);
    const int chunks = p.H / 8;
    auto layernorm = [&](auto midc, uint16_t *x_out, uint16_t *y_out, uint8_t *q_out, float s_q) __attribute__((always_inline)) {
        constexpr bool MID = decltype(midc)::value;
        const QuantStep step4 = quant_step<4>(s_q), step8 = quant_step<8>(s_q);
        lds_barrier();
        const int r = hw;
        const int64_t row = row0 + r;
        const bool in = r < rows;
        float v[MAXC][8], sums[2] = {0.0f, 0.0f};
        v4u raw[MAXC];
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            raw[i] = v4u{0, 0, 0, 0};
            if (hl + i * 32 < chunks) raw[i] = *reinterpret_cast<const v4u *>(tile + r * Cfg::PITCH + (hl + i * 32) * 16);
        }
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[i][2 * e] = half_bits_to_float((uint16_t)(raw[i][e] & 0xFFFFu));
                v[i][2 * e + 1] = half_bits_to_float((uint16_t)(raw[i][e] >> 16));
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) sums[MEET ? i : 0] += v[i][e];
        }
        const float mean = lane_reduce<32>(sums[0] + sums[1], AddF32()) / (float)p.H;
        float sqs[2] = {0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            if (hl + i * 32 < chunks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[i][e] -= mean;
                float &sq = sqs[MEET ? i : 0];
                sq = MEET || i == 0 ? add_squares<true>(sq, v[i]) : add_squares<false>(sq, v[i]);
            }
        }
        const float rstd = 1.0f / sqrtf(lane_reduce<32>(sqs[0] + sqs[1], AddF32()) / (float)p.H + p.eps);
        int csum = 0;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = hl + i * 32;
            uint32_t packed = 0;  // codes past the row: zero
            if (c < chunks) {
                float o[8];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const v4f gg = *reinterpret_cast<const v4f *>(affine + c * 8 + 4 * h), bb = *reinterpret_cast<const v4f *>(affine + Cfg::HCAP + c * 8 + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[4 * h + e] = v[i][4 * h + e] * rstd * gg[e] + bb[e];
                }
                const v4u y = {pack2_f16(o[0], o[1]), pack2_f16(o[2], o[3]), pack2_f16(o[4], o[5]), pack2_f16(o[6], o[7])};
                if (MID && FFN) *reinterpret_cast<v4u *>(tile + r * Cfg::PITCH + c * 16) = y;
                if (in) {
                    *reinterpret_cast<v4u *>(x_out + row * p.H + c * 8) = raw[i];
                    *reinterpret_cast<v4u *>(y_out + row * p.H + c * 8) = y;
                }
                if (MID || p.next_bits == 4) packed = quantize8<4>(o, step4).x;
                else if (q_out && in) *reinterpret_cast<uint2 *>(q_out + row * p.next_pitch + c * 8) = quantize8<8>(o, step8);
            }
            if (MID) {
                if (in && c * 8 < p.Hp) reinterpret_cast<uint32_t *>(q_out)[row * (p.Hp / 8) + c] = packed;
                if (FFN && c * 8 < Cfg::KH) *reinterpret_cast<uint2 *>(oph + token_operand_at(r, c * 8)) = token_operand(packed, csum);
            } else if (q_out && in && p.next_bits == 4 && c * 8 < p.next_pitch) {
                reinterpret_cast<uint32_t *>(q_out)[row * (p.next_pitch / 8) + c] = packed;
            }
        }
        if (MID && FFN) {
            const float total = lane_reduce<32>((float)csum, AddF32());
            if (hl == 0) corr[BM + r] = (int)total;
        }
    };

    // results of hidden columns: dequantized, added to the tile in place
    const int n_h = wave * 16 * GH;
    auto add_to_tile = [&](auto &acc, int ex, float s_x, bool biased) __attribute__((always_inline)) {
#pragma unroll
        for (int T = 0; T < GH; ++T) {
            __builtin_amdgcn_sched_barrier(0);
            v4f sc = *reinterpret_cast<const v4f *>(sc_lds + SCALES_H / 4 + 4 * GH * q + 4 * T);
            v4f bi = *reinterpret_cast<const v4f *>(sc_lds + SCALES_H / 4 + Cfg::NSH * 64 + 4 * GH * q + 4 * T);
            uint2 *const at = reinterpret_cast<uint2 *>(tile + t * Cfg::PITCH + (n_h + 4 * GH * q + 4 * T) * 2);
            const uint2 r = *at;
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[e] = (s_x * sc[e]) * 0.0625f;  // (the accumulators are 16 times the sums: exact)
                y[e] = __fmaf_rn((float)(acc[T][e] - ex), sc[e], biased ? bi[e] : 0.0f);
                // keep the binary32 rounding (see gemm_i4_epilogue)
                asm volatile("" : "+v"(y[e]));
            }
            y[0] += half_bits_to_float((uint16_t)(r.x & 0xFFFFu));
            y[1] += half_bits_to_float((uint16_t)(r.x >> 16));
            y[2] += half_bits_to_float((uint16_t)(r.y & 0xFFFFu));
            y[3] += half_bits_to_float((uint16_t)(r.y >> 16));
            *at = make_uint2(pack2_f16(y[0], y[1]), pack2_f16(y[2], y[3]));
        }
    };

    // ---- attention output ----
    uint32_t voff_h[GH][2], voff_f[GF][2];
    const int n_f = wave * 16 * GF;
    rows_of(IntC<GH>{}, n_h, p.H, pitch_h, voff_h);
    copy_affine(p.g1, p.be1);
    copy_scales(IntC<Cfg::NSH>{}, SCALES_H, n_h, p.H, p.sw_ao, p.b_ao);
    static_for<RH>([&](auto Tc) { copy(Tc, p.W_ao, 0, pitch_h, voff_h[decltype(Tc)::value]); });
    {
        const int r = hw;
        const bool in = r < rows;
        const int64_t row = row0 + r;
        v4u c = {0, 0, 0, 0}, h[MAXC];
        if (in && hl * 32 < p.Hp) c = *reinterpret_cast<const v4u *>(p.c1 + row * pitch_h + hl * 16);
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            h[i] = v4u{0, 0, 0, 0};
            if (in && hl + i * 32 < chunks) h[i] = *reinterpret_cast<const v4u *>(p.h_in + row * p.H + (hl + i * 32) * 8);
        }
        int csum = 0;
        if (hl * 32 < Cfg::KH) {
            const uint2 x0 = token_operand(c.x, csum), x1 = token_operand(c.y, csum), x2 = token_operand(c.z, csum), x3 = token_operand(c.w, csum);
            *reinterpret_cast<v4u *>(oph + token_operand_at(r, hl * 32)) = v4u{x0.x, x0.y, x1.x, x1.y};
            *reinterpret_cast<v4u *>(oph + token_operand_at(r, hl * 32 + 16)) = v4u{x2.x, x2.y, x3.x, x3.y};
        }
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if (hl + i * 32 < chunks) *reinterpret_cast<v4u *>(tile + r * Cfg::PITCH + (hl + i * 32) * 16) = h[i];
        const float total = lane_reduce<32>((float)csum, AddF32());
        if (hl == 0) {
            corr[r] = (int)total;
            corr[2 * BM + r] = 0;
        }
    }
    if constexpr (FFN) rows_of(IntC<GF>{}, n_f, p.F, pitch_h, voff_f);
    wait_vmcnt<0>();
    lds_barrier();
    take(IntC<0>{}, 0);
    const auto next_up = [&](auto nc) { copy(nc, p.W_up, 0, pitch_h, voff_f[decltype(nc)::value]); };
    {
        v4i acc[GH];
#pragma unroll
        for (int T = 0; T < GH; ++T) acc[T] = v4i{0, 0, 0, 0};
        units(IntC<GH>{}, IntC<RH>{}, IntC<FFN ? RF : 0>{}, acc, oph, units_h,
              [&](auto Tc, int k) { copy(IntC<decltype(Tc)::value % RH>{}, p.W_ao, k, pitch_h, voff_h[decltype(Tc)::value]); },
              [&] { if constexpr (FFN) copy_scales(IntC<Cfg::NSF>{}, SCALES_F, n_f, p.F, p.sw_up, p.b_up); }, next_up);
        add_to_tile(acc, 8 * corr[t], p.sx_ao, p.b_ao != nullptr);
    }
    layernorm(IntC<1>{}, p.u, p.h1, p.c2, p.sx_up);
    if constexpr (!FFN) return;
    lds_barrier();
    copy_affine(p.g2, p.be2);
    copy_scales(IntC<Cfg::NSH>{}, SCALES_H, n_h, p.H, p.sw_down, p.b_down);

    // ---- FFN, by chunks of its columns ----
    rows_of(IntC<GH>{}, n_h, p.H, pitch_f, voff_h);
    const int nchunks = (p.F + CF - 1) / CF;
    const QuantStep step = quant_step<4>(p.sx_down);
    v4i acc[GH];
    int csum = 0;
#pragma unroll
    for (int T = 0; T < GH; ++T) acc[T] = v4i{0, 0, 0, 0};
    for (int ch = 0; ch < nchunks; ++ch) {
        uint8_t *const opf = lds + Cfg::OPF_AT + (ch & 1) * Cfg::OPF_BYTES;
        const int kf = ch * (CF / 2);  // bytes of a row of W_down
        {
            v4i up[GF];
            const int ex = -8 * corr[BM + t];
#pragma unroll
            for (int T = 0; T < GF; ++T) up[T] = v4i{ex, ex, ex, ex};
            const int n = ch * CF + n_f + 4 * GF * q;
            units(IntC<GF>{}, IntC<RF>{}, IntC<RH>{}, up, oph, units_h,
                  [&](auto Tc, int k) { copy(IntC<decltype(Tc)::value % RF>{}, p.W_up, k, pitch_h, voff_f[decltype(Tc)::value]); }, [] {},
                  [&](auto nc) { copy(nc, p.W_down, kf, pitch_f, voff_h[decltype(nc)::value]); });
#pragma unroll
            for (int e8 = 0; e8 < GF / 2; ++e8) {
                __builtin_amdgcn_sched_barrier(0);
                const int c = n + 8 * e8;
                v4f sc[2], bi[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    sc[h] = *reinterpret_cast<const v4f *>(sc_lds + SCALES_F / 4 + 4 * GF * q + 8 * e8 + 4 * h);
                    bi[h] = *reinterpret_cast<const v4f *>(sc_lds + SCALES_F / 4 + Cfg::NSF * 64 + 4 * GF * q + 8 * e8 + 4 * h);
                }
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    y[e] = __fmaf_rn((float)up[2 * e8 + (e >> 2)][e & 3], (p.sx_up * sc[e >> 2][e & 3]) * 0.0625f, p.b_up ? bi[e >> 2][e & 3] : 0.0f);
                    asm volatile("" : "+v"(y[e]));
                    y[e] = gelu_erf(y[e]);
                }
                const uint32_t packed = c < p.F ? quantize8<4>(y, step).x : 0u;
                if (t < rows && c < p.Fp) reinterpret_cast<uint32_t *>(p.c3)[(row0 + t) * (p.Fp / 8) + (c >> 3)] = packed;
                *reinterpret_cast<uint2 *>(opf + token_operand_at(t, n_f + 4 * GF * q + 8 * e8)) = token_operand(packed, csum);
            }
        }
        if (ch == nchunks - 1) atomicAdd(&corr[2 * BM + t], csum);
        lds_barrier();
        const int left = (p.Fp - ch * CF + 255) / 256;
        const int units_f = left < CF / 256 ? left : CF / 256;
        if (ch + 1 < nchunks) rows_of(IntC<GF>{}, (ch + 1) * CF + n_f, p.F, pitch_h, voff_f);
        units(IntC<GH>{}, IntC<RH>{}, IntC<RF>{}, acc, opf, units_f,
              [&](auto Tc, int k) { copy(IntC<decltype(Tc)::value % RH>{}, p.W_down, kf + k, pitch_f, voff_h[decltype(Tc)::value]); },
              [&] { copy_scales(IntC<Cfg::NSF>{}, SCALES_F, (ch + 1) * CF + n_f, p.F, p.sw_up, p.b_up); }, next_up);
    }
    wait_vmcnt<0>();  // (what the last phase fetched for a next one is in before the workgroup's LDS can be another's)
    add_to_tile(acc, 8 * corr[2 * BM + t], p.sx_down, p.b_down != nullptr);
    layernorm(IntC<0>{}, p.d, p.h_out, p.q_next, p.s_next);
}

// p null: setup only
template <class Cfg, bool FFN>
static int launch_tail(const LayerTailParams *p, hipStream_t st)
{
    static PerDeviceOnce once;
    int64_t resident = 0;
    const int rc = resident_workgroups(once, layer_tail_kernel<Cfg, FFN>, Cfg::THREADS, Cfg::LDS_BYTES, 1, &resident);
    if (rc != MKQ_OK || !p) return rc;
    layer_tail_kernel<Cfg, FFN><<<(unsigned)ceil_div(p->M, Cfg::BM), Cfg::THREADS, Cfg::LDS_BYTES, st>>>(*p);
    return launch_status();
}
using TailWide = LayerTailCfg<3, 3, 10, 5>;    // chunks of 1280 FFN columns
using TailNarrow = LayerTailCfg<3, 3, 6, 3>;   // of 768
using OutputNorm = LayerTailCfg<6, 6, 2, 1>;   // up to 768 hidden columns, without the FFN

int run_layer_tail(const LayerTailParams &p, hipStream_t st)
{
    // the chunks whose columns add up to less (a chunk is multiplied whole), and the fewer of them
    static_assert(TailWide::CF == LAYER_TAIL_WIDE && TailNarrow::CF == LAYER_TAIL_NARROW, "");
    const int64_t wide = layer_tail_columns(p.F, TailWide::CF), narrow = layer_tail_columns(p.F, TailNarrow::CF);
    return wide <= narrow ? launch_tail<TailWide, true>(&p, st) : launch_tail<TailNarrow, true>(&p, st);
}

int run_output_norm(const LayerTailParams &p, hipStream_t st) { return launch_tail<OutputNorm, false>(&p, st); }

int setup_layer_tail()
{
    int rc = launch_tail<TailWide, true>(nullptr, nullptr);
    if (rc == MKQ_OK) rc = launch_tail<TailNarrow, true>(nullptr, nullptr);
    return rc != MKQ_OK ? rc : launch_tail<OutputNorm, false>(nullptr, nullptr);
}

}  // namespace mkq
