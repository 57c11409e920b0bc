// q, k, v = Lin_qkv(codes) and the attention core behind it in one launch, one workgroup of four waves per (sequence, head), for heads of
// at most 32 and sequences of at most 128 tokens: what the two launches share, the 6 bytes of q, k, v per token and hidden column, is
// written once and read by nobody, and one launch is gone.  Up to four tiles of 32 tokens times the head's columns of q, of k and of v,
// 32 each (dimensions past d_k repeat the last one's weights and are cleared behind the product).
// What bounds it is one workgroup's chain, with 384 of them for 32 sequences of 12 heads: of 16500 cycles (128 tokens, hidden size 312) set-up
// 2000, first stage out of memory 2100, product 2900, dequantization into LDS 2000, rows to memory 2500, softmax 2100, product with V
// 900, codes 1000 (these three with 32x32x16 products; the ones that give the held kernel's bits add 0.4 us to 11.1).  (Rows leave
// through LDS, neighbouring lanes with neighbouring pieces: straight from the result registers, a row to a lane, they took twice as long.)
// Of a layer of hidden size 312 it takes 4.5 us of 50 at 4096 tokens, 3.9 of 39 at 1024 (small_layer_attention_choice).  With heads of 64
// and hidden size 768 the chain is longer than what it saves: layers of 32 x 128 tokens 79.8 -> 79.3, padding-free of 440 40.1 -> 43.7.
#include "qkv_attention.h"

#include "gemm_i4_params.h"

namespace mkq {

typedef int v4i_4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t word_1 __attribute__((aligned(1)));

// KT: tiles of 32 tokens of the longest sequence
template <int KT>
struct QkvAttentionCfg {
    static constexpr int DKP = 32, THREADS = 256;
    static constexpr int STAGE_BYTES = (32 * KT + 3 * DKP) * 128;  // 256 codes of every token and channel
    // behind the product: q, k, v row by row, V transposed, scales and biases
    static constexpr int SCALE_AT = 3 * 32 * KT * DKP * 2 + DKP * (KT == 1 ? 64 : KT == 2 ? 128 : 256);
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
    static_assert(SCALE_AT + 2 * 3 * DKP * 4 <= LDS_BYTES, "");
};

// 16-byte chunk c of row r of q, K and V is kept at c ^ swz_rows(r): a product's fragment takes rows that differ in bits 0, 1, 3 and 4 of
// K, and in bits 0 to 3 of q, and each sixteen meet all 64 banks; so do eight neighbouring rows that are written.
__device__ __forceinline__ int swz_rows(int r) { return ((r >> 3) & 1) | (((r >> 2) ^ (r >> 4)) & 1) << 1; }

// VEC = 8: d_k % 8 == 0; 2: even
template <int VEC, int KT>
__global__ __launch_bounds__(256, 2) void qkv_attention_kernel(const QkvAttentionParams p, const XcdRuns runs)
{
    using Cfg = QkvAttentionCfg<KT>;
    constexpr int DKP = Cfg::DKP;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    const AttentionParams &a = p.att;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    // Uniform batches: an eighth of (sequence, head) to each XCD.  Padding-free ones: runs of heads (attention_runs), which read the same
    // codes and write the same lines.  us a layer of hidden size 312, heads one by one -> runs: 32 x 128 tokens 37.3 -> 34.5, 64 rising
    // from 8 to 128 54.4 -> 52.4, 64 of 2298 37.5 -> 36.9, 16 of 440 27.1 -> 27.1, 256 x 40 80.3 -> 80.8.
    const int bh = a.cu_seqlens ? xcd_run_index(blockIdx.x, runs) : xcd_index(blockIdx.x, gridDim.x);
    const int b = bh / a.heads, head = bh - b * a.heads;
    int64_t row0 = (int64_t)b * a.seq;
    int seq = a.seq;
    if (a.cu_seqlens) {
        const int first = __builtin_amdgcn_readfirstlane(a.cu_seqlens[b]);
        row0 = first;
        seq = __builtin_amdgcn_readfirstlane(a.cu_seqlens[b + 1]) - first;
    }
    seq = seq < 32 * KT ? seq : 32 * KT;  // (longer than the caller's bound on the lengths: not computed)
    if (seq <= 0) return;                 // the whole workgroup
    const int hidden = a.hidden, dk = a.dk, pitch = p.K / 2;
    constexpr float MASKED = -1.0e30f;  // the score of a key past the end of the sequence

    const QuantStep step = quant_step<4>(a.s_next);
    uint8_t *const codes = a.qout + ((row0 * a.q_pitch + head * dk) >> 1);
    // scale and bias of one of the workgroup's channels
    const int sn = tid < 3 * DKP ? tid : 3 * DKP - 1;
    const int s_at = sn / DKP * hidden + head * dk + (sn % DKP < dk ? sn % DKP : dk - 1);

    // NM: tiles of 32 tokens that are computed
    auto run = [&](auto nmc) __attribute__((always_inline)) {
        constexpr int NM = decltype(nmc)::value;
        // a wave has all three tiles of channels (q, k, v) of one of four token tiles, half of them of one of two, or one of the only one
        constexpr int WN = NM == 4 ? 1 : NM == 2 ? 2 : 4, TN = (3 + WN - 1) / WN;
        const int wm = wave / WN, wn = wave % WN;

        constexpr int AROWS = 32 * NM, STAGE = (AROWS + 3 * DKP) * 128, LPW = (AROWS + 3 * DKP) / 32;
        uint32_t voff[LPW];
#pragma unroll
        for (int c = 0; c < LPW; ++c) {
            const int row = 8 * (4 * c + wave) + (lane >> 3);
            const int chunk = (lane & 7) ^ swz<8>(row & 15);
            int r;
            if (4 * c * 8 < AROWS) {  // (the same for all: token rows come in whole turns of the four waves)
                r = row < seq ? row : seq - 1;
            } else {
                const int n = row - AROWS, d = n % DKP;
                r = n / DKP * hidden + head * dk + (d < dk ? d : dk - 1);
            }
            voff[c] = (uint32_t)r * (uint32_t)pitch + 16u * chunk;
        }
        const uint8_t *const A = p.c0 + row0 * pitch;
        auto copy = [&](int k, int slot) __attribute__((always_inline)) {
            const uint32_t at = lds0 + slot * STAGE + wave * 1024;
            static_for<LPW>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                uint32_t off = voff[c];
                // a row that ends with the first half line: that is read twice (and the second copy not used)
                if (k + 128 > pitch && (((lane >> 2) ^ (lane >> 5) ^ wave) & 1)) off -= 64;
                dma_copy16<c * 4096>((4 * c * 8 < AROWS ? A : p.W) + k, off, at);
            });
        };
        v16i acc[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0;
        const int m = (NM == 1 ? 0 : wm) * 32 + fr;  // the lane's token
        int wrow[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t) wrow[t] = AROWS + (t * WN + wn < 3 ? t * WN + wn : 0) * 32 + w_row_perm(fr);
        const int nk = (pitch + 127) / 128;
        const float s_reg = p.s_w[s_at], b_reg = (p.bias ? p.bias : p.s_w)[s_at];
        copy(0, 0);
        if (nk > 1) copy(128, 1);
        for (int s = 0; s < nk; ++s) {
            if (s + 1 < nk) wait_vmcnt<LPW>();
            else wait_vmcnt<0>();
            lds_barrier();
            const uint8_t *const st = lds + (s & 1) * STAGE;
            // two rounds of 64 codes at a time
            for (int r0 = 0; r0 < (s * 128 + 128 <= pitch ? 4 : 2); r0 += 2) {
#pragma unroll
                for (int r = r0; r < r0 + 2; ++r) {
                    const uint4 x = *reinterpret_cast<const uint4 *>(st + m * 128 + (((2 * r + fh) ^ swz<8>(m & 15)) * 16));
                    uint4 y[TN];
#pragma unroll
                    for (int t = 0; t < TN; ++t) y[t] = *reinterpret_cast<const uint4 *>(st + wrow[t] * 128 + (((2 * r + fh) ^ swz<8>(wrow[t] & 15)) * 16));
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const v4i xa = h ? widen(x.z, x.w) : widen(x.x, x.y);
#pragma unroll
                        for (int t = 0; t < TN; ++t)
                            acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(h ? widen(y[t].z, y[t].w) : widen(y[t].x, y[t].y), xa, acc[t], 0, 0, 0);
                    }
                }
            }
            if (s + 2 < nk) {
                lds_barrier();
                copy((s + 2) * 128, s & 1);
            }
        }

        // ---- q, k, v: dequantized and narrowed, to LDS ----
        constexpr int ROWB = DKP * 2, SMAX = 32 * NM;
        constexpr int VCHP = NM == 1 ? 4 : NM == 2 ? 8 : 16, VROW = VCHP * 16;
        uint8_t *const sQ = lds, *const sK = lds + SMAX * ROWB, *const sVt = lds + 3 * SMAX * ROWB;  // (V row by row between the last two)
        float *const scale = reinterpret_cast<float *>(lds + Cfg::SCALE_AT);
        lds_barrier();
        if (tid < 3 * DKP) {
            scale[tid] = (p.s_x * s_reg) * 0.00390625f;  // (the accumulators are 256 times the sums: exact)
            scale[3 * DKP + tid] = p.bias ? b_reg : 0.0f;
        }
        lds_barrier();
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const int part = t * WN + wn;
            if (part >= 3) continue;  // (uniform)
#pragma unroll
            for (int G = 0; G < 2; ++G) {
                const int d0 = 16 * G + 8 * fh;
                float sc[8], bi[8];
                load8(scale + part * DKP + d0, sc);
                load8(scale + 3 * DKP + part * DKP + d0, bi);
                uint32_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float y0 = __fmaf_rn((float)acc[t][8 * G + 2 * e], sc[2 * e], bi[2 * e]);
                    float y1 = __fmaf_rn((float)acc[t][8 * G + 2 * e + 1], sc[2 * e + 1], bi[2 * e + 1]);
                    // keep the binary32 rounding (see gemm_i4_epilogue)
                    asm volatile("" : "+v"(y0), "+v"(y1));
                    h[e] = d0 + 2 * e < dk ? pack2_f16(y0, y1) : 0;  // (d_k is even)
                }
                *reinterpret_cast<uint4 *>(sQ + (part * SMAX + m) * ROWB + (((d0 >> 3) ^ swz_rows(m)) * 16)) = make_uint4(h[0], h[1], h[2], h[3]);
                if (part == 2) {
                    // two neighbouring lanes have the same head dimensions of two neighbouring keys: each takes four of them for both
                    const bool odd = lane & 1;
                    const uint32_t own[2] = {odd ? h[2] : h[0], odd ? h[3] : h[1]};
                    const uint32_t give[2] = {odd ? h[0] : h[2], odd ? h[1] : h[3]};
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give[i], 0xB1, 0xF, 0xF, true);
                        const uint32_t even_key = odd ? got : own[i], odd_key = odd ? own[i] : got;
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const int d = d0 + (odd ? 4 : 0) + 2 * i + e;
                            const uint32_t v = e ? (even_key >> 16) | (odd_key & 0xFFFF0000u) : (even_key & 0xFFFFu) | (odd_key << 16);
                            *reinterpret_cast<uint32_t *>(sVt + d * VROW + (((m >> 3) ^ (swz_dims(d) & (VCHP - 1))) * 16) + (m & 6) * 2) = v;
                        }
                    }
                }
            }
        }
        lds_barrier();

        // rows to memory
        {
            constexpr int PPR = DKP / 8, TOTAL = 3 * SMAX * PPR;
            uint16_t *const to0 = p.qkv + row0 * 3 * hidden + head * dk;
#pragma unroll
            for (int i = 0; i < (TOTAL + 255) / 256; ++i) {
                const int idx = tid + i * 256, r = idx / PPR, c = idx % PPR;
                if (TOTAL % 256 != 0 && idx >= TOTAL) break;
                const int part = r / SMAX, mm = r % SMAX;
                const v4i_4 v = *reinterpret_cast<const v4i *>(sQ + r * ROWB + ((c ^ swz_rows(mm)) * 16));
                uint32_t *const to = reinterpret_cast<uint32_t *>(to0 + (uint32_t)mm * (uint32_t)(3 * hidden) + part * hidden + c * 8);
                if (mm < seq) {
                    if (c * 8 + 8 <= dk) {
                        *reinterpret_cast<v4i_4 *>(to) = v;  // (aligned to 4 bytes only where VEC = 2)
                    } else if (VEC != 8) {
                        if (c * 8 < dk) to[0] = v.x;
                        if (c * 8 + 2 < dk) to[1] = v.y;
                        if (c * 8 + 4 < dk) to[2] = v.z;
                    }
                }
            }
        }

        // ---- attention: two blocks of 16 queries to a wave, all keys at once, with the products, the sums and their order of
        // attention_held_kernel, so that a layer's bits are those of its two launches ----
        if (wave * 32 >= seq) return;  // (no barrier follows)
        const int lr = lane & 15, lg = lane >> 4;
        const int prow = 8 * (lr >> 2) + (lr & 3);  // row i = lr of a fragment of K or V^T, and 4 more in the second of a pair
        v4f sc[2][NM][2];  // scores: element e of part t of group g is key 32 g + 8 lg + 4 t + e
        v8h qf[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = wave * 32 + 16 * j + lr;
            qf[j] = *reinterpret_cast<const v8h *>(sQ + r * ROWB + ((lg ^ swz_rows(r)) * 16));
        }
        float m2[2][2] = {{MASKED, MASKED}, {MASKED, MASKED}};
#pragma unroll
        for (int g = 0; g < NM; ++g) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int r = g * 32 + prow + 4 * t;
                const v8h kf = *reinterpret_cast<const v8h *>(sK + r * ROWB + ((lg ^ swz_rows(r)) * 16));
#pragma unroll
                for (int j = 0; j < 2; ++j) sc[j][g][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qf[j], v4f{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            }
            if (g * 32 + 32 > seq) {  // (uniform) keys that do not exist
                const int keys = seq - g * 32 - 8 * lg;
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e) sc[j][g][t][e] = (4 * t + e < keys) ? sc[j][g][t][e] : MASKED;
            }
            // (median with infinity: a maximum that does not quiet its operand with a second instruction first)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) m2[j][t] = __builtin_amdgcn_fmed3f(m2[j][t], sc[j][g][t][e], __builtin_inff());
        }
        const float c_exp = (1.0f / sqrtf((float)dk)) * 1.4426950408889634f;
        float inv[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float mx = fmaxf(m2[j][0], m2[j][1]);
            mx = lane_pair<16>(mx, MaxF32());
            mx = lane_pair<32>(mx, MaxF32());
            const float shift = -mx * c_exp;
            float d2[2] = {0.0f, 0.0f};
#pragma unroll
            for (int g = 0; g < NM; ++g)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sc[j][g][t][e] = __builtin_amdgcn_exp2f(__fmaf_rn(sc[j][g][t][e], c_exp, shift));
                        d2[t] += sc[j][g][t][e];
                    }
            float den = d2[0] + d2[1];
            den = lane_pair<16>(den, AddF32());
            den = lane_pair<32>(den, AddF32());
            inv[j] = 1.0f / den;
        }

        v4f ot[2][2];  // element e of part dt is head dimension 8 lg + 4 dt + e
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) ot[j][dt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int g = 0; g < NM; ++g) {
            v8h pf[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[j][e] = (_Float16)(sc[j][g][e >> 2][e & 3] * inv[j]);
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                const int d = prow + 4 * dt;
                const v8h vf = *reinterpret_cast<const v8h *>(sVt + d * VROW + (((4 * g + lg) ^ (swz_dims(d) & (VCHP - 1))) * 16));
#pragma unroll
                for (int j = 0; j < 2; ++j) ot[j][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, pf[j], ot[j][dt], 0, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int qrow = wave * 32 + 16 * j + lr, d0 = 8 * lg;
            if (qrow >= seq) continue;
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = ot[j][e >> 2][e & 3];
            const uint32_t packed = quantize8<4>(o, step).x;
            uint8_t *const to = codes + (uint32_t)qrow * (uint32_t)(a.q_pitch / 2) + d0 / 2;
            if (d0 + 8 <= dk) *reinterpret_cast<word_1 *>(to) = packed;  // (aligned to 4 bytes where VEC = 8)
            else if (VEC != 8) {
                if (d0 < dk) to[0] = (uint8_t)packed;
                if (d0 + 2 < dk) to[1] = (uint8_t)(packed >> 8);
                if (d0 + 4 < dk) to[2] = (uint8_t)(packed >> 16);
            }
            if (lg == 0 && head == a.heads - 1) attention_pad_codes(a, row0 + qrow);
        }
    };
    if (KT == 1 || seq <= 32) run(IntC<1>{});
    else if (KT == 2 || seq <= 64) run(IntC<KT < 2 ? 1 : 2>{});
    else run(IntC<KT < 4 ? 1 : 4>{});
}

// p null: setup only
template <int VEC, int KT>
static int launch_qkv_attention(const QkvAttentionParams *p, hipStream_t st)
{
    using Cfg = QkvAttentionCfg<KT>;
    const auto kernel = qkv_attention_kernel<VEC, KT>;
    static PerDeviceOnce once;
    int64_t resident = 0;
    const int rc = resident_workgroups(once, kernel, Cfg::THREADS, Cfg::LDS_BYTES, 8, &resident);
    if (rc != MKQ_OK || !p) return rc;
    const int64_t sequence_heads = (int64_t)p->att.batch * p->att.heads;
    kernel<<<(unsigned)sequence_heads, Cfg::THREADS, Cfg::LDS_BYTES, st>>>(*p, attention_runs(sequence_heads, p->att.heads));
    return launch_status();
}

template <int VEC>
static int dispatch_qkv_attention(const QkvAttentionParams *p, int seq, hipStream_t st)
{
    if (seq <= 32) return launch_qkv_attention<VEC, 1>(p, st);
    return seq <= 64 ? launch_qkv_attention<VEC, 2>(p, st) : launch_qkv_attention<VEC, 4>(p, st);
}

int run_qkv_attention(const QkvAttentionParams &p, hipStream_t st)
{
    return (p.att.dk % 8) == 0 ? dispatch_qkv_attention<8>(&p, p.att.seq, st) : dispatch_qkv_attention<2>(&p, p.att.seq, st);
}

int setup_qkv_attention()
{
    for (const int seq : {32, 64, 128}) {
        int rc = dispatch_qkv_attention<8>(nullptr, seq, nullptr);
        if (rc == MKQ_OK) rc = dispatch_qkv_attention<2>(nullptr, seq, nullptr);
        if (rc != MKQ_OK) return rc;
    }
    return MKQ_OK;
}

}  // namespace mkq
