// Binary16 linear  y = a W^T + b  (binary32 accumulate) with the same epilogue options as the quantized
// linear: the 16-bit float baseline that the W4A4 layer is timed against.  It runs the tile kernel of the
// quantized linears (gemm_tile.h) with binary16 operands, v_mfma_f32_32x32x16_f16 and stages of one 128-byte
// line (64 values of k) per operand row; the smallest launches have a kernel of their own.
#include "gemm_tile.h"

namespace mkq {

template <class Cfg>
static int launch_f16_by_epilogue(const GemmI4Params &p, hipStream_t st)
{
    const bool gelu = p.act == MKQ_ACT_GELU;
    if ((p.N % 8) == 0 && !(p.residual && gelu)) {
        if (p.out_dtype == MKQ_F16 && p.residual) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, true, false>, 16>(p, st);
        if (p.out_dtype == MKQ_F16 && gelu) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, true>, 16>(p, st);
        if (p.out_dtype == MKQ_F16) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, false>, 16>(p, st);
        if (!p.residual && !gelu) return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F32, false, false>, 16>(p, st);
    }
    return launch_gemm_i4_dma_generic<Cfg, 16>(p, st);
}

// ---------------------------------------------------------------------------------
// Arguments of the split kernel: its launches are the smallest, and with the tile kernel's block of three times this
// size a launch took 0.2 us longer (M = 1024, K = 3072, N = 768 13.9 instead of 13.7).
struct GemmF16Params {
    const uint8_t *A;  // [M, K] binary16
    const uint8_t *W;  // [N, K] binary16
    int M, N, K;
    const float *bias;        // [N] or null
    const uint16_t *residual; // [M, N] binary16 or null
    int act;
    void *out;
    int out_dtype;  // MKQ_F32 or MKQ_F16
};
// The split kernel of the smallest launches: 64x64 tiles, 32x32 per wave, 64-wide k stages in rings of four, and the k loop
// shared by two groups of four waves, each with a ring of its own over one half of K (with at most one workgroup per CU a
// lone wave per SIMD is bound by its own instruction stream: M = 128, K = 3072, N = 768 takes 15.1 us on the tile kernel,
// 12.4 here); the second group's partial sums are added to the first group's through LDS before the epilogue.
struct SplitF16 {
    static constexpr int TILE = 64, S = 4, GROUPS = 2, WAVES = 4;  // waves per group, 2 x 2
    static constexpr int THREADS = GROUPS * WAVES * 64;
    static constexpr int RB = 128, CH = RB / 16;  // bytes and 16-byte chunks per row and stage
    static constexpr int STAGE_BYTES = 2 * TILE * RB;
    static constexpr int ROWS_PER_COPY = 1024 / RB;
    static constexpr int LPW = STAGE_BYTES / 1024 / WAVES;  // copies per wave and stage
    static constexpr int RING_BYTES = S * STAGE_BYTES;
    static constexpr int LDS_BYTES = GROUPS * RING_BYTES + WAVES * 4096;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS is 160 KiB per CU");
};

template <bool TAIL>  // epi_gelu_tail
__global__ __launch_bounds__(SplitF16::THREADS) void gemm_f16_kernel(const GemmF16Params p)
{
    using Cfg = SplitF16;
    constexpr int TILE = Cfg::TILE, RB = Cfg::RB, CH = Cfg::CH, S = Cfg::S, LPW = Cfg::LPW;

    extern __shared__ __attribute__((aligned(16))) uint8_t smem_all[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave_all / Cfg::WAVES, wave = wave_all % Cfg::WAVES;
    uint8_t *const smem = smem_all + grp * Cfg::RING_BYTES;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int wm = wave / 2, wn = wave % 2;
    const int fr = lane & 31, fh = lane >> 5;

    const int tiles_m = (p.M + TILE - 1) / TILE, tiles_n = (p.N + TILE - 1) / TILE;
    const int total_tiles = tiles_m * tiles_n;
    const uint32_t row_bytes = (uint32_t)p.K * 2;
    const int kt_count = (int)(row_bytes / (RB * Cfg::GROUPS));
    const int k_first = grp * kt_count * RB;
    const int my_tiles = (total_tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int steps = my_tiles * kt_count;

    uint32_t goff[LPW];
    const int c_row = lane / CH, c_slot = lane % CH;
    auto set_tile = [&](int tile) {
        int tm, tn;
        tile_coords(tile, tiles_m, tiles_n, TILE_GROUP, tm, tn);
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            const int row = (wave * LPW + q) * Cfg::ROWS_PER_COPY + c_row;
            const int chunk = c_slot ^ swz<CH>(row & 15);
            int g;
            if (row < TILE) {
                g = tm * TILE + row;
                g = g < p.M ? g : p.M - 1;
            } else {
                g = tn * TILE + (row - TILE);
                g = g < p.N ? g : p.N - 1;
            }
            goff[q] = (uint32_t)g * row_bytes + chunk * 16;
        }
    };
    int lt = blockIdx.x, lk = 0;
    set_tile(lt);
    auto copy_next = [&](int slot) {  // always issues LPW copies (dummy re-fetch past the end)
        const uint32_t dst = lds0 + slot * Cfg::STAGE_BYTES + wave * (LPW * 1024);
        const uint8_t *a_k = p.A + k_first + lk * RB;
        const uint8_t *w_k = p.W + k_first + lk * RB;
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            const bool is_a = (wave * LPW + q) * Cfg::ROWS_PER_COPY < TILE;
            dma_copy16<0>(is_a ? a_k : w_k, goff[q], dst + q * 1024);
        }
        if (++lk == kt_count) {
            lk = 0;
            if (lt + (int)gridDim.x < total_tiles) {
                lt += gridDim.x;
                set_tile(lt);
            }
        }
    };

    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

    const int row_a = wm * 32 + fr, row_w = wn * 32 + w_row_perm(fr);
    const int at_a = row_a * RB, at_w = (TILE + row_w) * RB;
    const int key_a = swz<CH>(row_a & 15), key_w = swz<CH>(row_w & 15);
    v8h frag_w[2], frag_a[2];
    auto read_step = [&](int stage_off, auto ksc, auto bc) {
        constexpr int ks = decltype(ksc)::value, b = decltype(bc)::value;
        const int c = ks * 2 + fh;
        frag_w[b] = *reinterpret_cast<const v8h *>(smem + stage_off + at_w + ((c ^ key_w) * 16));
        frag_a[b] = *reinterpret_cast<const v8h *>(smem + stage_off + at_a + ((c ^ key_a) * 16));
    };
    auto mfma_step = [&](auto bc) {
        constexpr int b = decltype(bc)::value;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(frag_w[b], frag_a[b], acc, 0, 0, 0);
    };

    // epilogue of one tile
    auto epilogue = [&](int tile) {
        int tile_m, tile_n;
        tile_coords(tile, tiles_m, tiles_n, TILE_GROUP, tile_m, tile_n);
        const bool vec_ok = (p.N % 8) == 0;
        static_for<2>([&](auto Gc) {
            constexpr int G = decltype(Gc)::value;
            const int nb = tile_n * TILE + wn * 32 + 16 * G + 8 * fh;
            if (nb >= p.N) return;
            const int nvalid = (p.N - nb) < 8 ? (p.N - nb) : 8;
            float bi[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) bi[e] = (p.bias && e < nvalid) ? p.bias[nb + e] : 0.0f;
            const int m = tile_m * TILE + wm * 32 + fr;
            if (m >= p.M) return;
            const int64_t o = (int64_t)m * p.N + nb;
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = acc[8 * G + e] + bi[e];
            if (p.residual) {
                const uint16_t *r = p.residual + o;
                if (vec_ok) {
                    const uint4 rr = *reinterpret_cast<const uint4 *>(r);
                    const uint32_t rwd[4] = {rr.x, rr.y, rr.z, rr.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        y[2 * e] += half_bits_to_float((uint16_t)(rwd[e] & 0xFFFFu));
                        y[2 * e + 1] += half_bits_to_float((uint16_t)(rwd[e] >> 16));
                    }
                } else {
                    for (int e = 0; e < nvalid; ++e) y[e] += half_bits_to_float(r[e]);
                }
            }
            if (TAIL || p.act == MKQ_ACT_GELU) {
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = TAIL ? gelu_erf_tail(y[e]) : gelu_erf(y[e]);
            }
            if (TAIL || p.out_dtype == MKQ_F32) {
                float *dst = (float *)p.out + o;
                if (vec_ok) {
                    *reinterpret_cast<float4 *>(dst) = make_float4(y[0], y[1], y[2], y[3]);
                    *reinterpret_cast<float4 *>(dst + 4) = make_float4(y[4], y[5], y[6], y[7]);
                } else {
                    for (int e = 0; e < nvalid; ++e) dst[e] = y[e];
                }
            } else {
                uint16_t *dst = (uint16_t *)p.out + o;
                if (vec_ok) {
                    *reinterpret_cast<uint4 *>(dst) = make_uint4(pack2_f16(y[0], y[1]), pack2_f16(y[2], y[3]),
                                                                 pack2_f16(y[4], y[5]), pack2_f16(y[6], y[7]));
                } else {
                    for (int e = 0; e < nvalid; ++e) dst[e] = float_to_half_bits(y[e]);
                }
            }
        });
    };

    // prologue
#pragma unroll
    for (int i = 0; i < S - 1; ++i) copy_next(i);
    wait_vmcnt<(S - 2) * LPW>();
    lds_barrier();
    read_step(0, IntC<0>{}, IntC<0>{});

    int ct = blockIdx.x, ck = 0, buf = 0;
    for (int s = 0; s < steps; ++s) {  // four k steps of 16 values per stage
        const int stage_off = buf * Cfg::STAGE_BYTES;
        const int nbuf = (buf + 1 == S) ? 0 : buf + 1;
        read_step(stage_off, IntC<1>{}, IntC<1>{});
        mfma_step(IntC<0>{});
        read_step(stage_off, IntC<2>{}, IntC<0>{});
        mfma_step(IntC<1>{});
        read_step(stage_off, IntC<3>{}, IntC<1>{});
        mfma_step(IntC<0>{});
        // stage s+1 readable; slot of stage s-1 refilled with stage s+S-1
        wait_vmcnt<(S - 3) * LPW>();
        lds_barrier();
        copy_next(buf == 0 ? S - 1 : buf - 1);
        read_step(nbuf * Cfg::STAGE_BYTES, IntC<0>{}, IntC<0>{});
        mfma_step(IntC<1>{});
        buf = nbuf;
        if (++ck == kt_count) {
            float *const xch = reinterpret_cast<float *>(smem_all + Cfg::GROUPS * Cfg::RING_BYTES) + wave * 1024 + lane * 4;
            if (grp == 1) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(xch + q * 256) =
                        make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
            }
            lds_barrier();
            if (grp == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 t = *reinterpret_cast<const float4 *>(xch + q * 256);
                    acc[4 * q] += t.x; acc[4 * q + 1] += t.y;
                    acc[4 * q + 2] += t.z; acc[4 * q + 3] += t.w;
                }
                epilogue(ct);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
            ck = 0;
            ct += gridDim.x;
        }
    }
    wait_vmcnt<0>();
}

template <bool TAIL>
static int launch_split_f16_as(const GemmI4Params &p, hipStream_t st)
{
    const int64_t tiles = ceil_div(p.M, SplitF16::TILE) * ceil_div(p.N, SplitF16::TILE);
    if (tiles > 0x7FFFFFFF) return MKQ_ERR_UNSUPPORTED;
    static PerDeviceOnce once;
    int64_t resident = 0;
    const int rc = resident_workgroups(once, gemm_f16_kernel<TAIL>, SplitF16::THREADS, SplitF16::LDS_BYTES, 1 << 20, &resident);
    if (rc != MKQ_OK || p.setup_only) return rc;
    const unsigned grid = (unsigned)(tiles < resident ? tiles : resident);
    const GemmF16Params q = {p.A, p.W, p.M, p.N, p.K, p.bias, (const uint16_t *)p.residual, p.act, p.out, p.out_dtype};
    gemm_f16_kernel<TAIL><<<grid, SplitF16::THREADS, SplitF16::LDS_BYTES, st>>>(q);
    return launch_status();
}
static int launch_split_f16(const GemmI4Params &p, hipStream_t st)
{
    return epi_gelu_tail(p.act, p.out_dtype) ? launch_split_f16_as<true>(p, st) : launch_split_f16_as<false>(p, st);
}

// K split between two wave groups applies, and there is at most one 64x64 tile per CU
static bool few_tiles(const GemmI4Params &p)
{
    return ceil_div(p.M, 64) * ceil_div(p.N, 64) <= 256 && (p.K % 128) == 0 && p.K >= 256;
}

// Tile choice, from sweeps over M = 32 .. 16384 at the BERT-base / BERT-large shapes (before: 128x128 tiles, one
// workgroup per CU, from 192 tiles on, and 64x64 below; us, old -> new):
//   4096 tokens, K = 768: N = 2304 31.9 -> 24.3, N = 768 14.3 -> 11.8, N = 3072 with GELU 39.8 -> 31.8;
//   K = 3072, N = 768 33.5 -> 28.8; 2298 tokens 22.0 -> 14.1, 9.4 -> 8.7, 26.8 -> 20.2, 28.8 -> 23.3;
//   16384 tokens, K = 1024, N = 4096 230 -> 153.  Over 1230 shapes (M = 1 .. 16384, 47 pairs of K and N with their
// epilogues) six are slower than before by more than 2 %, by 11 % at most (440 tokens, K = 1280, N = 5120 with GELU 13.7 -> 15.2).
enum { F16_SPLIT = 0, F16_64, F16_128_DEEP, F16_256x128, F16_128, F16_256, F16_128x96_DEEP, F16_256x192, F16_CONFIGS };
static int choose_f16(const GemmI4Params &p)
{
    const int64_t t128 = ceil_div(p.M, 128) * ceil_div(p.N, 128), t64 = ceil_div(p.M, 64) * ceil_div(p.N, 64);
    // at most one 64x64 tile per CU: two wave groups share the k loop (a lone wave per SIMD waits for its own loads)
    if (few_tiles(p)) return F16_SPLIT;
    // More than two 64x64 tiles per CU, but at most one of 128x96, whose deep ring covers the trip to memory: what a launch of this
    // size costs is its fullest CU, and 128x128 tiles leave a quarter of the chip idle where these leave none.  us, before -> here:
    // 4096 tokens, K = 3072, N = 768 26.5 -> 23.3, K = N = 768 with a residual 10.8 -> 9.9; 2560, K = 4096, N = 1024 32.6 -> 28.3;
    // 1024, K = 768, N = 2304 9.7 -> 8.9, N = 3072 with GELU 10.9 -> 10.3.  In a second round it loses (4352, K = 3072, N = 768 26.9 -> 41.1).
    if (f16_128x96(p.M, p.N, p.K, p.act == MKQ_ACT_GELU, p.residual != nullptr)) return F16_128x96_DEEP;
    // up to two 64x64 tiles per CU, three (all that fit) where the epilogue is a large share of the tile: 3072 tokens,
    // K = N = 768 with a residual 12.1 -> 11.3, 681 tokens, K = 768, N = 3072 with GELU 11.7 -> 10.9; without either the
    // 128x128 tiles win from two per CU on (1024 tokens, K = 768, N = 2304 10.5 -> 10.0)
    const bool long_epilogue = (p.residual || p.act == MKQ_ACT_GELU) && p.K <= 768;
    if (t64 <= (long_epilogue ? 768 : 512)) return F16_64;
    // about one 128x128 tile per CU: a deep ring, since nothing else covers the trip to memory
    if (t128 <= 256) return F16_128_DEEP;
    // one 256x128 tile of eight waves per CU in a single round
    if (ceil_div(p.M, 256) * ceil_div(p.N, 128) <= 256) return F16_256x128;
    // Several rounds: the tile whose rounds add up to the least.  256x256, one per CU, has the least traffic per product; two 128x128
    // workgroups per CU overlap one's epilogue with the other's k loop; 256x192, one per CU, is between them and fills rounds that
    // neither does.  A round takes about 18, 11.5 and 15 (and 2 for the first) at K = 768, and in that proportion at other K.  us,
    // without 256x192 -> with: 4096 tokens, K = 768, N = 3072 with GELU 26.0 -> 21.7, N = 2304 20.5 -> 17.8; 8192, N = 3072 46.9 -> 38.9;
    // 12288, K = 3072, N = 768 74.6 -> 54.4; 9216, K = 4096, N = 1024 91.0 -> 66.9; where it is not taken: 5632 tokens, K = 768,
    // N = 2304 24.4 and 31.6, 8192, K = 1024, N = 4096 56.9 and 65.4.
    const auto rounds = [](int64_t tiles, int64_t per_round) { return (double)ceil_div(tiles, per_round); };
    const int64_t t256 = ceil_div(p.M, 256) * ceil_div(p.N, 256);
    const double other = t256 >= 256 ? 18.0 * rounds(t256, 256) : 11.5 * rounds(t128, 512);
    if (15.0 * rounds(ceil_div(p.M, 256) * ceil_div(p.N, 192), 256) + 2.0 < other && f16_256x192_suits(p.N, p.K, p.residual != nullptr)) return F16_256x192;
    return t256 >= 256 ? F16_256 : F16_128;
}

static int run_config(const GemmI4Params &p, int cfg, hipStream_t st)
{
    switch (cfg) {
    case F16_SPLIT: return launch_split_f16(p, st);
    case F16_64: return launch_f16_by_epilogue<GemmI4DmaCfg<64, 64, 2, 2, 128, 3>>(p, st);
    case F16_128_DEEP: return launch_f16_by_epilogue<GemmI4DmaCfg<128, 128, 2, 2, 128, 4>>(p, st);
    case F16_256x128: return launch_f16_by_epilogue<GemmI4DmaCfg<256, 128, 4, 2, 128, 3>>(p, st);
    case F16_128: return launch_f16_by_epilogue<GemmI4DmaCfg<128, 128, 2, 2, 128, 2>>(p, st);
    case F16_128x96_DEEP: return launch_f16_by_epilogue<GemmI4DmaCfg<128, 96, 4, 1, 128, 4>>(p, st);
    case F16_256x192: return launch_f16_by_epilogue<GemmI4DmaCfg<256, 192, 4, 2, 128, 2>>(p, st);
    default: return launch_f16_by_epilogue<GemmI4DmaCfg<256, 256, 2, 4, 128, 2>>(p, st);
    }
}

int run_gemm_f16(const GemmI4Params &p, hipStream_t st) { return run_config(p, choose_f16(p), st); }

// once-per-device setup of every instantiation (nothing is launched)
int setup_gemm_f16()
{
    int rc = MKQ_OK;
    for (int cfg = 0; cfg < F16_CONFIGS; ++cfg)
        for (int e = 0; e < 5 && rc == MKQ_OK; ++e) {
            GemmI4Params p = {};
            p.M = p.N = p.K = 256;
            p.setup_only = true;
            p.out_dtype = e >= 3 ? MKQ_F32 : MKQ_F16;
            p.act = e == 2 || e == 4 ? MKQ_ACT_GELU : MKQ_ACT_NONE;
            if (e == 1) p.residual = &p;
            rc = run_config(p, cfg, nullptr);
        }
    return rc;
}

}  // namespace mkq

using namespace mkq;

extern "C" int mkq_linear_fp16(const void *a, const void *W, const float *bias, int64_t M, int64_t N,
                               int64_t K, void *out, int out_dtype, int act, const void *residual,
                               void *stream)
{
    if (out_dtype != MKQ_F32 && out_dtype != MKQ_F16) return MKQ_ERR_DTYPE;
    if (act != MKQ_ACT_NONE && act != MKQ_ACT_GELU) return MKQ_ERR_DTYPE;
    if (M < 0 || N <= 0 || K <= 0 || (K % 64) != 0) return MKQ_ERR_SHAPE;
    if (M == 0) return MKQ_OK;
    if (!a || !W || !out) return MKQ_ERR_NULL;
    if (!aligned16(a) || !aligned16(W) || !aligned16(out) || (bias && !aligned16(bias)) ||
        (residual && !aligned16(residual)))
        return MKQ_ERR_ALIGN;
    if (M > 0x7FFFFFFF || N > 0x7FFFFFFF || M * K * 2 > 0xFFFFFFFFLL || N * K * 2 > 0xFFFFFFFFLL)
        return MKQ_ERR_UNSUPPORTED;
    GemmI4Params p = {};
    p.A = (const uint8_t *)a; p.W = (const uint8_t *)W;
    p.M = (int)M; p.N = (int)N; p.K = (int)K;
    p.bias = bias; p.residual = residual; p.residual_dtype = MKQ_F16; p.act = act;
    p.out = out; p.out_dtype = out_dtype;
    p.by_rows = tiles_by_rows(p, 16);
    return run_gemm_f16(p, as_stream(stream));
}
