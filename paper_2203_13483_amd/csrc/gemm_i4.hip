// int4 x int4 -> int32 GEMM with fused dequantize / activation / requantize
// epilogue for gfx950 (CDNA4), the hot loop of the W4A4 linear layer.
//
// CDNA4 has no 4-bit integer MFMA, so nibbles are widened to int8 on the way from
// LDS to the matrix core.  The widening costs three VALU ops per eight codes: for
// a 32-bit word w of eight two's-complement nibbles,
//     hi = w & 0xF0F0F0F0          -> four int8 lanes equal to 16 * (odd codes)
//     lo = (w << 4) & 0xF0F0F0F0   -> four int8 lanes equal to 16 * (even codes)
// (the nibble's sign bit lands in bit 7 of its byte).  Both operands carry the
// factor 16, so the int32 accumulator holds exactly 256 * sum(a*w).  |sum| <= 64 K,
// so nothing overflows while 256 * 64 * K < 2^31, i.e. K < 131072.  The lo/hi split
// permutes k inside a word identically for both operands, which a dot product does
// not see.  The factor 256 is removed for free in the epilogue: the accumulator's
// low 8 bits are zero, so it has at most 18 significant bits and converts to
// binary32 exactly; the per-channel scale is pre-multiplied by 2^-8 (exact), and
// fma(256*sum, scale/256, bias) rounds the same real number as fma(sum, scale, bias).
//
// Data flow: packed rows of A [M, K/2] and W [N, K/2] (both K-contiguous) are
// fetched with 128-bit global loads into registers one stage ahead, written to
// LDS tiles of RB bytes per row (XOR-swizzled at 16-byte granularity so that the
// staging writes and the ds_read_b128 fragment reads are bank-conflict free), and
// each lane reads 16 bytes (32 codes) of one row, feeding two MFMA k-steps.
// W is the MFMA "A" operand and the activations the "B" operand; W rows are read
// in a permuted order so that a lane ends up with runs of 8 consecutive output
// channels of one token and stores them with one or two vector stores.
#include "gemm_tile.h"
#include "layer_tail.h"
#include "mkq_tuning.h"
#include "qkv_attention.h"

namespace mkq {

// few-token weight-streaming kernel (gemm_i4_stream.hip)
bool gemm_i4_stream_ok(const GemmI4Params &p);
int run_gemm_i4_stream(const GemmI4Params &p, const SplitKScratch *scr, int forced_ks, hipStream_t st);
int setup_gemm_i4_stream(const GemmI4Params &p, hipStream_t st);
int run_gemm_i4_wstream(const GemmI4Params &p, const SplitKScratch *scr, int forced_ks, int variant, hipStream_t st);
// quantizer and GEMM of a few tokens in one launch (gemm_small.hip)
bool small_quantizing_ok(const GemmI4Params &p, const void *a, int elem_bytes);
int run_gemm_i4_small(const GemmI4Params &p, const void *a, int a_dtype, hipStream_t st);
// tile kernels with 128-byte stage rows (gemm_lines.hip)
int run_gemm_i4_lines(const GemmI4Params &p, int epi, int cfg, hipStream_t st);
int run_gemm_i8_lines(const GemmI4Params &p, int epi, int cfg, hipStream_t st);
// few tokens and small linears (gemm_few.hip)
int run_gemm_few(const GemmI4Params &p, int bits, FewTile t, hipStream_t st);
int setup_gemm_few();
int gemm_i4_stream_slices(const GemmI4Params &p, const SplitKScratch *scr, int forced_ks);

template <class Cfg, bool FULL_STAGES, class Epi>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_i4_kernel(const GemmI4Params p)
{
    constexpr int BM = Cfg::BM, BN = Cfg::BN, RB = Cfg::RB, CH = Cfg::CH;
    constexpr int TM = Cfg::TM, TN = Cfg::TN, ROUNDS = Cfg::ROUNDS;
    constexpr int THREADS = Cfg::THREADS;

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
    const int fr = lane & 31;  // row inside a 32-row fragment
    const int fh = lane >> 5;  // which 16-byte half of a 32-byte k slice

    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    const int total_tiles = tiles_m * tiles_n;
    const int row_bytes = p.K / 2;
    const int kt_count = (row_bytes + RB - 1) / RB;

    // The workgroup is persistent: it owns tiles blockIdx.x, blockIdx.x + gridDim.x, ...
    // and runs ONE software pipeline over all their k stages, so the loads of a tile's
    // first stages are already in flight while the previous tile's epilogue runs.
    const int my_tiles = (total_tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int steps = my_tiles * kt_count;

    // --- staging: which 16-byte chunks this thread copies each stage -------------
    uint4 ra[Cfg::A_PER_T], rw[Cfg::W_PER_T];
    uint32_t ga[Cfg::A_PER_T], gw[Cfg::W_PER_T];  // byte offsets of the chunks at k = 0
    int sa[Cfg::A_PER_T], sw[Cfg::W_PER_T];
    const int my_c = (tid % CH) * 16;  // byte offset of this thread's chunk inside a stage row
#pragma unroll
    for (int i = 0; i < Cfg::A_PER_T; ++i) {
        const int idx = tid + i * THREADS;
        const int row = idx / CH, c = idx % CH;
        sa[i] = row * RB + ((c ^ swz<CH>(row & 15)) * 16);
    }
#pragma unroll
    for (int i = 0; i < Cfg::W_PER_T; ++i) {
        const int idx = tid + i * THREADS;
        const int row = idx / CH, c = idx % CH;
        sw[i] = BM * RB + row * RB + ((c ^ swz<CH>(row & 15)) * 16);
    }
    auto set_tile = [&](int tile) {
        int tm, tn;
        tile_coords(tile, tiles_m, tiles_n, TILE_GROUP, tm, tn);
#pragma unroll
        for (int i = 0; i < Cfg::A_PER_T; ++i) {
            const int idx = tid + i * THREADS;
            int gm = tm * BM + idx / CH;
            gm = gm < p.M ? gm : p.M - 1;  // rows past the edge re-read the last row; never stored
            ga[i] = (uint32_t)gm * (uint32_t)row_bytes + my_c;
        }
#pragma unroll
        for (int i = 0; i < Cfg::W_PER_T; ++i) {
            const int idx = tid + i * THREADS;
            int gn = tn * BN + idx / CH;
            gn = gn < p.N ? gn : p.N - 1;
            gw[i] = (uint32_t)gn * (uint32_t)row_bytes + my_c;
        }
    };

    int lt = blockIdx.x, lk = 0;  // load cursor: tile and k stage of the next stage to fetch
    set_tile(lt);
    auto load_next = [&]() {
        const int kb = lk * RB;
        const bool in = FULL_STAGES || (kb + my_c < row_bytes);
#pragma unroll
        for (int i = 0; i < Cfg::A_PER_T; ++i)
            ra[i] = in ? *reinterpret_cast<const uint4 *>(p.A + ga[i] + kb) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < Cfg::W_PER_T; ++i)
            rw[i] = in ? *reinterpret_cast<const uint4 *>(p.W + gw[i] + kb) : make_uint4(0, 0, 0, 0);
        if (++lk == kt_count) {
            lk = 0;
            lt += gridDim.x;
            if (lt < total_tiles) set_tile(lt);
        }
    };
    auto store_stage = [&](int buf) {
        uint8_t *base = smem + buf * Cfg::STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < Cfg::A_PER_T; ++i) *reinterpret_cast<uint4 *>(base + sa[i]) = ra[i];
#pragma unroll
        for (int i = 0; i < Cfg::W_PER_T; ++i) *reinterpret_cast<uint4 *>(base + sw[i]) = rw[i];
    };

    v16i acc[TM][TN];
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][t][v] = 0;

    // fragment read offsets (bytes inside a stage) and the lane's swizzle keys
    int offA[TM], offW[TN], keyA[TM], keyW[TN];
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int row = wm * Cfg::WTM + j * 32 + fr;
        offA[j] = row * RB;
        keyA[j] = swz<CH>(row & 15);
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int row = wn * Cfg::WTN + t * 32 + w_row_perm(fr);
        offW[t] = BM * RB + row * RB;
        keyW[t] = swz<CH>(row & 15);
    }

    auto compute_round = [&](const uint8_t *base, int r) {
        const int c = r * 2 + fh;
        uint4 fw[TN], fa[TM];
#pragma unroll
        for (int t = 0; t < TN; ++t)
            fw[t] = *reinterpret_cast<const uint4 *>(base + offW[t] + ((c ^ keyW[t]) * 16));
#pragma unroll
        for (int j = 0; j < TM; ++j)
            fa[j] = *reinterpret_cast<const uint4 *>(base + offA[j] + ((c ^ keyA[j]) * 16));
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            v4i wv[TN], av[TM];
#pragma unroll
            for (int t = 0; t < TN; ++t) wv[t] = ks ? widen(fw[t].z, fw[t].w) : widen(fw[t].x, fw[t].y);
#pragma unroll
            for (int j = 0; j < TM; ++j) av[j] = ks ? widen(fa[j].z, fa[j].w) : widen(fa[j].x, fa[j].y);
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[j][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wv[t], av[j], acc[j][t], 0, 0, 0);
        }
    };

    auto epilogue = [&](int tile) {
        int tile_m, tile_n;
        tile_coords(tile, tiles_m, tiles_n, TILE_GROUP, tile_m, tile_n);
        gemm_i4_epilogue<Cfg, Epi>(p, acc, tile_m * BM, tile_n * BN, wm, wn, fr, fh);
    };  // epilogue

    // --- main loop: LDS double buffer, registers hold the stage after next --------
    load_next();
    store_stage(0);
    if (steps > 1) load_next();
    lds_barrier();

    int ct = blockIdx.x, ck = 0;  // compute cursor
    for (int s = 0; s < steps; ++s) {
        const uint8_t *base = smem + (s & 1) * Cfg::STAGE_BYTES;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            compute_round(base, r);
            if (r == ROUNDS / 2 - 1) {
                // the other buffer was last read in the previous step, before its barrier
                if (s + 1 < steps) store_stage((s + 1) & 1);
                if (s + 2 < steps) load_next();
            }
        }
        lds_barrier();
        if (++ck == kt_count) {
            epilogue(ct);
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[j][t][v] = 0;
            ck = 0;
            ct += gridDim.x;
        }
    }
}

template <class Cfg, bool FULL, class Epi>
static int launch_one(const GemmI4Params &p, int64_t tiles, hipStream_t st)
{
    const size_t lds = 2 * (size_t)Cfg::STAGE_BYTES;
    static PerDeviceOnce once;  // per instantiation
    int64_t resident = 0;
    const int rc = resident_workgroups(once, gemm_i4_kernel<Cfg, FULL, Epi>, Cfg::THREADS, lds, 2, &resident);
    if (rc != MKQ_OK || p.setup_only) return rc;
    const unsigned grid = (unsigned)(tiles < resident ? tiles : resident);
    gemm_i4_kernel<Cfg, FULL, Epi><<<grid, Cfg::THREADS, lds, st>>>(p);
    return launch_status();
}

template <class Cfg>
static int launch_gemm_i4(const GemmI4Params &p, hipStream_t st)
{
    const int64_t tiles = ceil_div(p.M, Cfg::BM) * ceil_div(p.N, Cfg::BN);
    if (tiles > 0x7FFFFFFF) return MKQ_ERR_UNSUPPORTED;
    const bool full = ((p.K / 2) % Cfg::RB) == 0;
    if (epi_gelu_tail(p.act, p.out_dtype))
        return full ? launch_one<Cfg, true, EpiGeluTail>(p, tiles, st) : launch_one<Cfg, false, EpiGeluTail>(p, tiles, st);
    return full ? launch_one<Cfg, true, EpiGeneric>(p, tiles, st) : launch_one<Cfg, false, EpiGeneric>(p, tiles, st);
}

template <class Cfg>
static int launch_dma_by_epilogue(const GemmI4Params &p, int epi, hipStream_t st)
{
    switch (epi) {
    case EPI_F16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, false>>(p, st);
    case EPI_BF16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_BF16, false, false>>(p, st);
    case EPI_F32: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F32, false, false>>(p, st);
    case EPI_F16_RES16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, true, false>>(p, st);
    case EPI_I4_GELU: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, true>>(p, st);
    case EPI_I4: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, false>>(p, st);
    default: return launch_gemm_i4_dma_generic<Cfg>(p, st);
    }
}

// Tiles whose k loop is also split across workgroups (p.ks slices, partial sums through the caller's scratch).
template <class Cfg, int KS>
static int launch_xsplit_by_epilogue(const GemmI4Params &p, int epi, hipStream_t st)
{
    switch (epi) {
    case EPI_F16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, false>, 4, KS, true>(p, st);
    case EPI_BF16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_BF16, false, false>, 4, KS, true>(p, st);
    case EPI_F16_RES16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, true, false>, 4, KS, true>(p, st);
    case EPI_I4_GELU: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, true>, 4, KS, true>(p, st);
    default: return launch_gemm_i4_dma_generic<Cfg, 4, KS, true>(p, st);
    }
}

// Tiles with the k loop split between two wave groups of one workgroup.
template <class Cfg, int KS>
static int launch_ksplit_by_epilogue(const GemmI4Params &p, int epi, hipStream_t st)
{
    switch (epi) {
    case EPI_F16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, false>, 4, KS>(p, st);
    case EPI_BF16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_BF16, false, false>, 4, KS>(p, st);
    case EPI_F32: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F32, false, false>, 4, KS>(p, st);
    case EPI_F16_RES16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, true, false>, 4, KS>(p, st);
    case EPI_I4_GELU: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, true>, 4, KS>(p, st);
    case EPI_I4: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I4, false, false>, 4, KS>(p, st);
    default: return launch_gemm_i4_dma_generic<Cfg, 4, KS>(p, st);
    }
}

using DmaBig8 = GemmI4DmaCfg<256, 256, 2, 4, 64, 5>;   // 2 waves per SIMD, 128x64 per wave
using DmaMid = GemmI4DmaCfg<128, 128, 2, 2, 64, 4>;    // 64 KiB LDS: two workgroups per CU
using DmaSmall = GemmI4DmaCfg<64, 64, 2, 2, 64, 8>;

// Tile choice of the kernels with 64-byte stage rows, from sweeps over M = 256 .. 65536 at the BERT-base / BERT-large
// shapes (and 4096^2, 8192^2 weights).  Very large problems: 256x128 tiles, two workgroups per CU (18).  Few tiles: 64x64,
// four per CU (27; the launch is latency-bound, parallelism wins).  In between 128x128 with a three-stage ring,
// three per CU (29), or 128x64, four per CU (28), when 128x128 tiles would leave most of the 768 slots empty and
// the k loop is short.
static int choose_rows64(const GemmI4Params &p)
{
    const int64_t t128 = ceil_div(p.M, 128) * ceil_div(p.N, 128);
    const int64_t t128x64 = ceil_div(p.M, 128) * ceil_div(p.N, 64);
    const int64_t t256x128 = ceil_div(p.M, 256) * ceil_div(p.N, 128);
    const double ops = 2.0 * p.M * p.N * p.K;
    if (t256x128 >= 512 && ops >= 6e10) return 18;
    if (t128x64 <= 256) return 27;
    // GELU (and the code decision behind it) makes the epilogue a large share of a short tile: up to four 64x64
    // workgroups per CU spread it over all SIMDs (FFN-up at M = 1024: 9.2 instead of 10.4 us)
    if (p.act == MKQ_ACT_GELU && p.K < 2048 && ceil_div(p.M, 64) * ceil_div(p.N, 64) <= 1024) return 27;
    if (t128 >= 400 || p.K >= 2048) {
        // at most one 128x128 workgroup per CU and a long k loop: two wave groups share the tile's K; 6-14 % at
        // N = 768 / 1024, K = 3072 ... 8192, M = 2560 ... 5120
        if (t128 <= 256 && p.K >= 2048 && (p.K % 256) == 0) return 35;
        return 29;
    }
    return 28;
}

// Tile choice: where whole 256-code stages fit K, the kernels with 128-byte stage rows (43 .. 49 and 51, gemm_lines.hip) in the
// ranges where they are the faster ones.  From sweeps of every configuration at 1600 calls (K = 256 .. 8192, N = 40 ..
// 30522, M = 65 .. 65536; binary16, binary32, GELU, code and residual epilogues; M dense enough to meet full and ragged
// rounds of tiles).  (us, 64-byte -> 128-byte rows)  Of the calls with up to 256 tiles of 64x64 most are few_tile's: what comes here
// has K = 128 or 256, or K from 2048 on and pieces that eight waves do not share evenly.
static int choose_tiles(const GemmI4Params &p)
{
    const int rows64 = choose_rows64(p);
    if ((p.K % 256) != 0) return rows64;
    const int64_t t64 = ceil_div(p.M, 64) * ceil_div(p.N, 64), t128 = ceil_div(p.M, 128) * ceil_div(p.N, 128);
    const int64_t t256x128 = ceil_div(p.M, 256) * ceil_div(p.N, 128), t256 = ceil_div(p.M, 256) * ceil_div(p.N, 256);
    const bool gelu = p.act == MKQ_ACT_GELU, res = p.residual != nullptr, f32 = p.out_dtype == MKQ_F32;
    const bool codes = p.out_dtype == MKQ_I4;
    const bool split = (p.K % 512) == 0;  // two wave groups with whole stages each
    // The large tiles only where their epilogue has a compile-time instantiation and writes whole lines: their waves own 64
    // channels, and 16-bit rows of other lengths than a multiple of 64 start inside a line (M = 4096, K = 768, N = 2008
    // 11.2 -> 12.3, N = 2306 at M = 2048 24.5 -> 27.8; with N = 2304 12.4 -> 12.3)
    const bool fixed = classify_epilogue(p) != EPI_GENERIC && ((p.N % 64) == 0 || codes || res);
    if (rows64 == 18) {
        // 45, one 256x256 tile per CU and round: for code outputs (M = 8192, K = 1024, N = 4096 with GELU 52.2 -> 49.6) or a
        // long k loop (K = N = 4096 104.2 -> 99.5; K = 4096, N = 1024, M = 16384, a single round, 53.4 -> 49.5); at K <= 1024 a
        // plain epilogue, which nothing covers, eats the gain (f16, M = 12288 50.6 -> 52.0) until nine rounds (M = 65536 251
        // -> 247).  A last round that is less than five eighths full takes as long as a full one, where 18 fills it with one
        // workgroup per CU (M = 10240 with GELU 63.7 -> 68.6); residuals at short k and binary32 outputs lose everywhere
        // (M = 12288 65.7 -> 72.6).
        const int64_t last = t256 % 256;
        const bool many = t256 >= 9 * 256, full = many || last == 0 || last >= 160;
        return full && fixed && !f32 && (codes || p.K >= 2048 || (many && !res)) ? 45 : 18;
    }
    if (t64 <= 512 && ceil_div(p.M, 128) * ceil_div(p.N, 64) <= 256 && p.K >= 1024) {
        // few tiles and a long k loop, shared by the wave groups of a workgroup (a lone wave per SIMD is bound by its own
        // instruction stream): 47, 64x64: K = 2560, N = 1024, M = 963 8.7 -> 8.0; 48, 128x64: M = 2298, K = 3072, N = 768 12.5 -> 10.7
        if (split) return t64 <= 256 ? 47 : p.K >= 1536 ? 48 : 43;
        // an odd number of 256-code stages: a long loop can be shared in 64-byte rows
        return p.K >= 2048 ? rows64 : 43;
    }
    // 43, 64x64, up to three per CU: M = 4096, K = N = 768 with a residual 8.7 -> 8.1; M = 1024, N = 3072 with GELU 9.2 -> 8.6
    if (t64 <= 768 && (p.K < 1536 || (p.K < 2048 && (gelu || !split)))) return 43;
    // about one 128x128 tile per CU: 49, on eight waves (M = 1280, K = 768, N = 3072 with GELU 10.7 -> 9.6; M = 4096,
    // K = N = 1024 10.0 -> 9.5, where 43 with four 64x64 tiles per CU takes 10.5), or 46, two wave groups share the k loop
    // (M = 3072, K = 3072, N = 768 15.6 -> 14.4)
    if (t128 <= 256) {
        if (f32 && p.K < 1536) return rows64;  // (M = 1280, K = 768, N = 3072 10.2 -> 10.7)
        // 51, 128x96 with two wave groups, where one per CU holds all and CUs are left: three quarters of the work on the fullest CU
        // (K = 3072, N = 768, M = 3072 14.0 -> 13.1; K = 4096, N = 1024, M = 2560 16.9 -> 15.8; layers of 24 x 128 tokens 72.2 -> 70.2,
        // of 16 x 200 79.2 -> 77.9; with all 256 taken, 32 x 128, 78.6 -> 79.1)
        if (p.K >= (gelu ? 2048 : 1536)) return !split ? rows64 : fixed && ceil_div(p.M, 128) * ceil_div(p.N, 96) < 256 ? 51 : 46;
        return fixed ? 49 : rows64;
    }
    if (!fixed) return rows64;
    // one and a half rounds of 43 still beat two of anything larger where the epilogue is long (M = 1536, K = 768, N = 3072 with
    // GELU 13.0 -> 11.3; M = 6144, K = N = 768 with a residual 11.0 -> 10.2)
    if (t64 <= 1536 && ((gelu && p.K < 2048) || (res && p.K <= 1024 && t64 > 1024))) return 43;
    // 44, a single round of 256x128 tiles (M = 2298, K = 768, N = 2304 10.3 -> 9.5; M = 8192, K = 4096, N = 1024 37.3 -> 34.7);
    // in a second round nothing covers the first one's epilogue (M = 4096, K = 1024, N = 3072 15.4 -> 18.3)
    if (t256x128 <= (res && p.K <= 1024 ? 192 : 256) && t64 > 1024 && p.K >= (gelu ? 768 : 512) && !f32) return 44;
    return rows64;
}

// K split across workgroups of a tile kernel with BM x BN tiles and `groups` wave groups per workgroup: fills
// q.ks and the scratch pointers.  forced_ks: 0 = the largest power of two that keeps at least four 64-byte
// stages per wave group and pair, at most two (tile, slice) pairs per compute unit and partial sums that fit the scratch area.  Returns false when the
// split does not apply (no scratch, K does not divide, the partial sums or the tile count exceed the scratch).
static bool xsplit_plan(GemmI4Params &q, const SplitKScratch *scr, int BM, int BN, int groups, int forced_ks)
{
    if (!scr) return false;
    const int64_t tiles = ceil_div(q.M, BM) * ceil_div(q.N, BN);
    const int stages = q.K / 128 / groups;
    if ((q.K % (128 * groups)) != 0 || tiles > SPLITK_MAX_TILES) return false;
    int cus = 256;
    device_cus(&cus);
    int ks = forced_ks;
    if (ks <= 0) {
        ks = 1;
        while (ks < 32 && (stages % (2 * ks)) == 0 && stages / (2 * ks) >= 4 && tiles * 2 * ks <= 2 * cus &&
               (size_t)tiles * 2 * ks * BM * BN * sizeof(int32_t) <= scr->partial_bytes)
            ks *= 2;
    }
    if (ks < 1 || (stages % ks) != 0 || stages / ks < 2) return false;
    if ((size_t)tiles * ks * BM * BN * sizeof(int32_t) > scr->partial_bytes) return false;
    q.ks = ks;
    q.sk_counters = scr->counters;
    q.sk_partials = scr->partials;
    return true;
}

// forced_cfg: -1 = the library's own choice, otherwise one configuration by number (tuning interface);
// scr: scratch of a K split across workgroups, or null; forced_ks: 0 = automatic.
int run_gemm_i4(const GemmI4Params &p, hipStream_t st, int forced_cfg, const SplitKScratch *scr, int forced_ks)
{
    int cfg = forced_cfg;
    const bool dma_ok = (p.K % 128) == 0;  // whole 64-byte stages
    const int epi = classify_epilogue(p);
    if (cfg == 50) return gemm_i4_stream_ok(p) ? run_gemm_i4_stream(p, scr, forced_ks, st) : MKQ_ERR_UNSUPPORTED;
    if (cfg == 30) return (p.M <= 128 && (p.K % 256) == 0) ? run_gemm_few(p, 4, few_tile_or_largest(p.M, p.N, p.K / 2, 4), st) : MKQ_ERR_UNSUPPORTED;
    // 65 .. 128 tokens against a large weight matrix take the ring kernel with its shared activation stages (60 instead of 88 us at
    // K = N = 16384 with operands through registers)
    if (cfg < 0 && p.M > 64 && gemm_i4_stream_ok(p) && (int64_t)p.N * p.K >= ((int64_t)1 << 27))
        return run_gemm_i4_stream(p, scr, forced_ks, st);
    if (cfg < 0) {
        const FewTile few = few_choice(p.M, p.N, p.K / 2, 4);
        if (few != FEW_NONE) return run_gemm_few(p, 4, few, st);
    }
    if (cfg < 0) {
        if (!dma_ok) {
            cfg = 3;
        } else {
            cfg = choose_tiles(p);
        }
    }
    if (cfg >= 10 && !dma_ok) return MKQ_ERR_UNSUPPORTED;
    // few 64x64 tiles (at most two workgroups per CU) and a k loop long enough to halve, in 64-byte rows (an odd
    // number of 256-code stages): two wave groups per workgroup, with the deeper ring for a weight matrix of 4 MiB and more,
    // which comes from memory rather than from the caches on most calls
    if (forced_cfg < 0 && cfg == 27 && (p.K % 256) == 0 && p.K >= 2048) {
        const int64_t t64 = ceil_div(p.M, 64) * ceil_div(p.N, 64);
        if (t64 <= 512) cfg = t64 <= 256 && (int64_t)p.N * p.K >= ((int64_t)8 << 20) ? 31 : 33;
    }
    if ((cfg == 31 || cfg == 33 || cfg == 35) && (p.K % 256) != 0) return MKQ_ERR_UNSUPPORTED;
    if (cfg >= 60 && cfg <= 62) {  // tile kernels with the k loop also split across workgroups
        GemmI4Params q = p;
        if (cfg == 60) {
            if (!xsplit_plan(q, scr, 128, 128, 1, forced_ks)) return MKQ_ERR_UNSUPPORTED;
            return launch_xsplit_by_epilogue<GemmI4DmaCfg<128, 128, 2, 2, 64, 3>, 1>(q, epi, st);
        }
        if (cfg == 61) {
            if (!xsplit_plan(q, scr, 64, 64, 2, forced_ks)) return MKQ_ERR_UNSUPPORTED;
            return launch_xsplit_by_epilogue<GemmI4DmaCfg<64, 64, 2, 2, 64, 4>, 2>(q, epi, st);
        }
        if (!xsplit_plan(q, scr, 128, 64, 1, forced_ks)) return MKQ_ERR_UNSUPPORTED;
        return launch_xsplit_by_epilogue<GemmI4DmaCfg<128, 64, 2, 2, 64, 3>, 1>(q, epi, st);
    }
    if ((cfg >= 43 && cfg <= 49) || cfg == 51) return run_gemm_i4_lines(p, epi, cfg, st);
    switch (cfg) {
    case 2: return launch_gemm_i4<GemmI4Cfg<128, 128, 2, 2, 64>>(p, st);
    case 3: return launch_gemm_i4<GemmI4Cfg<64, 64, 2, 2, 64>>(p, st);
    case 11: return launch_dma_by_epilogue<DmaBig8>(p, epi, st);
    case 12: return launch_dma_by_epilogue<DmaMid>(p, epi, st);
    case 14: return launch_dma_by_epilogue<DmaSmall>(p, epi, st);
    case 18: return launch_dma_by_epilogue<GemmI4DmaCfg<256, 128, 2, 2, 64, 3>>(p, epi, st);
    case 19: return launch_dma_by_epilogue<GemmI4DmaCfg<128, 256, 2, 2, 64, 3>>(p, epi, st);
    case 20: return launch_dma_by_epilogue<GemmI4DmaCfg<256, 128, 2, 2, 32, 6>>(p, epi, st);
    case 27: return launch_dma_by_epilogue<GemmI4DmaCfg<64, 64, 2, 2, 64, 4>>(p, epi, st);
    case 28: return launch_dma_by_epilogue<GemmI4DmaCfg<128, 64, 2, 2, 64, 3>>(p, epi, st);
    case 29: return launch_dma_by_epilogue<GemmI4DmaCfg<128, 128, 2, 2, 64, 3>>(p, epi, st);
    case 31: return launch_ksplit_by_epilogue<GemmI4DmaCfg<64, 64, 2, 2, 64, 4>, 2>(p, epi, st);
    case 33: return launch_ksplit_by_epilogue<GemmI4DmaCfg<64, 64, 2, 2, 64, 3>, 2>(p, epi, st);
    case 35: return launch_ksplit_by_epilogue<GemmI4DmaCfg<128, 128, 2, 2, 64, 3>, 2>(p, epi, st);
    default: return MKQ_ERR_UNSUPPORTED;
    }
}

// 8-bit operands (W8A8 comparison path): [M, K] and [N, K] int8 codes, K a multiple of 64.
template <class Cfg>
static int launch_i8_by_epilogue(const GemmI4Params &p, int epi, hipStream_t st)
{
    switch (epi) {
    case EPI_F16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, false, false>, 8>(p, st);
    case EPI_BF16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_BF16, false, false>, 8>(p, st);
    case EPI_F32: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F32, false, false>, 8>(p, st);
    case EPI_F16_RES16: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_F16, true, false>, 8>(p, st);
    case EPI_I8_GELU: return launch_gemm_i4_dma<Cfg, EpiFixed<MKQ_I8, false, true>, 8>(p, st);
    default: return launch_gemm_i4_dma_generic<Cfg, 8>(p, st);
    }
}

// Tile choice of the 8-bit linear, from sweeps of every configuration at 2200 calls (as for 4 bits, with the general epilogue's
// forms; M to 65536; us, best 64-byte-row choice -> here):
//   47, 64x64, its long k loop shared by two wave groups: M = 440, K = 3072, N = 768 12.1 -> 8.4
//   43, 64x64, up to three per CU (M = 4096, K = 3072, N = 768 25.1 -> 20.3), and where the epilogue is long up to six (GELU,
//       M = 1280, K = 1024, N = 4096 17.1 -> 13.9) or four (residual, short k: M = 5120, K = N = 768 10.7 -> 9.3)
//   46, 128x128, two per CU: M = 1691, K = 768, N = 2304 8.3 -> 7.9; M = 2048, K = N = 2048 20.9 -> 13.0; M = 4096, K = 1024,
//       N = 3072 19.0 -> 18.5
//   44, a single round of 256x128: M = 2298, K = 768, N = 2304 13.7 -> 9.3; not for a residual at short k (its rows come late)
//       nor for binary32 until K = 1536 (M = 2560, K = 768, N = 3072 46 16.7, 44 19.6; M = 6144, K = 3072, N = 768 25.6, 23.5);
//       and very large problems, GELU and binary32 apart (K = N = 1536, M = 16384 50.4 -> 41.0; K = 1024, N = 4096, M = 32768
//       174 -> 161)
//   51, 128x96, a ring of four stages, one per CU and only one round, for a long k loop (K = 3072, N = 768, M = 4096 17.5 -> 15.2,
//       K = 4096, N = 1024, M = 2560 20.2 -> 17.8; at K = 768 43 is as fast, with GELU faster)
//   52, a single round of 256x192 where 128x128 tiles come in two of two per CU: GELU (K = 768, N = 3072, M = 4096 20.0 -> 17.5, K = 1024,
//       N = 4096, M = 2560 20.7 -> 18.7), residuals (K = N = 768, M = 12288 16.9 -> 15.5) and long k loops (K = 3072, N = 768, M = 12288
//       39.7 -> 32.7); plain outputs at short k between -4 and 8 %, and not taken
//   29, 64-byte rows, three per CU, where 46 would need a second, nearly empty round (M = 12288, K = N = 768 18.9 instead of
//       21.1), at short k (M = 12288, K = 256, N = 768 10.5 instead of 11.8) and for GELU over several rounds
static int choose_tiles_i8(const GemmI4Params &p)
{
    if ((p.K % 128) != 0) return choose_rows64(p);
    const int64_t t64 = ceil_div(p.M, 64) * ceil_div(p.N, 64), t128 = ceil_div(p.M, 128) * ceil_div(p.N, 128);
    const int64_t t256x128 = ceil_div(p.M, 256) * ceil_div(p.N, 128);
    const bool gelu = p.act == MKQ_ACT_GELU, res = p.residual != nullptr, f32 = p.out_dtype == MKQ_F32, whole = (p.N % 8) == 0;
    if (!gelu && t256x128 >= 512 && 2.0 * p.M * p.N * p.K >= 6e10) return whole && !f32 ? 44 : 18;
    if (t64 <= 256 && (p.K % 256) == 0 && p.K >= 2048) return 47;
    const bool fixed = classify_epilogue(p) != EPI_GENERIC && !f32;
    if (fixed && i8_128x96(p.M, p.N, p.K, gelu)) return 51;
    if (fixed && i8_256x192(p.M, p.N, p.K, gelu, res)) return 52;
    const bool general = p.K < 2048 && classify_epilogue(p) == EPI_GENERIC;
    if (t64 <= 768 || (gelu && p.K < 1536 && t64 <= (general && p.K < 768 ? 1024 : 1536)) ||
        (res && !f32 && p.K <= 1024 && t64 <= 1024))
        return 43;
    // The general epilogue, eight values of one token per lane: ragged rows and 32-bit values are stored piece by piece, and
    // the large tiles cover that badly (M = 1691, K = 768, N = 2306 21.1 -> 25.9); otherwise as below, 43 to a
    // larger count (codes, K = 768, N = 2304, M = 2048 28 12.8, 43 11.9) and 29 for GELU (M = 16384, N = 3072 18 108, 29 84)
    if (general) {
        if (!whole || f32) return choose_rows64(p);
        if (p.K >= 768 && t64 <= 1536) return 43;
        if (t256x128 <= 256) return t128 > 400 ? 44 : choose_rows64(p);
        return gelu ? 29 : choose_rows64(p);
    }
    if (t128 <= 256) return 46;
    if (t256x128 <= 256 && (!f32 || p.K >= 1536) && (!res || p.K >= 2048)) return 44;
    return t128 > 512 && (t128 <= 640 || p.K < 768 || (gelu && p.K < 1536)) ? 29 : 46;
}

int run_gemm_i8(const GemmI4Params &p, hipStream_t st, int forced_cfg = -1)
{
    if ((p.K % 64) != 0) return MKQ_ERR_UNSUPPORTED;
    if (forced_cfg == 30) return (p.M <= 64 && (p.K % 128) == 0) ? run_gemm_few(p, 8, few_tile_or_largest(p.M, p.N, p.K, 8), st) : MKQ_ERR_UNSUPPORTED;
    if (forced_cfg < 0) {
        const FewTile few = few_choice(p.M, p.N, p.K, 8);
        if (few != FEW_NONE) return run_gemm_few(p, 8, few, st);
    }
    int epi = classify_epilogue(p);
    if (epi == EPI_I4 || epi == EPI_I4_GELU) epi = EPI_GENERIC;
    const int cfg = forced_cfg >= 0 ? forced_cfg : choose_tiles_i8(p);
    if ((cfg >= 43 && cfg <= 47) || cfg == 51 || cfg == 52) return run_gemm_i8_lines(p, epi, cfg, st);
    switch (cfg) {
    case 18: return launch_i8_by_epilogue<GemmI4DmaCfg<256, 128, 2, 2, 64, 3>>(p, epi, st);
    case 29: return launch_i8_by_epilogue<GemmI4DmaCfg<128, 128, 2, 2, 64, 3>>(p, epi, st);
    case 28: return launch_i8_by_epilogue<GemmI4DmaCfg<128, 64, 2, 2, 64, 3>>(p, epi, st);
    default: return launch_i8_by_epilogue<GemmI4DmaCfg<64, 64, 2, 2, 64, 4>>(p, epi, st);
    }
}


// ---------------------------------------------------------------------------------
// Experimental: the same int4 x int4 -> exact integer contraction through the 6-bit float path of the
// matrix core.  Every code in [-8, 8] is an E3M2 value, products and sums of such values are exact in
// binary32 while |sum| < 2^24 (K < 2^18), and v_mfma_scale_f32_32x32x64_f8f6f4 with unit scales returns
// them exactly (checked by brute force in the tests).  Operands are stored as E3M2 codes, 6 bits each, in
// groups of 64 codes = 48 bytes: the 32 codes of half h of a group are one 192-bit MFMA operand of a lane,
// stored at bytes [16h, 16h + 16) and [32 + 8h, 40 + 8h) of the group, so that every lane fetches its
// operand with one aligned 16-byte and one aligned 8-byte LDS read.  No widening, and one MFMA covers 64
// codes of k.
// Tile 256 x 256, eight waves of 128 x 64, ring of 3 stages of 128 codes (96-byte rows = two container
// groups = two MFMA k steps, 48 KiB per stage, 48 wave copies of which every wave issues six); one
// persistent workgroup per CU.  The tile is this large and the stage rows this long because the route is
// bound by the number of 64-byte requests the global->LDS copies make, not by the matrix pipe: a 48-byte
// row segment straddles request boundaries (1.75 requests on average), a 96-byte one takes 1.5.
// (256 x 128 on four waves with a two-stage ring, two workgroups per CU, is the second shape.)
template <int BN_, int WGN_, int S_>
struct E3CfgT {
    static constexpr int BM = 256, BN = BN_, WGM = 2, WGN = WGN_, WAVES = WGM * WGN, THREADS = WAVES * 64;
    static constexpr int WTM = 128, WTN = 64, TM = 4, TN = 2;
    static_assert(BN == WGN * WTN, "waves of 128 x 64");
    // S slots keep S - 1 stages in flight: when a stage's second k step has been fetched by every wave its
    // slot is free for the stage S further on
    static constexpr int ROWB = 96, KSTEPS = 2, S = S_, STAGE_BYTES = (BM + BN) * ROWB, LDS_BYTES = S * STAGE_BYTES;
    static constexpr int CPR = ROWB / 16;                                   // 16-byte chunks per row
    static constexpr int A_COPIES = BM * CPR / 64, COPIES = (BM + BN) * CPR / 64, LPW = COPIES / WAVES;
    static_assert(COPIES % WAVES == 0 && (BM * CPR) % 64 == 0, "copies split evenly, none straddles A / W");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS is 160 KiB per CU");
};

template <class Cfg, class Epi>
__global__ __launch_bounds__(Cfg::THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_e3m2_kernel(const GemmI4Params p)
{
    constexpr int BM = Cfg::BM, BN = Cfg::BN, TM = Cfg::TM, TN = Cfg::TN, S = Cfg::S, ROWB = Cfg::ROWB;
    constexpr int LPW = Cfg::LPW, CPR = Cfg::CPR, WAVES = Cfg::WAVES;
    using Sh = EpiShuffle<Cfg>;
    static_assert(Cfg::WTN == 64 && Sh::NSL == 1, "one channel per lane in the scale copies");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
    const int fr = lane & 31, fh = lane >> 5;
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    const int total_tiles = tiles_m * tiles_n;
    const int row_bytes = p.K / 4 * 3;
    const int kt_count = p.K / 128;

    // The workgroup is persistent: it walks tiles blockIdx.x, blockIdx.x + gridDim.x, ... and its copies
    // run ahead of the arithmetic as one stream of stages across tile boundaries, so the first stages of
    // a tile are fetched while the previous tile is still being multiplied and stored.
    // Copy q of this wave is stage copy c = wave + WAVES * q: chunks 64c .. 64c + 63, chunk g = row g / CPR,
    // slot g % CPR.
    uint32_t goff[LPW];
    auto set_fetch_tile = [&](int t) {
        int tm, tn;
        tile_coords(t, tiles_m, tiles_n, TILE_GROUP, tm, tn);
        // (recomputed from the lane index at every tile change: kept across the k loop, the per-copy rows and
        // chunks would cost more registers than the wave has to spare)
        int l = lane;
        asm volatile("" : "+v"(l));
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            const int g = (wave + WAVES * q) * 64 + l;
            const int row = g / CPR, slot = g - row * CPR;
            // rows 8 .. 15 of every 16 hold their six chunks rotated by one: 16 consecutive rows then spread a
            // 16-byte column over all 64 banks (a row is 24 banks long)
            const int chunk = (slot + CPR - ((row >> 3) & 1)) % CPR;
            int src;
            if (row < BM) {
                src = tm * BM + row;
                src = src < p.M ? src : p.M - 1;  // rows past the edge re-read the last row; never stored
            } else {
                src = tn * BN + (row - BM);
                src = src < p.N ? src : p.N - 1;
            }
            goff[q] = (uint32_t)src * (uint32_t)row_bytes + chunk * 16;
        }
    };
    int ft = blockIdx.x, fk = 0;  // copy cursor: tile and stage; past the last tile it fetches that tile again
    set_fetch_tile(ft);
    auto issue = [&](int slot) {
        const int kb = fk * ROWB;
        const uint32_t dst = lds0 + slot * Cfg::STAGE_BYTES + wave * 1024;
        static_for<LPW>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const bool is_a = (wave + WAVES * q) < Cfg::A_COPIES;  // wave-uniform
            dma_copy16<q * WAVES * 1024>((is_a ? p.A : p.W) + kb, goff[q], dst);
        });
        if (++fk == kt_count) {
            fk = 0;
            if (ft + (int)gridDim.x < total_tiles) {
                ft += gridDim.x;
                set_fetch_tile(ft);
            }
        }
    };
    // s_w and bias of the wave's 64 channels of tile t, copied to the wave's 512 bytes beyond the ring; always
    // SC copies, so the number of copies in flight never depends on the arguments
    constexpr int SC = 2;
    float *const sc_lds = reinterpret_cast<float *>(smem + Cfg::LDS_BYTES + wave * Sh::SCALE_BYTES);
    auto issue_scales = [&](int t) {
        int tm, tn;
        tile_coords(t, tiles_m, tiles_n, TILE_GROUP, tm, tn);
        int n = tn * BN + wn * Cfg::WTN + lane;
        n = n < p.N ? n : p.N - 1;
        const uint32_t dst = lds0 + Cfg::LDS_BYTES + wave * Sh::SCALE_BYTES;
        dma_copy4<0>(reinterpret_cast<const uint8_t *>(p.s_w), (uint32_t)n * 4u, dst);
        dma_copy4<Sh::BIAS_AT * 4>(reinterpret_cast<const uint8_t *>(p.bias ? p.bias : p.s_w), (uint32_t)n * 4u, dst);
    };

    // fragment byte offsets inside a stage.  Logical chunk c of a row sits at chunk (c + rot) % 6, rot = bit 3
    // of the row.  K step r takes 16 bytes of chunk 3r + fh and 8 bytes (half fh) of chunk 3r + 2.
    // The rotation is the same for all row blocks of an operand (blocks are 32 rows apart), so one set of
    // offsets per operand serves every block with a constant added.
    int rdW[3], rdA[3];  // [0]: 16-byte read of k step 0 (k step 1: + 48), [1], [2]: the 8-byte reads
    auto offsets = [&](int row, int (&o)[3]) {
        const int rot = (row >> 3) & 1;
        o[0] = row * ROWB + (fh + rot) * 16;
        o[1] = row * ROWB + (2 + rot) * 16 + 8 * fh;
        o[2] = row * ROWB + (rot ? 0 : 80) + 8 * fh;
    };
    offsets(BM + wn * Cfg::WTN + w_row_perm(fr), rdW);
    offsets(wm * Cfg::WTM + fr, rdA);

    v16f acc[TM][TN];
    v8i fw[2][TN], fa[2][TM];  // fragments of two consecutive k steps
    // fragment of one operand row block: u = 0 .. TN-1: W blocks, TN .. TN+TM-1: A blocks
    auto read_one = [&](int sl, auto rc, auto bc, auto uc) {
        constexpr int r = decltype(rc)::value, b = decltype(bc)::value, u = decltype(uc)::value;
        const uint8_t *st = smem + sl * Cfg::STAGE_BYTES;
        if constexpr (u < TN) {
            const uint4 x = *reinterpret_cast<const uint4 *>(st + rdW[0] + (u * 32 * ROWB + r * 48));
            const uint2 y = *reinterpret_cast<const uint2 *>(st + rdW[1 + r] + u * 32 * ROWB);
            fw[b][u] = v8i{(int)x.x, (int)x.y, (int)x.z, (int)x.w, (int)y.x, (int)y.y, 0, 0};
        } else {
            constexpr int j = u - TN;
            const uint4 x = *reinterpret_cast<const uint4 *>(st + rdA[0] + (j * 32 * ROWB + r * 48));
            const uint2 y = *reinterpret_cast<const uint2 *>(st + rdA[1 + r] + j * 32 * ROWB);
            fa[b][j] = v8i{(int)x.x, (int)x.y, (int)x.z, (int)x.w, (int)y.x, (int)y.y, 0, 0};
        }
    };
    auto mfma_one = [&](auto bc, auto ic) {
        constexpr int b = decltype(bc)::value, i = decltype(ic)::value, j = i / TN, t = i % TN;
        acc[j][t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw[b][t], fa[b][j], acc[j][t], 3, 3, 0, 0x7f7f7f7f,
                                                                    0, 0x7f7f7f7f);
    };

    // Epilogue stores share the in-order vmcnt counter with the copies.  At the S - 2 stage boundaries that
    // follow an epilogue the wanted copies are older than its stores, so the stores may stay outstanding if
    // the wait allows for their exact number (known for interior tiles of the fixed epilogues).
    constexpr int SPU = Epi::generic ? 0 : (Epi::out == MKQ_F32 ? 2 : 1);
    constexpr int EPI_STORES = TN * 2 * TM * SPU;
    constexpr int N0 = (S - 2) * LPW, N1 = N0 + EPI_STORES + SC;
    constexpr bool ASYNC_STORES = !Epi::generic && S >= 3 && N1 <= 63;
    int stores_pending = 0;

    // prologue: S stages and the first tile's scales in flight, stage 0 landed, its first k step in registers
#pragma unroll
    for (int i = 0; i < S; ++i) issue(i);
    issue_scales(blockIdx.x);
    wait_vmcnt<(S - 1) * LPW + SC>();
    lds_barrier();
    static_for<TM + TN>([&](auto uc) { read_one(0, IntC<0>{}, IntC<0>{}, uc); });
    int slot = 0;
    for (int tile = blockIdx.x; tile < total_tiles; tile += gridDim.x) {
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][t][v] = 0.0f;
        for (int s = 0; s < kt_count; ++s) {
            const int nslot = (slot + 1 == S) ? 0 : slot + 1;
            // k step 0 of the stage; one fragment block of its k step 1 is fetched behind each of the first
            // six MFMAs
            static_for<TM * TN>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                mfma_one(IntC<0>{}, ic);
                if constexpr (i < TM + TN) read_one(slot, IntC<1>{}, IntC<1>{}, ic);
                __builtin_amdgcn_sched_barrier(0);
            });
            // two MFMAs of k step 1 keep the matrix pipe busy across the boundary
            mfma_one(IntC<1>{}, IntC<0>{});
            mfma_one(IntC<1>{}, IntC<1>{});
            __builtin_amdgcn_sched_barrier(0);
            // boundary: the next stage has landed (the S - 2 stages after it may still be in flight); past
            // the barrier every wave holds all of this stage in registers, so its slot takes the stage S
            // further on -- except behind a tile's last stage, where the slot first serves the epilogue
            if (ASYNC_STORES && stores_pending > 0) {
                wait_vmcnt<ASYNC_STORES ? N1 : 0>();
                --stores_pending;
            } else {
                wait_vmcnt<N0>();
            }
            lds_barrier();
            if (s + 1 < kt_count) issue(slot);
            __builtin_amdgcn_sched_barrier(0);
            static_for<TM * TN - 2>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                read_one(nslot, IntC<0>{}, IntC<0>{}, ic);
                mfma_one(IntC<1>{}, IntC<i + 2>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            slot = nslot;
        }

        const int done_slot = (slot == 0) ? S - 1 : slot - 1;  // idle: read by every wave, not yet refilled
        int tm, tn;
        tile_coords(tile, tiles_m, tiles_n, TILE_GROUP, tm, tn);
        constexpr bool LINES16 = EpiLines16<Cfg, Epi>::usable;
        if constexpr (LINES16) {
            // the scale copies are older than every stage copy issued during the tile; a one-stage tile
            // issues none
            if (kt_count < 2) wait_vmcnt<0>();
            gemm_epilogue_lines16<Cfg, Epi>(p, acc, tm * BM, tn * BN, wm, wn, lane,
                                            smem + done_slot * Cfg::STAGE_BYTES + wave * 4096, sc_lds);
        } else {
            v16i acci[TM][TN];
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acci[j][t][v] = (int)acc[j][t][v];  // exact: integers below 2^24
            if constexpr (Epi::generic) {
                gemm_i4_epilogue<Cfg, Epi>(p, acci, tm * BM, tn * BN, wm, wn, fr, fh);
            } else {
                if (kt_count < 2) wait_vmcnt<0>();
                gemm_i4_epilogue_rows<Cfg, Epi>(p, acci, tm * BM, tn * BN, wm, wn, lane,
                                                smem + done_slot * Cfg::STAGE_BYTES + wave * 4096, sc_lds);
            }
        }
        const bool interior = (tm + 1) * BM <= p.M && (tn + 1) * BN <= p.N;
        stores_pending = (ASYNC_STORES && interior) ? S - 2 : 0;
        lds_barrier();  // every wave is done with its share of the slot
        issue(done_slot);
        issue_scales(tile + (int)gridDim.x < total_tiles ? tile + (int)gridDim.x : tile);
        // the next stage's first k step is fetched again rather than kept in registers across the epilogue
        static_for<TM + TN>([&](auto uc) { read_one(slot, IntC<0>{}, IntC<0>{}, uc); });
    }
    wait_vmcnt<0>();  // the trailing copies must land before the LDS is released
}

template <class Cfg, class Epi>
static int launch_gemm_e3m2(const GemmI4Params &p, hipStream_t st)
{
    const int64_t tiles = ceil_div(p.M, Cfg::BM) * ceil_div(p.N, Cfg::BN);
    if (tiles > 0x7FFFFFFF) return MKQ_ERR_UNSUPPORTED;
    constexpr int lds = Cfg::LDS_BYTES + EpiShuffle<Cfg>::EXTRA_LDS;
    static_assert(lds <= 160 * 1024, "LDS is 160 KiB per CU");
    static PerDeviceOnce once;  // per instantiation
    int64_t resident = 0;
    const int rc = resident_workgroups(once, gemm_e3m2_kernel<Cfg, Epi>, Cfg::THREADS, lds, (160 * 1024) / lds, &resident);
    if (rc != MKQ_OK || p.setup_only) return rc;
    const unsigned grid = (unsigned)(tiles < resident ? tiles : resident);
    gemm_e3m2_kernel<Cfg, Epi><<<grid, Cfg::THREADS, lds, st>>>(p);
    return launch_status();
}

template <class Cfg>
static int launch_e3m2_by_epilogue(const GemmI4Params &p, hipStream_t st)
{
    switch (classify_epilogue(p)) {
    case EPI_F16: return launch_gemm_e3m2<Cfg, EpiFixed<MKQ_F16, false, false>>(p, st);
    case EPI_BF16: return launch_gemm_e3m2<Cfg, EpiFixed<MKQ_BF16, false, false>>(p, st);
    case EPI_F32: return launch_gemm_e3m2<Cfg, EpiFixed<MKQ_F32, false, false>>(p, st);
    }
    return epi_gelu_tail(p.act, p.out_dtype) ? launch_gemm_e3m2<Cfg, EpiGeluTail>(p, st) : launch_gemm_e3m2<Cfg, EpiGeneric>(p, st);
}

int run_gemm_e3m2(const GemmI4Params &p, hipStream_t st, int forced_cfg)
{
    // 256 x 256 tiles (one 8-wave workgroup per CU) make the fewest global->LDS requests per MFMA; 256 x 128
    // (two 4-wave workgroups per CU) overlap one tile's epilogue with the other's k loop
    if (forced_cfg == 41) return launch_e3m2_by_epilogue<E3CfgT<256, 4, 3>>(p, st);
    if (forced_cfg == 42) return launch_e3m2_by_epilogue<E3CfgT<128, 2, 2>>(p, st);
    // (with a short k loop the large tile wins only when every workgroup walks many tiles: 8 % at
    // M = 65536, N = 4096, K = 1024, sixteen tiles per CU)
    const int64_t t256 = ceil_div(p.M, 256) * ceil_div(p.N, 256);
    if (p.K >= 2048 || t256 >= 2048) return launch_e3m2_by_epilogue<E3CfgT<256, 4, 3>>(p, st);
    return launch_e3m2_by_epilogue<E3CfgT<128, 2, 2>>(p, st);
}

}  // namespace mkq

using namespace mkq;

extern "C" size_t mkq_linear_int4_workspace_bytes(int64_t M, int64_t N, int64_t K, int a_dtype)
{
    (void)N;
    if (a_dtype == MKQ_I4 || M <= 0 || K <= 0) return 0;
    return ((size_t)M * (size_t)(K / 2) + 255) & ~(size_t)255;
}

extern "C" size_t mkq_splitk_scratch_bytes(void) { return SPLITK_STATE_BYTES + MKQ_SPLITK_PARTIAL_BYTES; }

namespace mkq {

__global__ void clear_words_kernel(unsigned *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Splits a scratch area into ticket counters and room for partial sums.
static bool splitk_area(void *scratch, size_t bytes, SplitKScratch *out)
{
    if (!scratch || bytes <= SPLITK_STATE_BYTES + 65536) return false;
    out->counters = reinterpret_cast<unsigned *>(scratch);
    out->partials = reinterpret_cast<int32_t *>(reinterpret_cast<uint8_t *>(scratch) + SPLITK_STATE_BYTES);
    out->partial_bytes = bytes - SPLITK_STATE_BYTES;
    return true;
}

enum { W_CANONICAL = 0, W_STREAM = 1 };  // how the weight argument is laid out

// The linear on validated-or-not arguments; scr = scratch of a K split across workgroups or null.
static int linear_int4_run(const void *a, int a_dtype, float s_x, const uint8_t *Wq, const float *s_w,
                           const float *bias, int64_t M, int64_t N, int64_t K, void *out, int out_dtype,
                           const mkq_epilogue *epi, void *workspace, size_t workspace_bytes, void *stream,
                           const SplitKScratch *scr, int forced_cfg, int forced_ks, int w_layout = W_CANONICAL,
                           bool check_only = false)
{
    const bool stream_layout = w_layout == W_STREAM;
    const bool want_q = epi && epi->q_out;
    const bool want_acc = epi && epi->acc_out;
    if (a_dtype != MKQ_I4 && a_dtype != MKQ_F32 && a_dtype != MKQ_F16) return MKQ_ERR_DTYPE;
    if (out_dtype != MKQ_F32 && out_dtype != MKQ_F16 && out_dtype != MKQ_BF16 && out_dtype != MKQ_I4)
        return MKQ_ERR_DTYPE;
    if (epi) {
        if (epi->act != MKQ_ACT_NONE && epi->act != MKQ_ACT_GELU) return MKQ_ERR_DTYPE;
        if (epi->residual && epi->residual_dtype != MKQ_F32 && epi->residual_dtype != MKQ_F16)
            return MKQ_ERR_DTYPE;
    }
    const bool writes_codes = (out && out_dtype == MKQ_I4) || want_q;
    if (M < 0 || N <= 0 || K <= 0 || (K % 32) != 0) return MKQ_ERR_SHAPE;
    if (writes_codes && (N % 2) != 0) return MKQ_ERR_SHAPE;
    const int64_t q_pitch = epi ? epi->q_pitch : 0;
    if (q_pitch != 0 && (q_pitch < N || (q_pitch % 8) != 0 || q_pitch > 0x7FFFFFFF || (q_pitch != N && (N % 8) != 0)))
        return MKQ_ERR_SHAPE;
    if (!scale_ok(s_x)) return MKQ_ERR_SCALE;
    if (writes_codes && !scale_ok(epi ? epi->s_next : 0.0f)) return MKQ_ERR_SCALE;
    if (M == 0) return MKQ_OK;  // empty batch: pointers may be NULL
    if (!a || !Wq || !s_w) return MKQ_ERR_NULL;
    if (!out && !want_q && !want_acc) return MKQ_ERR_NULL;
    if (!aligned16(a) || !aligned16(Wq) || (out && !aligned16(out)) || !aligned16(s_w) ||
        (bias && !aligned16(bias)))
        return MKQ_ERR_ALIGN;
    if (epi && ((epi->residual && !aligned16(epi->residual)) || (epi->q_out && !aligned16(epi->q_out)) ||
                (epi->acc_out && !aligned16(epi->acc_out))))
        return MKQ_ERR_ALIGN;
    const size_t need = mkq_linear_int4_workspace_bytes(M, N, K, a_dtype);
    if (need && (!workspace || workspace_bytes < need || !aligned16(workspace))) return MKQ_ERR_WORKSPACE;
    // the kernel addresses operand bytes with 32-bit offsets
    if (K >= 131072 || M > 0x7FFFFFFF || N > 0x7FFFFFFF || M * (K / 2) > 0xFFFFFFFFLL ||
        N * (K / 2) > 0xFFFFFFFFLL)
        return MKQ_ERR_UNSUPPORTED;
    if (stream_layout && (M > 128 || (K % 256) != 0)) return MKQ_ERR_UNSUPPORTED;
    if (check_only) return MKQ_OK;

    GemmI4Params p;
    p.A = (a_dtype == MKQ_I4) ? (const uint8_t *)a : (const uint8_t *)workspace;
    p.W = Wq; p.M = (int)M; p.N = (int)N; p.K = (int)K;
    p.s_x = s_x; p.s_w = s_w; p.bias = bias;
    p.residual = epi ? epi->residual : nullptr;
    p.residual_dtype = epi ? epi->residual_dtype : MKQ_F32;
    p.act = epi ? epi->act : MKQ_ACT_NONE;
    p.out = out; p.out_dtype = out ? out_dtype : -1;
    p.s_next = epi ? epi->s_next : 1.0f;
    p.q_out = (epi && !(out && out_dtype == MKQ_I4)) ? epi->q_out : nullptr;
    p.acc_out = epi ? epi->acc_out : nullptr;
    p.q_pitch = (int)q_pitch;
    p.acc_shift = 8;
    p.acc_unit = 0.00390625f;
    p.by_rows = tiles_by_rows(p, 4);
    // a few sentences: quantizer and GEMM in one launch, which leaves the codes in the workspace as the two launches do
    if (a_dtype != MKQ_I4 && !stream_layout && forced_cfg < 0 && small_quantizing_ok(p, a, a_dtype == MKQ_F32 ? 4 : 2))
        return run_gemm_i4_small(p, a, a_dtype, as_stream(stream));
    // the kernel that will run is set up (and a forced configuration that does not apply is refused)
    // before anything is enqueued
    auto run = [&]() {
        return stream_layout ? run_gemm_i4_wstream(p, scr, forced_ks, forced_cfg, as_stream(stream))
                             : run_gemm_i4(p, as_stream(stream), forced_cfg, scr, forced_ks);
    };
    p.setup_only = true;
    int rc = run();
    if (rc != MKQ_OK) return rc;
    p.setup_only = false;
    if (a_dtype != MKQ_I4) {
        rc = mkq_quantize(a, a_dtype, M, K, K, s_x, (uint8_t *)workspace, stream);
        if (rc != MKQ_OK) return rc;
    }
    return run();
}

// scratch area named by the epilogue options, if any
static int epilogue_scratch(const mkq_epilogue *epi, SplitKScratch *scr, bool *have)
{
    *have = false;
    if (epi && epi->splitk_scratch) {
        if (!aligned16(epi->splitk_scratch)) return MKQ_ERR_ALIGN;
        if (epi->splitk_scratch_bytes < mkq_splitk_scratch_bytes()) return MKQ_ERR_WORKSPACE;
        *have = splitk_area(epi->splitk_scratch, epi->splitk_scratch_bytes, scr);
    }
    return MKQ_OK;
}

}  // namespace mkq

namespace mkq {
int setup_gemm_f16();  // gemm_f16.hip
int setup_attention();  // attention.hip
}

// Scratch of the entry point that allocates nothing (mkq_linear_int4_stream_static): ticket counters, then
// room for partial sums.  One copy per GPU, at its own address on each, held until the process ends; zero
// when the code object is loaded, and every call leaves the counters zero again.
static __device__ __align__(256) unsigned char scratch[SPLITK_STATE_BYTES + MKQ_SPLITK_PARTIAL_BYTES];

namespace mkq {
// Device address of `scratch` on the current device.  In host code the array's name is only a handle:
// the address that kernels may use comes from hipGetSymbolAddress, once per device.
static int static_scratch(void **ptr_out)
{
    static std::mutex mu;
    static void *ptr[MAX_DEVICES] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return MKQ_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) return MKQ_ERR_HIP;
        ptr[dev] = q;
    }
    *ptr_out = ptr[dev];
    return MKQ_OK;
}
}  // namespace mkq

extern "C" int mkq_init(void)
{
    GemmI4Params p = {};
    p.M = p.N = 256; p.K = 1024;
    p.setup_only = true;
    int rc = setup_gemm_i4_stream(p, nullptr);
    // (the configurations that split K across workgroups only look at the scratch area's size here)
    const SplitKScratch any_scratch = {reinterpret_cast<unsigned *>(16), reinterpret_cast<int32_t *>(16), (size_t)1 << 40};
    for (int cfg : {2, 3, 11, 12, 14, 18, 19, 20, 27, 28, 29, 31, 33, 35, 43, 44, 45, 46, 47, 48, 49, 51, 60, 61, 62}) {
        // one pass per epilogue class: the parameter block is made to classify as each in turn
        for (int e = 0; e < 8 && rc == MKQ_OK; ++e) {
            GemmI4Params q = p;
            q.out = &q; q.s_next = 1.0f;
            q.out_dtype = e == 0 ? MKQ_F16 : e == 1 ? MKQ_BF16 : e == 2 ? MKQ_F32 : e == 3 ? MKQ_F16 : e == 7 ? MKQ_F32 : MKQ_I4;
            if (e == 3) { q.residual = &q; q.residual_dtype = MKQ_F16; }
            if (e == 4 || e == 7) q.act = MKQ_ACT_GELU;
            if (e == 6) q.acc_out = reinterpret_cast<int32_t *>(&q);
            rc = run_gemm_i4(q, nullptr, cfg, cfg >= 60 ? &any_scratch : nullptr, 0);
            if (cfg < 10 && e == 0) e = 6;  // the register-staged kernel has two epilogues: one for all, and the last
        }
    }
    for (int cfg : {18, 29, 28, 27, 43, 44, 46, 47, 51, 52}) {  // the tile shapes of the 8-bit path
        for (int e = 0; e < 7 && rc == MKQ_OK; ++e) {
            GemmI4Params q = p;
            q.out = &q; q.s_next = 1.0f;
            q.out_dtype = e == 0 ? MKQ_F16 : e == 1 ? MKQ_BF16 : e == 2 ? MKQ_F32 : e == 3 ? MKQ_F16 : e == 4 ? MKQ_I8 : MKQ_F32;
            if (e == 3) { q.residual = &q; q.residual_dtype = MKQ_F16; }
            if (e == 4 || e == 6) q.act = MKQ_ACT_GELU;
            if (e == 5) q.acc_out = reinterpret_cast<int32_t *>(&q);
            rc = run_gemm_i8(q, nullptr, cfg);
        }
    }
    for (int cfg : {41, 42}) {
        for (int e = 0; e < 5 && rc == MKQ_OK; ++e) {
            GemmI4Params q = p;
            q.out = &q;
            q.out_dtype = e == 0 ? MKQ_F16 : e == 1 ? MKQ_BF16 : MKQ_F32;
            if (e == 3) q.acc_out = reinterpret_cast<int32_t *>(&q);
            if (e == 4) q.act = MKQ_ACT_GELU;
            rc = run_gemm_e3m2(q, nullptr, cfg);
        }
    }
    if (rc == MKQ_OK) rc = setup_gemm_few();
    if (rc == MKQ_OK) rc = setup_gemm_f16();
    if (rc == MKQ_OK) rc = setup_attention();
    if (rc == MKQ_OK) rc = setup_qkv_attention();
    if (rc == MKQ_OK) rc = setup_layer_tail();
    void *scratch_ptr = nullptr;
    if (rc == MKQ_OK) rc = static_scratch(&scratch_ptr);
    return rc;
}

extern "C" int mkq_splitk_scratch_init(void *scratch, size_t scratch_bytes, void *stream)
{
    if (!scratch) return MKQ_ERR_NULL;
    if (!aligned16(scratch)) return MKQ_ERR_ALIGN;
    if (scratch_bytes < mkq_splitk_scratch_bytes()) return MKQ_ERR_WORKSPACE;
    clear_words_kernel<<<SPLITK_MAX_TILES / 256, 256, 0, as_stream(stream)>>>((unsigned *)scratch, SPLITK_MAX_TILES);
    return launch_status();
}

extern "C" int mkq_linear_int4(const void *a, int a_dtype, float s_x, const uint8_t *Wq,
                               const float *s_w, const float *bias, int64_t M, int64_t N, int64_t K,
                               void *out, int out_dtype, const mkq_epilogue *epi, void *workspace,
                               size_t workspace_bytes, void *stream)
{
    SplitKScratch scr;
    bool have = false;
    const int rc = epilogue_scratch(epi, &scr, &have);
    if (rc != MKQ_OK) return rc;
    return linear_int4_run(a, a_dtype, s_x, Wq, s_w, bias, M, N, K, out, out_dtype, epi, workspace, workspace_bytes,
                           stream, have ? &scr : nullptr, -1, 0);
}

extern "C" int mkq_linear_int4_stream(const void *a, int a_dtype, float s_x, const uint8_t *Wq_stream,
                                      const float *s_w, const float *bias, int64_t M, int64_t N, int64_t K,
                                      void *out, int out_dtype, const mkq_epilogue *epi, void *workspace,
                                      size_t workspace_bytes, void *stream)
{
    SplitKScratch scr;
    bool have = false;
    const int rc = epilogue_scratch(epi, &scr, &have);
    if (rc != MKQ_OK) return rc;
    return linear_int4_run(a, a_dtype, s_x, Wq_stream, s_w, bias, M, N, K, out, out_dtype, epi, workspace,
                           workspace_bytes, stream, have ? &scr : nullptr, 0, 0, W_STREAM);
}

extern "C" int mkq_linear_int4_stream_static(const uint8_t *a, float s_x, const uint8_t *Wq_stream, const float *s_w,
                                             const float *bias, int64_t M, int64_t N, int64_t K, void *out,
                                             int out_dtype, const mkq_epilogue *epi, void *stream)
{
    // argument errors first, as everywhere; then the limits of the static area; only then the device
    int rc = linear_int4_run(a, MKQ_I4, s_x, Wq_stream, s_w, bias, M, N, K, out, out_dtype, epi, nullptr, 0, stream,
                             nullptr, 0, 0, W_STREAM, true);
    if (rc != MKQ_OK || M == 0) return rc;
    // the K split that mkq_linear_int4_stream would choose with room to spare must fit the static area
    GemmI4Params shape = {};
    shape.M = (int)M; shape.N = (int)N; shape.K = (int)K;
    SplitKScratch unbounded = {reinterpret_cast<unsigned *>(16), reinterpret_cast<int32_t *>(16), (size_t)1 << 60};
    const int tb = M <= 32 ? 1 : (M <= 64 ? 2 : 4);
    const int64_t tiles_n = ceil_div(N, 128);
    if (tiles_n > SPLITK_MAX_TILES) return MKQ_ERR_UNSUPPORTED;
    const int64_t ks = gemm_i4_stream_slices(shape, &unbounded, 0);
    if (ks > 1 && ks * tiles_n * 4 * tb * 4096 > (int64_t)MKQ_SPLITK_PARTIAL_BYTES) return MKQ_ERR_UNSUPPORTED;
    void *area = nullptr;
    rc = static_scratch(&area);
    if (rc != MKQ_OK) return rc;
    SplitKScratch scr;
    if (!splitk_area(area, SPLITK_STATE_BYTES + MKQ_SPLITK_PARTIAL_BYTES, &scr)) return MKQ_ERR_HIP;
    return linear_int4_run(a, MKQ_I4, s_x, Wq_stream, s_w, bias, M, N, K, out, out_dtype, epi, nullptr, 0, stream, &scr,
                           0, 0, W_STREAM);
}

extern "C" int mkq_tuning_linear_int4(const void *a, int a_dtype, float s_x, const uint8_t *Wq, const float *s_w,
                                      const float *bias, int64_t M, int64_t N, int64_t K, void *out, int out_dtype,
                                      const mkq_epilogue *epi, void *workspace, size_t workspace_bytes, void *stream,
                                      int config, int k_slices)
{
    SplitKScratch scr;
    bool have = false;
    const int rc = epilogue_scratch(epi, &scr, &have);
    if (rc != MKQ_OK) return rc;
    return linear_int4_run(a, a_dtype, s_x, Wq, s_w, bias, M, N, K, out, out_dtype, epi, workspace, workspace_bytes,
                           stream, have ? &scr : nullptr, config, k_slices);
}

extern "C" int mkq_tuning_linear_int4_stream(const void *a, int a_dtype, float s_x, const uint8_t *Wq_stream,
                                             const float *s_w, const float *bias, int64_t M, int64_t N, int64_t K,
                                             void *out, int out_dtype, const mkq_epilogue *epi, void *workspace,
                                             size_t workspace_bytes, void *stream, int prefetch_stages, int k_slices)
{
    if (prefetch_stages != 0 && prefetch_stages != 2 && prefetch_stages != 3 && prefetch_stages != 4 &&
        prefetch_stages != 6)
        return MKQ_ERR_UNSUPPORTED;
    SplitKScratch scr;
    bool have = false;
    const int rc = epilogue_scratch(epi, &scr, &have);
    if (rc != MKQ_OK) return rc;
    return linear_int4_run(a, a_dtype, s_x, Wq_stream, s_w, bias, M, N, K, out, out_dtype, epi, workspace,
                           workspace_bytes, stream, have ? &scr : nullptr, prefetch_stages, k_slices, W_STREAM);
}

static int linear_int8_run(const int8_t *a, float s_x, const int8_t *Wq, const float *s_w, const float *bias,
                           int64_t M, int64_t N, int64_t K, void *out, int out_dtype, const mkq_epilogue *epi,
                           void *stream, int forced_cfg)
{
    const bool want_acc = epi && epi->acc_out;
    if (out_dtype == MKQ_I4 || (epi && epi->q_out)) return MKQ_ERR_UNSUPPORTED;
    if (out_dtype != MKQ_F32 && out_dtype != MKQ_F16 && out_dtype != MKQ_BF16 && out_dtype != MKQ_I8)
        return MKQ_ERR_DTYPE;
    if (epi) {
        if (epi->act != MKQ_ACT_NONE && epi->act != MKQ_ACT_GELU) return MKQ_ERR_DTYPE;
        if (epi->residual && epi->residual_dtype != MKQ_F32 && epi->residual_dtype != MKQ_F16)
            return MKQ_ERR_DTYPE;
    }
    if (M < 0 || N <= 0 || K <= 0 || (K % 64) != 0) return MKQ_ERR_SHAPE;
    const int64_t q_pitch = epi ? epi->q_pitch : 0;
    if (q_pitch != 0 && (q_pitch < N || (q_pitch % 8) != 0 || q_pitch > 0x7FFFFFFF || (q_pitch != N && (N % 8) != 0)))
        return MKQ_ERR_SHAPE;
    if (!scale_ok(s_x)) return MKQ_ERR_SCALE;
    if (out && out_dtype == MKQ_I8 && !scale_ok(epi ? epi->s_next : 0.0f)) return MKQ_ERR_SCALE;
    if (M == 0) return MKQ_OK;
    if (!a || !Wq || !s_w) return MKQ_ERR_NULL;
    if (!out && !want_acc) return MKQ_ERR_NULL;
    if (!aligned16(a) || !aligned16(Wq) || (out && !aligned16(out)) || !aligned16(s_w) ||
        (bias && !aligned16(bias)))
        return MKQ_ERR_ALIGN;
    if (epi && ((epi->residual && !aligned16(epi->residual)) || (epi->acc_out && !aligned16(epi->acc_out))))
        return MKQ_ERR_ALIGN;
    // 32-bit byte offsets into the operands
    if (K >= 65536 || M > 0x7FFFFFFF || N > 0x7FFFFFFF || M * K > 0xFFFFFFFFLL || N * K > 0xFFFFFFFFLL)
        return MKQ_ERR_UNSUPPORTED;

    GemmI4Params p;
    p.A = (const uint8_t *)a; p.W = (const uint8_t *)Wq; p.M = (int)M; p.N = (int)N; p.K = (int)K;
    p.s_x = s_x; p.s_w = s_w; p.bias = bias;
    p.residual = epi ? epi->residual : nullptr;
    p.residual_dtype = epi ? epi->residual_dtype : MKQ_F32;
    p.act = epi ? epi->act : MKQ_ACT_NONE;
    p.out = out; p.out_dtype = out ? out_dtype : -1;
    p.s_next = (epi && out_dtype == MKQ_I8) ? epi->s_next : 1.0f;
    p.q_out = nullptr;
    p.acc_out = epi ? epi->acc_out : nullptr;
    p.q_pitch = (int)q_pitch;
    p.acc_shift = 0;   // byte operands enter the MFMA as they are
    p.acc_unit = 1.0f;
    p.by_rows = tiles_by_rows(p, 8);
    return run_gemm_i8(p, as_stream(stream), forced_cfg);
}

extern "C" int mkq_linear_int8(const int8_t *a, float s_x, const int8_t *Wq, const float *s_w,
                               const float *bias, int64_t M, int64_t N, int64_t K, void *out,
                               int out_dtype, const mkq_epilogue *epi, void *stream)
{
    return linear_int8_run(a, s_x, Wq, s_w, bias, M, N, K, out, out_dtype, epi, stream, -1);
}

extern "C" int mkq_tuning_linear_int8(const int8_t *a, float s_x, const int8_t *Wq, const float *s_w,
                                      const float *bias, int64_t M, int64_t N, int64_t K, void *out,
                                      int out_dtype, const mkq_epilogue *epi, void *stream, int config)
{
    if (config != -1 && config != 18 && config != 27 && config != 28 && config != 29 && config != 30 &&
        !(config >= 43 && config <= 47 && config != 45) && config != 51 && config != 52)
        return MKQ_ERR_UNSUPPORTED;
    return linear_int8_run(a, s_x, Wq, s_w, bias, M, N, K, out, out_dtype, epi, stream, config);
}

static int linear_int4_e3m2_run(const uint8_t *a, float s_x, const uint8_t *Wq, const float *s_w,
                                const float *bias, int64_t M, int64_t N, int64_t K, void *out, int out_dtype,
                                const mkq_epilogue *epi, void *stream, int forced_cfg)
{
    const bool want_q = epi && epi->q_out;
    const bool want_acc = epi && epi->acc_out;
    if (out_dtype != MKQ_F32 && out_dtype != MKQ_F16 && out_dtype != MKQ_BF16 && out_dtype != MKQ_I4)
        return MKQ_ERR_DTYPE;
    if (epi) {
        if (epi->act != MKQ_ACT_NONE && epi->act != MKQ_ACT_GELU) return MKQ_ERR_DTYPE;
        if (epi->residual && epi->residual_dtype != MKQ_F32 && epi->residual_dtype != MKQ_F16)
            return MKQ_ERR_DTYPE;
    }
    const bool writes_codes = (out && out_dtype == MKQ_I4) || want_q;
    if (M < 0 || N <= 0 || K <= 0 || (K % 128) != 0) return MKQ_ERR_SHAPE;
    if (writes_codes && (N % 2) != 0) return MKQ_ERR_SHAPE;
    const int64_t q_pitch = epi ? epi->q_pitch : 0;
    if (q_pitch != 0 && (q_pitch < N || (q_pitch % 8) != 0 || q_pitch > 0x7FFFFFFF || (q_pitch != N && (N % 8) != 0)))
        return MKQ_ERR_SHAPE;
    if (!scale_ok(s_x)) return MKQ_ERR_SCALE;
    if (writes_codes && !scale_ok(epi ? epi->s_next : 0.0f)) return MKQ_ERR_SCALE;
    if (M == 0) return MKQ_OK;
    if (!a || !Wq || !s_w) return MKQ_ERR_NULL;
    if (!out && !want_q && !want_acc) return MKQ_ERR_NULL;
    if (!aligned16(a) || !aligned16(Wq) || (out && !aligned16(out)) || !aligned16(s_w) || (bias && !aligned16(bias)))
        return MKQ_ERR_ALIGN;
    if (epi && ((epi->residual && !aligned16(epi->residual)) || (epi->q_out && !aligned16(epi->q_out)) ||
                (epi->acc_out && !aligned16(epi->acc_out))))
        return MKQ_ERR_ALIGN;
    // exact sums need |acc| <= 64 K < 2^24; 32-bit byte offsets
    if (K >= 262144 || M > 0x7FFFFFFF || N > 0x7FFFFFFF || M * (K / 4 * 3) > 0xFFFFFFFFLL ||
        N * (K / 4 * 3) > 0xFFFFFFFFLL)
        return MKQ_ERR_UNSUPPORTED;
    GemmI4Params p;
    p.A = a; p.W = Wq; p.M = (int)M; p.N = (int)N; p.K = (int)K;
    p.s_x = s_x; p.s_w = s_w; p.bias = bias;
    p.residual = epi ? epi->residual : nullptr;
    p.residual_dtype = epi ? epi->residual_dtype : MKQ_F32;
    p.act = epi ? epi->act : MKQ_ACT_NONE;
    p.out = out; p.out_dtype = out ? out_dtype : -1;
    p.s_next = epi ? epi->s_next : 1.0f;
    p.q_out = (epi && !(out && out_dtype == MKQ_I4)) ? epi->q_out : nullptr;
    p.acc_out = epi ? epi->acc_out : nullptr;
    p.q_pitch = (int)q_pitch;
    p.acc_shift = 0;
    p.acc_unit = 1.0f;
    return run_gemm_e3m2(p, as_stream(stream), forced_cfg);
}

extern "C" int mkq_linear_int4_e3m2(const uint8_t *a, float s_x, const uint8_t *Wq, const float *s_w,
                                    const float *bias, int64_t M, int64_t N, int64_t K, void *out, int out_dtype,
                                    const mkq_epilogue *epi, void *stream)
{
    return linear_int4_e3m2_run(a, s_x, Wq, s_w, bias, M, N, K, out, out_dtype, epi, stream, -1);
}

extern "C" int mkq_tuning_linear_int4_e3m2(const uint8_t *a, float s_x, const uint8_t *Wq, const float *s_w,
                                           const float *bias, int64_t M, int64_t N, int64_t K, void *out,
                                           int out_dtype, const mkq_epilogue *epi, void *stream, int config)
{
    return linear_int4_e3m2_run(a, s_x, Wq, s_w, bias, M, N, K, out, out_dtype, epi, stream, config);
}
