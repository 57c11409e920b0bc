// The tile kernel of the linears: persistent workgroups, a ring of LDS stages filled by direct global->LDS
// copies, operands of 4, 8 or 16 bits, and its launch.
#pragma once

#include "gemm_i4_params.h"

namespace mkq {

// ---------------------------------------------------------------------------------
// Fast path: direct global->LDS copies (global_load_lds_dwordx4) into a ring of S
// stage buffers.  Needs whole stages (K/2 a multiple of RB) because the copy cannot
// zero-fill.  A wave-level copy instruction writes 64 x 16 bytes to consecutive LDS
// addresses (M0 + 16 * lane), i.e. 1024/RB whole tile rows; the XOR swizzle is
// applied on the global side (a lane fetches chunk slot ^ swz(row) of its row), so
// every row is still read as one contiguous RB-byte segment.  The copies bypass the
// registers, which lets S-1 stages be in flight per wave -- several microseconds of
// prefetch, enough to cover HBM latency even for small tiles -- and the compiler
// does not see them, so waiting is explicit: s_waitcnt vmcnt(n) with n = the copies
// issued after the stage that is about to be read, then one workgroup barrier.
template <int BM_, int BN_, int WGM_, int WGN_, int RB_, int S_>
struct GemmI4DmaCfg : GemmI4Cfg<BM_, BN_, WGM_, WGN_, RB_> {
    using Base = GemmI4Cfg<BM_, BN_, WGM_, WGN_, RB_>;
    static constexpr int S = S_;
    static constexpr int WAVES = WGM_ * WGN_;
    static constexpr int ROWS_PER_COPY = 1024 / RB_;
    static constexpr int COPIES = Base::STAGE_BYTES / 1024;  // per stage, whole workgroup
    static constexpr int LPW = COPIES / WAVES;               // per stage, per wave
    static constexpr int LDS_BYTES = S * Base::STAGE_BYTES;
    // resident waves per SIMD the kernel is compiled for: as many workgroups as the LDS
    // holds (at most 2 are useful), one wave of each per SIMD per WAVES / 4
    // two (small per-wave tiles: up to four, 128 registers each then) resident workgroups
    static constexpr int WGS_FIT = 160 * 1024 / (LDS_BYTES + WAVES * 512);
    static constexpr int WGS_WANT = (Base::TM * Base::TN <= 2) ? 4 : (Base::TM * Base::TN <= 4 ? 3 : 2);
    static constexpr int WGS_PER_CU = WGS_FIT < 1 ? 1 : (WGS_FIT < WGS_WANT ? WGS_FIT : WGS_WANT);
    static constexpr int WAVES_PER_EU = (WGS_PER_CU * WAVES / 4 < 2 && RB_ == 128) ? 2 : WGS_PER_CU * WAVES / 4;
    static_assert(COPIES % WAVES == 0, "copies must divide evenly over the waves");
    static_assert(BM_ % ROWS_PER_COPY == 0, "a copy must not straddle the A / W boundary");
    // Which slot is refilled behind a stage's boundary.  OWN: the slot of the stage just read, which every wave holds
    // in registers by then; one more stage in flight from the same ring, what rings of two and three stages need.
    // Otherwise (64-byte stages, three stages and more) the slot of the stage before it, by copies that directly
    // follow the boundary: with the own slot these kernels were 0-10 % slower at short k loops (median 2.4 % of 162
    // shapes with 256x128 tiles, 2.8 % of 154 with 64x64 four-stage tiles of two wave groups).
    static constexpr bool OWN = RB_ != 64;
    // stages in flight right after a stage's copies are issued
    static constexpr int INFLIGHT = OWN ? S - 1 : S - 2;
    static_assert(RB_ == 32 || RB_ == 64 || RB_ == 128, "a stage is one, two or four 32-byte rounds");
    static_assert(S >= (OWN ? 2 : 3) && INFLIGHT * LPW <= 63, "vmcnt immediate is 6 bits");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS is 160 KiB per CU");
};

// Exchange buffer of the K split: per pass every wave of a non-first group hands over TPP of its
// 32x32 accumulator tiles (4 KiB each); tiles of 32x32 per wave need one pass, larger wave tiles go two
// tiles at a time so that the buffer fits beside the groups' rings.
template <class Cfg>
struct KSplitXch {
    static constexpr int TPP = (Cfg::TM * Cfg::TN % 2 == 0 && 2 * (Cfg::LDS_BYTES + EpiShuffle<Cfg>::EXTRA_LDS) +
                                                                  Cfg::WAVES * 8192 <= 160 * 1024) ? 2 : 1;
    static_assert((Cfg::TM * Cfg::TN) % TPP == 0, "whole passes");
    static constexpr int bytes(int ksplit) { return (ksplit - 1) * Cfg::WAVES * TPP * 4096; }
    static constexpr int lds(int ksplit)
    {
        return ksplit * (Cfg::LDS_BYTES + EpiShuffle<Cfg>::EXTRA_LDS) + bytes(ksplit);
    }
    // waves per SIMD the register allocator may assume: the configuration's own, except for split
    // workgroups of multi-tile waves, which are placed by their LDS footprint
    static constexpr int waves_per_eu(int ksplit)
    {
        return (ksplit == 1 || Cfg::TM * Cfg::TN == 1) ? Cfg::WAVES_PER_EU
                                                       : (160 * 1024 / lds(ksplit)) * Cfg::WAVES * ksplit / 4;
    }
};

// log2 of the wave-priority time slice, in shader cycles (0 = off); 2^15 measured best (2-4 %)
constexpr int PRIO_SLICE_LOG2 = 15;

// BITS = 4: nibble-packed operands, widened on the way to the matrix core.  BITS = 8: the
// operands are int8 codes already (the W8A8 comparison path): same ring, same epilogues, a
// 64-byte stage is then two k steps of 32 codes and nothing is widened.  BITS = 16: binary16 operands (the
// baseline linear): a 64-byte stage is two k steps of 16 values, the accumulators are binary32 and the
// epilogue adds the bias without a scale.
// KSPLIT = 2 or 4: the workgroup is that many groups of Cfg::WAVES waves, each running this
// pipeline with a ring of its own over one share of K (for launches with few tiles and a long
// k loop, where a lone wave per SIMD is bound by its own instruction stream); the other groups'
// partial accumulators meet the first group's in LDS at the end of a tile and the first group
// runs the epilogue.
// XS: the reduction over K of an output tile is, beyond that, cut into p.ks slices that different workgroups
// sum (few tokens against a weight matrix with few output channels give too few tiles to fill the chip).
// The persistent loop then runs over (tile, slice) pairs; at the end of a pair the workgroup stores its partial
// accumulators to the caller's scratch area and draws a ticket on the tile's counter, and the one that draws the
// last ticket adds the others' partials to its registers and runs the epilogue ("last ticket": nobody waits
// for anybody, so the grid drains in any scheduling order).  int32 addition is associative: same bits as unsplit.
template <class Cfg, class Epi, int BITS, int KSPLIT = 1, bool XS = false>
__global__ __launch_bounds__(Cfg::THREADS * KSPLIT)
__attribute__((amdgpu_waves_per_eu(KSplitXch<Cfg>::waves_per_eu(KSPLIT), KSplitXch<Cfg>::waves_per_eu(KSPLIT))))
void gemm_i4_dma_kernel(const GemmI4Params p)
{
    const int ks = XS ? p.ks : 1;
    static_assert(BITS == 4 || ((BITS == 8 || BITS == 16) && Cfg::RB >= 64), "stage rows");
    static_assert(BITS != 16 || (!XS && KSPLIT == 1), "partial sums across workgroups and wave groups are integers");
    constexpr bool SCALED = BITS != 16;  // the accumulator is a sum of codes
    using Acc = typename std::conditional<SCALED, v16i, v16f>::type;
    static_assert(KSPLIT == 1 || KSPLIT == 2 || KSPLIT == 4, "one, two or four wave groups");
    constexpr int BM = Cfg::BM, BN = Cfg::BN, RB = Cfg::RB, CH = Cfg::CH;
    constexpr int TM = Cfg::TM, TN = Cfg::TN;
    constexpr int S = Cfg::S, LPW = Cfg::LPW;
    constexpr int ROUNDS = Cfg::ROUNDS, INFLIGHT = Cfg::INFLIGHT;
    constexpr bool OWN = Cfg::OWN && ROUNDS > 1;  // (one-round stages refill their own slot in a loop of their own)

    extern __shared__ __attribute__((aligned(16))) uint8_t smem_all[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave_all / Cfg::WAVES;   // K half of this wave's group (0 when KSPLIT == 1)
    const int wave = wave_all % Cfg::WAVES;
    // per group: the ring, then the scale / bias area of the row epilogue; after the groups: the
    // exchange buffer of the K split
    constexpr int GROUP_LDS = Cfg::LDS_BYTES + EpiShuffle<Cfg>::EXTRA_LDS;
    uint8_t *const smem = smem_all + grp * GROUP_LDS;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
    const int fr = lane & 31, fh = lane >> 5;

    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    const int total_tiles = tiles_m * tiles_n * ks;     // (tile, slice) pairs: pair v is slice v % ks of tile v / ks
    const uint32_t row_bytes = (uint32_t)p.K / 8 * BITS;  // (below 4 GiB, beyond an int: K % 32 == 0)
    const int kt_count = (int)(row_bytes / (RB * KSPLIT)) / ks;  // stages per pair of this group
    // Persistent workgroup: pairs blockIdx.x, blockIdx.x + gridDim.x, ... run through ONE
    // software pipeline, so a tile's first stages are in flight during the previous
    // tile's epilogue.
    const int my_tiles = (total_tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int steps = my_tiles * kt_count;

    // copy q of this wave fills stage bytes [(wave*LPW + q) * 1024, +1024)
    uint32_t goff[LPW];  // byte offset (from A or W) of this lane's chunk at k = 0
    const int c_row = lane / CH;   // row inside the copy
    const int c_slot = lane % CH;  // 16-byte slot inside the row
    int k_first = 0;  // first byte, in a row, of this group's K range in the pair the copy cursor is in
    auto set_tile = [&](int pair) {
        int tm, tn;
        tile_coords(pair / ks, tiles_m, tiles_n, p.group_m, tm, tn);
        k_first = ((pair % ks) * KSPLIT + grp) * kt_count * RB;
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            const int row = (wave * LPW + q) * Cfg::ROWS_PER_COPY + c_row;  // stage row
            const int chunk = c_slot ^ swz<CH>(row & 15);
            int g;
            if (row < BM) {
                g = tm * BM + row;
                g = g < p.M ? g : p.M - 1;  // rows past the edge re-read the last row; never stored
            } else {
                g = tn * BN + (row - BM);
                g = g < p.N ? g : p.N - 1;
            }
            goff[q] = (uint32_t)g * row_bytes + chunk * 16;
        }
    };
    Acc acc[TM][TN];
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][t][v] = 0;

    // Per-lane LDS read offsets of every fragment for the two 64-code rounds of a stage.
    // Fragments are numbered W first (0 .. TN-1), then activations (TN .. TN+TM-1).
    constexpr int NF = TN + TM;
    constexpr int NMFMA = TM * TN;
    int rd[NF][ROUNDS];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int row = wn * Cfg::WTN + t * 32 + w_row_perm(fr);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) rd[t][r] = (BM + row) * RB + (((r * 2 + fh) ^ swz<CH>(row & 15)) * 16);
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int row = wm * Cfg::WTM + j * 32 + fr;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) rd[TN + j][r] = row * RB + (((r * 2 + fh) ^ swz<CH>(row & 15)) * 16);
    }

    // Software pipeline over k steps of 32 codes, two per 32-byte round of a stage.  A k step is
    // NMFMA "slots": one MFMA each, followed by its share of the VALU widening of the
    // NEXT step's operands and, in even steps, one LDS fragment read of the next 64-code
    // round (consumed a whole step later) and, behind the boundary, global->LDS copies.
    // Slots are fenced with scheduling barriers so the matrix pipe always has the next
    // MFMA queued while the wave's VALU work runs in the shadow of the current one.
    // rounds of fragments held; 8 and 16 bits: how many k steps ahead of its use a round is fetched
    constexpr int AHEAD = (BITS != 4 && ROUNDS == 4) ? 2 : 1, BUFS = 2 * AHEAD;
    constexpr int RDENS = AHEAD;  // a step's fetches are issued in its first 1 / RDENS
    uint32_t raw[BUFS][NF][4];

    // Steps of a stage, counted from its boundary (POST of them follow it, the others are the first ones of the
    // next iteration); OWN: a wave's copies into the slot just read are spread over SPREAD steps from the boundary on:
    // issued together, the 16 cycles that the address unit needs for each of them stall the wave and its matrix
    // pipe.  A two-stage ring waits for the copies at the next boundary, so they go out in its first half.
    constexpr int STEPS = BITS == 4 ? 2 * ROUNDS : ROUNDS;
    constexpr int POST = ROUNDS == 1 ? STEPS : BITS == 4 ? 2 : AHEAD;
    constexpr int SPREAD = !OWN ? 1 : (S >= 3 ? STEPS : (STEPS + 1) / 2);
    constexpr int FIRST = SPREAD <= POST ? LPW : POST * LPW / SPREAD;  // copies of the POST steps
    v4i wid[2][NF];          // widened operands of two k steps

    auto read_frag = [&](int stage_off, auto fc, auto rc, uint32_t(&dst)[4]) {
        constexpr int f = decltype(fc)::value, r = decltype(rc)::value;
        const uint4 v = *reinterpret_cast<const uint4 *>(smem + stage_off + rd[f][r]);
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
    };
    // register q of the widened operand: codes of word 2*ks + q/2, even (q even) or odd nibbles
    auto widen_reg = [&](const uint32_t(&src)[4], auto ksc, auto qc) -> int {
        constexpr int ks = decltype(ksc)::value, q = decltype(qc)::value;
        const uint32_t w = src[2 * ks + q / 2];
        return (int)(((q & 1) ? w : (w << 4)) & 0xF0F0F0F0u);
    };

    int lt = blockIdx.x, lk = 0;  // copy cursor
    set_tile(lt);
    // Per copy: one SALU op (M0 = LDS destination) and the copy itself.  The k offset
    // of the stage is folded into two base pointers that are advanced once per stage.
    const uint8_t *a_k = p.A + k_first, *w_k = p.W + k_first;
    const uint32_t lds_wave = lds0 + wave * (LPW * 1024);
    auto copy_one = [&](int slot, auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const bool is_a = (wave * LPW + q) * Cfg::ROWS_PER_COPY < BM;  // wave-uniform
        dma_copy16<q * 1024>(is_a ? a_k : w_k, goff[q], lds_wave + slot * Cfg::STAGE_BYTES);
    };
    // Always issues LPW copies per stage, so the number in flight never depends on where
    // the pipeline is: past the last stage it re-fetches the last tile's stages into
    // slots that are never read again.
    auto copy_advance = [&]() {
        a_k += RB;
        w_k += RB;
        if (++lk == kt_count) {
            lk = 0;
            if (lt + (int)gridDim.x < total_tiles) {
                lt += gridDim.x;
                set_tile(lt);
            }
            a_k = p.A + k_first;
            w_k = p.W + k_first;
        }
    };

    // the copies of MFMA slot i of the step that is step P from the boundary
    auto slot_copies = [&](auto pc, auto ic, int cslot, bool copy) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value, i = decltype(ic)::value, G = SPREAD * NMFMA, g = P * NMFMA + i;
        if constexpr (P < SPREAD) {
            constexpr int q0 = g * LPW / G, q1 = (g + 1) * LPW / G;
            if constexpr (q1 > q0) {
                if (P >= POST || copy) static_for<q1 - q0>([&](auto qc) { copy_one(cslot, IntC<q0 + decltype(qc)::value>{}); });
            }
        }
    };

    // One k step.  H = step inside the stage.  Operands: wid[H & 1]; widens the next
    // step's into wid[(H + 1) & 1] from raw[SRC] half KS; READ: fetch round RR of the
    // stage at rd_off into raw[RB_]; COPY: issue this wave's copies into ring slot cslot.
    auto k_step = [&](auto hc, int rd_off, int cslot, bool copy) {
        constexpr int H = decltype(hc)::value;
        constexpr int cb = H & 1, nb = cb ^ 1;
        constexpr int SRC = ((H + 1) / 2) & 1;            // raw buffer the next step is widened from
        constexpr int KS = (H + 1) & 1;                   // which half of it
        constexpr bool READ = (H & 1) == 0;
        constexpr int RDST = (H / 2 + 1) & 1;             // raw buffer the reads fill
        constexpr int RR = (H / 2 + 1) % ROUNDS;          // round they fetch
        static_for<NMFMA>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int j = i / TN, t = i % TN;
            if constexpr (Cfg::WAVES_PER_EU == 1) {
                // a single wave owns the SIMD's 512 registers: keep the accumulators in the
                // AGPR half by construction
                asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0"
                             : "+a"(acc[j][t]) : "v"(wid[cb][t]), "v"(wid[cb][TN + j]));
            } else {
                acc[j][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wid[cb][t], wid[cb][TN + j], acc[j][t], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (READ) {
                constexpr int f0 = i * NF / NMFMA, f1 = (i + 1) * NF / NMFMA;
                static_for<f1 - f0>([&](auto fc) {
                    constexpr int f = f0 + decltype(fc)::value;
                    read_frag(rd_off, IntC<f>{}, IntC<RR>{}, raw[RDST][f]);
                });
            }
            slot_copies(IntC<ROUNDS == 1 ? H & 1 : (H + 2) % STEPS>{}, ic, cslot, copy);
            constexpr int m0 = i * 4 * NF / NMFMA, m1 = (i + 1) * 4 * NF / NMFMA;
            static_for<m1 - m0>([&](auto mc) {
                constexpr int m = m0 + decltype(mc)::value;
                int w = widen_reg(raw[SRC][m / 4], IntC<KS>{}, IntC<m % 4>{});
                // pin the op to this slot: without a use here the optimizer sinks it to the
                // operand's first use, a whole k step (and possibly a branch) later
                asm volatile("" : "+v"(w));
                wid[nb][m / 4][m % 4] = w;
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // 8- and 16-bit operands: one k step per 32-byte round, ROUNDS per stage.  Step H multiplies the round in
    // raw[H % BUFS] while the round AHEAD steps later (of the next stage in the last AHEAD steps)
    // is fetched into its buffer.
    auto k_step8 = [&](auto hc, int rd_off, int cslot, bool copy) {
        constexpr int H = decltype(hc)::value;
        constexpr int B = H % BUFS, NB = (H + AHEAD) % BUFS;
        static_for<NMFMA>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int j = i / TN, t = i % TN;
            const v4i fw = {(int)raw[B][t][0], (int)raw[B][t][1], (int)raw[B][t][2], (int)raw[B][t][3]};
            const v4i fa = {(int)raw[B][TN + j][0], (int)raw[B][TN + j][1], (int)raw[B][TN + j][2],
                            (int)raw[B][TN + j][3]};
            if constexpr (BITS == 16)
                acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, fw), __builtin_bit_cast(v8h, fa),
                                                                   acc[j][t], 0, 0, 0);
            else
                acc[j][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw, fa, acc[j][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int f0 = min_i(i * RDENS * NF / NMFMA, NF), f1 = min_i((i + 1) * RDENS * NF / NMFMA, NF);
            static_for<f1 - f0>([&](auto fc) {
                constexpr int f = f0 + decltype(fc)::value;
                read_frag(rd_off, IntC<f>{}, IntC<(H + AHEAD) % ROUNDS>{}, raw[NB][f]);
            });
            slot_copies(IntC<(H + AHEAD) % STEPS>{}, ic, cslot, copy);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // prologue: put INFLIGHT stages and the FIRST copies of one more in flight, wait for stage 0, prime the
    // register pipeline
#pragma unroll
    for (int i = 0; i < INFLIGHT; ++i) {
        static_for<LPW>([&](auto qc) { copy_one(i, qc); });
        copy_advance();
    }
    static_for<FIRST>([&](auto qc) { copy_one(INFLIGHT, qc); });
    if constexpr (!OWN) copy_advance();
    wait_vmcnt<(INFLIGHT - 1) * LPW + FIRST>();
    lds_barrier();
    static_for<AHEAD>([&](auto rc) {
        static_for<NF>([&](auto fc) { read_frag(0, fc, rc, raw[decltype(rc)::value][decltype(fc)::value]); });
    });
    if constexpr (BITS == 4) {
        static_for<4 * NF>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            wid[0][m / 4][m % 4] = widen_reg(raw[0][m / 4], IntC<0>{}, IntC<m % 4>{});
        });
    }

    // Epilogue stores share the in-order vmcnt counter with the copies.  At the first
    // stage boundaries that follow an epilogue the wanted copies are older than those
    // stores, so the stores may stay outstanding if the wait allows for their
    // exact number; that number is only known at compile time for interior tiles of the
    // fixed epilogues.
    // (the row epilogue issues the same number of 16-byte-per-lane stores as the direct one,
    // and with a 16-bit residual its loads are all older than its first store only for the
    // direct path, so that variant waits for everything)
    constexpr int STORES_PER_UNIT = Epi::generic ? 0 : (Epi::out == MKQ_F32 ? 2 : 1);
    constexpr int EPI_STORES = TN * 2 * TM * STORES_PER_UNIT;
    constexpr bool ASYNC_STORES = !Epi::generic && ((INFLIGHT - 1) * LPW + EPI_STORES <= 63);
    int stores_pending = 0;  // boundaries left that may leave the epilogue's stores in flight

    // Stage boundary: the next stage becomes readable (INFLIGHT-1 younger stages may stay
    // in flight); past the barrier every wave is done with the slot that is refilled next.
    // Two workgroups share a CU and the SIMD arbiter always serves the older wave first: the
    // first-placed workgroup runs at full speed, the second in its gaps (and alone at the end).
    // Each workgroup therefore takes the higher wave priority in alternate time slices of the
    // CU's cycle counter, in opposite phase, so both progress at the same average rate.
    const unsigned prio_phase = (2 * blockIdx.x >= gridDim.x) ? 1u : 0u;
    unsigned long long tnow = 0;
    auto stage_boundary = [&]() {
        if constexpr (Cfg::WGS_PER_CU == 2 && PRIO_SLICE_LOG2 > 0) {
            const unsigned hi = __builtin_amdgcn_readfirstlane(((unsigned)(tnow >> PRIO_SLICE_LOG2) ^ prio_phase) & 1u);
            if (hi) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        if (ASYNC_STORES && stores_pending > 0) {
            wait_vmcnt<ASYNC_STORES ? (INFLIGHT - 1) * LPW + EPI_STORES : 0>();
            --stores_pending;
        } else {
            wait_vmcnt<(INFLIGHT - 1) * LPW>();
        }
        lds_barrier();
    };
    auto next_slot = [&](int b) { return (b + 1 == S) ? 0 : b + 1; };
    auto prev_slot = [&](int b) { return (b == 0) ? S - 1 : b - 1; };

    constexpr bool ROWS_EPI = !Epi::generic && EpiShuffle<Cfg>::usable;
    float *const sc_lds = reinterpret_cast<float *>(smem + Cfg::LDS_BYTES + wave * EpiShuffle<Cfg>::SCALE_BYTES);
    // copies s_w / bias of this wave's channels of tile `tile` to sc_lds
    auto stage_scales = [&](int pair) {
        int tm, tn;
        tile_coords(pair / ks, tiles_m, tiles_n, p.group_m, tm, tn);
        const uint32_t dst = lds0 + Cfg::LDS_BYTES + wave * EpiShuffle<Cfg>::SCALE_BYTES;
        static_for<EpiShuffle<Cfg>::NSL>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            int n = tn * BN + wn * Cfg::WTN + 64 * i + lane;
            n = n < p.N ? n : p.N - 1;
            if constexpr (SCALED) dma_copy4<256 * i>(reinterpret_cast<const uint8_t *>(p.s_w), (uint32_t)n * 4u, dst);
            if (p.bias)
                dma_copy4<EpiShuffle<Cfg>::BIAS_AT * 4 + 256 * i>(reinterpret_cast<const uint8_t *>(p.bias),
                                                                  (uint32_t)n * 4u, dst);
        });
    };

    // The copies are issued INFLIGHT stages before the tile ends (or at its first stage):
    // by the epilogue every vector memory operation still in flight is then younger.
    const int scale_stage = kt_count > INFLIGHT ? kt_count - INFLIGHT : 0;

    int ct = blockIdx.x, ck = 0;  // compute cursor
    int buf = 0;                  // ring slot of the stage being computed
    for (int s = 0; s < steps; s += ROUNDS == 1 ? 2 : 1) {
        if constexpr (Cfg::WGS_PER_CU == 2 && PRIO_SLICE_LOG2 > 0) tnow = __builtin_readcyclecounter();  // used at the boundary
        if constexpr (ROWS_EPI) {
            if (grp == 0 && ck == scale_stage) stage_scales(ct);
        }
        // OWN: a stage's slot is refilled from its boundary on, except behind a tile's last stage: there it first
        // serves the epilogue as scratch and each wave refills its share after that.
        const bool last = OWN && ck + 1 == kt_count;
        if constexpr (BITS != 4) {
            const int nbuf = next_slot(buf);
            const int pbuf = prev_slot(buf);
            static_for<ROUNDS - AHEAD>([&](auto hc) { k_step8(hc, buf * Cfg::STAGE_BYTES, pbuf, true); });
            if constexpr (OWN) copy_advance();
            stage_boundary();
            static_for<AHEAD>([&](auto hc) {
                k_step8(IntC<ROUNDS - AHEAD + decltype(hc)::value>{}, nbuf * Cfg::STAGE_BYTES, OWN ? buf : pbuf, !last);
            });
            if constexpr (!OWN) copy_advance();
            buf = nbuf;
            ck += 1;
        } else if constexpr (ROUNDS > 1) {
            // one stage of ROUNDS rounds: rounds 1 .. are fetched from the same stage, then the boundary,
            // then round 0 of the next stage while a slot is refilled
            const int nbuf = next_slot(buf);
            const int pbuf = prev_slot(buf);
            static_for<2 * ROUNDS - 2>([&](auto hc) { k_step(hc, buf * Cfg::STAGE_BYTES, pbuf, true); });
            if constexpr (OWN) copy_advance();
            stage_boundary();
            k_step(IntC<2 * ROUNDS - 2>{}, nbuf * Cfg::STAGE_BYTES, OWN ? buf : pbuf, !last);
            if constexpr (!OWN) copy_advance();
            k_step(IntC<2 * ROUNDS - 1>{}, 0, buf, !last);
            buf = nbuf;
            ck += 1;
        } else {
            // two 64-code stages (the raw / wid register buffers alternate, so the body is
            // unrolled twice); each stage's own slot is refilled at its boundary
            int nbuf = next_slot(buf);
            stage_boundary();
            k_step(IntC<0>{}, nbuf * Cfg::STAGE_BYTES, buf, true);
            copy_advance();
            k_step(IntC<1>{}, 0, 0, false);
            buf = nbuf;
            nbuf = next_slot(buf);
            stage_boundary();
            k_step(IntC<2>{}, nbuf * Cfg::STAGE_BYTES, buf, true);
            copy_advance();
            k_step(IntC<3>{}, 0, 0, false);
            buf = nbuf;
            ck += 2;
        }

        if (ck == kt_count) {
            int tile_m, tile_n;
            tile_coords(ct / ks, tiles_m, tiles_n, p.group_m, tile_m, tile_n);
            if constexpr (KSPLIT > 1) {
                // the other groups hand their partial sums over, KSplitXch<Cfg>::TPP 32x32 tiles of a wave
                // (16 registers per lane, 4 KiB per tile) per pass through the exchange buffer
                constexpr int TPP = KSplitXch<Cfg>::TPP, PASSES = TM * TN / TPP;
                int *const xch = reinterpret_cast<int *>(smem_all + KSPLIT * GROUP_LDS) + wave * (TPP * 1024) + lane * 4;
                static_for<PASSES>([&](auto pc) {
                    constexpr int pass = decltype(pc)::value;
                    if (pass > 0) lds_barrier();  // the first group has read the previous pass
                    if (grp > 0) {
                        static_for<TPP>([&](auto uc) {
                            constexpr int u = decltype(uc)::value, i = pass * TPP + u, j = i / TN, t = i % TN;
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                *reinterpret_cast<int4 *>(xch + (grp - 1) * (Cfg::WAVES * TPP * 1024) + u * 1024 + q * 256) =
                                    make_int4(acc[j][t][4 * q], acc[j][t][4 * q + 1], acc[j][t][4 * q + 2],
                                              acc[j][t][4 * q + 3]);
                        });
                    }
                    lds_barrier();
                    if (grp == 0) {
                        static_for<TPP>([&](auto uc) {
                            constexpr int u = decltype(uc)::value, i = pass * TPP + u, j = i / TN, t = i % TN;
#pragma unroll
                            for (int g = 0; g < KSPLIT - 1; ++g)
#pragma unroll
                                for (int q = 0; q < 4; ++q) {
                                    const int4 v = *reinterpret_cast<const int4 *>(
                                        xch + g * (Cfg::WAVES * TPP * 1024) + u * 1024 + q * 256);
                                    acc[j][t][4 * q] += v.x; acc[j][t][4 * q + 1] += v.y;
                                    acc[j][t][4 * q + 2] += v.z; acc[j][t][4 * q + 3] += v.w;
                                }
                        });
                    }
                });
            }
            bool finish = true;  // this workgroup runs the tile's epilogue
            if constexpr (XS) {
                if (ks > 1) {
                    // partial tile of a wave: TM * TN blocks of 16 registers x 64 lanes; register pair q of all
                    // lanes is one contiguous 512-byte piece.  Agent-scope relaxed atomics: the stores write
                    // through to memory and the loads do not hit a stale line of this XCD's L2.
                    const int tile = ct / ks, slice = ct % ks;
                    constexpr size_t WAVE_WORDS = (size_t)TM * TN * 8 * 64;  // 64-bit words
                    uint64_t *const area = reinterpret_cast<uint64_t *>(p.sk_partials);
                    if (grp == 0) {
                        uint64_t *const mine = area + ((size_t)(tile * ks + slice) * Cfg::WAVES + wave) * WAVE_WORDS + lane;
#pragma unroll
                        for (int j = 0; j < TM; ++j)
#pragma unroll
                            for (int t = 0; t < TN; ++t)
#pragma unroll
                                for (int q = 0; q < 8; ++q) {
                                    const uint64_t v = (uint64_t)(uint32_t)acc[j][t][2 * q] |
                                                       ((uint64_t)(uint32_t)acc[j][t][2 * q + 1] << 32);
                                    __hip_atomic_store(mine + ((j * TN + t) * 8 + q) * 64, v, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
                                }
                    }
                    wait_vmcnt<0>();   // this wave's partials have reached memory (and every copy in flight has landed)
                    __syncthreads();   // ... and every other wave's
                    // whether this workgroup drew the last ticket is told through the first word of the first
                    // group's ring slot of the stage just finished (idle until the next stage boundary)
                    volatile int *const xs_last =
                        reinterpret_cast<volatile int *>(smem_all + ((buf == 0) ? S - 1 : buf - 1) * Cfg::STAGE_BYTES);
                    if (tid == 0) {
                        const unsigned old = __hip_atomic_fetch_add(p.sk_counters + tile, 1u, __ATOMIC_RELAXED,
                                                                    __HIP_MEMORY_SCOPE_AGENT);
                        const int last = old == (unsigned)(ks - 1);
                        if (last) __hip_atomic_store(p.sk_counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        *xs_last = last;
                    }
                    __syncthreads();
                    finish = *xs_last != 0;
                    __syncthreads();  // (the slot serves the epilogue as scratch next)
                    if (finish && grp == 0) {
                        for (int o = 0; o < ks; ++o) {
                            if (o == slice) continue;
                            const uint64_t *theirs = area + ((size_t)(tile * ks + o) * Cfg::WAVES + wave) * WAVE_WORDS + lane;
#pragma unroll
                            for (int j = 0; j < TM; ++j)
#pragma unroll
                                for (int t = 0; t < TN; ++t)
#pragma unroll
                                    for (int q = 0; q < 8; ++q) {
                                        const uint64_t v = __hip_atomic_load(theirs + ((j * TN + t) * 8 + q) * 64,
                                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                        acc[j][t][2 * q] += (int)(uint32_t)v;
                                        acc[j][t][2 * q + 1] += (int)(uint32_t)(v >> 32);
                                    }
                        }
                    }
                }
            }
            if (grp == 0 && finish) {
                if constexpr (ROWS_EPI) {
                    // the slot of the stage just finished is idle (!OWN: until every wave has passed the next
                    // boundary): each wave shuffles through the share of it that it refills itself
                    const int done_slot = (buf == 0) ? S - 1 : buf - 1;
                    // the scale / bias copies have landed: only the stage copies issued after them (those of
                    // INFLIGHT boundaries, one less with OWN, fewer in a shorter tile) may be in flight
                    if (kt_count >= INFLIGHT) wait_vmcnt<(INFLIGHT - (OWN ? 1 : 0)) * LPW>();
                    else wait_vmcnt<OWN ? 0 : LPW>();
                    // plain 16-bit outputs of 64-channel waves take the line epilogue, without its register
                    // cache of the scales (with it this kernel spills)
                    if constexpr (EpiLines16<Cfg, Epi>::usable)
                        gemm_epilogue_lines16<Cfg, Epi, false, SCALED>(p, acc, tile_m * BM, tile_n * BN, wm, wn, lane,
                                                               smem + done_slot * Cfg::STAGE_BYTES +
                                                                   wave * EpiShuffle<Cfg>::REGION, sc_lds);
                    else
                        gemm_i4_epilogue_rows<Cfg, Epi, SCALED>(p, acc, tile_m * BM, tile_n * BN, wm, wn, lane,
                                                        smem + done_slot * Cfg::STAGE_BYTES +
                                                            wave * EpiShuffle<Cfg>::REGION, sc_lds);
                } else {
                    gemm_i4_epilogue<Cfg, Epi, SCALED>(p, acc, tile_m * BM, tile_n * BN, wm, wn, fr, fh);
                }
            }
            const bool interior = (tile_m + 1) * BM <= p.M && (tile_n + 1) * BN <= p.N;
            // (a group without stores must not count them in its waits)
            // (OWN: the copies of the slot refilled next come behind the stores, one boundary less)
            stores_pending = (ASYNC_STORES && interior && grp == 0 && finish) ? INFLIGHT - (OWN ? 1 : 0) : 0;
            if constexpr (OWN) {
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave is done with its scratch
                const int done = __builtin_amdgcn_readfirstlane(prev_slot(buf));
                static_for<FIRST>([&](auto qc) { copy_one(done, qc); });
            }
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
    wait_vmcnt<0>();  // the trailing dummy copies must land before the LDS is released
}

template <class Cfg, class Epi, int BITS = 4, int KSPLIT = 1, bool XS = false>
static int launch_gemm_i4_dma(const GemmI4Params &p, hipStream_t st)
{
    const int64_t tiles = ceil_div(p.M, Cfg::BM) * ceil_div(p.N, Cfg::BN) * (XS ? p.ks : 1);
    if (tiles > 0x7FFFFFFF) return MKQ_ERR_UNSUPPORTED;
    constexpr bool rows_epi = !Epi::generic && EpiShuffle<Cfg>::usable;
    constexpr size_t lds_kernel =
        KSPLIT == 1 ? Cfg::LDS_BYTES + (rows_epi ? EpiShuffle<Cfg>::EXTRA_LDS : 0)
                    : KSplitXch<Cfg>::lds(KSPLIT);
    static_assert(lds_kernel <= 160 * 1024, "LDS is 160 KiB per CU");
    const size_t lds = lds_kernel;
    static PerDeviceOnce once;  // per instantiation
    int64_t resident = 0;
    const int rc = resident_workgroups(once, gemm_i4_dma_kernel<Cfg, Epi, BITS, KSPLIT, XS>, Cfg::THREADS * KSPLIT, lds,
                                       1 << 20, &resident);
    if (rc != MKQ_OK || p.setup_only) return rc;
    const unsigned grid = (unsigned)(tiles < resident ? tiles : resident);
    GemmI4Params q = p;
    q.group_m = tile_group(p.by_rows, ceil_div(p.M, Cfg::BM));
    gemm_i4_dma_kernel<Cfg, Epi, BITS, KSPLIT, XS><<<grid, Cfg::THREADS * KSPLIT, lds, st>>>(q);
    return launch_status();
}

// With the epilogue that takes every option
template <class Cfg, int BITS = 4, int KSPLIT = 1, bool XS = false>
static int launch_gemm_i4_dma_generic(const GemmI4Params &p, hipStream_t st)
{
    if (epi_gelu_tail(p.act, p.out_dtype)) return launch_gemm_i4_dma<Cfg, EpiGeluTail, BITS, KSPLIT, XS>(p, st);
    return launch_gemm_i4_dma<Cfg, EpiGeneric, BITS, KSPLIT, XS>(p, st);
}

}  // namespace mkq
