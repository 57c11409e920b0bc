// Attention core of sequences of up to 512 keys with the scores held in registers between the softmax and the product
// with V, so that every score is computed and exponentiated once.  (The kernel for longer sequences goes over the keys
// twice, because the probabilities are normalized before they are narrowed to binary16.)
//
// One workgroup of eight waves per (sequence, head) and some of its blocks of 128 queries.  All keys and values of the
// head are staged in LDS once (V transposed).  A wave has 16 queries and all keys, and after the staging no wave waits for
// another, so that one's matrix products run beside the other's exponentials:
//   S^T = K Q^T                 (MFMA "A" = keys, "B" = queries: a lane has one query, and of every 32 keys the eight that
//                                its P operand takes, by the order in which the rows of K are read)
//   P = exp(S / sqrt(d_k) - max) / sum, in binary32, narrowed to binary16
//   O^T = V^T P^T               (rows of V^T in the same order: a lane ends with runs of eight head dimensions)
// The scores of 32 keys take 8 registers, those of 512 keys 128.
// What bounds it: the 6 KiB of q, k, v per token and 1024 hidden out of memory, all at the start of a round (10 of 38 us
// below), then vector issue: per score one exponential (16 cycles) and about 16 cycles of other operations, against 8 of
// matrix pipe.  us in a graph, over the keys twice -> here: 16 heads of 64, 16 x 512 tokens 56.5 -> 38.5, 4 x 512 22.3 -> 13.3,
// 32 x 256 32.0 -> 24.6, 20 x 384 44.2 -> 35.7; 12 heads of 26, 32 x 128 9.6 -> 7.2, 64 x 128 15.3 -> 10.7, 16 x 512 33.9 -> 29.5.
// Tried before it: 32 queries and half of the keys per wave, maxima and outputs exchanged by pairs of waves: 42 to 46 us at
// 16 x 512, 46 at 20 x 384 (the pairs run in step, so exponentials and matrix products do not overlap).
#include "attention.h"

namespace mkq {

// NG: groups of 32 keys
template <int DKP, int NG>
struct AttentionHeldCfg {
    static constexpr int THREADS = ATTENTION_HELD_THREADS, KEYS = 32 * NG;
    static constexpr int VROW = (KEYS + 127) / 128 * 256;  // bytes of a row of V^T: the swizzle moves within 16 chunks of 8 keys
    static constexpr int K_BYTES = KEYS * DKP * 2, V_BYTES = DKP * VROW;
    static constexpr int LDS_BYTES = K_BYTES + V_BYTES;
};

// 16-byte chunk c of key r is kept at c ^ swz_keys(r) (of V^T: swz_dims).  A fragment's sixteen rows
// differ in bits 0, 1, 3 and 4 (prow below); with these functions of just those bits they meet all 64 banks, and each eight of them 32.
// (Functions of bits 0 to 3, as for sixteen neighbouring rows, put them on half of the banks: us in a graph, 32 x 256 tokens, 16 heads
// of 64 27.4 -> 24.6, 32 x 200, 12 heads 22.4 -> 19.3, 20 x 384, 16 heads 37.4 -> 35.7.)
template <int CH>
__device__ __forceinline__ int swz_keys(int r)
{
    return CH == 8 ? ((r >> 1) & 1) | ((r >> 2) & 2) | (((r >> 4) ^ r) & 1) << 2 : ((r >> 3) & 1) | (((r >> 4) ^ (r >> 1)) & 1) << 1;
}

// DKP: head size rounded up to 32 or 64 (dimensions d_k .. DKP - 1 are staged as zeros and never stored).  VEC = 8: 16-byte
// accesses (d_k % 8 == 0); VEC = 2: 4-byte ones.  parts: workgroups per (sequence, head), from the host, 1 for up to 128 keys: the divisions
// by it are latency in front of the first load (64 x 64 tokens, 12 heads of 26, 8.4 -> 7.5 us in a graph, 32 x 128 7.6 -> 7.45).
template <int DKP, int VEC, int NG>
__global__ __launch_bounds__(512, NG <= 8 ? 4 : 2) void attention_held_kernel(const AttentionParams p, int per_wg, int parts, int first_half,
                                                                                const XcdRuns runs)
{
    using Cfg = AttentionHeldCfg<DKP, NG>;
    constexpr int THREADS = Cfg::THREADS, KEYS = Cfg::KEYS, ROWB = DKP * 2, CH = DKP / 8, VROW = Cfg::VROW, DS = DKP / 32;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint8_t *const sK = smem, *const sVt = smem + Cfg::K_BYTES;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    // uniform batches: an eighth of (sequence, head, part) to each XCD.  Padding-free ones: runs of heads, parts outermost (with the
    // parts of a head side by side, all first parts of two meet on every other XCD).  us, 16 heads of 64, 16 sequences to 512, an eighth
    // in one piece -> this with the longest shared: rising from 32 34.0 -> 25.5, random 33.5 -> 27.2, one of 512 and the others of
    // 64 31.0 -> 18.9, all of 230 13.1 -> 13.9, all of 512 38.2 -> 38.0
    int part, bh;
    bool share = false;  // the longest sequences by two workgroups
    if (p.cu_seqlens) {
        const unsigned sequence_heads = (unsigned)p.batch * p.heads;
        part = parts == 1 ? 0 : (int)(blockIdx.x / sequence_heads);
        bh = xcd_run_index(blockIdx.x - part * sequence_heads, runs);
        if (first_half) {
            // of the first 64 sequences, at most half are longest: these are shared, and where they are at most an eighth, their
            // second halves come before everything else (16 x 512 tokens, one sequence of 512 and the others of 64: second halves
            // last 22.3 us, first 18.6; 16 random lengths to 512, six of them longest, 27.3 and 31.2)
            const int n = p.batch < 64 ? p.batch : 64;
            const int32_t *const at = p.cu_seqlens + (lane < n ? lane : 0);
            const int many = __builtin_popcountll(__ballot(lane < n && at[1] - at[0] > (p.q_blocks - 1) * 128));
            share = 2 * many <= n;
            if (many && 8 * many <= n) part = 1 - part;
        }
    } else {
        const int block = xcd_index(blockIdx.x, gridDim.x);
        bh = parts == 1 ? block : block / parts;
        part = block - bh * parts;
    }
    const int b = bh / p.heads, head = bh % p.heads;
    const int64_t row0 = p.cu_seqlens ? (int64_t)p.cu_seqlens[b] : (int64_t)b * p.seq;
    int seq = p.cu_seqlens ? (p.cu_seqlens[b + 1] - p.cu_seqlens[b]) : p.seq;
    seq = seq < KEYS ? seq : KEYS;  // (longer than the caller's bound on the lengths: not computed)
    if (share && seq > (p.q_blocks - 1) * 128) per_wg = first_half;
    const int first = part * per_wg * 128;
    if (first >= seq) return;  // the whole workgroup: no barrier has been passed
    const int hidden = p.hidden, dk = p.dk, ld = 3 * hidden;

    // K row by row (swizzled 16-byte chunks), V transposed, [d][key]: a thread takes the same columns of two neighbouring
    // rows of V, so that an LDS write carries two keys of one head dimension.  All loads are issued before the first write.
    using Piece = typename std::conditional<VEC == 8, uint4, uint32_t>::type;
    constexpr int PPR = DKP / VEC;                                           // pieces per row
    constexpr int JOBS = KEYS * PPR, PER_T = (JOBS + THREADS - 1) / THREADS;  // pieces of K; per thread
    constexpr int PAIRS = JOBS / 2, PAIRS_T = (PAIRS + THREADS - 1) / THREADS;
    // the code is free of branches where at most the last 64 keys are short of KEYS (they are staged as copies of the last
    // row and masked)
    const bool full = seq > KEYS - 64;
    const int rows = full ? KEYS : (seq + 31) & ~31;
    // (offsets within a sequence in 32 bits: attention_route keeps longer ones away)
    auto fetch = [&](int r, int d, int col) __attribute__((always_inline)) {
        Piece v{};
        const uint8_t *const base = reinterpret_cast<const uint8_t *>(p.qkv + row0 * ld + head * dk + col);
        if (d < dk) v = *reinterpret_cast<const Piece *>(base + ((uint32_t)(r < seq ? r : seq - 1) * (uint32_t)ld + (uint32_t)d) * 2u);
        return v;
    };
    Piece kv[PER_T], vv[PAIRS_T][2];
#pragma unroll
    for (int i = 0; i < PER_T; ++i) {
        if (i * THREADS / PPR < rows) {  // (uniform)
            const int idx = tid + i * THREADS;
            kv[i] = fetch(idx / PPR, (idx % PPR) * VEC, hidden);
        }
    }
#pragma unroll
    for (int i = 0; i < PAIRS_T; ++i) {
        if (2 * (i * THREADS / PPR) < rows) {
            const int j = tid + i * THREADS;
#pragma unroll
            for (int k = 0; k < 2; ++k) vv[i][k] = fetch(2 * (j / PPR) + k, (j % PPR) * VEC, 2 * hidden);
        }
    }
    const int last = first + per_wg * 128 < seq ? first + per_wg * 128 : seq;
    const int qrow = wave * 16 + lr;  // within a block
    uint32_t qraw[DS][4];
    auto fetch_q = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            const int d = (ds * 4 + lg) * 8;
            if constexpr (VEC == 8) {
                const uint4 v = fetch(q, d, 0);
                qraw[ds][0] = v.x; qraw[ds][1] = v.y; qraw[ds][2] = v.z; qraw[ds][3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) qraw[ds][e] = fetch(q, d + 2 * e, 0);
            }
        }
    };
    fetch_q(first + qrow);
#pragma unroll
    for (int i = 0; i < PER_T; ++i) {
        if (i * THREADS / PPR < rows && (JOBS % THREADS == 0 || tid + i * THREADS < JOBS)) {
            const int idx = tid + i * THREADS, r = idx / PPR, d = (idx % PPR) * VEC;
            *reinterpret_cast<Piece *>(sK + r * ROWB + (((d >> 3) ^ swz_keys<CH>(r)) * 16) + (d & 7) * 2) = kv[i];
        }
    }
#pragma unroll
    for (int i = 0; i < PAIRS_T; ++i) {
        const int j = tid + i * THREADS;
        if (2 * (i * THREADS / PPR) < rows && (PAIRS % THREADS == 0 || j < PAIRS)) {
            const int r = 2 * (j / PPR), d0 = (j % PPR) * VEC;
            uint32_t w0[VEC / 2], w1[VEC / 2];
            if constexpr (VEC == 8) {
                w0[0] = vv[i][0].x; w0[1] = vv[i][0].y; w0[2] = vv[i][0].z; w0[3] = vv[i][0].w;
                w1[0] = vv[i][1].x; w1[1] = vv[i][1].y; w1[2] = vv[i][1].z; w1[3] = vv[i][1].w;
            } else {
                w0[0] = vv[i][0];
                w1[0] = vv[i][1];
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const int d = d0 + e;
                const uint32_t lo = (w0[e >> 1] >> (16 * (e & 1))) & 0xFFFFu, hi = (w1[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
                *reinterpret_cast<uint32_t *>(sVt + d * VROW + (((r >> 3) ^ swz_dims(d)) * 16) + (r & 7) * 2) = lo | (hi << 16);
            }
        }
    }
    __syncthreads();

    // exp(x / sqrt(d_k)) as exp2(x * c)
    const float c_exp = (1.0f / sqrtf((float)dk)) * 1.4426950408889634f;
    constexpr float MASKED = -1.0e30f;  // a key past the end of the sequence: exp2 gives 0
    // row i = lr of a K or V^T fragment: 8 (i / 4) + i % 4 of 32, and 4 more in the second of a pair
    const int prow = 8 * (lr >> 2) + (lr & 3);

    // This lane's chunks of its rows of K and V^T in the first group and part.  The swizzles leave out bit 2 of a row and the bits above 4,
    // so parts, groups and halves of a head's dimensions are constants away (chunk 4 g + lg of V^T: 4 (g % 4) under the swizzle, 16 (g / 4)
    // beyond).
    const int kat = prow * ROWB + ((lg ^ swz_keys<CH>(prow)) * 16), vat = prow * VROW + ((lg ^ swz_dims(prow)) * 16);
    v4f sc[NG][2];  // scores: element e of part t of group g is key 32 g + 8 lg + 4 t + e
    auto softmax = [&](auto fullc, float &mx, float &den) __attribute__((always_inline)) {
        constexpr bool FULL = fullc.value;
        constexpr int AHEAD = held_fetch_ahead(FULL, NG);
        auto exists = [&](int g) { return FULL || g * 32 < seq; };  // (uniform)
        v8h qf[DS];
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            const v4i packed = {(int)qraw[ds][0], (int)qraw[ds][1], (int)qraw[ds][2], (int)qraw[ds][3]};
            qf[ds] = __builtin_bit_cast(v8h, packed);
        }
        float m2[2] = {MASKED, MASKED};
        v8h kf[AHEAD + 1][2][DS];
        auto fetch_k = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int ds = 0; ds < DS; ++ds)
                    kf[g % (AHEAD + 1)][t][ds] = *reinterpret_cast<const v8h *>(sK + (kat ^ (ds * 64)) + (g * 32 + 4 * t) * ROWB);
        };
        auto scores = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                sc[g][t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) sc[g][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[g % (AHEAD + 1)][t][ds], qf[ds], sc[g][t], 0, 0, 0);
            }
        };
        auto maximum = [&](int g) __attribute__((always_inline)) {
            if ((!FULL || g >= NG - 2) && g * 32 + 32 > seq) {  // (uniform) keys that do not exist
                int keys = seq - g * 32 - 8 * lg;
                asm volatile("" : "+v"(keys));  // the comparisons stay here (masks carried through the loop spill)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sc[g][t][e] = (4 * t + e < keys) ? sc[g][t][e] : MASKED;
            }
            // (median with infinity: a maximum that does not quiet its operand with a second instruction first)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) m2[t] = __builtin_amdgcn_fmed3f(m2[t], sc[g][t][e], __builtin_inff());
        };
        if constexpr (AHEAD == 0) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (exists(g)) {
                    fetch_k(g);
                    scores(g);
                    maximum(g);
                }
                // (else the fragments of all groups are fetched at once: spills)
                if (NG == 8 || (NG < 8 ? g & 1 : (g & 3) == 3)) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            fetch_k(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g + 1 < NG) fetch_k(g + 1);
                scores(g);
                if (g > 0) maximum(g - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            maximum(NG - 1);
        }
        mx = fmaxf(m2[0], m2[1]);
        mx = lane_pair<16>(mx, MaxF32());
        mx = lane_pair<32>(mx, MaxF32());
        const float shift = -mx * c_exp;
        float d2[2] = {0.0f, 0.0f};
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (exists(g)) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sc[g][t][e] = __builtin_amdgcn_exp2f(__fmaf_rn(sc[g][t][e], c_exp, shift));
                        d2[t] += sc[g][t][e];
                    }
            }
        den = d2[0] + d2[1];
        den = lane_pair<16>(den, AddF32());
        den = lane_pair<32>(den, AddF32());
    };
    v4f ot[2 * DS];  // element e of part dt is head dimension 32 (dt / 2) + 8 lg + 4 (dt % 2) + e
    auto values = [&](auto fullc, float inv) __attribute__((always_inline)) {
        constexpr bool FULL = fullc.value;
        constexpr int AHEAD = held_fetch_ahead(FULL, NG);
        v8h vf[AHEAD + 1][2 * DS], pf[2];
        auto fetch_v = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int dt = 0; dt < 2 * DS; ++dt)
                vf[g % (AHEAD + 1)][dt] = *reinterpret_cast<const v8h *>(sVt + (vat ^ ((g & 3) * 64)) + (g >> 2) * 256 +
                                                                        ((dt / 2) * 32 + 4 * (dt % 2)) * VROW);
        };
        auto narrow = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[g % 2][e] = (_Float16)(sc[g][e >> 2][e & 3] * inv);
        };
        auto products = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int dt = 0; dt < 2 * DS; ++dt) ot[dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[g % (AHEAD + 1)][dt], pf[g % 2], ot[dt], 0, 0, 0);
        };
        if constexpr (AHEAD == 0) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (FULL || g * 32 < seq) {
                    fetch_v(g);
                    narrow(g);
                    products(g);
                }
                if (NG == 8 || (g & 1)) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            fetch_v(0);
            narrow(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g + 1 < NG) fetch_v(g + 1);
                products(g);
                if (g + 1 < NG) narrow(g + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    for (int q_base = first; q_base < last; q_base += 128) {
        const int q = q_base + qrow;
        if (q_base + wave * 16 >= seq) return;  // (uniform) no queries for this wave, here or further on; no barrier follows
        float mx, den;
        if (full) softmax(std::true_type(), mx, den);
        else softmax(std::false_type(), mx, den);
        const float inv = 1.0f / den;
#pragma unroll
        for (int dt = 0; dt < 2 * DS; ++dt) ot[dt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        if (full) values(std::true_type(), inv);
        else values(std::false_type(), inv);
        if (q_base + 128 < last) fetch_q(q + 128);
        if (q < seq) {
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                const int d0 = s * 32 + 8 * lg;
                float o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = ot[2 * s + (e >> 2)][e & 3];
                if (d0 < dk) attention_store<VEC>(p, row0 + q, head, d0, o);
            }
            if (lg == 0 && head == p.heads - 1) attention_pad_codes(p, row0 + q);
        }
    }
}

template <int DKP, int VEC, int NG>
static int launch_held(const AttentionParams *p, hipStream_t st)
{
    using Cfg = AttentionHeldCfg<DKP, NG>;
    const auto kernel = attention_held_kernel<DKP, VEC, NG>;
    static PerDeviceOnce once;
    int64_t resident = 0;
    const int rc = resident_workgroups(once, kernel, Cfg::THREADS, Cfg::LDS_BYTES, 1 << 20, &resident);
    if (rc != MKQ_OK || !p) return rc;
    const int64_t sequence_heads = (int64_t)p->batch * p->heads;
    const int per_wg = attention_held_blocks(sequence_heads, p->q_blocks, resident);
    const int first_half = p->cu_seqlens ? attention_held_first_half(sequence_heads, p->q_blocks, per_wg) : 0;
    const int parts = first_half ? 2 : (int)ceil_div(p->q_blocks, per_wg);
    const unsigned grid = (unsigned)(sequence_heads * parts);
    kernel<<<grid, Cfg::THREADS, Cfg::LDS_BYTES, st>>>(*p, per_wg, parts, first_half, attention_runs(sequence_heads, p->heads));
    return launch_status();
}

// p null: setup only
template <int DKP, int VEC>
static int dispatch_held(const AttentionParams *p, int ng, hipStream_t st)
{
    switch (ng) {
    case 2: return launch_held<DKP, VEC, 2>(p, st);
    case 4: return launch_held<DKP, VEC, 4>(p, st);
    case 6: return launch_held<DKP, VEC, 6>(p, st);
    case 8: return launch_held<DKP, VEC, 8>(p, st);
    case 10: return launch_held<DKP, VEC, 10>(p, st);
    case 12: return launch_held<DKP, VEC, 12>(p, st);
    case 14: return launch_held<DKP, VEC, 14>(p, st);
    default: return launch_held<DKP, VEC, 16>(p, st);
    }
}

int run_attention_held(const AttentionParams &p, hipStream_t st)
{
    const int ng = 2 * (int)ceil_div(p.seq, 64);
    if (p.dk > 32) return dispatch_held<64, 8>(&p, ng, st);
    return (p.dk % 8) == 0 ? dispatch_held<32, 8>(&p, ng, st) : dispatch_held<32, 2>(&p, ng, st);
}

int setup_attention()
{
    for (int ng = 2; ng <= 16; ng += 2) {
        int rc = dispatch_held<32, 8>(nullptr, ng, nullptr);
        if (rc == MKQ_OK) rc = dispatch_held<64, 8>(nullptr, ng, nullptr);
        if (rc == MKQ_OK) rc = dispatch_held<32, 2>(nullptr, ng, nullptr);
        if (rc != MKQ_OK) return rc;
    }
    return MKQ_OK;
}

}  // namespace mkq
