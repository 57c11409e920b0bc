// Rules of launches in plain arithmetic, without HIP, so that they can be checked on any machine.
#pragma once

#include <cstdint>

namespace mkq {

// Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  A kernel that takes its share of the tokens
// by xcd_index(blockIdx.x, gridDim.x) gives XCD x the x-th eighth of them, so it finds in its L2 what the kernel before,
// with the same rule, wrote there.  What another XCD wrote has to come through memory first: 16 MiB just written are read
// in 2 us by the XCDs that wrote them and in 9 by their neighbours.  (Which XCD a workgroup runs on decides only the time.)
constexpr int XCDS = 8;
constexpr int xcd_index(unsigned wg, unsigned total)
{
    const unsigned q = total / XCDS, r = total % XCDS, x = wg % XCDS;
    return (int)(x * q + (x < r ? x : r) + wg / XCDS);
}

// Where the shares are not alike (sequences of different lengths), an eighth of them in one piece can be most of the work:
// runs of neighbours go to one XCD after the other instead, and what is left of whole rounds one by one.
struct XcdRuns {
    unsigned length, whole;  // of a run; in whole rounds of eight runs
};
constexpr int xcd_run_index(unsigned wg, const XcdRuns &r)
{
    if (wg >= r.whole) return (int)wg;
    const unsigned x = wg % XCDS, j = wg / XCDS, k = j / r.length;
    return (int)((k * XCDS + x) * r.length + (j - k * r.length));
}
// Sequences times heads of a padding-free batch.  The heads of a sequence share lines of q, k, v and of the codes that are written,
// so up to a sequence's heads make a run, as long as there are eight runs for every XCD.  us in a graph, 12 heads, an eighth in
// one piece / one head at a time / these runs: 64 sequences, heads of 26, lengths rising from 8 to 128 9.9 / 9.7 / 8.9, all of 128
// 10.4 / 14.9 / 10.5; 32 sequences, heads of 64, rising from 16 to 256 21.1 / 16.8 / 17.0, falling 21.3 / 15.9 / 15.7.
// What it costs is near-equal lengths, where one piece is even and what the kernel before wrote is near: layers of the student
// on 32 sequences of about 60 tokens 78.7 -> 79.8, of 440 tokens 39.8 -> 40.0.  (One piece where the eighths have about as many
// tokens, decided from the offsets in the kernels, cost each launch 0.25 us and more.)
constexpr XcdRuns attention_runs(int64_t sequence_heads, int64_t heads)
{
    int64_t length = sequence_heads / (8 * XCDS);
    length = length < 1 ? 1 : length < heads ? length : heads;
    return {(unsigned)length, (unsigned)(sequence_heads / (length * XCDS) * (length * XCDS))};
}

// Work-items of a launch in one dimension: a product of grid and workgroup size that HIP takes
constexpr int64_t MAX_WORK_ITEMS = 0xFFFFFFFFLL;

// Which kernel an attention call takes.
enum AttentionRoute {
    ATTENTION_ONE_BLOCK,  // attention_kernel: all keys of a head at once, probabilities in registers
    ATTENTION_HELD,       // attention_held_kernel: scores of up to ATTENTION_HELD_KEYS keys held in registers
    ATTENTION_BLOCKS,     // attention_blocks_kernel: blocks of 128 keys, twice
};
constexpr int ATTENTION_HELD_KEYS = 512;
constexpr int ATTENTION_HELD_THREADS = 512;  // of a workgroup

// Up to 512 keys are held in registers between softmax and product with V; heads of 64 and up to 128 keys keep the one-block
// kernel, which fits more workgroups on a CU (64 x 128 tokens, 12 heads 13.0 us, held 14.6; 64 x 32 4.7, 7.4; with few
// workgroups held is ahead by 2 to 8 % of 6 us).  The kernel that goes over the keys twice is left with longer sequences,
// heads of 34 to 62 that are no multiple of 8, sequences whose rows of qkv (6 hidden bytes each) reach over 4 GiB, within
// which the held kernel's 32-bit offsets stay, and more heads than one workgroup of the held kernel each can be launched for
// (the other's are half as large).
constexpr AttentionRoute attention_route(int64_t batch, int64_t seq, int64_t hidden, int64_t heads, int64_t q_pitch)
{
    const int64_t dk = hidden / heads;
    if (dk == 64 && seq <= 128 && q_pitch == hidden) return ATTENTION_ONE_BLOCK;
    const bool held = seq <= ATTENTION_HELD_KEYS && (dk <= 32 || dk % 8 == 0) && seq * hidden * 6 <= 0xFFFFFFFFLL &&
                      batch * heads <= MAX_WORK_ITEMS / ATTENTION_HELD_THREADS;
    return held ? ATTENTION_HELD : ATTENTION_BLOCKS;
}

// Blocks of 128 queries per workgroup of the held kernel: more share one staging of the keys (about as long as half a block),
// fewer fill the last round of workgroups better.  sequence_heads: pairs of sequence and head (attention_route bounds them, so
// that one workgroup for each can be launched); resident: workgroups that the device runs at a time.
constexpr int attention_held_blocks(int64_t sequence_heads, int q_blocks, int64_t resident)
{
    int per_wg = q_blocks;
    int64_t best = -1;
    for (int c = 1; c <= q_blocks; ++c) {
        const int64_t wgs = sequence_heads * ((q_blocks + c - 1) / c);
        const int64_t cost = (wgs + resident - 1) / resident * (1 + 2 * c);
        if (wgs <= MAX_WORK_ITEMS / ATTENTION_HELD_THREADS && (best < 0 || cost < best)) { best = cost; per_wg = c; }
    }
    return per_wg;
}

// Padding-free batches: where attention_held_blocks lets one workgroup take a whole sequence, the longest ones (as many blocks
// as the bound on the lengths has) are shared by two if they are few, because the kernel would end with them.  Blocks of the first
// of the two; 0: never shared.  Whether they are few, the kernel sees from the lengths.
constexpr int attention_held_first_half(int64_t sequence_heads, int q_blocks, int per_wg)
{
    return q_blocks >= 2 && per_wg == q_blocks && 2 * sequence_heads <= MAX_WORK_ITEMS / ATTENTION_HELD_THREADS ? (q_blocks + 1) / 2 : 0;
}

// Groups of 32 keys by which the held kernel fetches fragments ahead of their products: with two waves on a SIMD the LDS answers too late
// otherwise (16 x 512 tokens, 16 heads of 64, 41.2 -> 38.2 us), with four the registers spill (32 x 256 27.8 -> 39.0).  Two groups
// gain nothing over one up to 384 keys and spill at 512.  Sequences with groups that do not exist take theirs one at a time, fetch,
// products and maximum under one condition: ahead, they would fetch the missing ones as well (20 sequences of 1500 tokens in all, at most 384,
// 16 heads of 16 8.7 -> 7.55, 12 x 288 of 2000 tokens, 12 heads of 26 10.8 -> 8.7).
constexpr int held_fetch_ahead(bool full, int groups) { return full && groups > 8 ? 1 : 0; }

// 4-bit layers of small hidden size (rows of codes, padding included, of up to 384) run in two launches and a quantizer instead of seven:
// their kernels take 4 to 12 us each, most of it the launch and one trip to memory.  us a layer, 4-bit, hidden size 312 with heads of 26,
// kernels of their own -> q, k, v with the attention -> what follows it in one launch as well:
//   1024 tokens 39.1 -> 35.2 -> 28.4, 4096 50.0 -> 45.6 -> 34.5, padding-free 2298 46.0 -> 45.0 -> 37.8; hidden 384, 4096 tokens
//   49.5 -> 45.3 -> 36.6; with fewer tokens only the first step is taken (small_layer_tail): 256 37.5 -> 34.1, padding-free 440 38.3 -> 34.2.
//   In a graph, where launches cost less, and with the few-token kernels for what is left to them: 256 32.7 -> 25.9, 440 31.6 -> 25.8,
//   1024 31.8 -> 29.5, 2298 44.3 -> 37.2, 4096 46.3 -> 34.9.
constexpr int64_t SMALL_LAYER_ROW = 384;
// q, k, v and the attention: any number of tokens (16384 of hidden size 312 109 -> 100, 65536 335 -> 292); one workgroup of 256 threads per
// (sequence, head) has to fit a launch.
constexpr bool small_layer_attention(int64_t batch, int64_t seq, int64_t hidden, int64_t heads, int64_t row)
{
    return row <= SMALL_LAYER_ROW && row % 128 == 0 && seq <= 128 && hidden / heads <= 32 && batch * heads <= MAX_WORK_ITEMS / 256;
}
// What a layer takes: that, where the attention would take the held kernel, whose sums it has in the same order (more heads than that
// one can be launched for sum otherwise), and where it is the faster one.  A head takes the room of 32 in its products and a sequence that
// of 32, 64 or 128 tokens, so what one launch saves is used up by that many workgroups' waste: sooner for small heads, and in padding-free
// batches, whose short sequences share one bound.  us a layer, kernels of their own / this:
//   hidden size 256, heads of 8: 16 x 128 tokens (512 workgroups) 25.6 / 24.1, 32 x 128 (1024) 31.8 / 32.7, 64 x 64 (2048) 31.7 / 33.8;
//     of 4, 200 sequences of at most 128, 12000 tokens in all (12800) 151.6 / 191.4
//   384, heads of 16: 32 x 128 (768) 43.7 / 42.6, 64 x 128 (1536) 74.4 / 75.0, 128 sequences of 4097 (3072) 67.6 / 74.1
//   312, heads of 26: 128 x 128 (1536) 104.8 / 100.0, 200 sequences of 12000 (2400) 97.1 / 99.9
constexpr bool small_layer_attention_choice(int64_t batch, int64_t seq, int64_t hidden, int64_t heads, int64_t row, bool padding_free)
{
    if (!small_layer_attention(batch, seq, hidden, heads, row) || attention_route(batch, seq, hidden, heads, row) != ATTENTION_HELD) return false;
    const int64_t tiles = seq <= 32 ? 1 : seq <= 64 ? 2 : 4, work = batch * heads * tiles, dk = hidden / heads;
    if (dk < 16) return work <= 2048;
    return work <= 4096 || (!padding_free && dk >= (tiles == 1 ? 24 : 26));
}
// The rest: one round of workgroups of 16 tokens on 256 CUs, each of which reads all weights and goes through the FFN's columns one chunk
// after the other (columns of a chunk, and what whole chunks of the better of the two sizes add up to).  In a second round the kernels of
// their own win, which read the weights once per 64 or 128 tokens: hidden size 384, 8192 tokens 63.5 -> 61.6, 16384 of 312 100 -> 105, 32768
// 163 -> 201.
constexpr int64_t LAYER_TAIL_WIDE = 1280, LAYER_TAIL_NARROW = 768;
constexpr int64_t layer_tail_columns(int64_t ffn, int64_t chunk) { return (ffn + chunk - 1) / chunk * chunk; }
// Its time is that of its columns at any token count, the others' grows with the tokens and, up to 1024 of them, hardly with the columns, so
// the line rises: 768 columns always, beyond 600 more than there are tokens, and 3840 at most.  us a layer from call to call, where seven
// launches cost the host about 25, kernels of their own / this, hidden size 312, heads of 26 (440: padding-free; 4096: in a graph):
//   tokens        16          128         440         1024        1536        2048        4096
//    768 columns  26.3 21.3   27.0 24.7   27.3 25.0   27.9 25.5   31.4 26.5   33.5 26.4   39.9 31.2
//   1280          25.0 25.0   27.2 28.5   28.2 28.7   30.6 29.0   32.2 30.0   35.3 30.1   44.6 35.1
//   1536          24.3 26.5   27.3 29.9   28.7 30.3   31.0 30.7   33.7 31.8   35.3 32.1   45.2 36.3
//   2304          23.7 31.5   28.2 35.4   29.2 36.0   33.7 36.8   35.2 37.7   40.3 38.2   50.1 41.2
//   3072          24.6 38.2   28.8 41.9   30.8 42.9   33.5 43.3   37.7 43.9   40.6 44.1   52.7 48.3
// (384 alike.  In a graph their own kernels cost less: 1280 columns 25.8 28.2 at 128 tokens, 28.8 29.5 at 1024, 30.1 30.4 at 1536;
// 3840 columns 49.2 51.3 at 3072, 57.2 53.1 at 3584.)
constexpr bool small_layer_tail(int64_t tokens, int64_t row, int64_t ffn_row)
{
    if (row > SMALL_LAYER_ROW || row % 128 != 0 || ffn_row % 128 != 0 || ffn_row > 3840 || tokens > 4096) return false;
    const int64_t wide = layer_tail_columns(ffn_row, LAYER_TAIL_WIDE), narrow = layer_tail_columns(ffn_row, LAYER_TAIL_NARROW);
    const int64_t columns = wide < narrow ? wide : narrow;
    return columns <= LAYER_TAIL_NARROW || columns <= tokens + 600;
}

// LayerNorm with one row per half wave (the kernels have 256 threads: eight rows), not per wave (four).  Up to D = 1024: where
// half waves leave fewer lanes idle (chunks of 8 values: up to 32, or 65 to 96, of which whole waves would use half
// and three quarters) and there are rows enough to fill the chip with them; a tie goes to whole waves, which have half the
// work per lane.  us in a graph, half -> whole waves: 2299 x 1024 4.31 -> 3.82, with codes 5.15 -> 4.52, 16384 x 1024 12.7 -> 11.9,
// with codes 14.8 -> 13.8, 2048 x 312 2.75 -> 2.56, 4099 x 512 3.46 -> 3.42; but 8192 x 768 5.93 -> 6.52, with codes 7.28 -> 8.09.
// And for more rows than can be launched four to a workgroup.
constexpr bool layernorm_half_waves(int64_t M, int64_t D)
{
    return D <= 1024 && M >= 2048 && (D <= 256 || (D > 512 && D <= 768) || (M + 3) / 4 > MAX_WORK_ITEMS / 256);
}

// 4-bit layers of medium hidden size: attention output and LayerNorm in one launch, 16 tokens and all columns to a workgroup, where these
// are one round on 256 CUs and LayerNorm alone would have its rows to half waves as well, so that its sums run in the same order.  us a
// layer of hidden size 768, before -> this: 2048 tokens 56.9 -> 56.1, 2298 66.5 -> 65.7, 3072 76.1 -> 73.6, two of 4096 162.2 -> 158.8;
// below, every workgroup's read of all weights costs more than the launch (1024 tokens 46.2 -> 46.9, 440 36.8 -> 38.3).  The FFN's second
// linear the same way: 16 tokens for each widening of four times the weights, 4096 tokens +1.3, 2048 +5.4.
constexpr bool output_norm(int64_t tokens, int64_t hidden, int64_t row)
{
    return row > 512 && row <= 768 && row % 128 == 0 && tokens <= 4096 && layernorm_half_waves(tokens, hidden);
}

// The kernels of few tokens and small linears (gemm_few.hip): tiles of channels x tokens; _LONG: waves take 128 bytes of a row at a
// time, not 64 (rows of 2048 bytes and more: M = 128, K = N = 4096 6.4 -> 5.8; at 1536 bytes M = 440, N = 768 5.1 -> 5.4).
enum FewTile { FEW_NONE = -1, FEW_16x16, FEW_16x32, FEW_32x32, FEW_32x64, FEW_64x64,
               FEW_16x16_LONG, FEW_16x32_LONG, FEW_32x32_LONG, FEW_32x64_LONG, FEW_64x64_LONG };
constexpr int64_t few_workgroups(int64_t M, int64_t N, int channels, int tokens)
{
    return ((N + channels - 1) / channels) * ((M + tokens - 1) / tokens);
}
// LDS of a workgroup: 16, 24, 32, 64 and 128 KiB for the five tiles, 32, 48, 64, 96 and 128 with the long pieces.
// Up to 16 tokens the smallest tile, up to 32 it or 32x32, however many workgroups there are: more tokens to a tile would only be
// padding.  Beyond, the smallest tile whose workgroups are about one round, because a second costs as much as the first: one per CU, or
// two (32x32 and 32x64 of rows below 1024 bytes; more than two of 32x32 fit and gain nothing).  Past that the persistent kernels take
// over (FEW_NONE), but for up to 64 tokens with rows of 2048 bytes and more, whose 64x64 tiles have any number.  us, 4 bits, binary16 out:
// K = N = 768, M = 640 (480 / 240 workgroups) 32x32 3.4, 32x64 3.6; M = 1024 (768 / 384 / 192) 4.5, 4.4, 64x64 4.6, the persistent 64x64
// 5.1; N = 2304, M = 440 (504 of 32x64) 4.6, persistent 4.8, M = 640 (720) 6.4, 5.7; K = 3072, N = 768, M = 1024 (384 / 192) 32x64 7.7,
// 64x64 6.7, persistent 7.7; K = N = 4096, M = 256 (256 of 64x64) 7.8, persistent 10.8, M = 440 (448) 13.8, 13.4.  8-bit operands need no
// widening, and the persistent kernels win earlier: K = 768, N = 3072, M = 320 (480 of 32x64) 5.5, persistent 5.0; K = 3072, N = 768,
// M = 1024 (192 of 64x64) 8.3, 7.6; in one round of 32x64 5.7 against 7.6 (M = 440).
constexpr FewTile few_tile(int64_t M, int64_t N, int64_t row_bytes, int bits)
{
    if (row_bytes % 64 != 0) return FEW_NONE;
    const bool deep = row_bytes >= 2048 && row_bytes % 128 == 0;
    auto kind = [&](FewTile t) { return deep ? (FewTile)(t + FEW_16x16_LONG) : t; };
    if (few_workgroups(M, N, 16, 16) > MAX_WORK_ITEMS / 512) return FEW_NONE;  // (of 512 threads)
    if (M <= 16) return kind(FEW_16x16);
    if (M <= 32) return kind(few_workgroups(M, N, 16, 32) <= (deep ? 256 : 512) ? FEW_16x32 : FEW_32x32);
    const int64_t two = row_bytes < 1024 ? 512 : 256;  // workgroups: two per CU where they are short
    if (few_workgroups(M, N, 32, 32) <= two) return kind(FEW_32x32);
    if (few_workgroups(M, N, 32, 64) <= (bits == 8 ? 256 : two)) return kind(FEW_32x64);
    // (M = 64, K = 768, N = 30522 14.8, persistent 11.9; K = 4096, N = 12288 16.7 -> 8.9)
    return (bits == 4 && few_workgroups(M, N, 64, 64) <= 256) || (M <= 64 && deep) ? kind(FEW_64x64) : FEW_NONE;
}
// What a call takes: that, but for shapes where it leaves waves idle and the persistent kernels are ahead.
constexpr FewTile few_choice(int64_t M, int64_t N, int64_t row_bytes, int bits)
{
    const FewTile t = few_tile(M, N, row_bytes, bits);
    // One or two pieces leave most waves without one, and a second 32x64 workgroup per CU is no gain any more (4 bits, K = 128, N = 936,
    // M = 1048, 510 workgroups 4.9, persistent 4.2; K = 256, N = 768, M = 1019 4.45, 4.2; but 59 tokens, N = 12288 4.4, 7.1)
    if (t == FEW_32x64 && (row_bytes == 64 || (row_bytes == 128 && M > 64)) && few_workgroups(M, N, 32, 64) > 256) return FEW_NONE;
    // Pieces of 64 bytes that are not the same number for all waves cost a round of them: K = 2304 (18 pieces), N = 936, M = 1032 (255
    // workgroups) 8.2, persistent 7.9, up to 208 of them 0.94 to 1.0 of its time; where that one's wave groups share K evenly it is ahead
    // sooner (K = 2560, N = 4096, M = 228, 256 workgroups 7.9, 7.45; up to 144 0.96 to 1.0).
    if (t == FEW_64x64 && row_bytes % 512 != 0 && few_workgroups(M, N, 64, 64) > (row_bytes % 256 == 0 ? 144 : 208)) return FEW_NONE;
    return t;
}
// Tiles of three parts, one per CU in one round: when an 8-bit linear takes 128x96 and 256x192.
constexpr int64_t tiles_of(int64_t M, int64_t N, int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
// 128x96: more than two 64x64 tiles per CU and a long k loop, with GELU, which nothing covers, a longer one (us, 43 -> 51: K = 1536, N = 256,
// M = 8653 with GELU 11.2 -> 11.75, N = 1024, M = 2372 11.9 -> 11.8, without 11.0 -> 9.8; K = 2048, N = 768, M = 3815 with GELU 14.6 -> 14.1).
constexpr bool i8_128x96(int64_t M, int64_t N, int64_t K, bool gelu)
{
    return K >= (gelu ? 2048 : 1536) && tiles_of(M, N, 64, 64) > 512 && tiles_of(M, N, 128, 96) <= 256;
}
// 256x192: where 128x128 tiles come in two rounds of two per CU, for GELU, residuals and long k loops.  At short k the epilogue is the tile and
// three 128x128 ones per CU share it out (us, 29 -> 52: K = 128, N = 768, M = 10942 with a residual 10.3 -> 11.35, with GELU 13.2 -> 14.5;
// K = 256, N = 6144, M = 1759 14.1 -> 15.3; K = 384, N = 1920, M = 6365 with GELU 18.0 -> 16.9, with a residual 16.8 -> 16.9; K = 512, N = 2304,
// M = 3615 15.1 -> 14.65), longer where a residual's rows end inside a line (K = 512, N = 936, M = 11546 17.4 -> 20.25; K = 1024, M = 8557
// 20.9 -> 20.5).
constexpr bool i8_256x192(int64_t M, int64_t N, int64_t K, bool gelu, bool residual)
{
    const bool takes = K >= 1536 || (gelu && K >= 384) || (residual && K >= (N % 64 != 0 ? 1024 : 512));
    return takes && tiles_of(M, N, 128, 128) > 512 && tiles_of(M, N, 256, 192) <= 256;
}
// The same of a binary16 linear.  128x96: as above, at any k but with a longer epilogue (us, before -> 128x96: K = 128, N = 512, M = 5204 with
// GELU 6.85 -> 7.25, K = 512, N = 936, M = 2223 with GELU 9.0 -> 9.3; K = 256, N = 936, M = 2593 with a residual 7.4 -> 7.65; K = 768 with GELU
// 4 % in its favour).
constexpr bool f16_128x96(int64_t M, int64_t N, int64_t K, bool gelu, bool residual)
{
    return K >= (gelu ? 640 : residual ? 384 : 0) && tiles_of(M, N, 64, 64) > 512 && tiles_of(M, N, 128, 96) <= 256;
}
// 256x192: not for a short k loop and a residual whose rows end inside a line (K = 384, N = 936, M = 11647 21.6 -> 23.4, K = 512, M = 11461
// 24.3 -> 25.4; K = 768, M = 11428 31.0 -> 29.6).  Otherwise the tile whose rounds add up to the least (choose_f16).
constexpr bool f16_256x192_suits(int64_t N, int64_t K, bool residual) { return !(residual && N % 64 != 0 && K < 768); }

// Which tiles an XCD has: by tokens, an eighth of them with all channels, where what kernels around the linear left of its activations
// in an L2 is worth more than weights that each XCD reads (M > N, or half of that if they are small beside it: 8-bit K = 5120, N = 768,
// M = 444 would take 9.3 instead of 7.3); or by channels, an eighth with all tokens.  Workgroups dealt one by one do the latter by
// themselves if the channel tiles are a multiple of 8; if not, every XCD reads everything, which costs as soon as that is more than its
// L2.  us, dealt one by one -> this: layers of hidden size 512 and 1024 tokens 36.5 -> 31.8, of 1536 44.0 -> 39.0, 8-bit ones of 256 and
// 2048 tokens 36.5 -> 29.7; 8-bit K = 4096, N = 64, M = 7379 12.9 -> 10.1, 4-bit K = 8192, N = 576, M = 1679 15.9 -> 13.2.  Finding the
// tile is 0.05 us of a launch (1 to 2 % of the smallest), so it is left out where it gives nothing.
struct FewOrder {
    unsigned inner, magic;  // tiles along the dimension that is gone through first, 0: the grid has both; i / inner = i * magic >> 20
    bool by_tokens;
};
constexpr FewOrder few_order(int64_t M, int64_t N, int64_t row_bytes, int channels, int tokens)
{
    const int64_t ct = (N + channels - 1) / channels, tt = (M + tokens - 1) / tokens;
    const bool by_tokens = M > N || (2 * M > N && N * row_bytes <= (3 << 19));
    const bool worth_it = by_tokens ? M * row_bytes >= (1 << 16) : tt > 2 && ct % XCDS != 0 && (M + N) * row_bytes > (4 << 20);
    if (tt == 1 || !worth_it) return {0, 0, false};
    const int64_t inner = by_tokens ? ct : tt;
    return {(unsigned)inner, ct * tt <= 512 ? (unsigned)(((1 << 20) + inner - 1) / inner) : 0, by_tokens};
}
struct FewPlace { int channels, tokens; };
constexpr FewPlace few_place(unsigned wg, unsigned total, const FewOrder &o)
{
    const unsigned i = (unsigned)xcd_index(wg, total), outer = o.magic ? i * o.magic >> 20 : i / o.inner, in = i - outer * o.inner;
    return o.by_tokens ? FewPlace{(int)in, (int)outer} : FewPlace{(int)outer, (int)in};
}
// where the kernels were asked for by number
constexpr FewTile few_tile_or_largest(int64_t M, int64_t N, int64_t row_bytes, int bits)
{
    const FewTile t = few_tile(M, N, row_bytes, bits);
    return t == FEW_NONE && row_bytes % 64 == 0 ? FEW_64x64 : t;
}

}  // namespace mkq
