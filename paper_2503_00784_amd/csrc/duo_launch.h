// Launch rules and index maps: plain arithmetic from sizes to launch shapes and places, without a word of HIP but for the qualifiers of what a
// kernel calls too, so that a program without a GPU can evaluate them.
#pragma once
#include <math.h>

#include <algorithm>

#include "../../include/duo_verify.h"

// Workgroups go to the eight dies in turn, each with an L2 of its own.  This turns workgroup b of n into a place such that every die gets a
// contiguous range of places: neighbours that write parts of the same 128-byte lines (channels of a query row, columns of the residual
// stream, partial sums of squares) then do so through one L2 instead of through eight.  Only speed depends on it.
// us, before and after: LM head of 33 rows x 32000 53.5 -> 49.5, x 128256 200 -> 191; O projection of 8 rows 9.0 -> 8.7; the whole 7B step of
// 8 rows 2829 -> 2806.  Not for the block kernel of prompt chunks (Q/K/V of 1024 rows 165 -> 175).
__host__ __device__ __forceinline__ int die_contiguous(int b, int n) {
    const int die = b & 7, q = n >> 3, r = n & 7;
    return die * q + (die < r ? die : r) + (b >> 3);
}

// Where the lo halves of a paired operand's rows lie (hi halves: row m).  Up to eight rows share one 16-row tile with their lo halves.
// Beyond that hi and lo halves occupy whole tiles, lo tile = hi tile + M/16 rounded up, so that a lane's hi and lo sums have the same position
// in their tiles; but where the last tile of a verify pass has one to eight rows it holds their lo halves too, eight rows further on (17, 33,
// 65 rows, a previously emitted token in front of the drafts: 3, 5, 9 tiles instead of 4, 6, 10).  What bounds the projections at
// 16..80 rows is the bytes that a compute unit takes in, weights and operand alike.
struct LoRows {
    int split, base;  // rows below split: base rows further on, the others eight
    __host__ __device__ __forceinline__ int operator()(int m) const { return m < split ? m + base : m + 8; }
};

// Rows of the A operand for M paired activations, hi and lo halves in whole tiles beyond eight rows: pair_rows each.
inline int pair_rows_for(int M) { return M <= 8 ? 8 : (M + 15) / 16 * 16; }
// The last tile holds its rows' lo halves too (see LoRows): up to sixteen rows the one-band kernels read whole tiles, prompt chunks of more
// than 80 rows are padded to larger blocks anyway.
inline bool half_tail(int M) { return M > 16 && M <= DUO_MAX_ROWS && (M - 1) % 16 < 8; }
inline int a_tiles_for(int M) { return (2 * pair_rows_for(M) + 15) / 16 - (half_tail(M) ? 1 : 0); }
inline LoRows lo_rows_for(int M) {
    const int pr = pair_rows_for(M);
    if (M <= 8) return LoRows{0, 0};
    return half_tail(M) ? LoRows{pr - 16, pr} : LoRows{pr, pr};
}

// Which row of an operand a workgroup prepares.  An operand buffer keeps 16 bytes of eight rows together in a 128-byte line, and workgroups go to
// the eight dies in turn, each with an L2 of its own: with one row after the other every line was written by eight dies, 16 bytes each.  So
// the eight workgroups of eight rows (a unit: the rows times one of several column ranges or heads) are eight places apart, on one die.  us, one
// row after the other against this: set-up of 1024 rows 29.2 -> 18.5, the reduce kernel at 300 / 520 / 900 rows of the 8B shape 11.0 / 17.1 / 14.1 ->
// 8.1 / 11.9 / 10.9, at 64 rows 4.6 -> 4.35, and the whole step of 64 rows 1219 -> 1204 (the end of a kernel writes its lines back).
__host__ __device__ __forceinline__ int unit_of(int b) { return b % 8 + b / 64 * 8; }
__host__ __device__ __forceinline__ int row_of_unit(int b) { return (b >> 3) % 8; }
__host__ __device__ __forceinline__ int unit_blocks(int units) { return (units + 7) / 8 * 64; }

// Rows times 2^parts_log2 column ranges.  A power of two: a division in front of the first load is a tenth of the reduce kernel's time
// where rows are short (3.45 against 3.75 us, 49 rows of 512 channels).
struct RowUnits {
    int M, parts_log2;
    __host__ __device__ __forceinline__ int blocks() const { return unit_blocks((M + 7) / 8 << parts_log2); }
    __host__ __device__ __forceinline__ int row(int b, int& part) const {  // M or more: none
        const int unit = unit_of(b);
        part = unit & ((1 << parts_log2) - 1);
        return (unit >> parts_log2) * 8 + row_of_unit(b);
    }
};

// Rows times heads, for the merge of attention chunks.
struct HeadUnits {
    int M, heads;
    __host__ __device__ __forceinline__ int blocks() const { return unit_blocks((M + 7) / 8 * heads); }
    __host__ __device__ __forceinline__ int row(int b, int& head) const {  // M or more, or heads or more: none
        const int unit = unit_of(b), groups = (M + 7) / 8;
        head = unit / groups;
        return (unit - head * groups) * 8 + row_of_unit(b);
    }
};

// Column ranges per row for residual_reduce_kernel, as a power of two: enough workgroups to fill the chip when there are few rows.
// (520 rows of the 8B shape: 4 ranges 11.9 us, 1 range 13.1; 400: 9.8 / 10.0.)
inline int reduce_parts_log2(int M, int d) {
    int p = M <= 32 ? 3 : 2;
    while (p > 0 && d % (64 << p) != 0) --p;
    return p;
}
// Attention of a prompt chunk: query tiles of attn_shared_kernel's workgroups (a tile per wave of a team) and chunks of keys.  A
// workgroup has a compute unit to itself and takes 6 us and, per ring stage of a block for each team, 1.02 us with two teams of four
// waves, 1.27 with two of five, 1.06 as one team of eight (heads of 128; of 64: 0.68 of it), about the same per tile and block: what
// decides is how evenly the groups of 4, 5 or 8 tiles fill the chip.  The late rows see the most keys and go first, so the launch takes its
// mean load or, where the last workgroups come as an odd few, (rounds + 1) times the length of those.  More than one chunk: the merge, 4 us
// and 1.5 us per million values.  In us with the merge, groups of four tiles
// alone against this choice: 32 heads, 640 rows behind 4000 keys 139 -> 108, behind 16000 420 -> 371; 40 heads, 200 rows behind 8000
// 110 -> 98; 8 heads x 8, 800 rows behind 8000 533 -> 478.  1024 rows behind 1024 keys on 32 heads keep them: 69, against 93 + 14 with two
// tiles per wave.
struct PromptAttention {
    int nwv, ksplit, chunks;
};
inline PromptAttention prompt_attention(int D, int Hkv, int group, int M, int P, int max_chunks) {
    constexpr int CUS = 256;
    static const struct {
        int nwv, ksplit;
        float stage;
    } shapes[] = {{8, 2, 1.02f}, {10, 2, 1.27f}, {8, 1, 1.06f}};
    const int NB = (P + M + 31) / 32, MQ = M * group;
    PromptAttention best{8, 2, 1};
    float best_cost = 1e30f;
    for (const auto& s : shapes) {
        const int rows = s.nwv / s.ksplit * 16, groups = (MQ + rows - 1) / rows;  // query rows of a workgroup, row groups
        const auto blocks_seen = [&](int z) { return std::min(NB, (P + (std::min(MQ, (z + 1) * rows) - 1) / group) / 32 + 1); };
        for (int t = 1; t <= max_chunks; ++t) {
            const int bl = std::max(2, (NB + t - 1) / t), n = (NB + bl - 1) / bl;  // blocks per chunk, chunks
            const float mean_stages = 0.5f * (float)(blocks_seen(0) + blocks_seen(groups - 1)) / (float)s.ksplit;  // all chunks of a row group
            float cost = (float)(Hkv * groups) * (6.f * (float)n + s.stage * mean_stages) / (float)CUS;
            for (int r = 0; r * CUS < Hkv * groups * n; ++r) {  // 256 r workgroups came first: the next one is the longest that is left
                const int seen = std::min(bl, blocks_seen(groups - 1 - r * CUS / (n * Hkv)));
                cost = std::max(cost, (float)(r + 1) * (6.f + s.stage * (float)((seen + s.ksplit - 1) / s.ksplit)));
            }
            if (D == 64) cost *= 0.68f;
            if (n > 1) cost += 4.f + 1.5e-6f * (float)n * (float)MQ * (float)Hkv * (float)D;
            if (cost < best_cost) {
                best_cost = cost;
                best = PromptAttention{s.nwv, s.ksplit, t};
            }
        }
    }
    return best;
}

// Attention of one pass: M rows behind P keys, `group` query heads for each of Hkv kv heads of D channels; `many`: a prompt chunk of more
// rows than a verify pass has.
struct AttnLaunch {
    bool small;                   // attn_small_kernel, otherwise attn_shared_kernel
    int nwv, ksplit, row_groups;  // attn_shared_kernel: consumer waves, teams; row groups (grid z)
    int chunk_blocks, chunks;     // 32-key blocks of a chunk; chunks (more than one: a second kernel merges them)
};

// Whether a short context of three or more query tiles is one chunk.  Against chunks and the merge, which adds about 3 us to a step (4.2 us by
// itself, of which one overlaps with its neighbours: whole layers with the one against the other): the more workgroups one chunk makes, the
// longer the context up to which it wins, and the blocks behind the prefix count less, since the early rows leave them out.  us, one chunk
// against the two kernels less 1 us, heads of 128, at 100 / 200 / 250 keys.  Three and four tiles: 64 rows on 1 head 9.5 / 10.6 / 10.8 against
// 10.2 / 9.4 / 9.7, on 32 9.9 / 10.9 / 11.1 against 11.7 / 11.6 / 11.8; 16 rows of four on 8 heads 9.6 / 11.6 / 12.8 against 9.5 / 9.7 / 9.8.
// More than eight: 64 rows of four on 1 head 10.5 / 12.1 / 12.2 against 9.8 / 9.7 / 9.8 (20 keys 9.4, 9.5), on 8 10.6 / 12.3 / 12.6 against 11.0 /
// 11.6 / 12.1, on 32 11.9 / 13.8 / 14.0 against 15.0 / 16.0 / 16.2.  Five to eight, one team of eight waves, at 60 / 90 keys: 32 rows of four on
// 8 heads 12.2 / 13.0 against 10.3 / 11.1, on 32 12.6 / 13.5 against 11.9 / 12.6, 16 rows of eight on 64 13.3 / 14.3 against 15.8 / 16.3.
// Heads of 64 take two thirds as long and so stay one chunk further: 64 rows of four on 1 head 6.9 at 100 and 8.4 at 200 against 7.2 and 7.3, 16
// rows of four on 8 heads 7.5 at 200 and 8.3 at 250 against 7.5 and 7.6.
inline bool attention_one_chunk(int D, int MqT, int ksplit, int wgs, int M, int P, int NB) {
    const int x = P / 32;  // blocks of the prefix alone
    if (ksplit == 1) return NB <= 5 && (D == 64 || wgs >= 40 || x <= (wgs >= 32 ? 1 : 0));
    if (NB > 10) return false;
    if (D == 64) return wgs >= 16 || NB <= 8;
    if (wgs >= 40) return true;
    if (MqT > 8) return wgs >= 12 && x <= 3;
    return x <= (wgs >= 32 ? 4 + M / 16 : 3);
}

inline AttnLaunch attention_launch(int D, int Hkv, int group, int M, int P, bool many, int max_chunks) {
    const int NB = (P + M + 31) / 32, MqT = (M * group + 15) / 16;  // blocks of keys, query tiles per kv head
    // One query tile per kv head on a short context: one workgroup of eight waves per kv head does the whole head without a loop, at
    // most 32 blocks.  Against chunks and their merge (less the 1 us of it that overlaps), heads of 128, 660 / 800 / 990 keys: 8 heads 10.5 / 11.6 /
    // 14.0 against 8.7 / 8.6 / 9.0 us, 32 10.8 / 11.8 / 14.4 against 9.5 / 9.3 / 10.1, 64 11.3 / 12.3 / 15.1 against 10.9 / 11.7 / 12.7, 96 12.0 /
    // 13.2 / 16.1 against 12.4 / 13.7 / 14.8; from there on the chunks are too few: 128 12.4 / 14.0 / 17.0 against 14.2 / 15.9 / 17.4, 256 17.9 / 20.2 /
    // 24.6 against 18.3 / 21.2 / 24.4 without a merge.  Up to 640 keys the smaller number of blocks per wave decides (400 keys on 32 heads 8.7
    // against 9.6), with heads of 64 all the way (990 keys 8.5 against 9.6).
    if (MqT == 1 && NB <= (D == 64 || Hkv > 96 ? 32 : Hkv > 64 ? 24 : 20)) return {true, 8, 1, 1, NB, 1};
    // Otherwise the kernel that stages K/V blocks in LDS for all query tiles, one query tile per wave.
    // Up to four tiles: two teams of waves share the blocks (two waves per SIMD: 20.7 against 23.2 us at 4 tiles,
    // 11.8 against 14.4 us at 2 tiles, measured on 32 heads x 4160 / 2080 keys).
    // 9..16 tiles (64 rows x a GQA group of 4): 27.3 against 28.2 us at 8192 keys; 17..20 tiles (65..80 rows) in the same shape
    // against two tiles per wave: 33.8 against 43.4 us at 8192 keys, 14.1 against 18.6 at 2048, 10.9 against 13.4 at 700.
    AttnLaunch at{false, MqT > 2 ? 8 : 4, (MqT <= 4 || MqT > 8) ? 2 : 1, 1, 0, 1};
    if (many) {
        const PromptAttention p = prompt_attention(D, Hkv, group, M, P, max_chunks);
        at.nwv = p.nwv;
        at.ksplit = p.ksplit;
        at.chunks = p.chunks;
    } else if (MqT == 5 && NB >= 64) {
        // five tiles (65..80 rows of a head without a group) on a long context: two teams of five against eight waves of which
        // five have a tile, 25.9 -> 22.3 us on 32 heads x 4161 keys, 17.9 -> 17.3 at 2127 (at 577 keys 9.1 -> 10.3: not there)
        at.nwv = 10;
        at.ksplit = 2;
    }
    bool few_heads = false;
    const int tiles = at.nwv / at.ksplit;
    at.row_groups = (MqT + tiles - 1) / tiles;
    if (!many) {
        // LDS (teams) or registers (nine waves) leave room for one workgroup per compute unit, so no more than 256 of them: measured best
        // for 4 tiles x 32 heads and 16 tiles x 8 heads (40 heads x 1032 keys: 240 against 280 workgroups 8.4 against 13.4 us).
        const int wgs = Hkv * at.row_groups;
        at.chunks = std::min(std::max(256 / wgs, 1), max_chunks);
        // On few heads a chunk more costs the merge what it saves the kernel: no more than about 1.5 sqrt(blocks).  Steps in us, as
        // many chunks as there are compute units (at most 64) against this.  Two kv heads of four, three layers, behind 4000 keys: 8 rows 122.2 ->
        // 112.2, 32 rows 147.1 -> 139.3, 64 rows 169.1 -> 162.5; behind 2000: 112.4 -> 108.4, 133.0 -> 131.2, 161.4 -> 158.3.  Twelve heads of 64, two
        // layers, behind 2000 / 6000 keys: 8 rows 103.5 -> 100.2, 106.3 -> 105.3.  Eight kv heads of 128 of four, two layers, behind 2000 / 6000
        // keys: 1 row 377.1 -> 375.5, 382.4 -> 379.5, 8 rows 403.4 -> 398.5, 407.4 -> 403.8.  One team (five to eight tiles) takes twice as long for a block:
        // 2 sqrt(blocks) and at least 16, 24 rows of those eight heads behind 1400 keys 442.0 -> 442.3 with 13, 445.3 with 10.  At least 12 for two teams: a
        // stage each up to 24 blocks (the kernel alone, 16 rows of two kv heads of four behind 700 keys, 5.3 us in 12 chunks, 6.3 in 6).
        const float root = sqrtf((float)NB);
        const int most = at.ksplit == 1 ? std::max(16, (int)(2.f * root)) : std::max(12, (int)(1.5f * root));
        few_heads = most < at.chunks;
        if (few_heads) at.chunks = most;
        // Two tiles on up to 512 keys, us, one chunk against chunks and merge, 32 heads of 128: 250 / 400 / 700 keys 9.0 / 9.6 / 13.4 against 9.9 /
        // 10.4 / 10.7.
        if (MqT == 2 ? NB <= 16 : MqT > 2 && attention_one_chunk(D, MqT, at.ksplit, wgs, M, P, NB)) at.chunks = 1;
    }
    at.chunk_blocks = std::max(2, (NB + at.chunks - 1) / at.chunks);
    // two teams take two blocks at a time: an odd one more costs them nothing and may save a chunk
    if (few_heads && at.ksplit == 2 && at.chunks > 1) at.chunk_blocks = (at.chunk_blocks + 1) / 2 * 2;
    at.chunks = (NB + at.chunk_blocks - 1) / at.chunk_blocks;
    return at;
}

// Whether the merge of attention chunks puts eight rows of a head into eight workgroups of a wave each or into one of eight waves.  Where the rows
// are few, one compute unit per wave: steps of 12 / 24 / 32 rows of three layers of two kv heads of four behind 6000 keys (64 chunks) 128.8 /
// 151.3 / 156.0 us with eight waves, 123.3 / 145.6 / 151.8 with one; twelve heads behind 1400 keys, 12 rows, 103.2 against 101.5.  From 64 rows of
// 32 heads on they are equal.
inline bool merge_spread(int M, int heads) { return (M + 7) / 8 * heads < 128; }
