// The library's own launch rules and index maps (plain arithmetic) for the tests to call.
#define __host__
#define __device__
#define __forceinline__ inline
#include "../paper_2503_00784_amd/csrc/duo_launch.h"

extern "C" {

int place(int b, int n) { return die_contiguous(b, n); }

int row_blocks(int M, int parts_log2) { return RowUnits{M, parts_log2}.blocks(); }
int row_of(int M, int parts_log2, int b, int* part) { return RowUnits{M, parts_log2}.row(b, *part); }
int head_blocks(int M, int heads) { return HeadUnits{M, heads}.blocks(); }
int head_row_of(int M, int heads, int b, int* head) { return HeadUnits{M, heads}.row(b, *head); }
int parts_of(int M, int d) { return 1 << reduce_parts_log2(M, d); }

int operand_tiles(int M) { return a_tiles_for(M); }
int shared_last_tile(int M) { return half_tail(M); }
int lo_row(int M, int m) { return lo_rows_for(M)(m); }

void attention(int D, int Hkv, int group, int M, int P, int many, int max_chunks, int* out) {
    const AttnLaunch a = attention_launch(D, Hkv, group, M, P, many != 0, max_chunks);
    const int v[] = {a.small, a.nwv, a.ksplit, a.row_groups, a.chunk_blocks, a.chunks};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}
}
