// Masked attention of the verify pass: every row attends to the shared prefix, the optional root
// token and the earlier tokens of its own draft sequence (independent sequences, Sec. 3.2).
//
// The prefix keys/values of one KV head are read ONCE for all rows and all query heads of the
// group, or once per row group where these are more query tiles than a workgroup takes: a workgroup takes one (kv head, key
// chunk, row group).  Per 32-key block a wave computes S^T = K Q^T and O^T += V^T P^T with MFMA:
//   - K and V^T tiles lie in the cache as MFMA operands; attn_small_kernel loads them straight into registers, attn_shared_kernel
//     puts them in LDS once for all query tiles of a row group (both with the non-temporal hint);
//   - the key permutation inside a block is chosen so that the S^T accumulator of a lane
//     already holds the eight consecutive keys its P^T operand needs: no cross-lane traffic
//     between the two products;
//   - queries and softmax weights enter the MFMAs as bf16 pairs (hi + lo), keys and values are the
//     cache's bf16;
//   - the softmax is online (running max / sum per row), reduced across the four lane groups by lane swaps.
// Chunk partials (max, sum, unnormalised O) go to scratch and are merged in chunk order by a small second kernel; where a head is one
// chunk (short prefixes) the same workgroup finishes it: one kernel per layer.
#pragma once
#include "duo_common.h"
#include "duo_gemm.h"

struct AttnArgs {
    const u16* q;  // queries as bf16 pairs: hi plane [rows][Hq*D], lo plane q_plane elements further on
    int ldq;
    size_t q_plane;
    const u16* kc;  // this layer: [Hkv] planes of max_seq * D elements, tiled (k_cache_offset)
    const u16* vc;  // this layer: [Hkv] planes of max_seq * D elements, tiled (v_cache_offset)
    int max_seq, group;
    RowPlan plan;
    int Ktot;             // P + M keys in play
    int chunk_blocks;     // 32-key blocks per chunk (attn_shared_kernel)
    int nchunks;
    int mq_pad;           // padded number of (row, query-head-in-group) pairs
    float scale_log2;     // log2(e) / sqrt(D)
    float* part;          // [Hkv][mq_pad][nchunks][D + 4]: O (unnormalised), max, sum
    u16* out;             // attention output, operand layout of the O projection (bf16 pairs)
    int out_tiles;
    LoRows lo_rows;
};

// 2^x by the hardware instruction alone: results below the normal range come out as zero; 2^0 is exactly 1 and 2^-inf exactly 0.
// Three and more query tiles take their softmax weights so: such a weight shows only next to values of 2^100 and more.  One and two tiles
// keep them (exp2f), as do the merges.
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

// The largest of the four lane groups' values (lanes c, c + 16, c + 32, c + 48), in all of them.  Lane swaps within the vector unit: the maximum of
// a block stands between its scores and its exponentials, and two dependent shuffles through the LDS crossbar, which eight waves keep busy
// with operand reads, are two trips there (1024 prompt rows behind 1024 keys on 32 heads 75.6 -> 74.0 us, 65 rows of eight groups of four
// behind 8192 keys 31.4 -> 30.3).
__device__ __forceinline__ float lane_groups_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Merge the chunk partials (at most 64) of one (row, query head), normalise, store as a bf16 pair
// (hi = operand row m, lo = operand row lo_rows(m)).  Called by one wave.  Lane cb takes chunk cb's
// max and sum (one load each instead of a chain of them), the maximum and the weighted sum are formed by
// fixed butterflies; the outputs are then added in chunk order, lane handling D/64 channels; the first eight
// chunks' outputs are requested together with the statistics, further ones four at a time.
template <int D>
__device__ __forceinline__ void attn_merge_row(const AttnArgs& a, int hk, int r, int lane) {
    const int m = r / a.group, gq = r % a.group;
    const float* pp = a.part + ((size_t)hk * a.mq_pad + r) * a.nchunks * (D + 4);
    const bool has = lane < a.nchunks;
    const float mc = has ? pp[(size_t)lane * (D + 4) + D] : -INFINITY;
    const float lc = has ? pp[(size_t)lane * (D + 4) + D + 1] : 0.f;
    // the first eight chunks' outputs are requested with the statistics (they do not depend on them)
    constexpr int PRE = 8;
    float vp[PRE][D / 64];
#pragma unroll
    for (int i = 0; i < PRE; ++i) {
        const int cb = i < a.nchunks ? i : a.nchunks - 1;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) vp[i][e] = pp[(size_t)cb * (D + 4) + lane + e * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
    float mx = mc;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    const float w = mc == -INFINITY ? 0.f : exp2f(mc - mx);  // this lane's chunk weight
    float L = lc * w;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) L += __shfl_xor(L, o, 64);
    float acc[D / 64];
#pragma unroll
    for (int e = 0; e < D / 64; ++e) acc[e] = 0.f;
#pragma unroll
    for (int i = 0; i < PRE; ++i) {
        const float wc = i < a.nchunks ? __shfl(w, i, 64) : 0.f;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) acc[e] += vp[i][e] * wc;
    }
    for (int cb0 = PRE; cb0 < a.nchunks; cb0 += 4) {
        float v[4][D / 64], wc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cb = cb0 + i < a.nchunks ? cb0 + i : a.nchunks - 1;
            wc[i] = cb0 + i < a.nchunks ? __shfl(w, cb, 64) : 0.f;
#pragma unroll
            for (int e = 0; e < D / 64; ++e) v[i][e] = pp[(size_t)cb * (D + 4) + lane + e * 64];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < D / 64; ++e) acc[e] += v[i][e] * wc[i];
    }
    const int col0 = (hk * a.group + gq) * D;
#pragma unroll
    for (int e = 0; e < D / 64; ++e) {
        const float o = acc[e] / L;
        u16 hi, lo;
        split_elem(o, hi, lo);
        const int col = col0 + lane + e * 64;
        a.out[operand_offset(m, col, a.out_tiles)] = hi;
        a.out[operand_offset(a.lo_rows(m), col, a.out_tiles)] = lo;
    }
}

// Short contexts (at most 8 * BATCH blocks of 32 keys, up to 16 query rows per kv head): the whole head
// in one workgroup of eight waves, no loop.  A wave requests the keys of ALL its blocks and the values
// of the first one at once, forms every score, requests the remaining values into the registers the
// keys just left, does one plain softmax over its keys and the P V products; then the waves are merged
// through LDS in one step and every wave writes one 16-channel tile of the normalised output.  One memory latency for the keys and
// one for the values, instead of one per block.
template <int D, int BATCH>
__global__ __launch_bounds__(512) void attn_small_kernel(AttnArgs a) {
    constexpr int KS = D / 32, DT = D / 16, NWV = 8;
    __shared__ f32x4 lds_o[NWV][DT * 64];
    __shared__ float lds_ml[NWV][2][16];

    const int hk = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    const int MQ = a.plan.M * a.group;

    const int r = c;  // column c of the one query tile is pair r = (row m, head gq of the group)
    const bool ok = r < MQ;
    const int m = ok ? r / a.group : 0, gq = ok ? r % a.group : 0;
    const int R = a.plan.R;
    const int vis_lo = !ok ? 0x7fffffff : (m < R ? 0 : R + ((m - R) / a.plan.k) * a.plan.k);
    const int vis_hi = ok ? m : -1;
    elem8 qf[KS], ql[KS];
    {
        const u16* qp = a.q + (size_t)m * a.ldq + (hk * a.group + gq) * D + g * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            Frag8 f;
            f.q = ok ? *reinterpret_cast<const u32x4*>(qp + ks * 32) : u32x4{0u, 0u, 0u, 0u};
            qf[ks] = f.v;
            f.q = ok ? *reinterpret_cast<const u32x4*>(qp + a.q_plane + ks * 32) : u32x4{0u, 0u, 0u, 0u};
            ql[ks] = f.v;
        }
    }
    const u16* kbase = a.kc + (size_t)hk * a.max_seq * D + lane * 8;
    const u16* vbase = a.vc + (size_t)hk * a.max_seq * D + lane * 8;
    const int NB = (a.Ktot + 31) / 32;
    // block b of this wave is global block wave + 8*b (round-robin keeps the waves within one block of each other)
    int nb = (NB - wave + NWV - 1) / NWV;
    nb = nb < 0 ? 0 : nb;

    elem8 kf[BATCH][2][KS], vf[BATCH][DT];
    auto load_v = [&](int b) {
        const int kb = (wave + NWV * b) * 32;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) vf[b][dt] = load_frag_stream(vbase + ((size_t)(kb >> 5) * DT + dt) * 512);
    };
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        if (b < nb) {
            const int blk = wave + NWV * b;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) kf[b][t][ks] = load_frag_stream(kbase + ((size_t)(blk * 2 + t) * KS + ks) * 512);
        }
    }
    if (nb > 0) load_v(0);
    __builtin_amdgcn_sched_barrier(0);

    float sc[BATCH][8];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sc[b][j] = -INFINITY;
        if (b < nb) {
            const int kb = (wave + NWV * b) * 32;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = mfma16(kf[b][t][ks], ql[ks], acc);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = mfma16(kf[b][t][ks], qf[ks], acc);
#pragma unroll
                for (int i = 0; i < 4; ++i) sc[b][t * 4 + i] = acc[i] * a.scale_log2;
            }
            if (kb + 32 > a.plan.P) {  // block touches draft slots or the end
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int mk = kb + g * 8 + j - a.plan.P;
                    const bool vis = (mk < R) | ((mk >= vis_lo) & (mk <= vis_hi));
                    sc[b][j] = vis ? sc[b][j] : -INFINITY;
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 1; b < BATCH; ++b)
        if (b < nb) load_v(b);
    __builtin_amdgcn_sched_barrier(0);

    // one softmax over all keys of this wave
    float mx = -INFINITY;
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
#pragma unroll
        for (int j = 0; j < 8; ++j) mx = fmaxf(mx, sc[b][j]);
    mx = lane_groups_max(mx);
    const float m_safe = mx == -INFINITY ? 0.f : mx;
    float m_run = mx, l_run = 0.f;
    f32x4 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        if (b < nb) {
            const int kb = (wave + NWV * b) * 32;
            if (kb + 32 > a.Ktot) {  // slots at or beyond Ktot may hold anything: zero their V
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    Frag8 f;
                    f.v = vf[b][dt];
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (kb + g * 8 + j >= a.Ktot) f.h[j] = 0;
                    vf[b][dt] = f.v;
                }
            }
            Frag8 pf, pl;  // softmax weights as bf16 pairs (hi + lo)
            float pw[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                pw[j] = exp2f(sc[b][j] - m_safe);
                l_run += pw[j];
            }
            split_elem8(pw, pf.q, pl.q);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                o[dt] = mfma16(vf[b][dt], pl.v, o[dt]);
                o[dt] = mfma16(vf[b][dt], pf.v, o[dt]);
            }
        }
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);

    // Merge of the eight waves in one step: every wave leaves its unnormalised output, maximum and sum in LDS;
    // after one barrier wave w combines channel tile w of all eight (in wave order), normalises and stores it.
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) lds_o[wave][dt * 64 + lane] = o[dt];
    if (g == 0) {
        lds_ml[wave][0][c] = m_run;
        lds_ml[wave][1][c] = l_run;
    }
    __syncthreads();
    if (wave >= DT || !ok) return;
    float mall = lds_ml[0][0][c];
#pragma unroll
    for (int w = 1; w < NWV; ++w) mall = fmaxf(mall, lds_ml[w][0][c]);
    float L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
        const float mw = lds_ml[w][0][c];
        const float sw = mw == -INFINITY ? 0.f : exp2f(mw - mall);
        L += lds_ml[w][1][c] * sw;
        acc += lds_o[w][wave * 64 + lane] * sw;
    }
    const int col0 = (hk * a.group + gq) * D;
    const float inv = 1.0f / L;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        u16 hi, lo;
        split_elem(acc[i] * inv, hi, lo);
        const int col = col0 + wave * 16 + g * 4 + i;
        a.out[operand_offset(m, col, a.out_tiles)] = hi;
        a.out[operand_offset(a.lo_rows(m), col, a.out_tiles)] = lo;
    }
}

// Two or more 16-row query tiles per kv head, or one on a long context.  (A kernel whose waves read their own keys for all query tiles was
// slower at every size: two tiles on 40 / 980 keys 9.0 / 20.4 us against 5.8 / 7.0 + 4.3 with the merge, one tile of 32 heads on 1400
// 8.4 against 7.2.)  A workgroup takes one (kv head, key chunk); each 32-key block of K and V^T is put
// in LDS once, in MFMA operand layout, and each of the NWV consumer waves owns one query tile and runs over all blocks of the
// chunk, so nothing is merged between waves.  One extra wave does nothing but move the blocks: 16-byte
// global -> LDS loads (no registers, no LDS store instructions) into a ring of three buffers, two blocks
// ahead of the MFMAs; its barriers are bare s_barrier instructions behind a counted wait.  One barrier per
// block hands a filled buffer over and takes a drained one back.
//
// With few query tiles (KSPLIT > 1) the NWV consumer waves are KSPLIT teams of TW = NWV / KSPLIT waves and a ring stage
// holds KSPLIT blocks: team z takes block z of every stage for the workgroup's TW query tiles, so that every SIMD holds
// KSPLIT waves whose matrix, vector and LDS instructions overlap; the teams' softmax states are merged in team order
// through LDS at the end (the same rescaled sum the chunk merge uses).

template <int N>
__device__ __forceinline__ void wait_vector_loads_but() {  // vmcnt(N); expcnt and lgkmcnt fields at their maxima
    static_assert(N >= 0 && N <= 63, "the memory counter has six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <int D, int NWV, int KSPLIT>
__global__ __launch_bounds__((NWV + 1) * 64) void attn_shared_kernel(AttnArgs a) {
    constexpr int KS = D / 32, DT = D / 16;
    constexpr int KT = 2 * KS;      // K tiles per block (2 key halves x KS)
    constexpr int TILES = KT + DT;  // 1 KiB tiles per block
    constexpr int NBUF = 3;
    constexpr int TW = NWV / KSPLIT;  // query-tile waves per team
    constexpr int STL = KSPLIT * TILES;  // tiles per ring stage: one block for every team
    static_assert(STL <= 63, "a stage's loads fit the producer's memory counter");
    static_assert(NWV % KSPLIT == 0, "teams of equal size");
    __shared__ u32x4 lds_kv[NBUF][STL * 64];
    __shared__ f32x4 lds_team_o[KSPLIT > 1 ? (KSPLIT - 1) * TW * DT * 64 : 1];
    __shared__ float lds_team_ml[KSPLIT > 1 ? (KSPLIT - 1) * TW * 2 * 64 : 1];

    const int cb = blockIdx.x, hk = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;  // scalar: MFMA ignores EXEC
    const int c = lane & 15, g = lane >> 4;
    const int NB = (a.Ktot + 31) / 32;
    const int b0 = cb * a.chunk_blocks;
    int nb = NB - b0;
    nb = nb < 0 ? 0 : (nb > a.chunk_blocks ? a.chunk_blocks : nb);
    // Row groups in reverse launch order: workgroups start in index order, and the late rows of a prompt chunk see the
    // most keys, so the longest-running groups go first.
    const int zg = (int)(gridDim.z - 1 - blockIdx.z);
    {
        // No row sees a key behind its own slot: the blocks behind the slot of this workgroup's last query row
        // are masked for all of its rows and are left out (a prompt chunk's early rows skip the chunk's late keys).
        const int r_last = min(a.plan.M * a.group, (zg + 1) * TW * 16) - 1;
        const int nb_vis = (a.plan.P + r_last / a.group) / 32 + 1 - b0;
        nb = nb_vis < nb ? (nb_vis < 0 ? 0 : nb_vis) : nb;
    }

    const int nst = (nb + KSPLIT - 1) / KSPLIT;  // ring stages
    if (wave == NWV) {
        // ---- producer.  The cache stores the tiles as they are needed (see k_cache_offset / v_cache_offset):
        // tile j < KT of a block is K tile (t = j / KS, ks = j % KS), otherwise V^T tile dt = j - KT; each is 1 KiB,
        // lane l takes bytes 16*l ..
        const u16* kbase = a.kc + (size_t)hk * a.max_seq * D + lane * 8;
        const u16* vbase = a.vc + (size_t)hk * a.max_seq * D + lane * 8;
        auto issue = [&](int st) {  // stage st: blocks st * KSPLIT .. + KSPLIT of the chunk, as far as it has them
            u32x4* dst = lds_kv[st % NBUF];
#pragma unroll
            for (int z = 0; z < KSPLIT; ++z) {
                const int ib = st * KSPLIT + z;
                if (ib >= nb) break;  // wave-uniform
                const int blk = b0 + ib;
#pragma unroll
                for (int j = 0; j < TILES; ++j) {
                    const u16* src = j < KT ? kbase + ((size_t)blk * KT + j) * 512 : vbase + ((size_t)blk * DT + (j - KT)) * 512;
                    // cache policy 2: the non-temporal hint.  Faster than ordinary loads also where several row groups read
                    // the same chunk: eight layers, 65 rows of four in five groups behind 8192 keys 1535 against 1553 us, 64 rows in
                    // one group behind 4096 1212 against 1236, one tile behind 901 784 / 796; prompt chunks of 1024 rows 6413 / 6391, where runs
                    // differ by 0.9 %, of 333 equal.
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                     (__attribute__((address_space(3))) void*)(dst + (z * TILES + j) * 64), 16, 0, 2);
                }
            }
        };
        // Only blocks of the chunk are requested, so the wait before a hand-over counts the blocks of the one stage that
        // may still be in flight: vmcnt(blocks * TILES), everything older has landed (expcnt, lgkmcnt fields at their maxima).
        static_assert(KSPLIT <= 2, "the waits below know stages of one or two blocks");
        auto wait_all_but_stage = [&](int st) {
            const int blocks = st < nst ? min(KSPLIT, nb - st * KSPLIT) : 0;
            if (blocks == 0) wait_vector_loads_but<0>();
            else if (blocks == 1) wait_vector_loads_but<TILES>();
            else wait_vector_loads_but<2 * TILES>();
        };
        if constexpr (NWV == 4) {
            // Up to two query tiles per kv head: the first two stages are requested without a branch (blocks past the chunk
            // or the context repeat the last block of the context and are not used).  Behind a branch around global -> LDS
            // loads the compiler waits for everything in flight, so stage 1 is otherwise requested only after stage 0 has
            // landed.  Measured on whole steps: 3.538 -> 3.517 ms at two tiles (32 rows, 32 heads), but 4.600 -> 4.607 ms
            // at four tiles and 5.088 -> 5.096 ms at sixteen, where the kernel alone is faster too: those keep the branches.
            auto issue_unconditionally = [&](int st) {
                u32x4* dst = lds_kv[st % NBUF];
#pragma unroll
                for (int z = 0; z < KSPLIT; ++z) {
                    const int blk = min(b0 + st * KSPLIT + z, NB - 1);
#pragma unroll
                    for (int j = 0; j < TILES; ++j) {
                        const u16* src = j < KT ? kbase + ((size_t)blk * KT + j) * 512 : vbase + ((size_t)blk * DT + (j - KT)) * 512;
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                         (__attribute__((address_space(3))) void*)(dst + (z * TILES + j) * 64), 16, 0, 2);
                    }
                }
            };
            issue_unconditionally(0);
            issue_unconditionally(1);
            wait_vector_loads_but<KSPLIT * TILES>();  // stage 0 has landed
        } else {
            if (nst > 0) issue(0);
            if (nst > 1) issue(1);
            wait_all_but_stage(1);  // stage 0 has landed
        }
        __builtin_amdgcn_s_barrier();
        for (int st = 0; st < nst; ++st) {
            if (st + 2 < nst) issue(st + 2);  // its buffer was drained in iteration st - 1
            wait_all_but_stage(st + 2);       // stage st + 1 has landed
            __builtin_amdgcn_s_barrier();
        }
        if (KSPLIT > 1) __builtin_amdgcn_s_barrier();  // the teams' hand-over
        return;
    }

    // ---- consumers
    const int MQ = a.plan.M * a.group;
    const int team = wave / TW, tw = wave - team * TW;
    const int tile = zg * TW + tw;  // this wave's query tile
    elem8 qf[KS], ql[KS];
    int vis_lo, vis_hi;
    {
        const int r = tile * 16 + c;
        const bool ok = r < MQ;
        const int m = ok ? r / a.group : 0, gq = ok ? r % a.group : 0;
        const int R = a.plan.R;
        vis_lo = !ok ? 0x7fffffff : (m < R ? 0 : R + ((m - R) / a.plan.k) * a.plan.k);
        vis_hi = ok ? m : -1;
        const u16* qp = a.q + (size_t)m * a.ldq + (hk * a.group + gq) * D + g * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            Frag8 f;
            f.q = ok ? *reinterpret_cast<const u32x4*>(qp + ks * 32) : u32x4{0u, 0u, 0u, 0u};
            qf[ks] = f.v;
            f.q = ok ? *reinterpret_cast<const u32x4*>(qp + a.q_plane + ks * 32) : u32x4{0u, 0u, 0u, 0u};
            ql[ks] = f.v;
        }
    }
    f32x4 o[DT];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto weight = [](float x) { return NWV == 4 ? exp2f(x) : exp2_raw(x); };  // four waves: up to two query tiles
    auto use_block = [&](const u32x4* buf, int kb) {
        const bool masked = kb + 32 > a.plan.P;  // block touches draft slots or the end
        const bool tail = kb + 32 > a.Ktot;      // slots at or beyond Ktot may hold anything: zero their V
        auto frag = [&](int j) {
            Frag8 f;
            f.q = buf[j * 64 + lane];
            return f;
        };
        float sc[8];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            elem8 kf[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = frag(t * KS + ks).v;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};  // lo and hi query parts into one accumulator; the scale comes with the exponent
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                acc = mfma16(kf[ks], ql[ks], acc);
                acc = mfma16(kf[ks], qf[ks], acc);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) sc[t * 4 + i] = acc[i];
        }
        Frag8 pf, pl;
        if (masked) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int mk = kb + g * 8 + j - a.plan.P;
                const bool vis = (mk < a.plan.R) | ((mk >= vis_lo) & (mk <= vis_hi));
                sc[j] = vis ? sc[j] : -INFINITY;
            }
        }
        float bm = sc[0];
#pragma unroll
        for (int j = 1; j < 8; ++j) bm = fmaxf(bm, sc[j]);
        const float m_new = fmaxf(m_run, lane_groups_max(bm) * a.scale_log2);  // the running maximum is kept in scaled units
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = weight(m_run - m_safe);
        m_run = m_new;
        float pw[8], ps = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            pw[j] = weight(fmaf(sc[j], a.scale_log2, -m_safe));
            ps += pw[j];
        }
        split_elem8(pw, pf.q, pl.q);  // softmax weights as bf16 pairs (hi + lo)
        l_run = l_run * alpha + ps;
        // the running maximum rarely moves after the first blocks: rescale only when some row's did
        if (__ballot(alpha != 1.0f) != 0) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = o[dt] * alpha;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            Frag8 vf = frag(KT + dt);
            if (tail) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (kb + g * 8 + e >= a.Ktot) vf.h[e] = 0;
            }
            const f32x4 acc = mfma16(vf.v, pl.v, o[dt]);
            o[dt] = mfma16(vf.v, pf.v, acc);
        }
    };

    // No row of this wave sees a key behind the slot of the wave's last query row: such blocks are masked for all of its
    // rows, so the wave leaves out their products and softmax (a prompt chunk's early rows against the chunk's late
    // keys: causal attention per query tile, not only per workgroup) and only keeps the ring's pace.
    // A wave without a query tile (the last of 3, 5 or 17 tiles) leaves out all of them.
    const int r_wave_last = min(MQ, (tile + 1) * 16) - 1;
    const int kb_last = tile * 16 < MQ ? a.plan.P + r_wave_last / a.group : -1;  // key slot of that row
    __syncthreads();  // block 0 is in LDS
    for (int st = 0; st < nst; ++st) {
        const int ib = st * KSPLIT + team;  // this team's block of the stage
        const int kb = (b0 + ib) * 32;
        if (ib < nb && kb <= kb_last) use_block(lds_kv[st % NBUF] + team * TILES * 64, kb);  // wave-uniform
        __syncthreads();  // stage st + 1 is in LDS; stage st's buffer may be refilled
    }
    if constexpr (KSPLIT > 1) {
        // teams 1 .. KSPLIT-1 hand their states (running maximum, this lane's part of the sum, output) to team 0
        if (team > 0) {
            const int slot = (team - 1) * TW + tw;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) lds_team_o[(slot * DT + dt) * 64 + lane] = o[dt];
            lds_team_ml[(slot * 2 + 0) * 64 + lane] = m_run;
            lds_team_ml[(slot * 2 + 1) * 64 + lane] = l_run;
        }
        __syncthreads();
        if (team > 0) return;
#pragma unroll
        for (int z = 1; z < KSPLIT; ++z) {  // team order
            const int slot = (z - 1) * TW + tw;
            const float mz = lds_team_ml[(slot * 2 + 0) * 64 + lane], lz = lds_team_ml[(slot * 2 + 1) * 64 + lane];
            const float m_new = fmaxf(m_run, mz);
            const float m_safe = m_new == -INFINITY ? 0.f : m_new;
            const float s0 = exp2f(m_run - m_safe), sz = exp2f(mz - m_safe);  // exp2(-inf) = 0: an empty state adds nothing
            m_run = m_new;
            l_run = l_run * s0 + lz * sz;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = o[dt] * s0 + lds_team_o[(slot * DT + dt) * 64 + lane] * sz;
        }
    }

    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    const int r = tile * 16 + c;
    if (r >= MQ) return;
    if (a.nchunks == 1) {
        const int m = r / a.group, col0 = (hk * a.group + r % a.group) * D;
        const float inv = 1.0f / l_run;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {  // four consecutive channels: 8 bytes of an operand chunk
            u32x2 hi, lo;
            split_elem4(o[dt] * inv, hi, lo);
            const int col = col0 + dt * 16 + g * 4;
            *reinterpret_cast<u32x2*>(a.out + operand_offset(m, col, a.out_tiles)) = hi;
            *reinterpret_cast<u32x2*>(a.out + operand_offset(a.lo_rows(m), col, a.out_tiles)) = lo;
        }
    } else {
        float* pp = a.part + (((size_t)hk * a.mq_pad + r) * a.nchunks + cb) * (D + 4);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4*>(pp + dt * 16 + g * 4) = o[dt];
        if (g == 0) {
            pp[D] = m_run;
            pp[D + 1] = l_run;
        }
    }
}

// Merge of the chunk partials when a head was split over several workgroups: one wave per (row, head).  Eight rows of one head share the
// 128-byte lines of the operand that the merge writes, so their waves are one workgroup or, with SPREAD, eight workgroups on one die.
template <int D, bool SPREAD>
__global__ __launch_bounds__(SPREAD ? 64 : 512) void attn_combine_kernel(AttnArgs a, HeadUnits units) {
    int head, m;
    if (SPREAD) {
        m = units.row(blockIdx.x, head);
    } else {
        const int groups = (a.plan.M + 7) >> 3;
        head = blockIdx.x / groups;
        m = (blockIdx.x - head * groups) * 8 + (threadIdx.x >> 6);
    }
    const int hk = head / a.group;
    if (head < units.heads && m < a.plan.M) attn_merge_row<D>(a, hk, m * a.group + head - hk * a.group, threadIdx.x & 63);
}
