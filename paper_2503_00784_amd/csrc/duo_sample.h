// Speculative sampling over the target logits (Alg. 2, Sec. 3.3) and the KV commit.
//
// All probabilities are evaluated in double from the fp32 logits, so that the accept decision
// u * q(t) < p(t) and the inverse-CDF draws are taken in the precision a plain reference uses;
// the volumes are tiny next to the weight stream (two passes over a few vocabulary rows).
//   sample_stats_kernel   max and normaliser of softmax(logits / T) for every row of logits, the vocabulary cut into
//                         slices for parallelism (caller-supplied logits only: in the verify step the LM head's
//                         epilogue leaves these statistics, one part per 32-column tile, see EpiLogitsStats, and
//                         sample_row_stats_kernel merges them)
//   sample_spread_kernel, sample_locate_kernel
//                         independent sequences, vocabularies of SPREAD_MIN_VOCAB entries and more: accept flags, leading
//                         accepts, then the correction token from norm(max(0, p - q)) or the bonus token from p
//   seq_stage_kernel, seq_tail_kernel, seq_locate_kernel
//                         the sequential first-token rule over the candidate sequences, with the running distribution
//                         replaced by its residual after each rejection: the call's own sequences, or (Alg. 2 as listed)
//                         new sequences behind a verified suffix; the same vocabularies
//   sample_finish_kernel, sample_paper_kernel, sample_deferred_kernel
//                         the same rules for small vocabularies, one workgroup per sequence or per call
//   commit_kernel         picks the sequence to keep, moves its accepted K/V next to the prefix
//
// T = 0 is the greedy limit of the same rule: softmax(logits / T) tends to the one-hot distribution at the
// largest logit (lowest id among equals), so a draft token is accepted exactly when it is that id, and every
// correction or bonus token is that id (p(t) in {0, 1} in u * q(t) < p(t); the residual of a one-hot p is the
// same one-hot unless q already puts all its mass there).  The statistics then hold the arg max instead of the
// normaliser; everything else runs unchanged on the one-hot p.
//
// Nucleus (top-p) restriction of the target distributions: nucleus_hist_kernel and nucleus_cut_kernel find, per judging
// row, the set of most probable tokens whose mass reaches top_p (equal probabilities by ascending id) as a threshold on
// the logit plus the last admitted id among the logits equal to it, and the kept mass; the kernels above then
// evaluate p'(v) = p(v) / kept mass inside the set and 0 outside.  Without it (nuc == nullptr) nothing changes.
#pragma once
#include "duo_common.h"

struct SampleArgs {
    const float* logits;  // fp32 [R + n*k][ld]
    int ld;
    const float* root_logits;  // fp32 [V], judges first tokens when R == 0
    int V, n, k, R, P;
    double T;               // temperature; 0 selects the greedy limit
    const int32_t* tokens;  // [n][k]
    const float* q;         // [n][k][V]
    const float* u;         // [n][k+1]
    // Softmax statistics of the judging rows, as partial results over slices of the vocabulary: per slice the max of
    // z = logit / T and sum exp(z - max) (greedy: the max logit and the lowest id that attains it).  stats_rows
    // [R + n*k][parts][2] belongs to the rows of `logits`: written by the LM head's epilogue (one part per 32-column
    // tile) or by sample_stats_kernel (STATS_SPLIT parts); stats_root [root_parts][2] to root_logits (R == 0).
    double* stats_rows;
    int parts;
    double* stats_root;
    int root_parts;  // STATS_SPLIT from sample_stats_kernel, ROOT_STATS_PARTS from the verify pass's first kernel
    int32_t* acc;           // [n][k] accept flags
    double* p_run;          // [V] running distribution of the sequential rule
    int32_t* accept_len;    // [n]
    int32_t* next_token;    // [n]
    int32_t* commit;        // [4]
    int32_t* status;
    const double* nuc;      // nucleus records [1 + n*k][4] (threshold key, last tied id, kept mass, -), or nullptr
    __device__ __forceinline__ int nuc_row(int i, int j) const { return j == 0 ? 0 : 1 + i * k + (j - 1); }
    // row of `logits` that judges draft (i, j), or -1 for root_logits
    __device__ __forceinline__ int judge_index(int i, int j) const { return j == 0 ? (R ? 0 : -1) : R + i * k + j - 1; }
    __device__ __forceinline__ const float* judge_row(int i, int j) const {
        if (j == 0) return R ? logits : root_logits;
        return logits + (size_t)(R + i * k + j - 1) * ld;
    }
    __device__ __forceinline__ bool greedy() const { return T == 0.0; }
    __device__ __forceinline__ int token(int i, int j) const {
        int t = tokens[i * k + j];
        return t < 0 ? 0 : (t >= V ? V - 1 : t);
    }
};

// The status word as the kernels before this one left it (they OR their flags in with device-scope atomics).  A pass
// whose status is not clean commits nothing: the device prefix length and every cache slot below it stay as they
// were, and the commit record reads {-1, 0, -1, unchanged prefix length}.
__device__ __forceinline__ int32_t status_now(int32_t* status) {
    return status ? __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
}
// commit record of a pass that failed on the device; P is the host's prefix length, used when there is no cache
__device__ __forceinline__ void write_failed_commit(int32_t* commit, const int32_t* prefix_len, int P) {
    commit[0] = -1;
    commit[1] = 0;
    commit[2] = -1;
    commit[3] = prefix_len ? *prefix_len : P;
}

// Logits as unsigned keys in the same order (-0 counted as +0), and the nucleus test of one token.
__device__ __forceinline__ uint32_t logit_key(float x) {
    const uint32_t b = __float_as_uint(x + 0.0f);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
struct Nucleus {
    bool on;
    uint32_t thr;  // kept: key > thr, or key == thr and id <= vcut
    int vcut;
    double inv;    // 1 / kept mass
    __device__ __forceinline__ bool keeps(float logit, int v) const {
        const uint32_t kx = logit_key(logit);
        return kx > thr || (kx == thr && v <= vcut);
    }
    // p (already normalised over the whole vocabulary) -> p'
    __device__ __forceinline__ double apply(double p, float logit, int v) const {
        return !on ? p : (keeps(logit, v) ? p * inv : 0.0);
    }
};
// NUC = false: the kernels are compiled without the restriction (nothing of it is left in their loops)
template <bool NUC>
__device__ __forceinline__ Nucleus nucleus_of(const SampleArgs& a, int i, int j) {
    if (!NUC || !a.nuc) return Nucleus{false, 0u, 0, 1.0};
    const double* e = a.nuc + (size_t)a.nuc_row(i, j) * 4;
    return Nucleus{true, (uint32_t)e[0], (int)e[1], 1.0 / e[2]};
}

constexpr int SAMPLE_THREADS = 1024;
constexpr int STATS_SPLIT = 8;        // workgroups per row of logits in sample_stats_kernel
constexpr int STATS_PER_THREAD = 16;  // values of a slice that a thread of it holds in registers
constexpr int ROOT_STATS_PARTS = 32;  // slices of the cached root logits when the verify pass's first kernel takes their statistics

__device__ __forceinline__ double block_sum_d(double v, double* sm) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < nw; ++w) t += sm[w];
    return t;
}
__device__ __forceinline__ double block_max_d(double v, double* sm) {
    v = wave_max(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    double t = sm[0];
    for (int w = 1; w < nw; ++w) t = fmax(t, sm[w]);
    return t;
}

// Statistics of one slice [v0, v1) of a row of logits (all 256 threads of the workgroup): zmax and Z as SampleArgs
// describes them.
__device__ __forceinline__ void slice_stats(const float* __restrict__ row, int v0, int v1, double T, double* sm, double& zmax,
                                            double& Z) {
    float lm = -INFINITY;
    for (int v = v0 + threadIdx.x; v < v1; v += 256) lm = fmaxf(lm, row[v]);
    if (T == 0.0) {  // Z: the lowest id of the slice that holds the slice's largest logit
        zmax = block_max_d((double)lm, sm);
        int first = 0x7fffffff;
        for (int v = v0 + threadIdx.x; v < v1; v += 256)
            if ((double)row[v] == zmax) first = min(first, v);
        Z = -block_max_d(-(double)first, sm);
    } else {
        zmax = block_max_d((double)lm, sm) / T;
        double s = 0.0;
        for (int v = v0 + threadIdx.x; v < v1; v += 256) s += exp((double)row[v] / T - zmax);
        Z = block_sum_d(s, sm);
    }
}

// grid (R + n*k + (R ? 0 : 1), STATS_SPLIT): slice sl of row r of `logits`, the last row index being root_logits when
// there is no root row.  Used when the logits come from the caller; the verify step's LM head leaves the same
// statistics itself (EpiLogitsStats in duo_gemm.h) and the pass's first kernel those of root_logits.  As the first kernel
// of a sampling-only call it also sets the status word (set_status): its first workgroup checks the draft tokens.
// A thread holds its share of the slice in registers between the maximum and the sum (up to STATS_PER_THREAD values, i.e. a
// vocabulary of 131072 with 1024 threads; longer slices are read twice): one trip to memory.  Bound by the latency of that trip, of
// the block sums and of the double-precision exponentials of few waves: 128256 entries and 65 rows 20.2 us with 1024 threads against 46
// with 256 that read the slice twice; but no more threads than a slice needs (see the launch).  At most 64 registers, so that two
// workgroups of 1024 fit a compute unit: 65 rows are 520 workgroups, three rounds of one per compute unit otherwise.
template <int TH>
__global__ __launch_bounds__(TH, 8) void sample_stats_kernel(SampleArgs a, int set_status) {
    __shared__ double sm[16];
    const int r = blockIdx.x, sl = blockIdx.y, rows = a.R + a.n * a.k, tid = threadIdx.x;
    const float* row = r < rows ? a.logits + (size_t)r * a.ld : a.root_logits;
    const int len = (a.V + STATS_SPLIT - 1) / STATS_SPLIT;
    const int v0 = min(a.V, sl * len), v1 = min(a.V, v0 + len);
    constexpr int PER = STATS_PER_THREAD;
    const bool in_regs = len <= PER * TH;
    float x[PER];
    float lm = -INFINITY;
    if (in_regs) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {  // beyond the slice: its first value again (a slice may be empty: any value of the row)
            const int v = v0 + tid + e * TH;
            x[e] = row[v < v1 ? v : 0];
        }
#pragma unroll
        for (int e = 0; e < PER; ++e) lm = v0 + tid + e * TH < v1 ? fmaxf(lm, x[e]) : lm;
    } else {
        for (int v = v0 + tid; v < v1; v += TH) lm = fmaxf(lm, row[v]);
    }
    if (set_status && r == 0 && sl == 0) {
        const int raw = tid < a.n * a.k ? a.tokens[tid] : 0;  // n * k is at most DUO_MAX_ROWS
        const int bad = __syncthreads_or(raw < 0 || raw >= a.V);
        if (tid == 0 && a.status) *a.status = bad ? 1 : 0;
    }
    double zmax = block_max_d((double)lm, sm), Z;
    if (a.greedy()) {  // Z: the lowest id of the slice that holds the slice's largest logit
        int first = 0x7fffffff;
        if (in_regs) {
#pragma unroll
            for (int e = PER - 1; e >= 0; --e)
                if (v0 + tid + e * TH < v1 && (double)x[e] == zmax) first = v0 + tid + e * TH;
        } else {
            for (int v = v0 + tid; v < v1; v += TH)
                if ((double)row[v] == zmax) first = min(first, v);
        }
        Z = -block_max_d(-(double)first, sm);
    } else {
        const double iT = 1.0 / a.T;  // a reciprocal instead of a division per entry: an ulp, as in TokenWeights
        zmax *= iT;
        double s = 0.0;
        if (in_regs) {
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                if (e * TH >= len) break;  // workgroup-uniform
                if (v0 + tid + e * TH < v1) s += exp((double)x[e] * iT - zmax);
            }
        } else {
            for (int v = v0 + tid; v < v1; v += TH) s += exp((double)row[v] * iT - zmax);
        }
        Z = block_sum_d(s, sm);
    }
    if (tid == 0) {
        double* st = (r < rows ? a.stats_rows + ((size_t)r * a.parts + sl) * 2 : a.stats_root + sl * 2);
        st[0] = zmax;
        st[1] = Z;
    }
}

// The merged statistics of the judging rows of one sequence, position j -> {zmax, Z} (greedy: {max logit, arg max}),
// kept in shared memory by the kernels below.
struct SeqStats {
    double (*t)[2];
};

// Merge of the partial statistics of one judging row (jr as judge_index returns it) by one wave: lanes stride over the
// parts, fixed butterflies (deterministic); every lane gets the result.
__device__ __forceinline__ void wave_row_stats(const SampleArgs& a, int jr, double& zmax, double& Z) {
    const int lane = threadIdx.x & 63;
    const double* pt = jr < 0 ? a.stats_root : a.stats_rows + (size_t)jr * a.parts * 2;
    const int np = jr < 0 ? a.root_parts : a.parts;
    double mx = -INFINITY;
#pragma unroll 4
    for (int p = lane; p < np; p += 64) mx = fmax(mx, pt[2 * p]);
    mx = wave_max(mx);
    if (a.greedy()) {  // the lowest id among the parts that hold the largest logit (parts are in id order)
        double first = 4.0e9;
        for (int p = lane; p < np; p += 64)
            if (pt[2 * p] == mx) first = fmin(first, pt[2 * p + 1]);
        Z = -wave_max(-first);
    } else {
        double sum = 0.0;
#pragma unroll 4
        for (int p = lane; p < np; p += 64)
            if (pt[2 * p + 1] > 0.0) sum += pt[2 * p + 1] * exp(pt[2 * p] - mx);
        Z = wave_sum(sum);
    }
    zmax = mx;
}

// The same for judging rows (i, j0 .. j1) into st.t[j], one wave per row.  All threads of the workgroup call it; ends
// with a barrier.
__device__ __forceinline__ void load_seq_stats(const SampleArgs& a, int i, int j0, int j1, const SeqStats& st) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    for (int j = j0 + wave; j <= j1; j += nw) {
        double mx, Z;
        wave_row_stats(a, a.judge_index(i, j), mx, Z);
        if (lane == 0) {
            st.t[j][0] = mx;
            st.t[j][1] = Z;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void merged_stats(const SeqStats& st, int j, double& zmax, double& Z) {
    zmax = st.t[j][0];
    Z = st.t[j][1];
}
__device__ __forceinline__ int merged_argmax(const SeqStats& st, int j) { return (int)st.t[j][1]; }

// p_run[v] = p(v) of judging distribution (i, j) for the whole vocabulary; ends with a barrier
template <bool NUC>
__device__ __forceinline__ void fill_running_distribution(const SampleArgs& a, const SeqStats& st, int i, int j) {
    const float* row = a.judge_row(i, j);
    if (a.greedy()) {
        const int amax = merged_argmax(st, j);
        for (int v = threadIdx.x; v < a.V; v += blockDim.x) a.p_run[v] = v == amax ? 1.0 : 0.0;
    } else {
        double zmax, Z;
        merged_stats(st, j, zmax, Z);
        const Nucleus nc = nucleus_of<NUC>(a, i, j);
        for (int v = threadIdx.x; v < a.V; v += blockDim.x)
            a.p_run[v] = nc.apply(exp((double)row[v] / a.T - zmax) / Z, row[v], v);
    }
    __syncthreads();
}

// ---- the nucleus of a judging row ------------------------------------------------------------------------------
// Row r: 0 = the root distribution, 1 + i*k + (j-1) = row (i, j).  Wanted is the last token, in order of decreasing
// logit and, among equal logits, ascending id, with which the mass reaches top_p * total.
//
// Masses are added as whole numbers, p in units of 2^-62: sums of whole numbers do not depend on their order, so LDS
// atomics give repeatable results, and the sums add no rounding of their own.  A single mass is what its double was: the
// error of exp and of the multiplication by 1/Z, a few 2^-53 of it, and 2^-63 for the step to a whole number, which is the larger of
// the two below p = 2^-10 or so.
//   1. every id goes into one of NUC_BINS bins of equal width in logit / T below the maximum (a monotone map, so the
//      bins are in order of decreasing probability; the last bin takes everything from e^-42.6 down), and each bin's
//      mass is added up: large vocabularies by nucleus_hist_kernel, G slices of a row on as many workgroups (the
//      exponentials are the work: 4.2 million for 33 rows of 128256), small ones inside nucleus_cut_kernel;
//   2. nucleus_cut_kernel, one workgroup per row: a scan over the bins finds the one in which the cut lies; its ids (a few
//      hundred of 128256) are collected and, as long as there are more than a wave's worth, divided once more into bins of
//      equal key range; the last few are ranked by one wave.
// Measured: 5 rows of 32000 107 -> 26 us, 33 rows of 128256 2587 -> 44 us, against a bitwise search of the threshold key by one
// workgroup per row (33 sums over the whole row).  What bounds it now: the exponentials of the first kernel and the chain of
// block-wide steps of the second.
constexpr int NUC_BINS = 2048;
constexpr double NUC_BINS_PER_NAT = 48.0;
constexpr int NUC_LIST = 2048;     // ids of one bin that are held in LDS; more (near-equal logits): passes over the row
constexpr int NUC_SUB = 1024;      // bins of a refinement
constexpr int NUC_SMALL_VOCAB = 8192;  // below: nucleus_cut_kernel<true> alone
constexpr double NUC_ONE = 4611686018427387904.0;  // 2^62
typedef unsigned long long u64;

struct NucRow {  // what both kernels evaluate a row with (the same expressions: equal masses in both)
    const float* row;
    double iT, zmax, iZ;
    __device__ __forceinline__ double below_max(float x) const { return fma(-(double)x, iT, zmax); }
    __device__ __forceinline__ u64 mass(double d) const {
        const double m = fma(exp(-d) * iZ, NUC_ONE, 0.5);
        return m >= 1.0 ? (u64)m : 0ull;  // NaN: none
    }
    __device__ __forceinline__ int bin(double d) const { return (int)fmin(fmax(d * NUC_BINS_PER_NAT, 0.0), (double)(NUC_BINS - 1)); }
};

// Scratch of the two kernels inside p_rows ([rows][V] doubles): hist [rows][G][NUC_BINS] masses, then the ids' bins
// [rows][bin_stride].
struct NucBuf {
    u64* hist;
    uint16_t* bins;
    int G, slice, bin_stride;
    const double* row_stats;  // merged statistics {zmax, Z} of judging row jr at [2 * (jr + 1)], or nullptr: merge the parts
};

// wave 0 leaves the row's statistics in sm[0..1]; every thread gets the row's evaluator (contains a barrier)
__device__ __forceinline__ NucRow nuc_row(const SampleArgs& a, const double* row_stats, int i, int j, double* sm) {
    const int jr = a.judge_index(i, j);
    if (threadIdx.x < 64) {
        double zmax, Z;
        if (row_stats) {
            zmax = row_stats[2 * (jr + 1)];
            Z = row_stats[2 * (jr + 1) + 1];
        } else {
            wave_row_stats(a, jr, zmax, Z);
        }
        if (threadIdx.x == 0) {
            sm[0] = zmax;
            sm[1] = Z;
        }
    }
    __syncthreads();
    return NucRow{a.judge_row(i, j), 1.0 / a.T, sm[0], 1.0 / sm[1]};
}

// grid (rows, G)
__global__ __launch_bounds__(512) void nucleus_hist_kernel(SampleArgs a, NucBuf b) {
    __shared__ u64 h[NUC_BINS];
    __shared__ double sm[2];
    const int r = blockIdx.x, tid = threadIdx.x;
    const int i = r == 0 ? 0 : (r - 1) / a.k, j = r == 0 ? 0 : (r - 1) % a.k + 1;
    for (int e = tid; e < NUC_BINS; e += 512) h[e] = 0ull;
    const NucRow n = nuc_row(a, b.row_stats, i, j, sm);  // its barrier also orders the zeros
    const int v0 = min(a.V, (int)blockIdx.y * b.slice), v1 = min(a.V, v0 + b.slice);
    uint16_t* bins = b.bins + (size_t)r * b.bin_stride;
#pragma unroll 4
    for (int v = v0 + tid; v < v1; v += 512) {
        const double d = n.below_max(n.row[v]);
        const int bin = n.bin(d);
        bins[v] = (uint16_t)bin;
        const u64 m = n.mass(d);
        if (m) atomicAdd(&h[bin], m);
    }
    __syncthreads();
    u64* out = b.hist + ((size_t)r * b.G + blockIdx.y) * NUC_BINS;
    for (int e = tid; e < NUC_BINS; e += 512) out[e] = h[e];
}

// Inclusive sum of v over the threads of a 1024-thread workgroup in thread order; `total` gets the sum of all.
__device__ __forceinline__ u64 block_scan_u64(u64 v, u64* sm, u64& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const u64 y = __shfl_up(v, o, 64);
        if (lane >= o) v += y;
    }
    __syncthreads();
    if (lane == 63) sm[wave] = v;
    __syncthreads();
    total = 0ull;
    u64 before = 0ull;
#pragma unroll
    for (int w = 0; w < SAMPLE_THREADS / 64; ++w) {
        if (w < wave) before += sm[w];
        total += sm[w];
    }
    return before + v;
}

// One workgroup per row.  FUSED: the bins of step 1 are filled here (V < NUC_SMALL_VOCAB), otherwise nucleus_hist_kernel
// has filled them.  nuc_out[r] = {threshold key, last admitted id among the keys equal to it, kept mass, 0}.
template <bool FUSED>
__global__ __launch_bounds__(SAMPLE_THREADS) void nucleus_cut_kernel(SampleArgs a, double top_p, NucBuf b, double* __restrict__ nuc_out) {
    __shared__ __align__(16) u64 h[NUC_BINS];   // also the refinements' masses [NUC_SUB] and counts
    __shared__ __align__(16) u64 list_c[NUC_LIST], list_m[NUC_LIST];  // (key, complement of the id) and mass of the collected ids
    __shared__ __align__(16) uint16_t own_bins[FUSED ? NUC_SMALL_VOCAB : 8];
    __shared__ u64 sm_w[SAMPLE_THREADS / 64], sm_before;
    __shared__ double sm[2];
    __shared__ int sm_bin, sm_count;
    __shared__ uint32_t sm_lo, sm_hi;
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = r == 0 ? 0 : (r - 1) / a.k, j = r == 0 ? 0 : (r - 1) % a.k + 1;
    if (tid == 0) {
        sm_bin = -1;
        sm_before = 0ull;
        sm_count = 0;
    }
    if (FUSED)
        for (int e = tid; e < NUC_BINS; e += SAMPLE_THREADS) h[e] = 0ull;
    const NucRow n = nuc_row(a, b.row_stats, i, j, sm);
    u64 m0 = 0ull, m1 = 0ull;  // masses of bins 2*tid, 2*tid + 1
    static_assert(NUC_BINS == 2 * SAMPLE_THREADS, "two bins per thread");
    if (FUSED) {
        for (int v = tid; v < a.V; v += SAMPLE_THREADS) {
            const double d = n.below_max(n.row[v]);
            const int bin = n.bin(d);
            own_bins[v] = (uint16_t)bin;
            const u64 m = n.mass(d);
            if (m) atomicAdd(&h[bin], m);
        }
        __syncthreads();
        m0 = h[2 * tid];
        m1 = h[2 * tid + 1];
    } else {
        const u64* hist = b.hist + (size_t)r * b.G * NUC_BINS + 2 * tid;
#pragma unroll 8
        for (int g = 0; g < b.G; ++g) {
            m0 += hist[(size_t)g * NUC_BINS];
            m1 += hist[(size_t)g * NUC_BINS + 1];
        }
    }
    u64 total;
    const u64 incl = block_scan_u64(m0 + m1, sm_w, total);
    // whole-number masses reach top_p * total exactly when they reach its ceiling (at least one token is kept)
    const double tgt = ceil(top_p * (double)total);
    const u64 target = tgt >= 1.0 ? (u64)tgt : 1ull;
    {
        const u64 before = incl - m0 - m1;
        if (before < target && target <= before + m0) {
            sm_bin = 2 * tid;
            sm_before = before;
        } else if (before + m0 < target && target <= incl) {
            sm_bin = 2 * tid + 1;
            sm_before = before + m0;
        }
    }
    __syncthreads();
    const int bin = sm_bin;
    double* e = nuc_out + (size_t)r * 4;
    if (bin < 0) {  // no mass at all (not-a-number or infinite logits): nothing is restricted
        if (tid == 0) {
            e[0] = 0.0;
            e[1] = (double)(a.V - 1);
            e[2] = 1.0;
            e[3] = 0.0;
        }
        return;
    }
    // Calls f(first id of eight, mask of those that lie in the bin) wherever there are any.  Every thread visits its own ids;
    // the loop has no barriers.
    const uint16_t* bins = b.bins + (size_t)r * b.bin_stride;
    auto eights_of_bin = [&](auto f) {
        const int eights = (a.V + 7) >> 3;  // bin_stride covers whole eights; ids past the vocabulary are masked out
#pragma unroll 4
        for (int c = tid; c < eights; c += SAMPLE_THREADS) {
            const u32x4 w = FUSED ? *reinterpret_cast<const u32x4*>(own_bins + c * 8) : *reinterpret_cast<const u32x4*>(bins + (size_t)c * 8);
            uint32_t hit = 0u;
#pragma unroll
            for (int q = 0; q < 8; ++q) hit |= (uint32_t)((int)((w[q >> 1] >> (16 * (q & 1))) & 0xffffu) == bin && c * 8 + q < a.V) << q;
            if (hit) f(c * 8, hit);
        }
    };
    auto each_of_bin = [&](auto f) {
        eights_of_bin([&](int v0, uint32_t hit) {
            for (; hit; hit &= hit - 1u) f(v0 + __ffs(hit) - 1);
        });
    };
    // First the ids alone (a load behind every hit would be a trip to memory for every wave and position), then, a thread per
    // id, their keys and masses.
    eights_of_bin([&](int v0, uint32_t hit) {
        int at = atomicAdd(&sm_count, __popc(hit));
        for (; hit; hit &= hit - 1u, ++at)
            if (at < NUC_LIST) list_c[at] = (u64)(v0 + __ffs(hit) - 1);
    });
    __syncthreads();
    for (int q = tid; q < min(sm_count, NUC_LIST); q += SAMPLE_THREADS) {
        const int v = (int)list_c[q];
        const float x = n.row[v];
        list_c[q] = ((u64)logit_key(x) << 32) | (uint32_t)~v;
        list_m[q] = n.mass(n.below_max(x));
    }
    __syncthreads();
    int count = sm_count;
    bool listed = count <= NUC_LIST;
    uint32_t klo = 0u, khi = 0xffffffffu;  // the ids still in question: those of the bin with klo <= key <= khi
    // Calls f(key, id, mass) for every id still in question.
    auto each_left = [&](auto f) {
        if (listed) {
            for (int q = tid; q < count; q += SAMPLE_THREADS) {
                const uint32_t key = (uint32_t)(list_c[q] >> 32);
                if (key >= klo && key <= khi) f(key, (int)~(uint32_t)list_c[q], list_m[q]);
            }
        } else {
            each_of_bin([&](int v) {
                const float x = n.row[v];
                const uint32_t key = logit_key(x);
                if (key >= klo && key <= khi) f(key, v, n.mass(n.below_max(x)));
            });
        }
    };
    u64* sub_m = h;
    uint32_t* sub_n = reinterpret_cast<uint32_t*>(h + NUC_SUB);
    int left = count;
    while (left > 64) {
        if (tid == 0) {
            sm_lo = 0xffffffffu;
            sm_hi = 0u;
        }
        sub_m[tid] = 0ull;
        sub_n[tid] = 0u;
        __syncthreads();
        uint32_t lo = 0xffffffffu, hi = 0u;
        each_left([&](uint32_t key, int, u64) {
            lo = min(lo, key);
            hi = max(hi, key);
        });
        if (lo <= hi) {
            atomicMin(&sm_lo, lo);
            atomicMax(&sm_hi, hi);
        }
        __syncthreads();
        klo = sm_lo;
        khi = sm_hi;
        if (klo == khi) break;  // equal logits only: the ids decide
        int sh = 0;
        while (((khi - klo) >> sh) >= (uint32_t)NUC_SUB) ++sh;
        each_left([&](uint32_t key, int, u64 m) {
            const int q = (int)((khi - key) >> sh);  // 0: the largest keys
            if (m) atomicAdd(&sub_m[q], m);
            atomicAdd(&sub_n[q], 1u);
        });
        const u64 before0 = sm_before;
        __syncthreads();
        static_assert(NUC_SUB == SAMPLE_THREADS, "one refinement bin per thread");
        u64 sub_total;
        const u64 m = sub_m[tid];
        const u64 in = block_scan_u64(m, sm_w, sub_total);
        if (tid == 0) sm_bin = -1;
        __syncthreads();
        if (before0 + in - m < target && target <= before0 + in) {
            sm_bin = tid;
            sm_before = before0 + in - m;
        }
        __syncthreads();
        if (sm_bin < 0) {  // cannot happen while both passes add the same masses; the smallest key then, and the loop ends
            khi = klo;
            break;
        }
        const uint32_t top = khi;
        khi = top - ((uint32_t)sm_bin << sh);
        klo = max(klo, (uint32_t)(khi - ((1u << sh) - 1u) > khi ? 0u : khi - ((1u << sh) - 1u)));
        left = (int)sub_n[sm_bin];
        __syncthreads();
    }
    const u64 before = sm_before;
    if (left > 64) {
        // equal logits, one key: as many of its ids, ascending, as the target still needs; contiguous ranges per thread
        const int per = (a.V + SAMPLE_THREADS - 1) / SAMPLE_THREADS;
        const int v0 = min(a.V, tid * per), v1 = min(a.V, v0 + per);
        u64 cnt = 0ull, m = 0ull;
        for (int v = v0; v < v1; ++v)
            if (logit_key(n.row[v]) == klo) {
                ++cnt;
                m = n.mass(n.below_max(n.row[v]));
            }
        u64 ties;
        const u64 upto = block_scan_u64(cnt, sm_w, ties);
        if (cnt) list_m[0] = m;  // every writer has the same value
        __syncthreads();
        m = list_m[0];
        u64 need = m ? (target - before + m - 1) / m : 1ull;
        need = need > ties ? ties : (need < 1ull ? 1ull : need);
        if (cnt && upto - cnt < need && need <= upto) {  // the need-th of them lies in this thread's range
            u64 seen = upto - cnt;
            for (int v = v0; v < v1; ++v)
                if (logit_key(n.row[v]) == klo && ++seen == need) {
                    e[0] = (double)klo;
                    e[1] = (double)v;
                    e[2] = (double)(before + need * m) / NUC_ONE;
                    e[3] = 0.0;
                }
        }
        return;
    }
    // at most 64 ids: to the front of the list (in registers meanwhile), then one wave ranks them
    __syncthreads();
    if (tid == 0) sm_count = 0;
    __syncthreads();
    u64* fin_c = h;
    u64* fin_m = h + 64;
    each_left([&](uint32_t key, int v, u64 m) {
        const int at = atomicAdd(&sm_count, 1);
        if (at < 64) {
            fin_c[at] = ((u64)key << 32) | (uint32_t)~v;
            fin_m[at] = m;
        }
    });
    __syncthreads();
    if (wave != 0) return;
    const int nf = min(sm_count, 64);
    const u64 c = lane < nf ? fin_c[lane] : 0ull, m = lane < nf ? fin_m[lane] : 0ull;
    u64 front = before;
    bool last = true;  // no id behind this one is still short of the target
    for (int q = 0; q < nf; ++q) {
        const u64 cq = fin_c[q];
        front += cq > c ? fin_m[q] : 0ull;
    }
    const bool in = lane < nf && front < target;  // the admitted ones
    for (int q = 0; q < nf; ++q)
        if (__shfl((int)in, q, 64) && fin_c[q] < c) last = false;
    if (in && last) {
        e[0] = (double)(uint32_t)(c >> 32);
        e[1] = (double)(int)~(uint32_t)c;
        e[2] = (double)(front + m) / NUC_ONE;
        e[3] = 0.0;
    }
}

// accept flags of sequence i, positions from..k-1 (one thread each), into acc[]; ends with a barrier
// the accept test u * q(t) < p(t) of draft (i, j)
template <bool NUC>
__device__ __forceinline__ int accept_flag(const SampleArgs& a, const SeqStats& st, int i, int j) {
    const float* row = a.judge_row(i, j);
    const int t = a.token(i, j);
    double p_t;
    if (a.greedy()) {
        p_t = t == merged_argmax(st, j) ? 1.0 : 0.0;
    } else {
        double zmax, Z;
        merged_stats(st, j, zmax, Z);
        p_t = nucleus_of<NUC>(a, i, j).apply(exp((double)row[t] / a.T - zmax) / Z, row[t], t);
    }
    const double lhs = (double)a.u[i * (a.k + 1) + j] * (double)a.q[((size_t)i * a.k + j) * a.V + t];
    return lhs < p_t ? 1 : 0;
}
template <bool NUC>
__device__ __forceinline__ void accept_flags(const SampleArgs& a, const SeqStats& st, int i, int from) {
    const int j = from + threadIdx.x;
    if (j < a.k) a.acc[i * a.k + j] = accept_flag<NUC>(a, st, i, j);
    __threadfence_block();
    __syncthreads();
}

// Inverse CDF over non-negative weights w(v), v ascending: smallest v whose running sum exceeds
// u * total.  Every wave owns a contiguous chunk of the vocabulary and reads it 64 consecutive ids at a
// time (coalesced; the loads of a chunk do not depend on each other).  First the chunk sums, added over
// the waves in index order, locate the chunk where the running sum crosses the target; then that wave
// alone narrows it down (lane segments, then a scan inside the crossing segment).
// Returns (to every thread) the token, or -1 if the total is zero.
template <class F>
__device__ int block_inverse_cdf(F w, int V, double u, double* sm_d, int* sm_i) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, nw = blockDim.x >> 6;
    const int chunk = ((V + nw - 1) / nw + 63) / 64 * 64;
    const int c0 = wave * chunk, c1 = min(V, c0 + chunk);
    double local = 0.0;
    int lastpos = -1;
#pragma unroll 4
    for (int v = c0 + lane; v < c1; v += 64) {
        const double x = w(v);
        local += x;
        if (x > 0.0) lastpos = v;
    }
    const double csum = wave_sum(local);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lastpos = max(lastpos, __shfl_xor(lastpos, o, 64));
    __syncthreads();
    if (lane == 0) {
        sm_d[wave] = csum;
        sm_i[4 + wave] = lastpos;
    }
    __syncthreads();
    double total = 0.0;
    for (int ww = 0; ww < nw; ++ww) total += sm_d[ww];
    if (!(total > 0.0)) return -1;
    const double target = u * total;
    // the first chunk whose inclusive sum exceeds the target, and the running sum before it
    int owner = -1, last_all = -1;
    double base = 0.0, run = 0.0;
    for (int ww = 0; ww < nw; ++ww) {
        if (owner < 0 && run + sm_d[ww] > target) {
            owner = ww;
            base = run;
        }
        run += sm_d[ww];
        last_all = max(last_all, sm_i[4 + ww]);
    }
    if (owner < 0) return last_all;  // rounding left no crossing: largest id with positive weight
    if (wave == owner) {
        // Lane l re-adds ids [c0 + l*per, +per) of the chunk; a scan over the lanes finds the lane whose
        // segment holds the crossing; the wave then walks that segment 64 ids at a time.
        const int per = chunk >> 6;
        const int s0 = c0 + lane * per, s1 = min(c1, s0 + per);
        double seg = 0.0;
#pragma unroll 4
        for (int v = s0; v < s1; ++v) seg += w(v);
        double incl = seg;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        const unsigned long long hit = __ballot(base + incl > target);
        int tok = -1;
        if (hit) {
            const int hl = __ffsll((long long)hit) - 1;
            double before = base + __shfl(incl - seg, hl, 64);  // running sum in front of that segment
            const int h0 = c0 + hl * per, h1 = min(c1, h0 + per);
            for (int v0 = h0; v0 < h1 && tok < 0; v0 += 64) {
                const int v = v0 + lane;
                const double x = v < h1 ? w(v) : 0.0;
                double ix = x;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const double y = __shfl_up(ix, o, 64);
                    if (lane >= o) ix += y;
                }
                const unsigned long long h2 = __ballot(before + ix > target);
                if (h2) tok = v0 + __ffsll((long long)h2) - 1;
                before += __shfl(ix, 63, 64);
            }
        }
        // the chunk sum crossed but, in this summation order, no prefix did: its last positive id
        if (lane == 0) sm_i[2] = tok >= 0 ? tok : sm_i[4 + wave];
    }
    __syncthreads();
    return sm_i[2];
}

// Correction / bonus token of sequence i after `a` accepted drafts.
template <bool NUC>
__device__ int finish_token(const SampleArgs& a, const SeqStats& st, int i, int acc_len, double* sm_d, int* sm_i) {
    const float* row = a.judge_row(i, acc_len);
    if (a.greedy()) {  // one-hot p: same two draws over the one-hot weights
        const int amax = merged_argmax(st, acc_len);
        const double ug = (double)a.u[i * (a.k + 1) + a.k];
        auto pg = [=](int v) { return v == amax ? 1.0 : 0.0; };
        if (acc_len < a.k) {
            const float* qrow = a.q + ((size_t)i * a.k + acc_len) * a.V;
            auto rg = [=](int v) { return fmax((v == amax ? 1.0 : 0.0) - (double)qrow[v], 0.0); };
            const int tok = block_inverse_cdf(rg, a.V, ug, sm_d, sm_i);
            if (tok >= 0) return tok;
        }
        return block_inverse_cdf(pg, a.V, ug, sm_d, sm_i);
    }
    double zmax, Z;
    merged_stats(st, acc_len, zmax, Z);
    // reciprocals once per call instead of two divisions per vocabulary entry (the single workgroup is
    // bound by its double-precision arithmetic); the results differ from the quotients by an ulp at most
    const double iT = 1.0 / a.T, iZ = 1.0 / Z;
    const double u = (double)a.u[i * (a.k + 1) + a.k];
    const Nucleus nc = nucleus_of<NUC>(a, i, acc_len);
    auto pw = [=](int v) { return nc.apply(exp((double)row[v] * iT - zmax) * iZ, row[v], v); };
    if (acc_len < a.k) {
        const float* qrow = a.q + ((size_t)i * a.k + acc_len) * a.V;
        auto rw = [=](int v) { return fmax(nc.apply(exp((double)row[v] * iT - zmax) * iZ, row[v], v) - (double)qrow[v], 0.0); };
        const int tok = block_inverse_cdf(rw, a.V, u, sm_d, sm_i);
        if (tok >= 0) return tok;  // else: the residual vanished (p == q), fall back to p
    }
    return block_inverse_cdf(pw, a.V, u, sm_d, sm_i);
}

__device__ __forceinline__ int leading_accepts(const SampleArgs& a, int i, int from) {
    int n = from;
    while (n < a.k && a.acc[i * a.k + n]) ++n;
    return n;
}

// self_commit (single-sequence calls): also write the commit record and advance the device prefix length, which
// otherwise commit_kernel does after choosing among the sequences.
template <bool NUC>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_finish_kernel(SampleArgs a, int self_commit, int32_t* prefix_len) {
    __shared__ double sm_d[16];
    __shared__ int sm_i[4 + 16];
    __shared__ double sm_st[DUO_MAX_ROWS + 1][2];
    const SeqStats st{sm_st};
    const int i = blockIdx.x;
    load_seq_stats(a, i, 0, a.k, st);
    accept_flags<NUC>(a, st, i, 0);
    const int acc_len = leading_accepts(a, i, 0);
    const int tok = finish_token<NUC>(a, st, i, acc_len, sm_d, sm_i);
    if (threadIdx.x == 0) {
        a.accept_len[i] = acc_len;
        a.next_token[i] = tok;
        if (self_commit) {
            if (status_now(a.status) != 0) {
                write_failed_commit(a.commit, prefix_len, a.P);
            } else {
                a.commit[0] = 0;
                a.commit[1] = acc_len;
                a.commit[2] = tok;
                a.commit[3] = a.P + a.R + acc_len;
                if (prefix_len) *prefix_len = a.P + a.R + acc_len;
            }
        }
    }
}

// ---- the same rule for large vocabularies, spread over the chip ----------------------------------------------
// sample_finish_kernel is one workgroup per sequence and bound by its double-precision arithmetic: the merge of the
// rows' partial statistics (vocab / 32 parts per row after the LM head) and the pass over the vocabulary behind the
// correction token each evaluate tens of thousands of exponentials on one compute unit (27 us at 32000 entries, 87 us at
// 128256).  Three small kernels do the same work on many:
//   sample_row_stats_kernel   one workgroup per judging row: its merged statistics {zmax, Z}
//   sample_spread_kernel      grid (sequence, slice of the vocabulary): accept flags and leading accepts (every slice
//                             repeats them: k exponentials), then the sums of the correction weights max(0, p - q)
//                             and of p over the slice's 16 wave chunks, with the last id of positive weight in each
//   sample_locate_kernel      one wave per sequence: the chunk in which the running sum crosses u * total (chunk sums
//                             added in index order), the id inside it, the commit record of a single sequence
// Their scratch (SpreadBuf) lies in p_run, which this rule does not use otherwise.
struct SpreadBuf {
    // [R + n*k + 1][2], row judge_index + 1: written by sample_row_stats_kernel behind an LM head (vocab / 32 parts per
    // row); nullptr when the caller's logits were the input (STATS_SPLIT parts: the kernels merge the rows they need)
    double* row_stats;
    double* sums;       // [n][chunks][2]: correction weights, target probabilities
    int32_t* last;      // [n][chunks][2]
    int G, chunk;       // slices per sequence; ids per wave chunk (a multiple of 64); chunks = 16 * G
    __host__ __device__ int chunks() const { return 16 * G; }
};
constexpr int SPREAD_MIN_VOCAB = 8192;   // below: sample_finish_kernel
constexpr int SPREAD_MAX_GROUPS = 128;   // n * G at most: the records fit SPREAD_MIN_VOCAB doubles
constexpr int SPREAD_MAX_SLICES = 32;

__global__ __launch_bounds__(256) void sample_row_stats_kernel(SampleArgs a, double* __restrict__ row_stats) {
    __shared__ double sm[16];
    const int jr = (int)blockIdx.x - 1;
    if (jr < 0 && a.R) return;  // a root row judges the first tokens: the cached root logits are not in play
    const double* pt = jr < 0 ? a.stats_root : a.stats_rows + (size_t)jr * a.parts * 2;
    const int np = jr < 0 ? a.root_parts : a.parts;
    // a thread's parts stay in registers between the two passes, all of their loads in flight together (up to
    // 256 * PER parts, i.e. a vocabulary of 131072 behind the LM head; more: the passes re-read them)
    constexpr int PER = 16;
    const bool in_regs = np <= 256 * PER;
    double pm[PER], pz[PER];
    if (in_regs) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int p = threadIdx.x + 256 * e;
            const int pc = p < np ? p : np - 1;
            pm[e] = pt[2 * pc];
            pz[e] = pt[2 * pc + 1];
            if (p >= np) {
                pm[e] = -INFINITY;
                pz[e] = 0.0;
            }
        }
    }
    double mx = -INFINITY;
    if (in_regs) {
#pragma unroll
        for (int e = 0; e < PER; ++e) mx = fmax(mx, pm[e]);
    } else {
#pragma unroll 4
        for (int p = threadIdx.x; p < np; p += 256) mx = fmax(mx, pt[2 * p]);
    }
    mx = block_max_d(mx, sm);
    double Z;
    if (a.greedy()) {  // the lowest id among the parts that hold the largest logit
        double first = 4.0e9;
        if (in_regs) {
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (pm[e] == mx) first = fmin(first, pz[e]);
        } else {
            for (int p = threadIdx.x; p < np; p += 256)
                if (pt[2 * p] == mx) first = fmin(first, pt[2 * p + 1]);
        }
        Z = -block_max_d(-first, sm);
    } else {
        double sum = 0.0;
        if (in_regs) {
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (pz[e] > 0.0) sum += pz[e] * exp(pm[e] - mx);
        } else {
#pragma unroll 4
            for (int p = threadIdx.x; p < np; p += 256)
                if (pt[2 * p + 1] > 0.0) sum += pt[2 * p + 1] * exp(pt[2 * p] - mx);
        }
        Z = block_sum_d(sum, sm);
    }
    if (threadIdx.x == 0) {
        row_stats[2 * blockIdx.x] = mx;
        row_stats[2 * blockIdx.x + 1] = Z;
    }
}

// statistics of one judging row for one wave: the merged ones, or the parts merged here
__device__ __forceinline__ void row_stats_of(const SampleArgs& a, const double* row_stats, int jr, double& zmax, double& Z) {
    if (row_stats) {
        zmax = row_stats[2 * (jr + 1)];
        Z = row_stats[2 * (jr + 1) + 1];
    } else {
        wave_row_stats(a, jr, zmax, Z);
    }
}

// p(v) of judging row (i, j) and the correction weight max(0, p(v) - q(v)) behind a rejection at j < k
template <bool NUC>
struct TokenWeights {
    const float* row;
    const float* qrow;  // nullptr: no draft distribution at this position (bonus token)
    double iT, zmax, iZ;
    int amax;  // greedy: the one-hot id; -1 otherwise
    Nucleus nc;
    // row_zmax, row_Z: the row's merged statistics (greedy: row_Z is the arg max)
    __device__ __forceinline__ TokenWeights(const SampleArgs& a, int i, int j, double row_zmax, double row_Z) {
        row = a.judge_row(i, j);
        qrow = j < a.k ? a.q + ((size_t)i * a.k + j) * a.V : nullptr;
        amax = a.greedy() ? (int)row_Z : -1;
        iT = a.greedy() ? 0.0 : 1.0 / a.T;  // reciprocals once instead of two divisions per entry (an ulp at most)
        zmax = row_zmax;
        iZ = a.greedy() ? 0.0 : 1.0 / row_Z;
        nc = nucleus_of<NUC>(a, i, j);
    }
    __device__ __forceinline__ double p(int v) const {
        if (amax >= 0) return v == amax ? 1.0 : 0.0;
        return nc.apply(exp((double)row[v] * iT - zmax) * iZ, row[v], v);
    }
    __device__ __forceinline__ double r(double pv, int v) const { return fmax(pv - (double)qrow[v], 0.0); }
};

// One wave: the sums of both kinds of weights, f(v, p, r) with p the target probability and r the correction weight, over
// wave chunk c of the vocabulary, and the last id of positive weight of each (-1: none): sums = {r, p}, last = {r, p}.
template <class F>
__device__ __forceinline__ void wave_chunk_sums(F f, int V, int c, int chunk, double* sums, int32_t* last) {
    const int lane = threadIdx.x & 63;
    const int c0 = min(V, c * chunk), c1 = min(V, c0 + chunk);
    double sum_r = 0.0, sum_p = 0.0;
    int last_r = -1, last_p = -1;
#pragma unroll 4
    for (int v = c0 + lane; v < c1; v += 64) {
        double pv, rv;
        f(v, pv, rv);
        sum_p += pv;
        sum_r += rv;
        if (pv > 0.0) last_p = v;
        if (rv > 0.0) last_r = v;
    }
    sum_r = wave_sum(sum_r);
    sum_p = wave_sum(sum_p);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        last_r = max(last_r, __shfl_xor(last_r, o, 64));
        last_p = max(last_p, __shfl_xor(last_p, o, 64));
    }
    if (lane == 0) {
        sums[0] = sum_r;
        sums[1] = sum_p;
        last[0] = last_r;
        last[1] = last_p;
    }
}

template <bool NUC>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_spread_kernel(SampleArgs a, SpreadBuf b) {
    __shared__ double sm_st[DUO_MAX_ROWS + 1][2];
    __shared__ int sm_acc[DUO_MAX_ROWS];
    const SeqStats st{sm_st};
    const int i = blockIdx.x, g = blockIdx.y;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (b.row_stats) {
        if (tid <= a.k) {
            const double* rs = b.row_stats + 2 * (a.judge_index(i, tid) + 1);
            sm_st[tid][0] = rs[0];
            sm_st[tid][1] = rs[1];
        }
        __syncthreads();
    } else {
        load_seq_stats(a, i, 0, a.k, st);
    }
    if (tid < a.k) sm_acc[tid] = accept_flag<NUC>(a, st, i, tid);
    __syncthreads();
    int acc_len = 0;
    while (acc_len < a.k && sm_acc[acc_len]) ++acc_len;
    if (g == 0 && tid == 0) a.accept_len[i] = acc_len;
    const TokenWeights<NUC> w(a, i, acc_len, sm_st[acc_len][0], sm_st[acc_len][1]);
    const int c = g * 16 + wave;
    const size_t e = ((size_t)i * b.chunks() + c) * 2;
    if (w.qrow) wave_chunk_sums([&](int v, double& p, double& r) { p = w.p(v); r = w.r(p, v); }, a.V, c, b.chunk, b.sums + e, b.last + e);
    else wave_chunk_sums([&](int v, double& p, double& r) { p = w.p(v); r = 0.0; }, a.V, c, b.chunk, b.sums + e, b.last + e);
}

// One wave.  Inverse CDF over the weights whose chunk sums (x[g]: chunk 64 * g + lane, zero beyond the last chunk) and
// last ids of positive weight (lp[g], -1 for none) were left by sample_spread_kernel: smallest id whose running sum
// (chunks in index order, then lane segments of the crossing chunk, then single ids) exceeds u * total; the largest id
// of positive weight where rounding leaves no crossing; -1 if the total is zero.
constexpr int SPREAD_GROUPS64 = SPREAD_MAX_SLICES * 16 / 64;
template <class F>
__device__ int wave_inverse_cdf(F w, int V, double u, const double (&x)[SPREAD_GROUPS64], const int (&lp)[SPREAD_GROUPS64], int chunks,
                                int chunk) {
    const int lane = threadIdx.x & 63;
    // Running sums over the chunks, 64 at a time: an inclusive scan over the lanes on top of the sum of the groups in
    // front.  The total is the last running sum of the same arithmetic, so the search ends on it.
    double incl[SPREAD_GROUPS64], front[SPREAD_GROUPS64], total = 0.0;
    int last_all = -1;
#pragma unroll
    for (int g = 0; g < SPREAD_GROUPS64; ++g) {
        incl[g] = x[g];
        front[g] = total;
        if (g * 64 >= chunks) continue;  // wave-uniform: no chunk in this group
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double y = __shfl_up(incl[g], o, 64);
            if (lane >= o) incl[g] += y;
        }
        total += __shfl(incl[g], 63, 64);
        int l = lp[g];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) l = max(l, __shfl_xor(l, o, 64));
        last_all = max(last_all, l);
    }
    if (!(total > 0.0)) return -1;
    const double target = u * total;
    int owner = -1, owner_last = -1;
    double base = 0.0;
#pragma unroll
    for (int g = 0; g < SPREAD_GROUPS64; ++g) {
        const unsigned long long hit = __ballot(x[g] > 0.0 && front[g] + incl[g] > target);
        if (owner < 0 && hit) {
            const int hl = __ffsll((long long)hit) - 1;
            owner = g * 64 + hl;
            base = front[g] + __shfl(incl[g] - x[g], hl, 64);  // running sum in front of that chunk
            owner_last = __shfl(lp[g], hl, 64);
        }
    }
    if (owner < 0) return last_all;
    const int c0 = min(V, owner * chunk), c1 = min(V, c0 + chunk);
    const int per = chunk >> 6;
    const int s0 = min(c1, c0 + lane * per), s1 = min(c1, s0 + per);
    double seg = 0.0;
#pragma unroll 4
    for (int v = s0; v < s1; ++v) seg += w(v);
    double sincl = seg;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(sincl, o, 64);
        if (lane >= o) sincl += y;
    }
    const unsigned long long hit = __ballot(base + sincl > target);
    int tok = -1;
    if (hit) {
        const int hl = __ffsll((long long)hit) - 1;
        double before = base + __shfl(sincl - seg, hl, 64);  // running sum in front of that segment
        const int h0 = min(c1, c0 + hl * per), h1 = min(c1, h0 + per);
        for (int v0 = h0; v0 < h1 && tok < 0; v0 += 64) {
            const int v = v0 + lane;
            const double x = v < h1 ? w(v) : 0.0;
            double ix = x;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const double y = __shfl_up(ix, o, 64);
                if (lane >= o) ix += y;
            }
            const unsigned long long h2 = __ballot(before + ix > target);
            if (h2) tok = v0 + __ffsll((long long)h2) - 1;
            before += __shfl(ix, 63, 64);
        }
    }
    // the chunk sum crossed but, in this summation order, no prefix did: its last positive id
    return tok >= 0 ? tok : owner_last;
}

template <bool NUC>
__global__ __launch_bounds__(64) void sample_locate_kernel(SampleArgs a, SpreadBuf b, int self_commit, int32_t* prefix_len) {
    const int i = blockIdx.x;
    // the chunk records of both kinds of weights are requested before anything is known about the sequence
    const double* sums = b.sums + (size_t)i * b.chunks() * 2;
    const int32_t* last = b.last + (size_t)i * b.chunks() * 2;
    double xr[SPREAD_GROUPS64], xp[SPREAD_GROUPS64];
    int lr[SPREAD_GROUPS64], lq[SPREAD_GROUPS64];
#pragma unroll
    for (int g = 0; g < SPREAD_GROUPS64; ++g) {
        const int c = g * 64 + (int)threadIdx.x;
        const bool in = c < b.chunks();
        const int cc = in ? c : 0;
        xr[g] = sums[cc * 2];
        xp[g] = sums[cc * 2 + 1];
        lr[g] = last[cc * 2];
        lq[g] = last[cc * 2 + 1];
        if (!in) {
            xr[g] = 0.0;
            xp[g] = 0.0;
            lr[g] = -1;
            lq[g] = -1;
        }
    }
    const int acc_len = a.accept_len[i];
    double row_zmax, row_Z;
    row_stats_of(a, b.row_stats, a.judge_index(i, acc_len), row_zmax, row_Z);
    const TokenWeights<NUC> w(a, i, acc_len, row_zmax, row_Z);
    const double u = (double)a.u[i * (a.k + 1) + a.k];
    int tok = -1;
    if (w.qrow) {
        auto rw = [&](int v) { return w.r(w.p(v), v); };
        tok = wave_inverse_cdf(rw, a.V, u, xr, lr, b.chunks(), b.chunk);
    }
    if (tok < 0) {  // bonus token, or the residual vanished (p == q): draw from p
        auto pw = [&](int v) { return w.p(v); };
        tok = wave_inverse_cdf(pw, a.V, u, xp, lq, b.chunks(), b.chunk);
    }
    if (threadIdx.x == 0) {
        a.next_token[i] = tok;
        if (self_commit) {
            if (status_now(a.status) != 0) {
                write_failed_commit(a.commit, prefix_len, a.P);
            } else {
                a.commit[0] = 0;
                a.commit[1] = acc_len;
                a.commit[2] = tok;
                a.commit[3] = a.P + a.R + acc_len;
                if (prefix_len) *prefix_len = a.P + a.R + acc_len;
            }
        }
    }
}

// The sequential first-token rule of Alg. 2 over s candidate sequences: p_run (already filled with the
// judging distribution) is tested against each first token in index order and replaced by its normalised
// residual after every rejection.  Returns the accepted sequence or -1 (same value in every thread).
// Candidate i has token first_tok[i * tok_stride], draft distribution first_q + i * q_stride, uniform
// first_u[i * u_stride].
__device__ int sequential_first_tokens(double* p_run, int V, int s, const int32_t* first_tok, int tok_stride,
                                       const float* first_q, size_t q_stride, const float* first_u, int u_stride,
                                       double* sm_d) {
    const int tid = threadIdx.x;
    for (int i = 0; i < s; ++i) {
        int t = first_tok[i * tok_stride];
        t = t < 0 ? 0 : (t >= V ? V - 1 : t);
        const float* qrow = first_q + (size_t)i * q_stride;
        const double lhs = (double)first_u[i * u_stride] * (double)qrow[t];
        if (lhs < p_run[t]) return i;  // same value in every thread
        double sum = 0.0;
        for (int v = tid; v < V; v += SAMPLE_THREADS) sum += fmax(p_run[v] - (double)qrow[v], 0.0);
        const double Rm = block_sum_d(sum, sm_d);
        if (Rm > 0.0)
            for (int v = tid; v < V; v += SAMPLE_THREADS) p_run[v] = fmax(p_run[v] - (double)qrow[v], 0.0) / Rm;
        __syncthreads();
    }
    return -1;
}

template <bool NUC>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_paper_kernel(SampleArgs a) {
    __shared__ double sm_d[16];
    __shared__ int sm_i[4 + 16];
    __shared__ double sm_st[DUO_MAX_ROWS + 1][2];
    const SeqStats st{sm_st};
    const int tid = threadIdx.x;
    load_seq_stats(a, 0, 0, 0, st);  // the distribution that judges every first token
    fill_running_distribution<NUC>(a, st, 0, 0);
    const int sel = sequential_first_tokens(a.p_run, a.V, a.n, a.tokens, a.k, a.q, (size_t)a.k * a.V, a.u, a.k + 1, sm_d);
    int acc_len = 0, tok;
    if (sel < 0) {
        const double* pr = a.p_run;
        auto pw = [=](int v) { return pr[v]; };
        tok = block_inverse_cdf(pw, a.V, (double)a.u[(a.n - 1) * (a.k + 1) + a.k], sm_d, sm_i);
    } else {
        load_seq_stats(a, sel, 1, a.k, st);  // the rows of the selected sequence
        accept_flags<NUC>(a, st, sel, 1);
        acc_len = leading_accepts(a, sel, 1);
        tok = finish_token<NUC>(a, st, sel, acc_len, sm_d, sm_i);
    }
    for (int i = tid; i < a.n; i += SAMPLE_THREADS) {
        a.accept_len[i] = sel < 0 ? 0 : (i < sel ? 0 : (i == sel ? acc_len : -1));
        a.next_token[i] = i == sel ? tok : -1;
    }
    if (tid == 0) {
        a.commit[0] = sel;
        a.commit[1] = acc_len;
        a.commit[2] = tok;
        a.commit[3] = a.P + a.R + acc_len;
    }
}

// Alg. 2 as listed (one round of the pipelined loop): the k = l rows of the single sequence are the
// unverified suffix; after it, only the first tokens of s new sequences are judged.  One workgroup.
struct DeferredArgs {
    const int32_t* first_tokens;  // [s]
    const float* first_probs;     // [s][V]
    const float* uniforms_first;  // [s]
    int s;
    int32_t* prefix_len;  // device prefix length to advance, may be NULL (sampling only)
};

template <bool NUC>
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_deferred_kernel(SampleArgs a, DeferredArgs d) {
    __shared__ double sm_d[16];
    __shared__ int sm_i[4 + 16];
    __shared__ double sm_st[DUO_MAX_ROWS + 1][2];
    const SeqStats st{sm_st};
    const int tid = threadIdx.x;
    if (tid < d.s && a.status) {
        const int t = d.first_tokens[tid];
        if (t < 0 || t >= a.V) atomicOr(a.status, 1);
    }
    load_seq_stats(a, 0, 0, a.k, st);
    accept_flags<NUC>(a, st, 0, 0);
    const int acc_len = leading_accepts(a, 0, 0);
    int sel = -1, tok = -1;
    if (acc_len < a.k) {
        tok = finish_token<NUC>(a, st, 0, acc_len, sm_d, sm_i);  // residual draw at the first rejection
    } else {
        fill_running_distribution<NUC>(a, st, 0, a.k);  // the distribution after the last scored token
        sel = sequential_first_tokens(a.p_run, a.V, d.s, d.first_tokens, 1, d.first_probs, (size_t)a.V, d.uniforms_first, 1,
                                      sm_d);
        if (sel < 0) {
            const double* pr = a.p_run;
            auto pw = [=](int v) { return pr[v]; };
            tok = block_inverse_cdf(pw, a.V, (double)a.u[a.k], sm_d, sm_i);
        }
    }
    if (tid == 0) {  // the flags of this kernel's own token check were set before the barriers above
        a.accept_len[0] = acc_len;
        a.next_token[0] = tok;
        if (status_now(a.status) != 0) {
            write_failed_commit(a.commit, d.prefix_len, a.P);
        } else {
            a.commit[0] = sel;
            a.commit[1] = acc_len;
            a.commit[2] = tok;
            a.commit[3] = a.P + a.R + acc_len;
            if (d.prefix_len) *d.prefix_len = a.P + a.R + acc_len;
        }
    }
}

// ---- the sequential first-token rule for large vocabularies, spread over the chip --------------------------------
// sample_paper_kernel and sample_deferred_kernel are one workgroup, whose compute unit evaluates the vocabulary's
// double-precision exponentials and makes two passes over it per rejected candidate (128256 entries, four candidates:
// 395 us behind an LM head).  Here candidate i is judged by launch i (seq_stage_kernel) on G workgroups, each a slice of the
// vocabulary.  Every workgroup takes the decision for itself, from the same numbers; on a rejection it adds up its slice
// of the residual max(0, p_i - q_i), whose total the next launch needs for p_{i+1} = residual / total.  The running
// distribution itself is kept nowhere: an entry of p_i is evaluated from the logit, the draft distributions rejected so far and
// their totals, which for a handful of candidates is less work than a pass through memory.  Launches behind the decision
// return at once but cost 3 us each all the same, so there are at most b.stages of them, one per 8192 entries of the
// vocabulary, three at least and no more than SEQ_STAGES, and seq_tail_kernel, one workgroup with the running distribution in memory, judges the
// candidates beyond (a single one gets a launch of its own instead).  seq_locate_kernel draws the token from the sums of the launch that
// decided and writes the results.
struct SeqArgs {
    const int32_t* tok;  // candidate i: first token tok[i * tok_stride], draft distribution q + i * q_stride, uniform u[i * u_stride]
    int tok_stride;
    const float* q;
    size_t q_stride;
    const float* u;
    int u_stride;
    int s;
    int deferred;         // 0: the candidates are the call's n sequences; 1: Alg. 2 as listed (see DeferredArgs)
    int32_t* prefix_len;  // device prefix length (may be NULL); advanced here in the deferred form, by commit_kernel otherwise
};
constexpr int SEQ_MIN_VOCAB = 12288;  // below, and with more candidates up to 28672: sample_paper_kernel, sample_deferred_kernel
constexpr int SEQ_STAGES = 8;

struct SeqBuf {
    double* row_stats;  // merged statistics, or nullptr (see SpreadBuf)
    double* inv_total;  // [SEQ_STAGES] 1 / total of candidate i's residual; 0: the residual vanished, p_i stays
    int32_t* rec;       // [SEQ_STAGES + 1][8] what is known after launch i: {kind, selected, accepted length, launch, token}
    double* sums;       // [2][chunks][2] by launch parity: chunk sums as in SpreadBuf
    int32_t* last;      // [2][chunks][2]
    int G, chunk;
    int stages;         // launches of seq_stage_kernel when there are more candidates than that
    __host__ __device__ int chunks() const { return 16 * G; }
};
constexpr int SEQ_OPEN = 0;   // every candidate so far was rejected
constexpr int SEQ_DRAW = 1;   // the token is drawn from the sums of TokenWeights(selected or 0, accepted length)
constexpr int SEQ_TAKEN = 2;  // deferred: a candidate was accepted, no token
constexpr int SEQ_DONE = 3;   // the tail drew the token

// p_m(v) after the rejection of candidates 0 .. m-1
template <bool NUC>
struct ChainWeights {
    const TokenWeights<NUC>& base;
    const SeqArgs& d;
    const double* inv_total;
    int m;
    __device__ __forceinline__ double p(int v) const {
        double x = base.p(v);
        for (int i = 0; i < m; ++i) {
            const double c = inv_total[i];
            if (c > 0.0) x = fmax(x - (double)d.q[(size_t)i * d.q_stride + v], 0.0) * c;
        }
        return x;
    }
};

// total of a launch's residual chunk sums, by one wave in a fixed order -> its reciprocal, 0 where there is none
__device__ __forceinline__ double seq_inv_total(const SeqBuf& b, int launch) {
    const double* sums = b.sums + (size_t)(launch & 1) * b.chunks() * 2;
    double t = 0.0;
    for (int c = threadIdx.x & 63; c < b.chunks(); c += 64) t += sums[2 * c];
    t = wave_sum(t);
    return t > 0.0 ? 1.0 / t : 0.0;
}
__device__ __forceinline__ void seq_record(int32_t* rec, int kind, int sel, int acc_len, int launch, int tok) {
    rec[0] = kind;
    rec[1] = sel;
    rec[2] = acc_len;
    rec[3] = launch;
    rec[4] = tok;
}
__device__ __forceinline__ int first_token(const SeqArgs& d, int i, int V) {
    const int t = d.tok[i * d.tok_stride];
    return t < 0 ? 0 : (t >= V ? V - 1 : t);
}

// Rows j0 .. j1 of sequence i in st, then the leading accepts from position j0 on (same value in every thread).
template <bool NUC>
__device__ __forceinline__ int seq_accepts(const SampleArgs& a, const double* row_stats, int i, int j0, const SeqStats& st, int* sm_acc) {
    const int tid = threadIdx.x;
    if (row_stats) {
        if (tid >= j0 && tid <= a.k) {
            const double* rs = row_stats + 2 * (a.judge_index(i, tid) + 1);
            st.t[tid][0] = rs[0];
            st.t[tid][1] = rs[1];
        }
        __syncthreads();
    } else {
        load_seq_stats(a, i, j0, a.k, st);
    }
    if (tid >= j0 && tid < a.k) sm_acc[tid] = accept_flag<NUC>(a, st, i, tid);
    __syncthreads();
    int n = j0;
    while (n < a.k && sm_acc[n]) ++n;
    return n;
}

// grid (G): launch number `stage`, 0 .. min(candidates, b.stages) - 1 (deferred without candidates: launch 0 alone)
template <bool NUC>
__global__ __launch_bounds__(SAMPLE_THREADS) void seq_stage_kernel(SampleArgs a, SeqArgs d, SeqBuf b, int stage) {
    __shared__ double sm_st[DUO_MAX_ROWS + 1][2];
    __shared__ int sm_acc[DUO_MAX_ROWS];
    __shared__ double sm_inv[SEQ_STAGES], sm_row[2];
    const SeqStats st{sm_st};
    const int g = blockIdx.x, tid = threadIdx.x, wave = tid >> 6;
    const bool lead = g == 0 && tid == 0;
    int32_t* rec = b.rec + stage * 8;
    if (stage > 0) {
        const int32_t* prev = rec - 8;
        if (prev[0] != SEQ_OPEN) {  // same value in every thread of every workgroup
            if (lead) seq_record(rec, prev[0], prev[1], prev[2], prev[3], prev[4]);
            return;
        }
    } else if (d.deferred && g == 0 && tid < d.s && a.status) {
        const int t = d.tok[tid * d.tok_stride];
        if (t < 0 || t >= a.V) atomicOr(a.status, 1);
    }
    const int c = g * 16 + wave;
    const size_t e = ((size_t)(stage & 1) * b.chunks() + c) * 2;
    auto token_sums = [&](const TokenWeights<NUC>& w) {
        if (w.qrow) wave_chunk_sums([&](int v, double& p, double& r) { p = w.p(v); r = w.r(p, v); }, a.V, c, b.chunk, b.sums + e, b.last + e);
        else wave_chunk_sums([&](int v, double& p, double& r) { p = w.p(v); r = 0.0; }, a.V, c, b.chunk, b.sums + e, b.last + e);
    };
    if (d.deferred && stage == 0) {  // the unverified suffix comes first
        const int acc_len = seq_accepts<NUC>(a, b.row_stats, 0, 0, st, sm_acc);
        if (acc_len < a.k) {
            token_sums(TokenWeights<NUC>(a, 0, acc_len, sm_st[acc_len][0], sm_st[acc_len][1]));
            if (lead) seq_record(rec, SEQ_DRAW, -1, acc_len, stage, -1);
            return;
        }
    }
    const int jj = d.deferred ? a.k : 0;  // the row that judges the candidates
    if (wave == 0) {
        double zmax, Z;
        row_stats_of(a, b.row_stats, a.judge_index(0, jj), zmax, Z);
        if (tid == 0) {
            sm_row[0] = zmax;
            sm_row[1] = Z;
        }
    } else if (wave == 1 && stage > 0) {
        const double inv = seq_inv_total(b, stage - 1);
        if ((tid & 63) == 0) {
            sm_inv[stage - 1] = inv;
            if (g == 0) b.inv_total[stage - 1] = inv;
        }
    } else if (wave == 2 && (tid & 63) < stage - 1) {
        sm_inv[tid & 63] = b.inv_total[tid & 63];
    }
    __syncthreads();
    const TokenWeights<NUC> base(a, 0, jj, sm_row[0], sm_row[1]);
    const ChainWeights<NUC> w{base, d, sm_inv, stage};
    if (stage >= d.s) {  // no candidates at all (deferred): the token is drawn from the judging distribution
        wave_chunk_sums([&](int v, double& p, double& r) { p = w.p(v); r = 0.0; }, a.V, c, b.chunk, b.sums + e, b.last + e);
        if (lead) seq_record(rec, SEQ_OPEN, -1, jj, stage, -1);
        return;
    }
    const float* qrow = d.q + (size_t)stage * d.q_stride;
    const int t = first_token(d, stage, a.V);
    if ((double)d.u[stage * d.u_stride] * (double)qrow[t] < w.p(t)) {  // accepted; same outcome in every thread
        if (d.deferred) {
            if (lead) seq_record(rec, SEQ_TAKEN, stage, jj, stage, -1);
            return;
        }
        const int acc_len = seq_accepts<NUC>(a, b.row_stats, stage, 1, st, sm_acc);
        token_sums(TokenWeights<NUC>(a, stage, acc_len, sm_st[acc_len][0], sm_st[acc_len][1]));
        if (lead) seq_record(rec, SEQ_DRAW, stage, acc_len, stage, -1);
        return;
    }
    wave_chunk_sums([&](int v, double& p, double& r) { p = w.p(v); r = fmax(p - (double)qrow[v], 0.0); }, a.V, c, b.chunk, b.sums + e,
                    b.last + e);
    if (lead) seq_record(rec, SEQ_OPEN, -1, jj, stage, -1);
}

// More than b.stages candidates, none of the first b.stages accepted: the others one by one, the running distribution in
// p_run.  One workgroup.  The launches' scratch lies in p_run too: what is needed of it is read first, and the record of the
// outcome is written when the running distribution has served.
template <bool NUC>
__global__ __launch_bounds__(SAMPLE_THREADS) void seq_tail_kernel(SampleArgs a, SeqArgs d, SeqBuf b) {
    __shared__ double sm_d[16];
    __shared__ int sm_i[4 + 16];
    __shared__ double sm_st[DUO_MAX_ROWS + 1][2], sm_all[DUO_MAX_ROWS + 2][2];
    __shared__ double sm_inv[SEQ_STAGES], sm_row[2];
    const SeqStats st{sm_st};
    const int tid = threadIdx.x, wave = tid >> 6;
    int32_t* rec = b.rec + b.stages * 8;
    const int32_t* prev = rec - 8;
    if (prev[0] != SEQ_OPEN) {
        if (tid == 0) seq_record(rec, prev[0], prev[1], prev[2], prev[3], prev[4]);
        return;
    }
    const int jj = d.deferred ? a.k : 0;
    if (wave == 0) {
        double zmax, Z;
        row_stats_of(a, b.row_stats, a.judge_index(0, jj), zmax, Z);
        if (tid == 0) {
            sm_row[0] = zmax;
            sm_row[1] = Z;
        }
    } else if (wave == 1) {
        const double inv = seq_inv_total(b, b.stages - 1);
        if ((tid & 63) == 0) sm_inv[b.stages - 1] = inv;
    } else if (wave == 2 && (tid & 63) < b.stages - 1) {
        sm_inv[tid & 63] = b.inv_total[tid & 63];
    }
    if (b.row_stats && tid <= a.R + a.n * a.k) {
        sm_all[tid][0] = b.row_stats[2 * tid];
        sm_all[tid][1] = b.row_stats[2 * tid + 1];
    }
    __syncthreads();
    {
        const TokenWeights<NUC> base(a, 0, jj, sm_row[0], sm_row[1]);
        const ChainWeights<NUC> w{base, d, sm_inv, b.stages};
        for (int v = tid; v < a.V; v += SAMPLE_THREADS) a.p_run[v] = w.p(v);
    }
    __syncthreads();
    int sel = sequential_first_tokens(a.p_run, a.V, d.s - b.stages, d.tok + b.stages * d.tok_stride, d.tok_stride,
                                      d.q + (size_t)b.stages * d.q_stride, d.q_stride, d.u + b.stages * d.u_stride, d.u_stride, sm_d);
    int acc_len = jj, tok = -1;
    if (sel < 0) {
        const double* pr = a.p_run;
        auto pw = [=](int v) { return pr[v]; };
        tok = block_inverse_cdf(pw, a.V, (double)a.u[(a.n - 1) * (a.k + 1) + a.k], sm_d, sm_i);
    } else {
        sel += b.stages;
        if (!d.deferred) {
            if (b.row_stats) {
                if (tid >= 1 && tid <= a.k) {
                    sm_st[tid][0] = sm_all[a.judge_index(sel, tid) + 1][0];
                    sm_st[tid][1] = sm_all[a.judge_index(sel, tid) + 1][1];
                }
                __syncthreads();
            } else {
                load_seq_stats(a, sel, 1, a.k, st);
            }
            accept_flags<NUC>(a, st, sel, 1);
            acc_len = leading_accepts(a, sel, 1);
            tok = finish_token<NUC>(a, st, sel, acc_len, sm_d, sm_i);
        }
    }
    __syncthreads();  // nobody reads the running distribution any more
    if (tid == 0) seq_record(rec, SEQ_DONE, sel, acc_len, b.stages, tok);
}

// One wave.  `rec`: the record of the last launch (or the tail's); launches: stage launches made.
template <bool NUC>
__global__ __launch_bounds__(64) void seq_locate_kernel(SampleArgs a, SeqArgs d, SeqBuf b, const int32_t* rec, int launches) {
    const int lane = threadIdx.x;
    const int kind = rec[0], sel = rec[1], acc_len = rec[2], launch = rec[3];
    int tok = rec[4];
    if (kind == SEQ_OPEN || kind == SEQ_DRAW) {
        const double* sums = b.sums + (size_t)(launch & 1) * b.chunks() * 2;
        const int32_t* last = b.last + (size_t)(launch & 1) * b.chunks() * 2;
        double xr[SPREAD_GROUPS64], xp[SPREAD_GROUPS64];
        int lr[SPREAD_GROUPS64], lq[SPREAD_GROUPS64];
#pragma unroll
        for (int g = 0; g < SPREAD_GROUPS64; ++g) {
            const int c = g * 64 + lane;
            const bool in = c < b.chunks();
            const int cc = in ? c : 0;
            xr[g] = in ? sums[cc * 2] : 0.0;
            xp[g] = in ? sums[cc * 2 + 1] : 0.0;
            lr[g] = in ? last[cc * 2] : -1;
            lq[g] = in ? last[cc * 2 + 1] : -1;
        }
        const bool open = kind == SEQ_OPEN;
        const int i = open ? 0 : max(sel, 0), j = open ? (d.deferred ? a.k : 0) : acc_len;
        double zmax, Z;
        row_stats_of(a, b.row_stats, a.judge_index(i, j), zmax, Z);
        const TokenWeights<NUC> w(a, i, j, zmax, Z);
        const ChainWeights<NUC> ch{w, d, b.inv_total, open ? launches - 1 : 0};
        const float* qrow = open ? (d.s > 0 ? d.q + (size_t)(launches - 1) * d.q_stride : nullptr) : w.qrow;
        const int ui = open ? a.n - 1 : i;
        const double u = (double)a.u[ui * (a.k + 1) + a.k];
        auto pw = [&](int v) { return ch.p(v); };
        if (qrow) {
            auto rw = [&](int v) { return fmax(ch.p(v) - (double)qrow[v], 0.0); };
            tok = wave_inverse_cdf(rw, a.V, u, xr, lr, b.chunks(), b.chunk);
        }
        if (tok < 0) tok = wave_inverse_cdf(pw, a.V, u, xp, lq, b.chunks(), b.chunk);  // nothing to subtract, or the residual vanished
    }
    if (d.deferred) {
        if (lane == 0) {
            a.accept_len[0] = acc_len;
            a.next_token[0] = tok;
        }
    } else {
        for (int i = lane; i < a.n; i += 64) {
            a.accept_len[i] = sel < 0 ? 0 : (i < sel ? 0 : (i == sel ? acc_len : -1));
            a.next_token[i] = i == sel ? tok : -1;
        }
    }
    if (lane == 0) {
        if (status_now(a.status) != 0) {
            write_failed_commit(a.commit, d.prefix_len, a.P);
        } else {
            a.commit[0] = sel;
            a.commit[1] = acc_len;
            a.commit[2] = tok;
            a.commit[3] = a.P + a.R + acc_len;
            if (d.deferred && d.prefix_len) *d.prefix_len = a.P + a.R + acc_len;
        }
    }
}

struct CommitArgs {
    u16* kc;  // [L][Hkv] planes of max_seq * D elements, tiled layouts (k_cache_offset, v_cache_offset)
    u16* vc;
    int Hkv, D, max_seq;
    int P, R, n, k, mode;
    const int32_t* accept_len;
    const int32_t* next_token;
    int32_t* commit;
    int32_t* prefix_len;  // may be NULL (sampling only)
    int32_t* status;
};

// grid (Hkv, L) for the copy; (1, 1) when there is no cache.  In longest mode every workgroup
// recomputes the (cheap) selection; workgroup (0, 0) publishes it.  A pass whose status word is not clean moves
// nothing and leaves the prefix length alone.
__global__ __launch_bounds__(256) void commit_kernel(CommitArgs a) {
    if (status_now(a.status) != 0) {  // same value in every workgroup: all flags were set by earlier kernels
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) write_failed_commit(a.commit, a.prefix_len, a.P);
        return;
    }
    int sel, len, tok;
    if (a.mode == 0) {
        sel = 0;
        len = a.accept_len[0];
        for (int i = 1; i < a.n; ++i)
            if (a.accept_len[i] > len) {
                len = a.accept_len[i];
                sel = i;
            }
        tok = a.next_token[sel];
    } else {
        sel = a.commit[0];
        len = a.commit[1];
        tok = a.commit[2];
    }
    const int newP = a.P + a.R + len;
    if (a.kc && sel > 0 && len > 0) {
        const int hk = blockIdx.x, l = blockIdx.y;
        const int src = a.P + a.R + sel * a.k, dst = a.P + a.R;
        u16* kp = a.kc + ((size_t)l * a.Hkv + hk) * a.max_seq * a.D;
        u16* vp = a.vc + ((size_t)l * a.Hkv + hk) * a.max_seq * a.D;
        // source rows [src, src + len) and destination rows [dst, dst + len) never overlap: src - dst = sel * k >= len
        for (int e = threadIdx.x; e < len * a.D; e += 256) {
            const int j = e / a.D, d = e - j * a.D;
            kp[k_cache_offset(a.D, dst + j, d)] = kp[k_cache_offset(a.D, src + j, d)];
            vp[v_cache_offset(a.D, dst + j, d)] = vp[v_cache_offset(a.D, src + j, d)];
        }
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        if (a.mode == 0) {
            a.commit[0] = sel;
            a.commit[1] = len;
            a.commit[2] = tok;
            a.commit[3] = newP;
        }
        if (a.prefix_len) *a.prefix_len = newP;
    }
}

// Prefill bookkeeping: all m rows join the prefix, the last row's logits become the root logits.  Nothing is
// changed when the pass's status word is not clean.
__global__ void prefill_finish_kernel(const float* __restrict__ last_logits, float* __restrict__ root_logits, int V,
                                      int32_t* prefix_len, int newP, int32_t* status) {
    if (status_now(status) != 0) return;
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < V) root_logits[v] = last_logits[v];
    if (v == 0) *prefix_len = newP;
}
