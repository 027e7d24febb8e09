// Statistical draft model at the bottom of the cascade: Max-Gram matching with a bigram
// fallback (Section 3.3, Appendix A).  Integer-only; one workgroup per sequence.
#include "csd_internal.h"

#define DRAFT_THREADS 256
#define FIT_THREADS 1024

// Max over the first `waves` waves of the workgroup of a 64-bit key; every thread of them gets the result.
__device__ __forceinline__ unsigned long long block_max_u64(unsigned long long v, unsigned long long *red, int waves) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        unsigned long long other = __shfl_xor(v, o, 64);
        v = other > v ? other : v;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    unsigned long long t = red[0];
    for (int i = 1; i < waves; i++) t = red[i] > t ? red[i] : t;
    return t;
}

// Rows with room for more than DRAFT_FEW tokens take workgroups of 1024 threads, which bring a sequence of up to DRAFT_LDS tokens to LDS: every
// thread compares positions backwards, a chain of dependent reads that cost a trip to L2 each where they go to memory (4000 tokens 6.1 us with
// 256 threads that read memory, 4.8 in LDS with 1024; 8000 tokens 10.0 and 5.9).  Longer sequences are read where they are (20000 tokens, 256 and 1024
// threads 21.3 and 9.6).  Up to DRAFT_FEW tokens 256 threads that read memory are the faster form (500 tokens 2.7 us against 4.2, 2040 3.7 against
// 4.4), and in a row with room for more the other waves leave at once (500 tokens 2.9 and 4.1).
#define DRAFT_LONG_THREADS 1024
#define DRAFT_FEW 2048
#define DRAFT_LDS 8192

// Each thread scores candidate match ends e = tid, tid + threads, ... <= len - 2 by comparing
// backwards against the suffix; the key (match length, ~e) makes the block maximum the
// longest match and, among equals, the left-most end.
__device__ __forceinline__ unsigned long long match_key(const int32_t *s, int len, int32_t max_match, int threads) {
    unsigned long long best = 0ull;
    for (int e = threadIdx.x; e <= len - 2; e += threads) {
        int r = 0;
        while (r <= e && (max_match <= 0 || r < max_match) && s[e - r] == s[len - 1 - r]) r++;
        if (r > 0) {
            unsigned long long key = ((unsigned long long)(uint32_t)r << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)e);
            best = key > best ? key : best;
        }
    }
    return best;
}
// How many threads of a workgroup of T work on a sequence of `len` tokens: the others leave.
template <int T>
__device__ __forceinline__ int draft_threads(int len) { return T > DRAFT_THREADS && len <= DRAFT_FEW ? DRAFT_THREADS : T; }
// The first tokens of a row, requested before the length is known: a pass over a row that no cache holds waits for memory once, not twice.
template <int T>
struct DraftEarly {
    static constexpr int N = T > DRAFT_THREADS ? 4 : DRAFT_FEW / T;
    int32_t v[N];
    __device__ __forceinline__ void request(const int32_t *s, int32_t stride) {
#pragma unroll
        for (int i = 0; i < N; i++) v[i] = s[min(i * T + (int)threadIdx.x, stride - 1)];
    }
};
// The longest match of the suffix of s[0 .. len); every one of the first `threads` threads (no others are left) gets the key (0: none).
template <int T>
__device__ __forceinline__ unsigned long long draft_match(const int32_t *s, const DraftEarly<T> &early, int len, int32_t max_match, int threads) {
    __shared__ unsigned long long red[T / 64];
    unsigned long long best;
    if (T > DRAFT_THREADS && len > DRAFT_FEW && len <= DRAFT_LDS) {      // uniform
        __shared__ int32_t row[T > DRAFT_THREADS ? DRAFT_LDS : 1];
#pragma unroll
        for (int i = 0; i < early.N; i++)
            if (i * T + (int)threadIdx.x < len) row[i * T + threadIdx.x] = early.v[i];
        for (int x = early.N * T + threadIdx.x; x < len; x += T) row[x] = s[x];
        __syncthreads();
        best = match_key(row, len, max_match, T);
    } else {
        best = match_key(s, len, max_match, threads);
#pragma unroll
        for (int i = 0; i < early.N; i++) asm volatile("" : : "v"(early.v[i]));          // (read for the caches)
    }
    return block_max_u64(best, red, threads / 64);
}

template <int T>
__global__ __launch_bounds__(T) void k_bigram_draft(
    const int32_t *__restrict__ ctx, const int32_t *__restrict__ ctx_len, int32_t ctx_stride,
    const int32_t *__restrict__ next_table, int32_t vocab, int32_t k, int32_t max_match,
    int32_t *__restrict__ out_tokens, int32_t *__restrict__ out_match_len) {
    const int b = blockIdx.x;
    const int32_t *s = ctx + (size_t)b * ctx_stride;
    DraftEarly<T> early;
    early.request(s, ctx_stride);
    int len = ctx_len[b];
    int32_t *out = out_tokens + (size_t)b * k;
    if (len < 1 || len > ctx_stride) {   // device-side guard: no valid context
        for (int j = threadIdx.x; j < k; j += T) out[j] = -1;
        if (out_match_len && threadIdx.x == 0) out_match_len[b] = 0;
        return;
    }
    const int threads = draft_threads<T>(len);
    if ((int)threadIdx.x >= threads) return;
    const unsigned long long best = draft_match<T>(s, early, len, max_match, threads);
    const int mlen = (int)(best >> 32);
    if (out_match_len && threadIdx.x == 0) out_match_len[b] = mlen;
    if (mlen == 0) {
        if (threadIdx.x == 0) {          // bigram chain from the last token
            int32_t cur = s[len - 1];
            for (int j = 0; j < k; j++) {
                cur = (cur >= 0 && cur < vocab) ? next_table[cur] : -1;
                out[j] = cur;
            }
        }
        return;
    }
    const int e = (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull));
    const int period = len - (e + 1);   // >= 1: the sequence extended by its own draft repeats with this period
    for (int j = threadIdx.x; j < k; j += threads) out[j] = s[e + 1 + (j % period)];
}

// k_bigram_draft that appends its drafts to the context itself (device-resident cascade control): sequences whose
// drafts in flight already number `need` or more (counted from start_len) are left alone.
template <int T>
__global__ __launch_bounds__(T) void k_bigram_draft_append(
    int32_t *ctx, int32_t ctx_stride, int32_t *__restrict__ ctx_len, const int32_t *__restrict__ next_table,
    int32_t vocab, int32_t k, int32_t max_match, const int32_t *__restrict__ gate, uint8_t *__restrict__ q_onehot_tab,
    const int32_t *__restrict__ q_base, int32_t q_stride) {
    const int b = blockIdx.x;
    int32_t *s = ctx + (size_t)b * ctx_stride;
    DraftEarly<T> early;
    early.request(s, ctx_stride);
    const int len = ctx_len[b];
    bool active = len >= 1 && len + k < ctx_stride && (!gate || gate[b] >= 0);
    if (active && q_onehot_tab && (len - q_base[b] < 0 || len + k - q_base[b] > q_stride)) active = false;
    if (!active) return;                                     // uniform over the workgroup
    const int threads = draft_threads<T>(len);
    if ((int)threadIdx.x >= threads) return;
    const unsigned long long best = draft_match<T>(s, early, len, max_match, threads);   // (its barriers: every thread has read the context by now)
    const int mlen = (int)(best >> 32);
    int32_t *out = s + len;
    if (mlen == 0) {
        if (threadIdx.x == 0) {                              // bigram chain from the last token
            int32_t cur = s[len - 1];
            for (int j = 0; j < k; j++) {
                cur = (cur >= 0 && cur < vocab) ? next_table[cur] : -1;
                out[j] = cur;
            }
        }
    } else {
        const int e = (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull));
        const int period = len - (e + 1);                    // sources s[e + 1 ..  len - 1] lie before the drafts
        for (int j = threadIdx.x; j < k; j += threads) out[j] = s[e + 1 + (j % period)];
    }
    if (q_onehot_tab)
        for (int j = threadIdx.x; j < k; j += threads) q_onehot_tab[(size_t)b * q_stride + len + j - q_base[b]] = 1;
    if (threadIdx.x == 0) ctx_len[b] = len + k;
}

// gate[b] = ctx_len[b] when sequence b still needs tokens in the loop that started at loop_start[b] (fewer than `need`
// exist) and the enclosing step is itself active (parent_gate null or >= 0); else -1.  A step gated with this value
// reviews drafts that start at that position.
__global__ void k_cascade_gate(const int32_t *__restrict__ ctx_len, const int32_t *__restrict__ loop_start, int32_t need,
                               const int32_t *__restrict__ parent_gate, int32_t B, int32_t *__restrict__ gate) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const bool on = (!parent_gate || parent_gate[b] >= 0) && (!loop_start || ctx_len[b] - loop_start[b] < need);
    gate[b] = on ? ctx_len[b] : -1;
}

// Max-Gram with the haystack apart from the needle (Appendix A's own signature: the encoder's ids are searched
// for the longest suffix of the decoder's ids).  Candidate match ends are all haystack positions; the key is
// the same (match length, ~end).  The continuation is copied while the haystack lasts (out_n_copied of the k
// tokens: what Appendix A returns); the rest chains the bigram table from the last token so far.
__global__ __launch_bounds__(DRAFT_THREADS) void k_maxgram_enc(
    const int32_t *__restrict__ hay, const int32_t *__restrict__ hay_len, int32_t hay_stride,
    const int32_t *__restrict__ needle, const int32_t *__restrict__ needle_len, int32_t needle_stride,
    const int32_t *__restrict__ next_table, int32_t vocab, int32_t k, int32_t max_match,
    int32_t *__restrict__ out_tokens, int32_t *__restrict__ out_match_len, int32_t *__restrict__ out_n_copied) {
    __shared__ unsigned long long red[DRAFT_THREADS / 64];
    const int b = blockIdx.x;
    const int32_t *h = hay + (size_t)b * hay_stride;
    const int32_t *s = needle + (size_t)b * needle_stride;
    const int hl = hay_len[b], len = needle_len[b];
    int32_t *out = out_tokens + (size_t)b * k;
    if (len < 1 || len > needle_stride || hl < 0 || hl > hay_stride) {   // device-side guard: no valid input
        for (int j = threadIdx.x; j < k; j += blockDim.x) out[j] = -1;
        if (threadIdx.x == 0) {
            if (out_match_len) out_match_len[b] = 0;
            if (out_n_copied) out_n_copied[b] = 0;
        }
        return;
    }
    unsigned long long best = 0ull;
    for (int e = threadIdx.x; e < hl; e += blockDim.x) {
        int r = 0;
        while (r <= e && r < len && (max_match <= 0 || r < max_match) && h[e - r] == s[len - 1 - r]) r++;
        if (r > 0) {
            unsigned long long key = ((unsigned long long)(uint32_t)r << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)e);
            best = key > best ? key : best;
        }
    }
    best = block_max_u64(best, red, DRAFT_THREADS / 64);
    const int mlen = (int)(best >> 32);
    const int e = mlen ? (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull)) : hl - 1;
    const int n_copied = mlen ? min(k, hl - 1 - e) : 0;
    for (int j = threadIdx.x; j < n_copied; j += blockDim.x) out[j] = h[e + 1 + j];
    if (threadIdx.x == 0) {
        if (out_match_len) out_match_len[b] = mlen;
        if (out_n_copied) out_n_copied[b] = n_copied;
        int32_t cur = n_copied > 0 ? h[e + n_copied] : s[len - 1];
        for (int j = n_copied; j < k; j++) {
            cur = (cur >= 0 && cur < vocab) ? next_table[cur] : -1;
            out[j] = cur;
        }
    }
}

// Bigram fit, one workgroup, everything in LDS.  A hash table over positions gives every pair (s[i], s[i+1]) one
// representative position, where its occurrences are counted and the last one is noted: key = count << 13 | last
// position.  A second pass of the same table over the first tokens gives the pair with the largest key per token, which
// is the fitted successor.  Linear probing over at least 1.5 slots per position, so a probe always finds its key or a free slot;
// three where they fit, since a wave waits for its longest probe: 4000 tokens 15.6 us with 1.5, 9.4 with three.
// Latency of a few dependent LDS operations per position bounds it, eight positions per thread at most (all probes of a
// thread in flight together, turn by turn: 30 us, the turns cost more than the latency they hide).
#define FIT_MAX 8192
#define FIT_EMPTY (-1)
#define FIT_SLOTS ((uint32_t)FIT_MAX * 3 / 2)
struct FitShared {
    int32_t s[FIT_MAX];
    union {                             // representative position, or FIT_EMPTY
        int32_t slot[FIT_SLOTS];
        int4 slot4[FIT_SLOTS / 4];
    };
    uint32_t key[FIT_MAX];              // of the pair whose representative is this position
    uint32_t best[FIT_MAX];             // largest key among the pairs whose first token has this representative
};
__device__ __forceinline__ uint32_t fit_hash(uint32_t a, uint32_t b, uint32_t n_slots) {
    uint32_t h = a * 0x9E3779B1u + b * 0x85EBCA77u;
    h = (h ^ (h >> 15)) * 0x2C1B3C6Du;
    return __umulhi(h ^ (h >> 13), n_slots);
}
// The representative of position i among the positions with the same first token (PAIR: and the same second one).
template <bool PAIR>
__device__ __forceinline__ int fit_representative(FitShared &S, int i, uint32_t n_slots) {
    const int32_t a = S.s[i], b = PAIR ? S.s[i + 1] : 0;
    uint32_t h = fit_hash((uint32_t)a, (uint32_t)b, n_slots);
    for (;;) {
        const int r = atomicCAS(&S.slot[h], FIT_EMPTY, i);
        if (r == FIT_EMPTY) return i;
        if (S.s[r] == a && (!PAIR || S.s[r + 1] == b)) return r;
        if (++h == n_slots) h = 0;
    }
}
__global__ __launch_bounds__(FIT_THREADS) void k_bigram_fit(const int32_t *__restrict__ s, int32_t n, int32_t vocab,
                                                            int32_t *__restrict__ next_table) {
    __shared__ FitShared S;
    constexpr int PER = FIT_MAX / FIT_THREADS;
    const uint32_t n_slots = min(3u * (uint32_t)n + 1u, FIT_SLOTS);
    for (int i = threadIdx.x; i < n; i += FIT_THREADS) {
        S.s[i] = s[i];
        S.key[i] = S.best[i] = 0u;
    }
    for (uint32_t i = threadIdx.x; i < (n_slots + 3) / 4; i += FIT_THREADS) S.slot4[i] = make_int4(FIT_EMPTY, FIT_EMPTY, FIT_EMPTY, FIT_EMPTY);
    __syncthreads();
    int rep[PER];                                            // of this thread's positions; -1: not a pair of known tokens
#pragma unroll
    for (int p = 0; p < PER; p++) {
        const int i = p * FIT_THREADS + (int)threadIdx.x;
        rep[p] = -1;
        if (i < n - 1 && (uint32_t)S.s[i] < (uint32_t)vocab && (uint32_t)S.s[i + 1] < (uint32_t)vocab) {
            rep[p] = fit_representative<true>(S, i, n_slots);
            atomicAdd(&S.key[rep[p]], 1u << 13);
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; p++)
        if (rep[p] >= 0)                                     // (the count no longer changes; only the position below it does)
            atomicMax(&S.key[rep[p]], (S.key[rep[p]] & ~(uint32_t)(FIT_MAX - 1)) | (uint32_t)(p * FIT_THREADS + (int)threadIdx.x));
    for (uint32_t i = threadIdx.x; i < (n_slots + 3) / 4; i += FIT_THREADS) S.slot4[i] = make_int4(FIT_EMPTY, FIT_EMPTY, FIT_EMPTY, FIT_EMPTY);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; p++) {
        const int i = p * FIT_THREADS + (int)threadIdx.x;
        if (rep[p] == i) {                                   // one thread per pair
            rep[p] = fit_representative<false>(S, i, n_slots);
            atomicMax(&S.best[rep[p]], S.key[i]);
        } else {
            rep[p] = -1;
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; p++) {
        const int i = p * FIT_THREADS + (int)threadIdx.x;
        if (rep[p] == i) next_table[S.s[i]] = S.s[(S.best[i] & (uint32_t)(FIT_MAX - 1)) + 1];
    }
}

extern "C" int32_t csd_bigram_fit(const int32_t *tokens, int32_t n, int32_t vocab, int32_t *next_table, void *stream) {
    if (!tokens || !next_table) return CSD_ENULL;
    if (n < 0 || vocab < 1) return CSD_EINVAL;
    if (n > FIT_MAX) return CSD_ESHAPE;
    if (n < 2) return CSD_OK;
    hipLaunchKernelGGL(k_bigram_fit, dim3(1), dim3(FIT_THREADS), 0, (hipStream_t)stream, tokens, n, vocab, next_table);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

extern "C" int32_t csd_bigram_draft(const int32_t *ctx, const int32_t *ctx_len, int32_t B, int32_t ctx_stride,
                                    const int32_t *next_table, int32_t vocab, int32_t k, int32_t max_match,
                                    int32_t *out_tokens, int32_t *out_match_len, void *stream) {
    if (!ctx || !ctx_len || !next_table) return CSD_ENULL;
    if (B < 0 || k < 0 || vocab < 1 || ctx_stride < 1) return CSD_EINVAL;
    if (k > 0 && !out_tokens) return CSD_ENULL;
    if (B == 0 || (k == 0 && !out_match_len)) return CSD_OK;   // k == 0 still reports match lengths
    const bool few = ctx_stride <= DRAFT_FEW;
    hipLaunchKernelGGL((few ? k_bigram_draft<DRAFT_THREADS> : k_bigram_draft<DRAFT_LONG_THREADS>), dim3(B), dim3(few ? DRAFT_THREADS : DRAFT_LONG_THREADS), 0,
                       (hipStream_t)stream, ctx, ctx_len, ctx_stride, next_table, vocab, k, max_match, out_tokens, out_match_len);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

extern "C" int32_t csd_maxgram_draft(const int32_t *haystack, const int32_t *haystack_len, int32_t haystack_stride,
                                     const int32_t *needle, const int32_t *needle_len, int32_t needle_stride, int32_t B,
                                     const int32_t *next_table, int32_t vocab, int32_t k, int32_t max_match,
                                     int32_t *out_tokens, int32_t *out_match_len, int32_t *out_n_copied, void *stream) {
    if (!haystack || !haystack_len || !needle || !needle_len || !next_table) return CSD_ENULL;
    if (B < 0 || k < 0 || vocab < 1 || haystack_stride < 1 || needle_stride < 1) return CSD_EINVAL;
    if (k > 0 && !out_tokens) return CSD_ENULL;
    if (B == 0 || (k == 0 && !out_match_len && !out_n_copied)) return CSD_OK;
    hipLaunchKernelGGL(k_maxgram_enc, dim3(B), dim3(DRAFT_THREADS), 0, (hipStream_t)stream, haystack, haystack_len,
                       haystack_stride, needle, needle_len, needle_stride, next_table, vocab, k, max_match, out_tokens,
                       out_match_len, out_n_copied);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

extern "C" int32_t csd_bigram_draft_append(int32_t *ctx, int32_t ctx_stride, int32_t *ctx_len, int32_t B,
                                           const int32_t *next_table, int32_t vocab, int32_t k, int32_t max_match,
                                           const int32_t *gate, uint8_t *q_onehot_tab, const int32_t *q_base,
                                           int32_t q_stride, void *stream) {
    if (!ctx || !ctx_len || !next_table) return CSD_ENULL;
    if (B < 0 || k < 0 || vocab < 1 || ctx_stride < 1) return CSD_EINVAL;
    if (q_onehot_tab && (!q_base || q_stride < 1)) return CSD_EINVAL;
    if (B == 0) return CSD_OK;
    const bool few = ctx_stride <= DRAFT_FEW;
    hipLaunchKernelGGL((few ? k_bigram_draft_append<DRAFT_THREADS> : k_bigram_draft_append<DRAFT_LONG_THREADS>), dim3(B),
                       dim3(few ? DRAFT_THREADS : DRAFT_LONG_THREADS), 0, (hipStream_t)stream, ctx, ctx_stride, ctx_len, next_table, vocab, k, max_match,
                       gate, q_onehot_tab, q_base, q_stride);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

extern "C" int32_t csd_cascade_gate(const int32_t *ctx_len, const int32_t *loop_start, int32_t need, const int32_t *parent_gate,
                                    int32_t B, int32_t *gate, void *stream) {
    if (!ctx_len || !gate) return CSD_ENULL;
    if (B < 0) return CSD_EINVAL;
    if (B == 0) return CSD_OK;
    hipLaunchKernelGGL(k_cascade_gate, dim3((B + 63) / 64), dim3(64), 0, (hipStream_t)stream, ctx_len, loop_start, need, parent_gate,
                       B, gate);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}
