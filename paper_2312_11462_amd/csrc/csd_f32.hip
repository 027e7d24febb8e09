// Forward of fp32 models (arch 0) and the GEMM of every model that is not on the matrix cores: row-major weights, fp32
// activations.
//
// Such models are small (tests, the tiny configuration), so a launch is bound by the chain of memory round trips of a
// thread, not by bandwidth.  One thread per output column that walks all of K takes K dependent rounds (41 us a launch at
// the tiny shape, K = 64 and 256); here K is split over the eight waves of a workgroup, a wave requests eight rows of its
// slice at once, the eight partial sums meet in LDS, and whatever follows a GEMM (rotary embedding and cache append, residual
// sum, gated activation, the scale of the folded norm) runs on them in the same kernel, which computes the norm of its input
// rows along the way: five launches per layer of 3 to 6 us.  Tiny shape, verify step, before the small models got a form of their own
// (below; the tiny shape runs here only while the profile is on): 363 -> 67 us.
#include <cmath>

#include <type_traits>

#include "csd_internal.h"

#define FG_WAVES 8
#define FG_THREADS (FG_WAVES * 64)
#define FG_ROWS 8             /* block rows per workgroup: one per wave in the epilogue */

enum { FG_PART = 0, FG_QKV = 1, FG_RESID = 2, FG_GU = 3, FG_LOGITS = 4 };

struct F32Gemm {
    const void *W;            // [K][N] row-major
    int K, N, M;
    const float *src;         // [M][K]
    const float *gain;        // folded norm: the input is src * gain, the sums are scaled by 1 / rms(src row); or null
    float eps;
    float *out;               // FG_PART, FG_LOGITS: [M][N]; FG_RESID: added to [M][N]; FG_GU: [M][N / 2]
    // FG_QKV
    int m, layer;
    const int32_t *cache_len;
    KvGeom geo;
    const float2 *rope;       // [M][dh / 2]
    float *q, *kv;
};

// Which column of the matrix a lane takes; -1: none.  QKV: the first workgroups take 32 rotary pairs of q each (lane l and
// lane l + 32 the two halves of a pair), the next ones those of k, the rest 64 columns of v; gate|up: 32 features, the
// gate column in lane l, the up column in lane l + 32.
template <int EPI>
__device__ __forceinline__ int fg_column(const F32Gemm &P, int bx, int lane) {
    if (EPI == FG_QKV) {
        const int hd = P.geo.H * P.geo.dh, half = P.geo.dh / 2, nb = (hd / 2 + 31) / 32;
        if (bx < 2 * nb) {
            const int pair = bx % nb * 32 + (lane & 31);
            return pair < hd / 2 ? bx / nb * hd + pair / half * P.geo.dh + pair % half + (lane >> 5) * half : -1;
        }
        const int c = (bx - 2 * nb) * 64 + lane;
        return c < hd ? 2 * hd + c : -1;
    }
    if (EPI == FG_GU) {
        const int j = bx * 32 + (lane & 31);
        return j < P.N / 2 ? j + (lane >> 5) * (P.N / 2) : -1;
    }
    const int c = bx * 64 + lane;
    return c < P.N ? c : -1;
}

template <typename TW, int EPI, bool NORM>
__global__ __launch_bounds__(FG_THREADS) void k_f32_gemm(const F32Gemm P) {
    __shared__ float red[FG_WAVES][FG_ROWS][64];
    __shared__ float red_ss[FG_WAVES][FG_ROWS];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r0 = blockIdx.y * FG_ROWS;
    const int col = fg_column<EPI>(P, blockIdx.x, lane);
    const TW *__restrict__ W = (const TW *)P.W + max(col, 0);
    const float *__restrict__ src = P.src;
    const float *__restrict__ gain = P.gain;
    const int k0 = (int)((long long)P.K * w / FG_WAVES), k1 = (int)((long long)P.K * (w + 1) / FG_WAVES);
    float acc[FG_ROWS], ss[FG_ROWS];
    size_t ro[FG_ROWS];                                      // rows past the block are read as its last one
#pragma unroll
    for (int r = 0; r < FG_ROWS; r++) {
        acc[r] = ss[r] = 0.f;
        ro[r] = (size_t)min(r0 + r, P.M - 1) * P.K;
    }
    int k = k0;
    for (; k + 8 <= k1; k += 8) {
        float wv[8], gv[8];
#pragma unroll
        for (int j = 0; j < 8; j++) wv[j] = to_f32<TW>(W[(size_t)(k + j) * P.N]);
#pragma unroll
        for (int j = 0; j < 8; j++) gv[j] = NORM ? gain[k + j] : 1.f;
#pragma unroll
        for (int r = 0; r < FG_ROWS; r++)
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const float a = src[ro[r] + k + j];
                if (NORM) ss[r] = fmaf(a, a, ss[r]);
                acc[r] = fmaf(NORM ? a * gv[j] : a, wv[j], acc[r]);
            }
    }
    for (; k < k1; k++) {
        const float wv = to_f32<TW>(W[(size_t)k * P.N]), gv = NORM ? gain[k] : 1.f;
#pragma unroll
        for (int r = 0; r < FG_ROWS; r++) {
            const float a = src[ro[r] + k];
            if (NORM) ss[r] = fmaf(a, a, ss[r]);
            acc[r] = fmaf(NORM ? a * gv : a, wv, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < FG_ROWS; r++) red[w][r][lane] = acc[r];
    if (NORM && lane == 0) {
#pragma unroll
        for (int r = 0; r < FG_ROWS; r++) red_ss[w][r] = ss[r];
    }
    __syncthreads();
    const int row = r0 + w;                                  // wave w: row w of the workgroup, uniform
    if (row >= P.M) return;
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < FG_WAVES; i++) v += red[i][w][lane];
    if (NORM) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < FG_WAVES; i++) s += red_ss[i][w];
        v *= rsqrtf(s / (float)P.K + P.eps);
    }
    const float other = EPI == FG_QKV || EPI == FG_GU ? __shfl_xor(v, 32, 64) : 0.f;
    if (col < 0) return;
    if (EPI == FG_PART || EPI == FG_LOGITS) {
        P.out[(size_t)row * P.N + col] = v;
    } else if (EPI == FG_RESID) {
        P.out[(size_t)row * P.N + col] += v;
    } else if (EPI == FG_GU) {
        if (lane < 32) P.out[(size_t)row * (P.N / 2) + col] = v / (1.0f + expf(-v)) * other;
    } else {
        const int dh = P.geo.dh, half = dh / 2, hd = P.geo.H * dh;
        const int region = col / hd, c = col % hd, hh = c / dh, x = c % dh;
        const int b = row / P.m, pos = P.cache_len[b] + row % P.m;
        if (region < 2) {
            const float2 cs = P.rope[(size_t)row * half + x % half];
            v = lane < 32 ? v * cs.x - other * cs.y : other * cs.y + v * cs.x;
        }
        if (region == 0)
            P.q[(size_t)row * hd + c] = v;
        else if (pos >= 0 && pos < P.geo.seq_pad) {
            if (region == 1)
                P.kv[kv_k_off(P.geo, P.layer, b, hh) + (size_t)pos * dh + x] = v;
            else
                P.kv[kv_v_off(P.geo, P.layer, b, hh) + kv_v_idx(P.geo, x, pos)] = v;
        }
    }
}

// h[r] = E[token[r]] and the rotary table of the call's positions
__global__ __launch_bounds__(256) void k_f32_embed(const int32_t *__restrict__ tokens, const float *__restrict__ E, int V, int d,
                                                   float *__restrict__ h, const int32_t *__restrict__ cache_len, int m, int dh,
                                                   float theta, float2 *__restrict__ rope, const int32_t *__restrict__ depth) {
    const int r = blockIdx.x, tok = tokens[r];
    const bool ok = tok >= 0 && tok < V;
    for (int x = threadIdx.x; x < d; x += blockDim.x) h[(size_t)r * d + x] = ok ? E[(size_t)tok * d + x] : 0.f;
    // the position of a row: where it sits in a plain block, how far it is from row 0 in a tree block
    const int pos = cache_len[r / m] + (depth ? depth[r] : r % m), half = dh / 2;
    for (int x = threadIdx.x; x < half; x += blockDim.x) {
        const double ang = (double)pos * pow((double)theta, -2.0 * (double)x / (double)dh);
        rope[(size_t)r * half + x] = float2{(float)cos(ang), (float)sin(ang)};
    }
}

// ------------------------------------------------------------------------------- small models: a layer per launch
//
// Where every matrix is at most 1024 columns wide and 32 K values large, a launch is latency and little else (3 to 6 us for 64 x 64
// products), so one workgroup of 1024 threads takes a block row through everything between two appends to the cache: attention of the
// row over all heads, O, gate|up, down, and the QKV projection of the next layer (the LM head after the last).  What bounds it is the
// chain of LDS steps and barriers, and the instruction fetches of code that runs once: with every loop unrolled and integer divisions
// (25 KB) a layer took 20.8 us, in 11 KB 12.6.  The weights of a product are requested one product ahead, a thread holding up to 32 values of
// one column.  Tiny shape (64 features, 4 heads, 256 hidden, 512 tokens, 2 layers), verify step with 5 rows: 66 us in five launches per
// layer, 40 in one.  With up to twice the values per thread (the second set of instances), the forward alone, 5 rows over 32 cached: 128 features, 4 heads
// of 16, 128 hidden, 256 tokens 49 us in five launches per layer, 31 in one; 96, 4 of 16, 160, 340: 50 and 31 (tiny shape: 46 and 30).
#define FR_THREADS 1024
#define FR_X (FR_THREADS + 64)        /* an input row, zero past its end up to a multiple of the slices */
struct RowProduct {
    const float *W;                   // row-major [K][N]
    int K, N, S, kper;                // S = FR_THREADS / N slices of kper = ceil(K / S) values
};
// x / n for 0 <= x < 2048, 1 <= n <= 1024: the quotient is at least 1 / 2048 away from the next whole number, the product within 2^-22 of it
__device__ __forceinline__ int small_div(int x, int n) { return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)n)); }
struct F32Row {
    RowProduct o, gu, down, next;     // this layer's O, gate|up, down; the next product (QKV, or the LM head)
    const float *ffn_gain, *next_gain;
    int layer, keys_pad;              // layer: of the attention; QKV appends to layer + 1
    int head_threads, pv_slices;      // FR_THREADS / n_heads, FR_THREADS / hd
    float eps, scale, theta;
    float *h, *q;                     // [M][d], [M][hd]
    float *kv;
    KvGeom geo;
    float2 *rope;                     // [M][dh / 2]
    const int32_t *depth;             // FIRST
    int V;
    const unsigned long long *anc;
    float *logits;                    // LAST
};

// A row times a K x N matrix (N <= FR_THREADS): thread (slice s of K, column c).  At most PER values of the column per thread.
template <int PER>
struct RowSlice {
    float w[PER];
    int k0, c, s;
    __device__ __forceinline__ void load(const RowProduct &Q) {
        const int N = Q.N, K = Q.K, S = Q.S;
        s = small_div(threadIdx.x, N);
        c = threadIdx.x - s * N;
        k0 = s * Q.kper;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(Q.W), 0, K * N * 4, 0x00020000);
        // (rows past the slice are not used, rows past the matrix are outside the buffer and read as 0, and so is all of a thread
        // without a slice: no load is under a branch)
        int off = s < S ? (k0 * N + c) * 4 : (int)0x80000000;
#pragma unroll
        for (int j = 0; j < PER; j++) {
            w[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
            off += N * 4;
        }
    }
    // partial sums to red[s][c], in four chains
    __device__ __forceinline__ void apply(const RowProduct &Q, const float *x, float *red) const {
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        const float *xs = x + (s < Q.S ? k0 : 0);
#pragma unroll
        for (int j = 0; j < PER; j++)
            if (j < Q.kper) a[j & 3] = fmaf(xs[j], w[j], a[j & 3]);      // (uniform)
        if (s < Q.S) red[s * Q.N + c] = (a[0] + a[1]) + (a[2] + a[3]);
    }
    static __device__ __forceinline__ float sum(const RowProduct &Q, const float *red, int col) {
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        int i = 0;
#pragma unroll 1
        for (; i + 4 <= Q.S; i += 4)
#pragma unroll
            for (int u = 0; u < 4; u++) a[u] += red[(i + u) * Q.N + col];
#pragma unroll 1
        for (; i < Q.S; i++) a[i & 1] += red[i * Q.N + col];
        return (a[0] + a[1]) + (a[2] + a[3]);
    }
};

// The same with four columns per thread and a quarter of the values of each: a load brings a kilobyte per wave instead of 256 bytes, and a
// compute unit's loads are what the wide products take their time for.  N a multiple of 4 and at least 64 (at most 64 slices: x is
// zero that far past its end), W aligned to 16 bytes; red holds 4 * FR_THREADS floats.  Tiny shape, 5 rows over 32 and 9 over 400 cached: 37.7 -> 36.6 and 48.8
// -> 47.4 us per step.
template <int PER>
struct RowSlice4 {
    f32x4 w[PER / 4];
    int k0, c, s;
    static __device__ __forceinline__ int slices(const RowProduct &Q) { return __builtin_amdgcn_readfirstlane(small_div(FR_THREADS, Q.N / 4)); }
    static __device__ __forceinline__ int values(const RowProduct &Q) { return __builtin_amdgcn_readfirstlane(small_div(Q.K + slices(Q) - 1, slices(Q))); }
    __device__ __forceinline__ void load(const RowProduct &Q) {
        const int N = Q.N, S = slices(Q);
        s = small_div(threadIdx.x, N / 4);
        c = (threadIdx.x - s * (N / 4)) * 4;
        k0 = s * values(Q);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(Q.W), 0, Q.K * N * 4, 0x00020000);
        int off = s < S ? (k0 * N + c) * 4 : (int)0x80000000;        // (as in RowSlice)
#pragma unroll
        for (int j = 0; j < PER / 4; j++) {
            w[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
            off += N * 4;
        }
    }
    __device__ __forceinline__ void apply(const RowProduct &Q, const float *x, float *red) const {
        f32x4 a[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        const int S = slices(Q), n = values(Q);
        const float *xs = x + (s < S ? k0 : 0);
#pragma unroll
        for (int j = 0; j < PER / 4; j++)
            if (j < n) {                                             // (uniform)
#pragma unroll
                for (int i = 0; i < 4; i++) a[j & 1][i] = fmaf(xs[j], w[j][i], a[j & 1][i]);
            }
        if (s < S) *reinterpret_cast<f32x4 *>(red + s * Q.N + c) = a[0] + a[1];
    }
    static __device__ __forceinline__ float sum(const RowProduct &Q, const float *red, int col) {
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        const int S = slices(Q);
        int i = 0;
#pragma unroll 1
        for (; i + 4 <= S; i += 4)
#pragma unroll
            for (int u = 0; u < 4; u++) a[u] += red[(i + u) * Q.N + col];
#pragma unroll 1
        for (; i < S; i++) a[i & 1] += red[i * Q.N + col];
        return (a[0] + a[1]) + (a[2] + a[3]);
    }
};

// PO, PN: most values per thread of the O projection and of the next product.  VEC: gate|up and the next product four columns per thread.
// What the first loads need comes ahead of the structure, in registers when a wave starts (see kc_gemm in csd_chain.hip): w0, w1 the O and
// gate|up matrices, or (FIRST) w0 the QKV matrix, q the tokens and h the embedding.
template <bool FIRST, bool LAST, int PO, int PN, bool VEC>
__global__ __launch_bounds__(FR_THREADS) void k_f32_row(const float *w0, const float *w1, const float *q0, const float *h0, const int32_t *cache_len,
                                                        int d, int hd, int F, int m, const F32Row P) {
    extern __shared__ __align__(16) float fr_smem[];             // (RowSlice4 stores four floats at a time)
    __shared__ float x[FR_X], red[FR_THREADS], hs[FR_THREADS], y[FR_THREADS], wave_red[2 * (FR_THREADS / 64)];
    float *sc = fr_smem;                                         // scores [H][keys_pad]; behind the attention, VEC: partial sums
    float *wide = VEC ? fr_smem : red;
    using Wide32 = typename std::conditional<VEC, RowSlice4<32>, RowSlice<32>>::type;
    using WideN = typename std::conditional<VEC, RowSlice4<PN>, RowSlice<PN>>::type;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = blockIdx.x;
    const int dh = P.geo.dh, H = P.geo.H, half = dh / 2;
    const int b = r / m, i = r % m;
    auto product = [](const float *W, int K, int N) {            // as the host makes them (K + S <= 1024 + 64)
        const int S = small_div(FR_THREADS, N);
        return RowProduct{W, K, N, S, small_div(K + S - 1, S)};
    };
    auto put_x = [&](int K, float v) {                           // x[0 .. K) = v of thread k, zeros behind
        if (tid < K) x[tid] = v;
        if (tid < 64) x[K + tid] = 0.f;
    };
    // 1 / rms of the row whose entries the threads below d hold
    auto row_rstd = [&](float v) {
        float ss = wave_sum(tid < d ? v * v : 0.f);
        if (lane == 0) wave_red[wv] = ss;
        __syncthreads();
        ss = 0.f;
#pragma unroll 1
        for (int u = 0; u < (d + 63) / 64; u++) ss += wave_red[u];
        return rsqrtf(ss / (float)d + P.eps);
    };
    const int t0 = cache_len[b];
    WideN wn;
    float hv = 0.f;                                              // this thread's entry of the residual stream
    if constexpr (FIRST) {
        wn.load(product(w0, d, 3 * hd));
        const int tok = reinterpret_cast<const int32_t *>(q0)[r];
        if (tid < d) hv = tok >= 0 && tok < P.V ? h0[(size_t)tok * d + tid] : 0.f;
        // the position of a row: where it sits in a plain block, how far it is from row 0 in a tree block
        const int pos = t0 + (P.depth ? P.depth[r] : i);
        if (tid < half) {
            const double ang = (double)pos * pow((double)P.theta, -2.0 * (double)tid / (double)dh);
            P.rope[(size_t)r * half + tid] = float2{(float)cos(ang), (float)sin(ang)};
        }
    } else {
        RowSlice<PO> wo;
        Wide32 wg;
        wo.load(product(w0, hd, d));
        wg.load(product(w1, d, 2 * F));
        // ---- attention of the row, all heads (the keys of a head as k_attn_simple takes them)
        if (tid < hd) y[tid] = q0[(size_t)r * hd + tid];
        if (tid < d) hv = h0[(size_t)r * d + tid];
        const int qpos = t0 + i, nk = max(1, min(qpos + 1, P.geo.seq_pad));
        const unsigned long long anc_row = P.anc ? P.anc[r] : 0ull;
        const float *kc = P.kv + kv_k_off(P.geo, P.layer, b, 0), *vc = P.kv + kv_v_off(P.geo, P.layer, b, 0);
        const size_t he = kv_head_elems(P.geo);
        // the first key of the thread (16 values of it) and its first values, requested before anything is waited for: one trip past the
        // caches instead of three in a row (rows up to the padded cache exist; those past the last key are not used: one row over 8 cached ones is 0.1 us
        // of 11.3 per layer slower for it, five rows are 0.2 faster, over 200 cached ones all are)
        const int G = P.head_threads, hq = small_div(tid, G), j0 = tid - hq * G;
        f32x4 kfirst[4];
#pragma unroll
        for (int u = 0; u < 4; u++) kfirst[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (dh % 16 == 0 && hq < H && j0 < P.geo.seq_pad) {
#pragma unroll
            for (int u = 0; u < 4; u++) kfirst[u] = *reinterpret_cast<const f32x4 *>(kc + hq * he + (size_t)j0 * dh + 4 * u);
        }
        const int S = P.pv_slices, pc = small_div(tid, S), ps = tid - pc * S;  // slices of the keys next to each other: V is contiguous in them
        const int ph = pc < hd ? small_div(pc, dh) : 0, pe = pc - ph * dh;
        float vfirst[4];
#pragma unroll
        for (int u = 0; u < 4; u++) vfirst[u] = pc < hd && ps + u * S < P.geo.seq_pad ? vc[ph * he + kv_v_idx(P.geo, pe, ps + u * S)] : 0.f;
        __syncthreads();
        if (hq < H) {
            const float *kh = kc + hq * he, *qr = y + hq * dh;
#pragma unroll 1
            for (int j = j0; j < nk; j += G) {
                const float *kr = kh + (size_t)j * dh;
                float s = 0.f;
                if (dh % 16 == 0) {
#pragma unroll 1
                    for (int e = 0; e < dh; e += 16) {
                        f32x4 kk[4];
                        if (j == j0 && e == 0) {
#pragma unroll
                            for (int u = 0; u < 4; u++) kk[u] = kfirst[u];
                        } else {
#pragma unroll
                            for (int u = 0; u < 4; u++) kk[u] = *reinterpret_cast<const f32x4 *>(kr + e + 4 * u);
                        }
#pragma unroll
                        for (int u = 0; u < 16; u++) s = fmaf(qr[e + u], kk[u / 4][u % 4], s);
                    }
                } else {
#pragma unroll 1
                    for (int e = 0; e < dh; e++) s = fmaf(qr[e], kr[e], s);
                }
                s *= P.scale;
                if (P.anc && !tree_sees(anc_row, j, t0)) s = -INFINITY;   // a row of the block that is not above this one
                sc[hq * P.keys_pad + j] = s;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int hh = wv; hh < H; hh += FR_THREADS / 64) {       // a wave per head
            float *row = sc + hh * P.keys_pad;
            float mx = -INFINITY, z = 0.f;
#pragma unroll 1
            for (int j = lane; j < nk; j += 64) mx = fmaxf(mx, row[j]);
            mx = wave_max(mx);
#pragma unroll 1
            for (int j = lane; j < nk; j += 64) {
                const float e = expf(row[j] - mx);
                row[j] = e;
                z += e;
            }
            z = wave_sum(z);
            if (lane == 0) hs[hh] = 1.0f / z;
        }
        __syncthreads();
        {
            float o = 0.f;
            if (pc < hd) {
                const float *row = sc + ph * P.keys_pad, *vr = vc + ph * he;
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (ps + u * S < nk) o = fmaf(row[ps + u * S], vfirst[u], o);
#pragma unroll 4
                for (int j = ps + 4 * S; j < nk; j += S) o = fmaf(row[j], vr[kv_v_idx(P.geo, pe, j)], o);
                red[ps * hd + pc] = o;
            }
            __syncthreads();
            o = 0.f;
            if (tid < hd) {
#pragma unroll 4
                for (int u = 0; u < S; u++) o += red[u * hd + tid];
                o *= hs[small_div(tid, dh)];
            }
            put_x(hd, o);
            __syncthreads();
        }
        // ---- O, residual
        RowSlice<16> wd;
        wo.apply(P.o, x, red);
        wd.load(P.down);
        __syncthreads();
        if (tid < d) hv += wo.sum(P.o, red, tid);
        float rstd = row_rstd(hv);                               // (its barrier: red and x have been read)
        put_x(d, tid < d ? hv * P.ffn_gain[tid] : 0.f);
        __syncthreads();
        // ---- gate|up, activation
        wg.apply(P.gu, x, wide);
        wn.load(P.next);
        __syncthreads();
        float f = 0.f;
        if (tid < F) {
            const float gt = wg.sum(P.gu, wide, tid) * rstd, up = wg.sum(P.gu, wide, F + tid) * rstd;
            f = gt / (1.0f + expf(-gt)) * up;
        }
        put_x(F, f);
        __syncthreads();
        // ---- down, residual
        wd.apply(P.down, x, red);
        __syncthreads();
        if (tid < d) hv += wd.sum(P.down, red, tid);
    }
    if (tid < d) P.h[(size_t)r * d + tid] = hv;
    const float rstd = row_rstd(hv);
    put_x(d, tid < d ? hv * P.next_gain[tid] : 0.f);
    __syncthreads();
    wn.apply(P.next, x, wide);
    __syncthreads();
    float v = 0.f;
    if (tid < P.next.N) v = wn.sum(P.next, wide, tid) * rstd;
    if constexpr (LAST) {
        if (tid < P.next.N) P.logits[(size_t)r * P.next.N + tid] = v;
    } else {
        y[tid] = v;
        __syncthreads();
        if (tid >= P.next.N) return;
        const int region = small_div(tid, hd), c = tid - region * hd, hh = small_div(c, dh), e = c - hh * dh;
        if (region < 2) {
            const float2 cs = P.rope[(size_t)r * half + (e < half ? e : e - half)];   // (FIRST: written by this workgroup before its barriers)
            const float other = y[e < half ? tid + half : tid - half];
            v = e < half ? v * cs.x - other * cs.y : other * cs.y + v * cs.x;
        }
        const int pos = t0 + i, layer = FIRST ? 0 : P.layer + 1;
        if (region == 0)
            P.q[(size_t)r * hd + c] = v;
        else if (pos >= 0 && pos < P.geo.seq_pad) {
            if (region == 1)
                P.kv[kv_k_off(P.geo, layer, b, hh) + (size_t)pos * dh + e] = v;
            else
                P.kv[kv_v_off(P.geo, layer, b, hh) + kv_v_idx(P.geo, e, pos)] = v;
        }
    }
}

// ------------------------------------------------------------------------------- host driver

template <typename TW, int EPI, bool NORM>
static int32_t f32_launch(const F32Gemm &P, hipStream_t st) {
    int gx = (P.N + 63) / 64;
    if (EPI == FG_QKV) {
        const int hd = P.N / 3;
        gx = 2 * ((hd / 2 + 31) / 32) + (hd + 63) / 64;
    } else if (EPI == FG_GU) {
        gx = (P.N / 2 + 31) / 32;
    }
    hipLaunchKernelGGL((k_f32_gemm<TW, EPI, NORM>), dim3(gx, (P.M + FG_ROWS - 1) / FG_ROWS), dim3(FG_THREADS), 0, st, P);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

static F32Gemm f32_args(const GemmW &w, const float *src, int M) {
    F32Gemm P{};
    P.W = w.data;
    P.K = w.K;
    P.N = w.N;
    P.M = M;
    P.src = src;
    return P;
}

int32_t csd_f32_part(const csd_model *mod, const GemmW &w, const float *act, int M, hipStream_t st) {
    F32Gemm P = f32_args(w, act, M);
    P.out = mod->part;
    return mod->cfg.dtype == CSD_DTYPE_BF16 ? f32_launch<bf16_t, FG_PART, false>(P, st) : f32_launch<float, FG_PART, false>(P, st);
}

// Whether the launch of a layer per row takes the model and the call: every product's columns over the threads, at most 32 values
// of a column in each, at most one workgroup per compute unit, the scores of a row in LDS.  Not while the profile is on (see csd_prof_enable):
// one launch is GEMM, attention and the rest at once, and its classes cannot be told apart.
// And only where it is the faster form when the cache is full.  One compute unit does the attention of a row over all heads, where k_attn_simple has a
// workgroup per head: its keys and values take longer than what four launches a layer cost once heads x features x keys is large, and sooner where a
// head's keys are not read 16 values at a time.  Forward of two layers of 32 features in us, this form / five launches per layer, one row of a
// block, full cache: 4 heads of 16, 500 / 2000 / 2600 keys 37 / 48, 73 / 76, 88 / 88; 8 of 16, 120 / 250 / 376 keys 33 / 41, 42 / 43, 51 / 47; 3 of 64,
// 120 / 376 keys 41 / 49, 71 / 67; 8 of 8, 184 / 376 keys 38 / 40, 51 / 43; 3 of 30, 120 / 376 keys 37 / 45, 63 / 54; 1 of 128, 2600 / 10500 keys
// 248 / 441, 926 / 1648; 16 of 16 with 5 rows, 56 / 120 keys 42 / 46, 57 / 47.  More rows gain more (256 rows, 4 of 16, 500 / 2600 keys 43 / 82, 98 / 215).
// Four columns per thread (RowSlice4) where the two wide products of a launch (the first launch has one) come in 36 slices of K together or
// fewer: the partial sums are added one after the other, and narrow products have many of them.  Forward of four layers, 5 rows over 8 cached, one
// column / four columns, in us, by gate|up and QKV slices: 32 + 42 (32 features, FFN 64) 47.5 / 50.6; 32 + 21 (64, 64) 47.1 / 48.6; 21 + 21 (64, 96) 47.9 / 48.4;
// 16 + 28 (48, 128) 47.9 / 47.9; 16 + 21 (64, 128) 47.7 / 48.0; 14 + 21 (64, 144) 49.5 / 48.6; 10 + 21 (64, 192) 50.3 / 48.6; 8 + 21 (32, 256) 49.0 / 48.1; 8 + 21 (64,
// 256) 50.9 / 48.4; 16 + 10 (64, 128, heads of 128 together) 53.3 / 50.8; 10 + 14 (24, 192) 51.0 / 50.6.
#define FR_VEC_SLICES 36
static bool row_product_fits(int K, int N, int per) { return N >= 16 && N <= FR_THREADS && (K + FR_THREADS / N - 1) / (FR_THREADS / N) <= per; }
static bool row_attention_fits(int H, int dh, int keys) {
    const long long hd = (long long)H * dh;
    if ((long long)H * keys > 11000) return false;
    if (dh % 16 == 0) return H == 1 || hd <= 64 || hd * keys <= 24576;
    return hd * keys <= 12288;
}
static bool f32_rows_fit(const csd_model *mod, int M) {
    const csd_model_cfg &c = mod->cfg;
    const int d = c.d_model, hd = mod->hd, F = c.d_ffn;
    return !mod->prof && M <= 256 && row_attention_fits(c.n_heads, c.head_dim, mod->seq_pad) && row_product_fits(hd, d, 8) &&
           row_product_fits(d, 2 * F, 32) && row_product_fits(F, d, 16) && row_product_fits(d, 3 * hd, 32) && row_product_fits(d, c.vocab, 32);
}
static int32_t f32_rows_enqueue(csd_model *mod, void *kv, const int32_t *tokens, const int32_t *cache_len, int M, int m, float *logits,
                                hipStream_t st) {
    const csd_model_cfg &c = mod->cfg;
    const int d = c.d_model, L = c.n_layers;
    F32Row P{};
    auto product = [](const GemmW &w) {
        const int S = FR_THREADS / w.N;
        return RowProduct{(const float *)w.data, w.K, w.N, S, (w.K + S - 1) / S};
    };
    P.head_threads = FR_THREADS / c.n_heads;
    P.pv_slices = FR_THREADS / mod->hd;
    P.keys_pad = mod->seq_pad;
    P.eps = c.rms_eps;
    P.scale = 1.0f / sqrtf((float)c.head_dim);
    P.theta = c.rope_theta;
    P.h = mod->h;
    P.q = (float *)mod->qbuf;
    P.kv = (float *)kv;
    P.geo = KvGeom{c.max_batch, c.n_heads, c.head_dim, mod->seq_pad, L, mod->kperm ? 1 : 0};
    P.rope = mod->rope;
    P.V = c.vocab;
    P.logits = logits;
    if (mod->tree_call) P.depth = mod->tree_depth, P.anc = mod->tree_anc;
    const size_t scores = sizeof(float) * (size_t)c.n_heads * mod->seq_pad;
    const bool few = row_product_fits(mod->hd, d, 4) && row_product_fits(d, 3 * mod->hd, 16);
    for (int l = -1; l < L; l++) {                               // layer l, and the QKV projection of the next one
        const GemmW &next = l + 1 < L ? mod->layers[l + 1].qkv : mod->lm;
        P.next = product(next);
        P.next_gain = l + 1 < L ? mod->layers[l + 1].attn_norm : mod->final_norm;
        P.layer = l;
        if (l >= 0) {
            const LayerW &lw = mod->layers[l];
            P.o = product(lw.o);
            P.gu = product(lw.gu);
            P.down = product(lw.down);
            P.ffn_gain = lw.ffn_norm;
        }
        const int hd = mod->hd, F = c.d_ffn;
        auto four = [](const RowProduct &Q) { return Q.N % 4 == 0 && Q.N >= 64 && (uintptr_t)Q.W % 16 == 0; };
        auto slices = [](const RowProduct &Q) { return FR_THREADS / (Q.N / 4); };
        const bool vec = four(P.next) && (l < 0 || four(P.gu)) && slices(P.next) + (l < 0 ? FR_VEC_SLICES / 2 : slices(P.gu)) <= FR_VEC_SLICES;
        const size_t wide = sizeof(float) * 4 * FR_THREADS, lds = vec && scores < wide ? wide : scores;
#define FR_LAUNCH(FIRST, LAST, PN, W0, W1, Q0, H0)                                                                                       \
    {                                                                                                                                    \
        auto *kernel = few ? (vec ? k_f32_row<FIRST, LAST, 4, PN, true> : k_f32_row<FIRST, LAST, 4, PN, false>)                          \
                           : (vec ? k_f32_row<FIRST, LAST, 8, 32, true> : k_f32_row<FIRST, LAST, 8, 32, false>);                         \
        hipLaunchKernelGGL(kernel, dim3(M), dim3(FR_THREADS), lds, st, W0, W1, Q0, H0, cache_len, d, hd, F, m, P);                        \
    }
        if (l < 0)
            FR_LAUNCH(true, false, 16, P.next.W, (const float *)nullptr, (const float *)tokens, (const float *)mod->embed)
        else if (l + 1 < L)
            FR_LAUNCH(false, false, 16, P.o.W, P.gu.W, P.q, P.h)
        else
            FR_LAUNCH(false, true, 32, P.o.W, P.gu.W, P.q, P.h)
#undef FR_LAUNCH
        CSD_LAUNCH_CHECK();
        if (mod->trace)
            CSD_HIP(hipMemcpyAsync(mod->trace + (size_t)(l + 1) * M * d, mod->h, sizeof(float) * (size_t)M * d, hipMemcpyDeviceToDevice, st));
    }
    return CSD_OK;
}

int32_t csd_f32_enqueue(csd_model *mod, void *kv, const int32_t *tokens, const int32_t *cache_len, int32_t B, int32_t m,
                        float *logits, hipStream_t st) {
    const csd_model_cfg &c = mod->cfg;
    const int M = B * m, d = c.d_model, L = c.n_layers;
    if (f32_rows_fit(mod, M)) return f32_rows_enqueue(mod, kv, tokens, cache_len, M, m, logits, st);
    const KvGeom geo{c.max_batch, c.n_heads, c.head_dim, mod->seq_pad, L, mod->kperm ? 1 : 0};
    float *act = (float *)mod->act;
    const float scale = 1.0f / sqrtf((float)c.head_dim);
    int32_t rc;
    auto gemm = [&](const GemmW &w, const float *src, const float *gain, float *out) {
        F32Gemm P = f32_args(w, src, M);
        P.gain = gain;
        P.eps = c.rms_eps;
        P.out = out;
        return P;
    };
#define F32_STEP(CLS, CALL)                              \
    {                                                    \
        ProfScope ps(mod, st, CLS);                      \
        if ((rc = (CALL)) != CSD_OK) return rc;          \
    }
    {
        ProfScope ps(mod, st, CSD_PROF_OTHER);
        hipLaunchKernelGGL(k_f32_embed, dim3(M), dim3(256), 0, st, tokens, (const float *)mod->embed, c.vocab, d, mod->h, cache_len, m,
                           c.head_dim, c.rope_theta, mod->rope, mod->tree_call ? mod->tree_depth : nullptr);
        CSD_LAUNCH_CHECK();
    }
    if (mod->trace) CSD_HIP(hipMemcpyAsync(mod->trace, mod->h, sizeof(float) * (size_t)M * d, hipMemcpyDeviceToDevice, st));
    AttnMode am;
    if (mod->tree_call) am.anc = mod->tree_anc;
    for (int l = 0; l < L; l++) {
        const LayerW &lw = mod->layers[l];
        F32Gemm Q = gemm(lw.qkv, mod->h, lw.attn_norm, nullptr);
        Q.m = m;
        Q.layer = l;
        Q.cache_len = cache_len;
        Q.geo = geo;
        Q.rope = mod->rope;
        Q.q = (float *)mod->qbuf;
        Q.kv = (float *)kv;
        F32_STEP(CSD_PROF_GEMM, (f32_launch<float, FG_QKV, true>(Q, st)))
        // (brackets itself for the profile: brackets do not nest)
        if ((rc = csd_attn_simple_f32(mod, geo, (const float *)kv, cache_len, B, m, l, scale, am, st)) != CSD_OK) return rc;
        F32_STEP(CSD_PROF_GEMM, (f32_launch<float, FG_RESID, false>(gemm(lw.o, act, nullptr, mod->h), st)))
        F32_STEP(CSD_PROF_GEMM, (f32_launch<float, FG_GU, true>(gemm(lw.gu, mod->h, lw.ffn_norm, act), st)))
        F32_STEP(CSD_PROF_GEMM, (f32_launch<float, FG_RESID, false>(gemm(lw.down, act, nullptr, mod->h), st)))
        if (mod->trace)
            CSD_HIP(hipMemcpyAsync(mod->trace + (size_t)(l + 1) * M * d, mod->h, sizeof(float) * (size_t)M * d,
                                   hipMemcpyDeviceToDevice, st));
    }
    F32_STEP(CSD_PROF_GEMM, (f32_launch<float, FG_LOGITS, true>(gemm(mod->lm, mod->h, mod->final_norm, logits), st)))
#undef F32_STEP
    return CSD_OK;
}
