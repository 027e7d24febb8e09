// Forward of fp32 models (arch 0) and the GEMM of every model that is not on the matrix cores: row-major weights, fp32
// activations.
//
// Such models are small (tests, the tiny configuration), so a launch is bound by the chain of memory round trips of a
// thread, not by bandwidth.  One thread per output column that walks all of K takes K dependent rounds (41 us a launch at
// the tiny shape, K = 64 and 256); here K is split over the eight waves of a workgroup, a wave requests eight rows of its
// slice at once, the eight partial sums meet in LDS, and whatever follows a GEMM (rotary embedding and cache append, residual
// sum, gated activation, the scale of the folded norm) runs on them in the same kernel, which computes the norm of its input
// rows along the way: five launches per layer of 3 to 6 us.  Tiny shape, verify step: 363 -> 67 us.
#include <cmath>

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

int32_t csd_f32_enqueue(csd_model *mod, void *kv, const int32_t *tokens, const int32_t *cache_len, int32_t B, int32_t m,
                        float *logits, hipStream_t st) {
    const csd_model_cfg &c = mod->cfg;
    const int M = B * m, d = c.d_model, L = c.n_layers;
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
