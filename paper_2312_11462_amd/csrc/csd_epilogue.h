// What the GEMM kernels with their epilogue inside share: the arguments of a launch, the stores of the two bf16 planes, and
// the epilogues themselves (rotary embedding and cache append, residual, gated activation, logits).
#pragma once

#include "csd_internal.h"

#define CH_OOB ((int)0x80000000)     /* buffer offset beyond any buffer: loads give 0 and touch no memory */
#define CH_SC1 16                    /* device scope: data for, or from, workgroups on other compute dies (stores write through) */

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_GU = 2, EPI_LOGITS = 3 };

struct ChainGemm {
    const u32x4 *Wp;          // tiles [N/16][KS][64 lanes][8 bf16]
    int KS, n_units, wbytes;  // k-steps of 32; units a workgroup owns whole (a tile; gate|up: a gate tile and its up tile)
    const bf16_t *a;          // input planes (hi, lo), fragment order (act_tiled_idx)
    int a_plane_bytes, mtp, M;
    const float *ssq_in;      // [n_ssq][ssq_rows]: sum of squares of the input's source rows per 16-feature tile (folded norm) or null
    int n_ssq, ssq_rows;      // ssq_rows: 16 * (row tiles of the call), for ssq_in and ssq_out alike
    float inv_d, eps;
    // EPI_RESID: residual stream, next norm's gain, output planes + sums of squares
    float *h;
    const float *gain;
    bf16_t *out;              // output planes (EPI_RESID, EPI_GU), fragment order
    int out_plane_bytes;
    float *ssq_out;
    int d;
    // EPI_QKV
    int m, hd, dh, layer;
    KvGeom geo;
    const int32_t *cache_len;
    const float2 *rope;       // (cos, sin) [M][dh/2] or null
    bf16_t *q;                // rotated queries, two row-major planes [..][hd]
    int q_plane_bytes;
    bf16_t *kv;
    int gelu;                 // EPI_GU: tanh-GELU instead of SiLU
    float *logits;            // EPI_LOGITS [M][V]
    int V;
    const int32_t *live;      // per sequence of m rows the rows that are needed (csd_review_ctx), or null: all
};

// A buffer descriptor must sit in scalar registers.  Base addresses here are the same in every lane, but the
// compiler cannot always prove it (64-bit address arithmetic on workgroup indices may end up in vector
// registers) and then wraps every access in a loop over the distinct descriptors: say so explicitly.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ch_rsrc(const void *p, size_t bytes) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    const int n = __builtin_amdgcn_readfirstlane((int)(bytes > 0x7FFFFFFFull ? 0x7FFFFFFFull : bytes));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((unsigned long long)hi << 32) | lo), 0, n, 0x00020000);
}

__device__ __forceinline__ void split4(const float *v, u32x2 &hi, u32x2 &lo) {
#pragma unroll
    for (int w = 0; w < 2; w++) {
        const uint32_t hh = pack_bf16x2(v[2 * w], v[2 * w + 1]);
        hi[w] = hh;
        lo[w] = pack_bf16x2(v[2 * w] - __uint_as_float(hh << 16), v[2 * w + 1] - __uint_as_float(hh & 0xFFFF0000u));
    }
}

// Four consecutive columns of one row into the two planes of a fragment-ordered activation buffer.
template <int AUX = CH_SC1>
__device__ __forceinline__ void store_planes4(bf16_t *out, int plane_bytes, int mtp, int row, int col, const float *v) {
    u32x2 hi, lo;
    split4(v, hi, lo);
    const int off = (int)(act_tiled_idx(row, col, mtp) * 2);
    const __amdgpu_buffer_rsrc_t r = ch_rsrc(out, (size_t)2 * plane_bytes);
    __builtin_amdgcn_raw_buffer_store_b64(hi, r, off, 0, AUX);
    __builtin_amdgcn_raw_buffer_store_b64(lo, r, off + plane_bytes, 0, AUX);
}

// What the epilogue of one (tile, row tile) needs besides the sums, fetched before the main loop.
struct EpiIn {
    f32x4 hcur, gcur;
    float2 cs[4];
    int pos;
};

// The epilogue of one output tile (gate|up: a gate tile and its up tile) for the 16 rows of one row tile, on complete,
// rstd-scaled sums v (AUX: cache policy of the stores).  row: this lane's block row; T: global index of the (first) tile.  No workgroup barrier inside.
template <int EPI, int AUX = CH_SC1>
__device__ __forceinline__ void gemm_epilogue(const ChainGemm &P, const f32x4 *v, const EpiIn &E, int row, int T, int g) {
    constexpr int UT = EPI == EPI_GU ? 2 : 1;
    const bool valid = row < P.M;
    if (EPI == EPI_RESID) {
        const f32x4 hv = E.hcur + v[0];
        float ss = hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2] + hv[3] * hv[3];
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (!valid) return;
        const int col = T * 16 + 4 * g;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hv), ch_rsrc(P.h, (size_t)P.M * P.d * 4),
                                               (int)(((size_t)row * P.d + col) * 4), 0, AUX);
        const float o[4] = {hv[0] * E.gcur[0], hv[1] * E.gcur[1], hv[2] * E.gcur[2], hv[3] * E.gcur[3]};
        store_planes4<AUX>(P.out, P.out_plane_bytes, P.mtp, row, col, o);
        if (g == 0)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, ss),
                                                  ch_rsrc(P.ssq_out, (size_t)(P.d / 16) * P.ssq_rows * 4), (T * P.ssq_rows + row) * 4, 0, AUX);
    } else if (EPI == EPI_GU) {
        if (!valid) return;
        float o[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float gt = v[0][r], up = v[UT - 1][r];
            const float a = P.gelu ? 0.5f * gt * (1.0f + tanhf(0.7978845608028654f * (gt + 0.044715f * gt * gt * gt)))
                                   : gt / (1.0f + expf(-gt));
            o[r] = a * up;
        }
        store_planes4<AUX>(P.out, P.out_plane_bytes, P.mtp, row, (T / 2) * 16 + 4 * g, o);
    } else if (EPI == EPI_LOGITS) {
        if (!valid) return;
        *reinterpret_cast<f32x4 *>(P.logits + (size_t)row * P.V + T * 16 + 4 * g) = v[0];
    } else {   // EPI_QKV
        const int tiles_per_region = P.hd / 16, tiles_per_head = P.dh / 16;
        const int region = T / tiles_per_region, tr = T % tiles_per_region;
        const int head = tr / tiles_per_head, ti = tr % tiles_per_head;
        const int b = valid ? row / P.m : 0;
        const int pos = E.pos;
        if (region < 2) {
            // tiles of q and k hold whole rotary pairs: lane groups 0, 1 the first-half entries 8 ti .. 8 ti + 7,
            // groups 2, 3 their partners; one exchange across the wave brings the pair together
            float o[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float other = __shfl_xor(v[0][r], 32, 64);
                const float c = E.cs[r].x, s = E.cs[r].y;
                o[r] = g < 2 ? v[0][r] * c - other * s : other * s + v[0][r] * c;
            }
            if (!valid) return;
            const int p0 = 16 * ti + 4 * g;                    // place inside the head, pair order
            if (region == 0) {
                u32x2 hi, lo;
                split4(o, hi, lo);
                const __amdgpu_buffer_rsrc_t rq = ch_rsrc(P.q, (size_t)2 * P.q_plane_bytes);
                const int off = (int)(((size_t)row * P.hd + head * P.dh + p0) * 2);
                __builtin_amdgcn_raw_buffer_store_b64(hi, rq, off, 0, AUX);
                __builtin_amdgcn_raw_buffer_store_b64(lo, rq, off + P.q_plane_bytes, 0, AUX);
            } else if (pos >= 0 && pos < P.geo.seq_pad) {
                u32x2 kk;
                kk[0] = pack_bf16x2(o[0], o[1]);
                kk[1] = pack_bf16x2(o[2], o[3]);
                // (the sequence, hence the head's region, differs from lane to lane: one descriptor for the layer's
                // keys, the rest in the per-lane offset; written through, the attention step may run on another die)
                const size_t he = kv_head_elems(P.geo);
                __builtin_amdgcn_raw_buffer_store_b64(kk, ch_rsrc(P.kv + kv_k_off(P.geo, P.layer, 0, 0), (size_t)P.geo.Bmax * P.geo.H * he * 2),
                                                      (int)((((size_t)b * P.geo.H + head) * he + (size_t)pos * P.dh + p0) * 2), 0, AUX);
            }
        } else if (valid && pos >= 0 && pos < P.geo.seq_pad) {
            const size_t he = kv_head_elems(P.geo);
            const __amdgpu_buffer_rsrc_t rv = ch_rsrc(P.kv + kv_v_off(P.geo, P.layer, 0, 0), (size_t)P.geo.Bmax * P.geo.H * he * 2);
#pragma unroll
            for (int r = 0; r < 4; r++)
                __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(v[0][r]), rv,
                                                      (int)((((size_t)b * P.geo.H + head) * he + kv_v_idx(P.geo, 16 * ti + 4 * g + r, pos)) * 2), 0,
                                                      AUX);
        }
    }
}
