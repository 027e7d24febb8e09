// Review forward for blocks of up to 32 rows (Section 2: one run of the reviewer scores every drafted
// position): five launches per layer, no split-K partial sums in memory, no epilogue kernels.
//
//   QKV GEMM   -> rotate q, k; q to the query buffer; K, V appended to the cache   (epilogue)
//   attention  -> key chunks in parallel, merged by the last chunk to finish
//   O GEMM     -> h += ; (h * gain) as the next GEMM's input; sum of squares per tile (epilogue)
//   gate|up    -> silu(rstd * gate) * (rstd * up) as the next GEMM's input              (epilogue)
//   down GEMM  -> h += ; (h * gain); sum of squares per tile                            (epilogue)
//
// A GEMM workgroup owns a few whole 16-feature output tiles (for one or two 16-row tiles of the block) and
// splits K over its eight waves; every wave
// streams its own K slice of the pre-tiled weights through a register ring and multiplies it with the
// activation fragments of the same slice (read from L2: no two waves need the same ones), the eight
// partial tiles are added in LDS in wave order (deterministic), and the epilogue runs in the same kernel
// on complete sums.  RMSNorm is folded around the GEMM: rmsnorm(h) * g @ W = rstd(row) * ((h * g) @ W);
// the producer of h writes h * g and one sum of squares per (row, 16-feature tile), the consumer's
// epilogue scales its output rows by 1 / sqrt(sum / d + eps).
#include <cmath>
#include <type_traits>

#include "csd_warm.h"

#define CH_WAVES 8
#define CH_THREADS (CH_WAVES * 64)
// This wave's share of a GEMM: the workgroup's tiles [t0, t0 + nt) (nt <= NT), the wave's k-steps [ks0, ks1).
struct GemmShare {
    int t0, nt, ks0, ks1;
};
template <int EPI>
__device__ __forceinline__ GemmShare gemm_share(const ChainGemm &P, int wg, int G, int w) {
    constexpr int UT = EPI == EPI_GU ? 2 : 1;
    // Workgroups go to the eight compute dies round-robin, and what a die can pull from memory is what bounds the
    // launch: the units are dealt so that every die gets the same number (consecutive shares to the workgroups of one
    // die), not merely every workgroup within one of the next (688 units over 256 workgroups gave three dies 96 units
    // and five dies 80, and the launch lasted as long as the dies with 96).
    if (G % 8 == 0) wg = (wg & 7) * (G >> 3) + (wg >> 3);
    const int u0 = (int)((long long)P.n_units * wg / G), u1 = (int)((long long)P.n_units * (wg + 1) / G);
    return GemmShare{u0 * UT, (u1 - u0) * UT, P.KS * w / CH_WAVES, P.KS * (w + 1) / CH_WAVES};
}

// Every load of the GEMM is issued unconditionally (what must not be read gets an offset beyond the buffer),
// so the compiler can count the loads in flight and wait for exactly the oldest.
template <int NT>
__device__ __forceinline__ void gemm_load_w(u32x4 (&W)[NT], const ChainGemm &P, const GemmShare &S, __amdgpu_buffer_rsrc_t rw, int ks,
                                            int lane) {
    const bool in = ks < S.ks1;   // uniform
#pragma unroll
    for (int j = 0; j < NT; j++) {
        const bool tv = in && j < S.nt;
        W[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, tv ? lane * 16 : CH_OOB,
                                                                              tv ? ((S.t0 + j) * P.KS + ks) * 1024 : 0, 2));
    }
}
// Activation fragments of MT row tiles: the hi and the lo plane of each, or, with HALF, of a last tile of at most eight rows one fragment
// for both: hi in its columns 0 to 7, lo in 8 to 15 (their sums meet after the reduction).  A launch over few rows is bound by the loads a
// compute unit can issue (some 25 cycles per KB, whatever arrives) as much as by HBM, and a k-step of one tile is then two loads and one
// matrix instruction instead of three and two: steps of the 7B shape with 6 rows 3130 -> 3090 us, of the T5 shape with 5 rows 2786 -> 2735.
template <int MT, bool HALF>
__device__ __forceinline__ void gemm_load_a(u32x4 (&A)[2 * MT - HALF], const ChainGemm &P, const GemmShare &S, __amdgpu_buffer_rsrc_t ra, int ks,
                                            const int (&voff_a)[MT]) {
    const bool in = ks < S.ks1;   // uniform
#pragma unroll
    for (int f = 0; f < 2 * MT - HALF; f++) {
        const int mt = f / 2;
        A[f] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             ra, in ? voff_a[mt] : CH_OOB, in ? (f & 1 ? P.a_plane_bytes : 0) + (ks * P.mtp + mt) * 1024 : 0, 0));
    }
}

// The first R k-steps of a wave's weight stream: they depend on nothing the other workgroups produce, so a
// kernel that runs several GEMMs may issue them before the device-wide barrier in front of the GEMM.
template <int NT, int R>
__device__ __forceinline__ void gemm_prefetch(u32x4 (&Wr)[R][NT], const ChainGemm &P, const GemmShare &S) {
    const __amdgpu_buffer_rsrc_t rw = ch_rsrc(P.Wp, (size_t)P.wbytes);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < R; r++) gemm_load_w<NT>(Wr[r], P, S, rw, S.ks0 + r, lane);
}

// The GEMM of one workgroup after gemm_prefetch: the wave's k-steps through the rings for MT row tiles of 16 rows, the
// eight partial tiles added in LDS in wave order (one row tile at a time), the epilogue.  LDS: red [8 waves][NT][64 lanes]
// 16-byte words, then [8 waves][16 MT rows] floats.  Every wave of the workgroup must call it (it holds workgroup barriers).
template <int NT, int R, int EPI, int MT, bool HALF>
__device__ __forceinline__ void gemm_run(u32x4 (&Wr)[R][NT], const ChainGemm &P, const GemmShare &S, char *smem) {
    f32x4 *red = reinterpret_cast<f32x4 *>(smem);
    float *rs_part = reinterpret_cast<float *>(smem + (size_t)CH_WAVES * NT * 64 * 16);
    constexpr int UT = EPI == EPI_GU ? 2 : 1;
    const int lane = threadIdx.x & 63, t = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t0 = S.t0, nt = S.nt, ks0 = S.ks0, ks1 = S.ks1;
    const __amdgpu_buffer_rsrc_t rw = ch_rsrc(P.Wp, (size_t)P.wbytes);
    const __amdgpu_buffer_rsrc_t ra = ch_rsrc(P.a, (size_t)2 * P.a_plane_bytes);
    int voff_a[MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++) voff_a[mt] = mt * 16 + t < P.M ? (4 * t + g) * 16 : CH_OOB;
    if (HALF) voff_a[MT - 1] = (MT - 1) * 16 + (t & 7) < P.M ? (4 * (t & 7) + g) * 16 + (t < 8 ? 0 : P.a_plane_bytes) : CH_OOB;

    // partial sums of squares of the rows behind the folded norm: wave w, lane group g take every 32nd tile.
    // Eight independent loads per row tile and turn (a dependent chain of them would hold up the rings behind it).
    float ssq[MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++) ssq[mt] = 0.f;
    if (P.ssq_in) {
        const __amdgpu_buffer_rsrc_t rq = ch_rsrc(P.ssq_in, (size_t)P.n_ssq * P.ssq_rows * 4);
        for (int base = 0; base < P.n_ssq; base += 8 * 4 * CH_WAVES) {
            float sv[MT][8];
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int n = 0; n < 8; n++) {
                    const int i = base + n * 4 * CH_WAVES + w * 4 + g;
                    sv[mt][n] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                              rq, i < P.n_ssq ? (i * P.ssq_rows + mt * 16 + t) * 4 : CH_OOB, 0, 0));
                }
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int n = 0; n < 8; n++) ssq[mt] += sv[mt][n];
        }
    }
    u32x4 Ar[R][2 * MT - HALF];
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int j = 0; j < NT; j++) acc[mt][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < R; r++) gemm_load_a<MT, HALF>(Ar[r], P, S, ra, ks0 + r, voff_a);

    // epilogue inputs that do not depend on the sums: fetched now, used after the reduction
    EpiIn E[MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        const int row = mt * 16 + t;
        E[mt].hcur = E[mt].gcur = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; r++) E[mt].cs[r] = float2{1.f, 0.f};
        E[mt].pos = -1;
        if (EPI == EPI_RESID && w < nt && row < P.M) {
            const int col = (t0 + w) * 16 + 4 * g;
            E[mt].hcur = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ch_rsrc(P.h, (size_t)P.M * P.d * 4),
                                                                                        (int)(((size_t)row * P.d + col) * 4), 0, 0));
            E[mt].gcur = *reinterpret_cast<const f32x4 *>(P.gain + col);
        }
        if (EPI == EPI_QKV && w < nt && row < P.M) {
            const int ti = ((t0 + w) % (P.hd / 16)) % (P.dh / 16);
            E[mt].pos = P.cache_len[row / P.m] + row % P.m;
            if (P.rope && (t0 + w) < 2 * (P.hd / 16)) {
#pragma unroll
                for (int r = 0; r < 4; r++) E[mt].cs[r] = P.rope[(size_t)row * (P.dh / 2) + 8 * ti + 4 * (g & 1) + r];
            }
        }
    }
    if (P.ssq_in) {
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            float s = ssq[mt];
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (g == 0) rs_part[(w * MT + mt) * 16 + t] = s;
        }
    }

    // The last turn of the rings requests nothing: a load that brings nothing still takes some 25 cycles of the compute unit's memory pipeline, and
    // the rings' depth in loads past the end was 1 us of a launch (160M shape 367 -> 335 us per step, 7B shape 2926 -> 2883, T5 shape
    // 2565 -> 2518, 7B shape, 20 rows 3678 -> 3536).
    auto step = [&](int r) {
#pragma unroll
        for (int f = 0; f < 2 * MT - HALF; f++)
#pragma unroll
            for (int j = 0; j < NT; j++)
                acc[f / 2][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, Wr[r][j]),
                                                                        __builtin_bit_cast(bf16x8, Ar[r][f]), acc[f / 2][j], 0, 0, 0);
    };
    for (int ks = ks0; ks + R < ks1; ks += R) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            step(r);
            gemm_load_w<NT>(Wr[r], P, S, rw, ks + r + R, lane);
            gemm_load_a<MT, HALF>(Ar[r], P, S, ra, ks + r + R, voff_a);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) step(r);                         // (k-steps past the end hold zeros)

    // ------------------------------------------------------------------ reduction and epilogue, a row tile at a time:
    // wave e takes unit e
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        if (mt > 0) __syncthreads();                           // the sums of the row tile before have been read
#pragma unroll
        for (int j = 0; j < NT; j++) red[(w * NT + j) * 64 + lane] = acc[mt][j];
        __syncthreads();
        if (w * UT < nt) {
            float rstd = 1.f;
            if (P.ssq_in) {
                float s = 0.f;
#pragma unroll
                for (int i = 0; i < CH_WAVES; i++) s += rs_part[(i * MT + mt) * 16 + t];
                rstd = rsqrtf(s * P.inv_d + P.eps);
            }
            f32x4 v[UT];
#pragma unroll
            for (int x = 0; x < UT; x++) {
                v[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < CH_WAVES; i++) v[x] += red[(i * NT + w * UT + x) * 64 + lane];
                if (HALF && mt == MT - 1) {                    // row t: column t (hi) + column t + 8 (lo)
#pragma unroll
                    for (int i = 0; i < 4; i++) v[x][i] += across_half_row(v[x][i]);
                }
                v[x] *= rstd;
            }
            gemm_epilogue<EPI>(P, v, E[mt], mt * 16 + t, t0 + w * UT, g);
        }
    }
}

// LIVE: a review of one sequence that the device may have skipped (a separate form: the look costs a plain step 0.7 %)
//
// What the first loads need comes as plain arguments ahead of the structure: the build asks for 14 dwords of them to be in registers when a
// wave starts (build.py), where the structure is a cold read of memory in front of everything else.  The kernels of the small-block forward
// begin with it 64 to 196 times in a row per step: with kc_gemm's alone 160M shape 400 -> 378 us per step, 7B shape 3061 -> 2986, T5 shape 2640 -> 2562;
// with the attention's too 374, 2963 and 2562.
template <int NT, int R, int EPI, int MT, bool HALF, bool LIVE>
__global__ __launch_bounds__(CH_THREADS) void kc_gemm(const u32x4 *Wp, int KS, int n_units, int wbytes, int G, const bf16_t *a, int a_plane_bytes,
                                                      int mtp, int M, const int32_t *live, const ChainGemm rest) {
    extern __shared__ __align__(16) char ch_smem[];
    ChainGemm P = rest;
    P.Wp = Wp;
    P.KS = KS;
    P.n_units = n_units;
    P.wbytes = wbytes;
    P.a = a;
    P.a_plane_bytes = a_plane_bytes;
    P.mtp = mtp;
    P.M = M;
    P.live = live;
    const GemmShare S = gemm_share<EPI>(P, blockIdx.x, G, __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)));
    u32x4 Wr[R][NT];
    gemm_prefetch<NT, R>(Wr, P, S);
    if (LIVE && P.live[0] == 0) return;                      // (the first weights are on their way meanwhile)
    gemm_run<NT, R, EPI, MT, HALF>(Wr, P, S, ch_smem);
}

// Causal attention of a block of up to 16 rows over the cached prefix, one launch per layer.  A workgroup
// of four waves takes 128 keys of one (sequence, head): each wave one 32-key tile with both products on the
// matrix cores, transposed so that no operand passes through LDS (S^T = K q^T, O^T = V^T P^T; V is cached
// transposed), the four softmax states are merged in LDS, and the workgroup writes one partial state per
// chunk.  The last workgroup of a (sequence, head) to finish (an arrival counter) merges the chunks and
// writes the rows as the O projection's input; the counter is back at zero when the kernel ends.
#define CA_KEYS 128
#define CA_MAX_CHUNKS 128     /* the merge keeps a weight per (chunk, row) in LDS: sequences of up to 16384 cached rows */
struct AttnArgs {
    const bf16_t *q;          // rotated queries, two row-major planes [..][hd]
    int q_plane, m;
    const int32_t *cache_len;
    KvGeom geo;
    const bf16_t *k, *v;      // the layer's keys and values
    float scale;
    float *part;              // chunk states [B][H][chunks_max][16 rows][DH + 4]
    int chunks_max;
    int chunk_slots;          // chunks the grid holds (workgroups past them read ahead, see csd_warm.h)
    unsigned *counters;       // arrivals per (sequence, head): zero between launches
    const unsigned long long *anc;   // tree block: per block row the rows it sees (see AttnMode), or null
    const float *bias_hd;     // arch 1 self-attention: [H][128] bias by distance query - key (127: that or more), or null
    int fixed_nk;             // > 0 (arch 1 cross-attention): every row sees keys [0, fixed_nk), whatever cache_len says
    bf16_t *out;              // merged rows: the O projection's input planes, fragment order
    int out_plane_bytes, mtp;
    const int32_t *live;      // as in ChainGemm: rows of a sequence past these are neither attended nor written (from then on they and their
                              // K/V rows hold anything, and no other row looks at them)
};
// The arguments that the first loads need come ahead of the structure, in registers when a wave starts (see kc_gemm).
template <int DH>
__device__ __forceinline__ AttnArgs attn_args(const bf16_t *k, const bf16_t *v, const bf16_t *q, const int32_t *cache_len, const int32_t *live,
                                              int q_plane, int H, int seq_pad, int rows_slots, const AttnArgs &rest) {
    AttnArgs A = rest;
    A.k = k;
    A.v = v;
    A.q = q;
    A.cache_len = cache_len;
    A.live = live;
    A.q_plane = q_plane;
    A.geo.H = H;
    A.geo.seq_pad = seq_pad;
    A.geo.dh = DH;
    A.m = rows_slots & 31;                                   // (up to 16 rows)
    A.chunk_slots = rows_slots >> 5;
    return A;
}
#define CA_ARGS(A) (A).k, (A).v, (A).q, (A).cache_len, (A).live, (A).q_plane, (A).geo.H, (A).geo.seq_pad, (A).m | (A).chunk_slots << 5, A
template <int DH>
struct AttnLds {
    f32x4 o[4][DH / 16][64];
    float m[4][16], l[4][16];
    float w[4][CA_MAX_CHUNKS * 16];                          // weights of the merge, every wave its own
    unsigned old;
    unsigned pad[3];
};

// One chunk of one (sequence, head) by a group of four waves (gtid = thread index in the group, 0 .. 255).
// Holds three workgroup barriers whatever `have` says, so groups with and without an item stay in step.
template <int DH, bool LIVE>
__device__ __forceinline__ void attn_item(const AttnArgs &A, AttnLds<DH> &L, bool have, int c, int hh, int b, int gtid) {
    constexpr int PS = DH + 4;                               // floats per partial row: DH outputs, max, sum, pad
    constexpr int DT = DH / 16;
    const KvGeom &geo = A.geo;
    const int m = LIVE ? min(A.m, A.live[b]) : A.m, stride = A.m;
    if (LIVE && m <= 0) return;                              // a skipped sequence: no workgroup of it arrives
    const int lane = gtid & 63, col = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(gtid >> 6);
    const int hd = geo.H * DH;
    const int kb = c * CA_KEYS + wv * 32;                    // this wave's 32 keys
    // Every load is issued before the cached length is known (their addresses do not depend on it; rows past
    // the end are masked below, rows past the cache are outside the buffer and read as zeros).
    const size_t head_bytes = have ? kv_head_elems(geo) * 2 : 0;
    const __amdgpu_buffer_rsrc_t rk = ch_rsrc(A.k + ((size_t)b * geo.H + hh) * kv_head_elems(geo), head_bytes);
    const __amdgpu_buffer_rsrc_t rv = ch_rsrc(A.v + ((size_t)b * geo.H + hh) * kv_head_elems(geo), head_bytes);
    const __amdgpu_buffer_rsrc_t rqb = ch_rsrc(A.q, have ? (size_t)4 * A.q_plane : 0);
    u32x4 qf[DH / 32][2], kf[2][DH / 32], vf[DT];
#pragma unroll
    for (int s = 0; s < DH / 32; s++) {
        const int qo = col < m ? (int)(((size_t)(b * stride + col) * hd + hh * DH + s * 32 + 8 * g) * 2) : CH_OOB;
        qf[s][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rqb, qo, 0, 0));
        qf[s][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rqb, qo, A.q_plane * 2, 0));
    }
    // A operands.  K: A-row r of tile T is key kb + 8 (r / 4) + 4 T + r % 4, so lane group g ends up with the
    // scores of keys kb + 8 g .. + 7; V^T: row = feature dt * 16 + col, 8 consecutive keys per lane.
#pragma unroll
    for (int T = 0; T < 2; T++) {
        const int key = kb + 8 * (col >> 2) + 4 * T + (col & 3);
#pragma unroll
        for (int s = 0; s < DH / 32; s++)
            kf[T][s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, (key * DH + 8 * g + s * 32) * 2, 0, 0));
    }
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
        vf[dt] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, (int)(kv_v_idx(geo, dt * 16 + col, kb + 8 * g) * 2), 0, 0));
    const bool causal = A.fixed_nk <= 0;
    const int t = (have && causal) ? A.cache_len[b] : 0;
    const int nk = max(0, min(causal ? t + m : A.fixed_nk, geo.seq_pad));   // cache rows in play for this block
    const int nch = (nk + CA_KEYS - 1) / CA_KEYS;
    const bool active = have && c < nch;                     // a chunk past the end is not counted
    const int qpos = t + col;                                // block row `col` sees cache rows 0 .. qpos
    const unsigned long long anc_row = (A.anc && have && col < m) ? A.anc[b * stride + col] : 0ull;
    float bias[8];                                           // requested ahead of the scores they are added to
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int dist = qpos - (kb + 8 * g + j);
        bias[j] = (A.bias_hd && have && dist >= 0) ? A.bias_hd[hh * 128 + min(dist, 127)] : 0.f;
    }
    float mrun = -INFINITY, lrun = 0.f;
    f32x4 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++) oacc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (active && kb < nk) {                                 // uniform over the wave
        f32x4 sT[2];
#pragma unroll
        for (int T = 0; T < 2; T++) {
            sT[T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < DH / 32; s++) {
                sT[T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[T][s]),
                                                                __builtin_bit_cast(bf16x8, qf[s][0]), sT[T], 0, 0, 0);
                sT[T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[T][s]),
                                                                __builtin_bit_cast(bf16x8, qf[s][1]), sT[T], 0, 0, 0);
            }
        }
        float sv[8], mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int key = kb + 8 * g + j;
            const bool seen = (A.anc ? tree_sees(anc_row, key, t) : (!causal || key <= qpos)) && key < nk;
            sv[j] = seen ? sT[j >> 2][j & 3] * A.scale + bias[j] : -INFINITY;
            mx = fmaxf(mx, sv[j]);
        }
        mx = groups_max(mx);
        float pv[8], psum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            pv[j] = (sv[j] == -INFINITY) ? 0.f : expf(sv[j] - mx);
            psum += pv[j];
        }
        psum = groups_sum(psum);
        mrun = mx;
        lrun = psum;
        u32x4 pf, pl;                                        // hi and lo planes of the probabilities
#pragma unroll
        for (int w2 = 0; w2 < 4; w2++) {
            const uint32_t hpk = pack_bf16x2(pv[2 * w2], pv[2 * w2 + 1]);
            pf[w2] = hpk;
            pl[w2] = pack_bf16x2(pv[2 * w2] - __uint_as_float(hpk << 16), pv[2 * w2 + 1] - __uint_as_float(hpk & 0xFFFF0000u));
        }
        const bool tail = kb + 32 > nk;                      // rows past nk may hold anything: zero them
#pragma unroll
        for (int dt = 0; dt < DT; dt++) {
            u32x4 v = vf[dt];
            if (tail) {
#pragma unroll
                for (int w2 = 0; w2 < 4; w2++) {
                    const int k0 = kb + 8 * g + 2 * w2;
                    v[w2] &= (k0 < nk ? 0x0000FFFFu : 0u) | (k0 + 1 < nk ? 0xFFFF0000u : 0u);
                }
            }
            oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pf), oacc[dt], 0, 0, 0);
            oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pl), oacc[dt], 0, 0, 0);
        }
    }
    // ---- the four tiles of the chunk, merged in LDS; wave wv writes output tiles wv, wv + 4, ...
#pragma unroll
    for (int dt = 0; dt < DT; dt++) L.o[wv][dt][lane] = oacc[dt];
    if (g == 0) {
        L.m[wv][col] = mrun;
        L.l[wv][col] = lrun;
    }
    __syncthreads();
    if (active) {
        float mstar = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; i++) mstar = fmaxf(mstar, L.m[i][col]);
        float wgt[4], lsum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            wgt[i] = L.m[i][col] == -INFINITY ? 0.f : expf(L.m[i][col] - mstar);
            lsum += wgt[i] * L.l[i][col];
        }
        float *po = A.part + (((size_t)b * geo.H + hh) * A.chunks_max + c) * 16 * PS;
        const __amdgpu_buffer_rsrc_t rp = ch_rsrc(po, (size_t)16 * PS * 4);
        for (int dt = wv; dt < DT; dt += 4) {
            f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; i++) o += L.o[i][dt][lane] * wgt[i];
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rp, (col * PS + dt * 16 + 4 * g) * 4, 0, CH_SC1);
        }
        if (wv == 0 && g == 0) {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, mstar), rp, (col * PS + DH) * 4, 0, CH_SC1);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, lsum), rp, (col * PS + DH + 1) * 4, 0, CH_SC1);
        }
    }
    // ---- arrival: the stores above are acknowledged before the counter moves
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)
    __syncthreads();
    unsigned *cnt = A.counters + b * geo.H + hh;
    if (gtid == 0) L.old = active ? __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0xFFFFFFFFu;
    __syncthreads();
    // ---- last to arrive: merge the chunk states of this (sequence, head).  Workgroups on other compute dies wrote them through to memory
    // (CH_SC1).  The loads are of device scope too: a line outlives the end of a kernel in an L2 (see csd_warm.h), and a die that merged this
    // head in an earlier layer has read the same addresses.  (160M shape of 24 layers, 2000 cached rows 625 -> 632 us per step, with an acquire
    // fence in front of plain loads 654; 700 rows 589 all three.)
    const bool last = active && L.old == (unsigned)(nch - 1);
    const float *pbase = A.part + ((size_t)b * geo.H + hh) * A.chunks_max * 16 * PS;
    const __amdgpu_buffer_rsrc_t rm = ch_rsrc(pbase, last ? (size_t)A.chunks_max * 16 * PS * 4 : 0);
    // out[r][x] = sum_c weight[c][r] * acc_c[r][x] with weight[c][r] = e^(m_c - m*) / sum_c l_c e^(m_c - m*).  A thread takes four
    // features of every RG-th row; the accumulators of sixteen chunks are requested together, and the first such batch before the states, so that
    // the common case is one memory round trip (one feature of four rows per thread was four times the loads, some 25 cycles of the compute unit each:
    // 7B shape, 1024 / 2000 cached rows, 2976 -> 2925 and 3479 -> 3342 us per step, 160M shape 393 -> 375, T5 shape, 1500 rows, 2909 -> 2863).  Every wave makes all
    // the weights for itself, lane (c % 4, r): no barrier, and up to 16 chunks without a loop over them.
    const int x = gtid % (DH / 4) * 4;
    constexpr int RG = 256 / (DH / 4);
    const int r_first = gtid / (DH / 4);
    f32x4 ac[16];
    auto load_acc = [&](int r_, int c0) {                    // (the scalar offset operand must be uniform: the per-thread part is the vector offset)
#pragma unroll
        for (int u = 0; u < 16; u++)
            ac[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rm, (r_ < m && c0 + u < nch) ? (((c0 + u) * 16 + r_) * PS + x) * 4 : CH_OOB, 0, CH_SC1));
    };
    float *wgt_c = L.w[wv];
    if (last) {
        load_acc(r_first, 0);
        float mc[4], lc[4], mst = -INFINITY, den = 0.f;
        auto states = [&](int c0) {                              // chunks c0 .. c0 + 15 of row `col`
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int cc = c0 + 4 * j + g, o = cc < nch ? (cc * 16 + col) * PS * 4 : CH_OOB;
                mc[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, o, DH * 4, CH_SC1));
                lc[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, o, (DH + 1) * 4, CH_SC1));
            }
#pragma unroll
            for (int j = 0; j < 4; j++)
                if (c0 + 4 * j + g >= nch) mc[j] = -INFINITY, lc[j] = 0.f;
        };
        for (int c0 = (nch - 1) / 16 * 16; c0 >= 0; c0 -= 16) {  // (the first sixteen last: their states stay in registers)
            states(c0);
#pragma unroll
            for (int j = 0; j < 4; j++) mst = fmaxf(mst, mc[j]);
        }
        mst = groups_max(mst);
        for (int c0 = 0; c0 < nch; c0 += 16) {
            if (c0 != 0) states(c0);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const float e = mc[j] == -INFINITY ? 0.f : expf(mc[j] - mst);
                den += e * lc[j];
                if (c0 + 4 * j + g < CA_MAX_CHUNKS) wgt_c[(c0 + 4 * j + g) * 16 + col] = e;
            }
        }
        den = groups_sum(den);
        const float inv = den > 0.f ? 1.0f / den : 0.f;
        for (int cc = g; cc < nch; cc += 4) wgt_c[cc * 16 + col] *= inv;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // read by the other lanes
        for (int r = r_first; r < m; r += RG) {
            f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int c0 = 0; c0 < nch; c0 += 16) {
                if (r != r_first || c0 != 0) load_acc(r, c0);
#pragma unroll
                for (int u = 0; u < 16; u++)
                    if (c0 + u < nch) num += ac[u] * wgt_c[(c0 + u) * 16 + r];
            }
            const float v[4] = {num[0], num[1], num[2], num[3]};
            store_planes4(A.out, A.out_plane_bytes, A.mtp, b * stride + r, hh * DH + x, v);
        }
        if (gtid == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Causal attention of a block of up to 16 rows over the cached prefix, one launch per layer.  A workgroup
// of four waves takes 128 keys of one (sequence, head): each wave one 32-key tile with both products on the
// matrix cores, transposed so that no operand passes through LDS (S^T = K q^T, O^T = V^T P^T; V is cached
// transposed), the four softmax states are merged in LDS, and the workgroup writes one partial state per
// chunk.  The last workgroup of a (sequence, head) to finish (an arrival counter) merges the chunks and
// writes the rows as the O projection's input; the counter is back at zero when the kernel ends.
template <int DH, bool LIVE, class WARM>
__global__ __launch_bounds__(256) void kc_attn(const bf16_t *k, const bf16_t *v, const bf16_t *q, const int32_t *cache_len, const int32_t *live, int q_plane,
                                               int H, int seq_pad, int rows_slots, const AttnArgs rest, const WARM Wm) {
    __shared__ __align__(16) AttnLds<DH> L;
    const AttnArgs A = attn_args<DH>(k, v, q, cache_len, live, q_plane, H, seq_pad, rows_slots, rest);
    if constexpr (!std::is_same<WARM, NoWarm>::value)
        if (__builtin_expect((int)blockIdx.z >= A.chunk_slots, 0)) {
            const int per_z = gridDim.x * gridDim.y, e = (blockIdx.z - A.chunk_slots) * per_z + blockIdx.y * gridDim.x + blockIdx.x;
            if (!(LIVE && A.live[blockIdx.y] <= 0)) l2_warm(Wm, e, A.chunk_slots * per_z + e, &L);
            return;
        }
    // Grid (head, sequence, chunk): the last chunk of a head holds little besides the block's own rows, and with the chunk
    // index slowest those short workgroups are dispatched after every long one has a compute unit of its own.
    attn_item<DH, LIVE>(A, L, true, blockIdx.z, blockIdx.x, blockIdx.y, threadIdx.x);
}

// The same for caches short enough that one workgroup of sixteen waves reads all of a (sequence, head): a 32-key tile per
// wave and turn, and the sixteen states meet in LDS.  No chunk state leaves the compute unit, so the write, the arrival
// counter and the read back of kc_attn's chunks (four trips through the fabric in a row) fall away.  Measured per launch
// against kc_attn (one sequence): heads of 64, 100 keys 5.4 us against 9.4, 500 keys 8.0 against 9.9, 700 keys 9.3 against 10.1, 1024
// keys 12.4 against 10.7; heads of 128, 100 keys 7.1
// against 9.9, 250 keys 8.4 against 10.1, 380 keys 9.8 against 10.1, 440 keys 11.5 against 10.7 (four sequences: 11.6 against 13.4).
// With heads of 128 the registers (128 per wave) hold a tile and the query or a tile and the output, not all three: one turn.
#define CA_ONE_NW 16
template <int DH, int NW>
struct AttnOneLds {
    f32x4 o[NW][DH / 16][64];
    float m[NW][16], l[NW][16], w[NW][16];
};
template <int DH, int NW, bool BIAS, bool LIVE, class WARM>
__global__ __launch_bounds__(NW * 64) void kc_attn_one(const bf16_t *k, const bf16_t *v, const bf16_t *q, const int32_t *cache_len, const int32_t *live, int q_plane,
                                                       int H, int seq_pad, int rows_slots, const AttnArgs rest, const WARM Wm) {
    extern __shared__ __align__(16) char one_smem[];
    const AttnArgs A = attn_args<DH>(k, v, q, cache_len, live, q_plane, H, seq_pad, rows_slots, rest);
    if constexpr (!std::is_same<WARM, NoWarm>::value)
        if (__builtin_expect(blockIdx.z > 0, 0)) {
            const int per_z = gridDim.x * gridDim.y, e = (blockIdx.z - 1) * per_z + blockIdx.y * gridDim.x + blockIdx.x;
            if (!(LIVE && A.live[blockIdx.y] <= 0)) l2_warm(Wm, e, per_z + e, one_smem);
            return;
        }
    AttnOneLds<DH, NW> &L = *reinterpret_cast<AttnOneLds<DH, NW> *>(one_smem);
    constexpr int DT = DH / 16;
    const KvGeom &geo = A.geo;
    const int hh = blockIdx.x, b = blockIdx.y;
    const int m = LIVE ? min(A.m, A.live[b]) : A.m, stride = A.m;
    if (LIVE && m <= 0) return;                              // a skipped sequence
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int hd = geo.H * DH;
    const size_t head_bytes = kv_head_elems(geo) * 2;
    const __amdgpu_buffer_rsrc_t rk = ch_rsrc(A.k + ((size_t)b * geo.H + hh) * kv_head_elems(geo), head_bytes);
    const __amdgpu_buffer_rsrc_t rv = ch_rsrc(A.v + ((size_t)b * geo.H + hh) * kv_head_elems(geo), head_bytes);
    const __amdgpu_buffer_rsrc_t rqb = ch_rsrc(A.q, (size_t)4 * A.q_plane);
    struct Tile {
        u32x4 k[2][DH / 32], v[DT];
    } ta;
    // Operand layout as in attn_item.
    auto load = [&](Tile &T, int tile) {
        const int kb = tile * 32;
#pragma unroll
        for (int t2 = 0; t2 < 2; t2++) {
            const int key = kb + 8 * (col >> 2) + 4 * t2 + (col & 3);
#pragma unroll
            for (int s = 0; s < DH / 32; s++)
                T.k[t2][s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, (key * DH + 8 * g + s * 32) * 2, 0, 0));
        }
#pragma unroll
        for (int dt = 0; dt < DT; dt++)
            T.v[dt] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                    rv, (int)(kv_v_idx(geo, dt * 16 + col, kb + 8 * g) * 2), 0, 0));
    };
    load(ta, wv);                                      // before the cached length is known: masked below
    u32x4 qf[DH / 32][2];
#pragma unroll
    for (int s = 0; s < DH / 32; s++) {
        const int qo = col < m ? (int)(((size_t)(b * stride + col) * hd + hh * DH + s * 32 + 8 * g) * 2) : CH_OOB;
        qf[s][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rqb, qo, 0, 0));
        qf[s][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rqb, qo, A.q_plane * 2, 0));
    }
    const bool causal = A.fixed_nk <= 0;
    const int t = causal ? A.cache_len[b] : 0;
    const int nk = max(0, min(causal ? t + m : A.fixed_nk, geo.seq_pad));   // cache rows in play for this block
    const int n_tiles = (nk + 31) / 32;
    const int qpos = t + col;                                // block row `col` sees cache rows 0 .. qpos
    const unsigned long long anc_row = (A.anc && col < m) ? A.anc[b * stride + col] : 0ull;
    float mrun = -INFINITY, lrun = 0.f;
    f32x4 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++) oacc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fold = [&](const Tile &T, int tile) {
        const int kb = tile * 32;
        float bias[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int dist = qpos - (kb + 8 * g + j);
            bias[j] = (BIAS && dist >= 0) ? A.bias_hd[hh * 128 + min(dist, 127)] : 0.f;
        }
        f32x4 sT[2];
#pragma unroll
        for (int t2 = 0; t2 < 2; t2++) {
            sT[t2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < DH / 32; s++) {
                sT[t2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, T.k[t2][s]),
                                                                 __builtin_bit_cast(bf16x8, qf[s][0]), sT[t2], 0, 0, 0);
                sT[t2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, T.k[t2][s]),
                                                                 __builtin_bit_cast(bf16x8, qf[s][1]), sT[t2], 0, 0, 0);
            }
        }
        float sv[8], mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int key = kb + 8 * g + j;
            const bool seen = (A.anc ? tree_sees(anc_row, key, t) : (!causal || key <= qpos)) && key < nk;
            sv[j] = seen ? sT[j >> 2][j & 3] * A.scale + bias[j] : -INFINITY;
            mx = fmaxf(mx, sv[j]);
        }
        mx = groups_max(mx);
        const float mnew = fmaxf(mrun, mx);
        const float alpha = mnew == -INFINITY ? 1.0f : expf(mrun - mnew);
        float pv[8], psum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            pv[j] = (sv[j] == -INFINITY) ? 0.f : expf(sv[j] - mnew);
            psum += pv[j];
        }
        psum = groups_sum(psum);
        lrun = lrun * alpha + psum;
        mrun = mnew;
        u32x4 pf, pl;                                        // hi and lo planes of the probabilities
#pragma unroll
        for (int w2 = 0; w2 < 4; w2++) {
            const uint32_t hpk = pack_bf16x2(pv[2 * w2], pv[2 * w2 + 1]);
            pf[w2] = hpk;
            pl[w2] = pack_bf16x2(pv[2 * w2] - __uint_as_float(hpk << 16), pv[2 * w2 + 1] - __uint_as_float(hpk & 0xFFFF0000u));
        }
        const bool tail = kb + 32 > nk;                      // rows past nk may hold anything: zero them
#pragma unroll
        for (int dt = 0; dt < DT; dt++) {
            u32x4 v = T.v[dt];
            if (tail) {
#pragma unroll
                for (int w2 = 0; w2 < 4; w2++) {
                    const int k0 = kb + 8 * g + 2 * w2;
                    v[w2] &= (k0 < nk ? 0x0000FFFFu : 0u) | (k0 + 1 < nk ? 0xFFFF0000u : 0u);
                }
            }
            oacc[dt] = oacc[dt] * alpha;
            oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pf), oacc[dt], 0, 0, 0);
            oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pl), oacc[dt], 0, 0, 0);
        }
    };
    if constexpr (DH == 128) {
        if (wv < n_tiles) fold(ta, wv);
    } else {
        // (a uniform branch: a load past the end brings nothing and takes its place in the memory pipeline all the same: 160M shape 332 -> 329 us per
        // step, T5 shape 2496 -> 2473)
        for (int tile = wv; tile < n_tiles; tile += NW) {
            fold(ta, tile);
            if (tile + NW < n_tiles) load(ta, tile + NW);
        }
    }
    // ---- the waves' states, merged in LDS
    if (col < m) {
#pragma unroll
        for (int dt = 0; dt < DT; dt++) L.o[wv][dt][lane] = oacc[dt];
    }
    if (g == 0) {
        L.m[wv][col] = mrun;
        L.l[wv][col] = lrun;
    }
    __syncthreads();
    if (threadIdx.x < NW * 16) {
        const int i = threadIdx.x >> 4, r = threadIdx.x & 15;
        float mst = -INFINITY;
#pragma unroll
        for (int x = 0; x < NW; x++) mst = fmaxf(mst, L.m[x][r]);
        L.w[i][r] = L.m[i][r] == -INFINITY ? 0.f : expf(L.m[i][r] - mst);
    }
    __syncthreads();
    for (int dt = wv; dt < DT; dt += NW) {
        if (col >= m) break;
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int i = 0; i < NW; i++) {                       // waves in order
            o += L.o[i][dt][lane] * L.w[i][col];
            den += L.l[i][col] * L.w[i][col];
        }
        if (den == 0.f) den = 1.f;                           // (no key seen: the sums are 0)
        const float v[4] = {o[0] / den, o[1] / den, o[2] / den, o[3] / den};
        store_planes4(A.out, A.out_plane_bytes, A.mtp, b * stride + col, hh * DH + dt * 16 + 4 * g, v);
    }
}

// h[r] = E[token[r]]; (h * gain) as the first GEMM's input, the sums of squares per 16-feature tile, and the
// rotary table of the call's positions.  One workgroup per block row, one thread per 16-feature tile.
// A wave of its own makes the table (double precision, a long chain) while the others take the row.
#define CE_ROW 256
__global__ __launch_bounds__(CE_ROW + 64) void kc_embed(const int32_t *__restrict__ tokens, const bf16_t *__restrict__ E, int V, int d,
                                                const float *__restrict__ gain, float *__restrict__ h, bf16_t *__restrict__ out,
                                                int out_plane_bytes, int mtp, float *__restrict__ ssq_out,
                                                int ssq_rows, const int32_t *__restrict__ cache_len, int m, int dh, float theta,
                                                float2 *__restrict__ rope, const int32_t *__restrict__ depth) {
    const int r = blockIdx.x;
    const int tok = tokens[r];
    const bool ok = tok >= 0 && tok < V;
    for (int T = (int)threadIdx.x < CE_ROW ? (int)threadIdx.x : d; T < d / 16; T += CE_ROW) {
        float ss = 0.f;
#pragma unroll
        for (int c4 = 0; c4 < 4; c4++) {
            const int col = T * 16 + c4 * 4;
            u32x2 e = u32x2{0u, 0u};
            if (ok) e = *reinterpret_cast<const u32x2 *>(E + (size_t)tok * d + col);
            const f32x4 hv = f32x4{__uint_as_float(e[0] << 16), __uint_as_float(e[0] & 0xFFFF0000u), __uint_as_float(e[1] << 16),
                                   __uint_as_float(e[1] & 0xFFFF0000u)};
            *reinterpret_cast<f32x4 *>(h + (size_t)r * d + col) = hv;
            const f32x4 gv = *reinterpret_cast<const f32x4 *>(gain + col);
            const float o[4] = {hv[0] * gv[0], hv[1] * gv[1], hv[2] * gv[2], hv[3] * gv[3]};
            store_planes4(out, out_plane_bytes, mtp, r, col, o);
            ss += (hv[0] * hv[0] + hv[1] * hv[1]) + (hv[2] * hv[2] + hv[3] * hv[3]);
        }
        ssq_out[T * ssq_rows + r] = ss;
    }
    if (theta > 0.f && threadIdx.x >= CE_ROW) {
        // the position of a row: where it sits in a plain block, how far it is from row 0 in a tree block
        const int pos = cache_len[r / m] + (depth ? depth[r] : r % m), half = dh / 2;
        for (int x = (int)threadIdx.x - CE_ROW; x < half; x += 64) {
            const double ang = (double)pos * pow((double)theta, -2.0 * (double)x / (double)dh);
            rope[(size_t)r * half + x] = float2{(float)cos(ang), (float)sin(ang)};
        }
    }
}

// ------------------------------------------------------------------------------- host driver

// keys (padded cache rows) up to which one workgroup per (sequence, head) takes them: see kc_attn_one.  A workgroup fills a
// compute unit, so more than one per unit run in rounds, each of them with the whole latency, however few the keys: four layers
// with heads of 128, 512 workgroups, a cache of 448 rows with 40 in use 108 us against 65 with the kernels of csd_attention.hip, 1024
// workgroups 198 against 74; heads of 64, 512 workgroups, 40 of 832 rows 63 against 53, 2048 workgroups 218 against 69.  256
// workgroups, 40 / 220 / 440 of 448 rows: 52 / 51 / 60 us against 61 / 74 / 95.
// Heads of 128: the few workgroups of one sequence lose to kc_attn's chunks on more compute units above 384 rows (32 workgroups, 440
// keys 11.5 us against 10.7); from 64 on the four chunks of up to 448 rows would be as many workgroups as there are compute
// units, and one turn of this form wins: steps of the 7B shape
// with 384 rows in use of 448, 4 / 6 / 8 sequences 3416 / 3981 / 4227 us against 3501 / 4110 / 4439.
#define CA_ONE_KEYS_128_FEW 384
#define CA_ONE_KEYS_128 448          /* at most 32 * CA_ONE_NW: one turn */
#define CA_ONE_KEYS_64 832
#define CA_ONE_GROUPS 256
static bool attn_one_fits(const csd_model *mod, int B, int keys_pad) {
    const int groups = mod->cfg.n_heads * B;
    const int most = mod->cfg.head_dim == 64 ? CA_ONE_KEYS_64 : groups < 64 ? CA_ONE_KEYS_128_FEW : CA_ONE_KEYS_128;
    return groups <= CA_ONE_GROUPS && keys_pad <= most;
}
template <int DH, bool BIAS, class WARM>
static void attn_one_launch(const AttnArgs &A, const WARM &Wm, const dim3 &grid, hipStream_t st) {
    hipLaunchKernelGGL((A.live ? kc_attn_one<DH, CA_ONE_NW, BIAS, true, WARM> : kc_attn_one<DH, CA_ONE_NW, BIAS, false, WARM>), grid,
                       dim3(CA_ONE_NW * 64), sizeof(AttnOneLds<DH, CA_ONE_NW>), st, CA_ARGS(A), Wm);
}
template <int DH, class WARM>
static void attn_launch_dh(const AttnArgs &A, const WARM &Wm, bool one, const dim3 &grid, hipStream_t st) {
    if (!one)
        hipLaunchKernelGGL((A.live ? kc_attn<DH, true, WARM> : kc_attn<DH, false, WARM>), grid, dim3(256), 0, st, CA_ARGS(A), Wm);
    else if (A.bias_hd)
        attn_one_launch<DH, true>(A, Wm, grid, st);
    else
        attn_one_launch<DH, false>(A, Wm, grid, st);
}

// a workgroup per compute unit, or as many more as keep a workgroup's tiles to eight
static int chain_groups(int n_units, int ut) {
    int G = n_units < 256 ? n_units : 256;
    if ((n_units + G - 1) / G * ut > 8) G = (n_units * ut + 7) / 8;
    return G;
}

// What the workgroups added to an attention launch read (csd_warm.h), us per step without them and with them:
// - all the matrices behind it up to the next layer, where these are 20 MB at most (160M shape, 15.3 MB: 512 cached rows 396 -> 375, 14 of the MB 377, 8 of
//   them 389; 100 rows 327 -> 307; chunks of 1024 rows 421 -> 402; with the next layer's QKV too, before arguments came in registers, 398 -> 425);
// - else, beside one workgroup per head, as much of the first (and so on) as 30 MB, from 256 cache rows on (T5 shape, 33.6 MB: 14 MB 2612, 24 MB 2570,
//   30 MB 2551, none 2649; 7B shape, 300 rows 2991 -> 2969), 14 MB with fewer, where the attention is shorter (7B shape, 100 rows 2772 -> 2784, with
//   30 MB 2836; T5 shape, 20 rows and 40 encoder rows 2529 -> 2493, with 30 MB 2525);
//   (In between, 27 to 76 MB: models of 1024 to 2048 features, 100 cached rows 1 to 4 % of a step shorter with it, 700 rows 0 to 8 %, 2000 rows the same;
//   arch 1 of 2048 features 1 % shorter with 100 rows, 1 to 2 % longer with 700 and 2000.  Small layers of a model that does not fit the memory-side
//   cache lose with a short cache: 24 layers of the 160M shape, 340 MB, 584 -> 611 with 100 rows, 600 -> 608 with 200, 623 -> 614 with 300, 644 -> 614
//   with 500; 12 layers of it 299 -> 273 with 100.)
// - beside the chunks of large models nothing: their own loads keep the memory busy (7B shape, 1024 rows 2963 against 2960 with 14 MB, 2967 with
//   16; two sequences of 700 rows 3198 against 3257).
// 96 workgroups of 16 waves, 128 of 4: 184 and 224 are no faster, half as many are (T5 shape, 30 MB 2805 us), and no more than fit on the chip with the launch's own.
#define WARM_LAYER (20u << 20)
#define WARM_MOST (30u << 20)
#define WARM_SHORT (14u << 20)
#define WARM_LONG_KEYS 256
static int warm_plan(L2Warm &Wm, const GemmW *const *mats, int n, bool one, int keys_pad, int per_z, int used) {
    Wm = L2Warm{};
    size_t left = 0;
    for (int i = 0; i < n; i++) left += (size_t)mats[i]->K * mats[i]->N * 2;
    if (left > WARM_LAYER) left = !one ? 0 : keys_pad >= WARM_LONG_KEYS ? WARM_MOST : WARM_SHORT;
    const int want = one ? 96 : 128, room = (one ? 256 : 512) - used;
    int z = (want + per_z - 1) / per_z;
    if (z * per_z > room) z = room > 0 ? room / per_z : 0;
    if (!left || z * per_z < 8) return 0;
    for (int i = 0; i < n && i < L2_WARM_MATS; i++) {
        const GemmW &w = *mats[i];
        const int ut = i == 1 ? 2 : 1;                       // O, gate|up, down
        L2Warm::Mat m{w.data, (int)((size_t)w.K * w.N * 2), w.K / 32, w.N / 16 / ut, ut, 0};
        const size_t step = (size_t)w.N / 16 * 8 * 1024;     // one k-step of every wave
        const size_t most = (size_t)(m.KS + 7) / 8, fit = left / step;
        m.keep = chain_groups(m.units, ut) % 8 ? 0 : (int)(fit < most ? fit : most);
        left -= m.keep * step < left ? m.keep * step : left;
        Wm.mat[i] = m;
    }
    Wm.groups = z * per_z / 8 * 8;
    return z;
}

// mats: the matrices of the GEMMs behind this launch (the output projection, then gate|up and down where they come next)
static int32_t attn_launch_small(const csd_model *mod, AttnArgs A, const GemmW *const *mats, int n_mats, int keys_pad, int B, hipStream_t st) {
    const int H = mod->cfg.n_heads;
    const bool one = attn_one_fits(mod, B, keys_pad);
    A.chunk_slots = (keys_pad + CA_KEYS - 1) / CA_KEYS;
    L2Warm Wm;
    const int wz = warm_plan(Wm, mats, n_mats, one, keys_pad, H * B, H * B * (one ? 1 : A.chunk_slots));
    const dim3 grid(H, B, (one ? 1 : A.chunk_slots) + wz);           // chunk index slowest: see kc_attn
    if (mod->cfg.head_dim == 128)
        wz ? attn_launch_dh<128>(A, Wm, one, grid, st) : attn_launch_dh<128>(A, NoWarm{}, one, grid, st);
    else
        wz ? attn_launch_dh<64>(A, Wm, one, grid, st) : attn_launch_dh<64>(A, NoWarm{}, one, grid, st);
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

#define CH_MT_MAX 2          /* row tiles of 16 rows a launch covers: blocks of up to 32 rows */

// Tiles per workgroup.  (The QKV epilogue holds the most state: eight tiles with two row tiles do not fit the registers, and a model
// whose QKV matrix has more than 6 * 256 column tiles takes the per-operation kernels for such blocks.)
#define CH_FOR_ALL_NT(X, EPI, MT) X(1, EPI, MT) X(2, EPI, MT) X(3, EPI, MT) X(4, EPI, MT) X(6, EPI, MT) X(8, EPI, MT)
#define CH_FOR_QKV_TALL(X, MT) X(1, EPI_QKV, MT) X(2, EPI_QKV, MT) X(3, EPI_QKV, MT) X(4, EPI_QKV, MT) X(6, EPI_QKV, MT)
#define CH_FOR_GU(X, MT) X(2, EPI_GU, MT) X(4, EPI_GU, MT) X(6, EPI_GU, MT) X(8, EPI_GU, MT)

// Depth of the rings.  Two row tiles: the accumulators and the activation ring take more registers.  One row tile of at most eight rows: the
// activation ring is half as wide.  Per launch of the 7B shape with 6 rows: QKV (3 tiles) 18.6 / 19.0 / 18.1 / 18.8 us with rings of 4 / 6 / 8 / 10, gate|up (6)
// 31.7 / 31.1 / 31.4 / 31.7 with 2 / 3 / 4 / 5, O and down (1) 13.2 / 13.4 / 13.4 with 4 / 6 / 8, LM head (8) 42.2 to 43 with 2 to 4.
// Short sums take rings of three at most: a ring deeper than a wave's k-steps requests what is past the end (160M shape: 3 k-steps per wave, 12 for down;
// QKV 4.6 -> 4.3 us, gate|up 5.2 -> 4.5, the step 338 -> 324).  The line, K = 4096, is where the 7B shape prefers the deeper rings.  Below it, at 6 to 12
// k-steps per wave, where nothing is requested past the end, rings of three are 0 to 3 % of a step faster (1536, 2048 and 3072 features, 9 rows 340 -> 334, 292 ->
// 283, 254 -> 253 us) but with arch 1 of 2048 features, where they are 1 to 2 % slower (9 rows 377 -> 383).
#define CH_SHORT_KS (16 * CH_WAVES)
static constexpr int ch_ring(int nt, int mt, bool half, bool short_k) {
    const int r = mt == 2 ? (nt == 1 ? 4 : nt == 2 ? 3 : 2) : nt == 3 ? (half ? 8 : 4) : nt == 6 ? (half ? 3 : 2) : nt == 2 ? 6 : nt == 8 ? 2 : 4;
    return short_k && (r > 3 || (nt == 8 && mt == 1)) ? 3 : r;
}

template <int NT, int EPI, int MT>
static constexpr int chain_lds() { return CH_WAVES * NT * 64 * 16 + CH_WAVES * MT * 16 * 4; }
template <int NT, int EPI, int MT, bool HALF, bool SHORT, bool LIVE>
static constexpr auto *chain_kernel() { return kc_gemm<NT, ch_ring(NT, MT, HALF, SHORT), EPI, MT, HALF, LIVE>; }

template <int NT, int EPI, int MT, bool HALF, bool SHORT>
static hipError_t chain_allow_lds() {
    const hipError_t e = hipFuncSetAttribute((const void *)chain_kernel<NT, EPI, MT, HALF, SHORT, false>(), hipFuncAttributeMaxDynamicSharedMemorySize,
                                             chain_lds<NT, EPI, MT>());
    if (MT > 1 || e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)chain_kernel<NT, EPI, MT, HALF, SHORT, MT == 1>(), hipFuncAttributeMaxDynamicSharedMemorySize,
                               chain_lds<NT, EPI, MT>());
}

int32_t csd_chain_setup() {
#define CH_ALLOW(NT, EPI, MT)                                   \
    CSD_HIP((chain_allow_lds<NT, EPI, MT, false, false>()));    \
    CSD_HIP((chain_allow_lds<NT, EPI, MT, false, true>()));     \
    CSD_HIP((chain_allow_lds<NT, EPI, MT, true, false>()));     \
    CSD_HIP((chain_allow_lds<NT, EPI, MT, true, true>()));
    CH_FOR_ALL_NT(CH_ALLOW, EPI_QKV, 1)
    CH_FOR_ALL_NT(CH_ALLOW, EPI_RESID, 1)
    CH_FOR_ALL_NT(CH_ALLOW, EPI_LOGITS, 1)
    CH_FOR_GU(CH_ALLOW, 1)
    CH_FOR_QKV_TALL(CH_ALLOW, 2)
    CH_FOR_ALL_NT(CH_ALLOW, EPI_RESID, 2)
    CH_FOR_ALL_NT(CH_ALLOW, EPI_LOGITS, 2)
    CH_FOR_GU(CH_ALLOW, 2)
#undef CH_ALLOW
#define CA_ALLOW_ONE(DH, BIAS, LIVE, WARM)                                                                                         \
    CSD_HIP(hipFuncSetAttribute((const void *)kc_attn_one<DH, CA_ONE_NW, BIAS, LIVE, WARM>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                (int)sizeof(AttnOneLds<DH, CA_ONE_NW>)));
#define CA_ALLOW(DH, BIAS) \
    CA_ALLOW_ONE(DH, BIAS, false, NoWarm) CA_ALLOW_ONE(DH, BIAS, true, NoWarm) CA_ALLOW_ONE(DH, BIAS, false, L2Warm) CA_ALLOW_ONE(DH, BIAS, true, L2Warm)
    CA_ALLOW(128, false)
    CA_ALLOW(128, true)
    CA_ALLOW(64, false)
    CA_ALLOW(64, true)
#undef CA_ALLOW
#undef CA_ALLOW_ONE
    return CSD_OK;
}

template <int NT, int EPI, int MT, bool HALF, bool SHORT>
static void chain_launch_one(const ChainGemm &P, int G, hipStream_t st) {
    const bool live = MT == 1 && P.live && P.M == P.m;
    auto *kernel = live ? chain_kernel<NT, EPI, MT, HALF, SHORT, MT == 1>() : chain_kernel<NT, EPI, MT, HALF, SHORT, false>();
    hipLaunchKernelGGL(kernel, dim3(G), dim3(CH_THREADS), (chain_lds<NT, EPI, MT>()), st, P.Wp, P.KS, P.n_units, P.wbytes, G, P.a, P.a_plane_bytes, P.mtp,
                       P.M, P.live, P);
}

template <int EPI, int MT>
static int32_t chain_launch_mt(ChainGemm &P, int G, int per, hipStream_t st) {
    const bool half = (P.M - 1) % 16 < 8, short_k = P.KS < CH_SHORT_KS;
#define CH_LAUNCH(NT, E, MT_)                                                                                                                \
    if (per <= NT) {                                                                                                                        \
        if (half)                                                                                                                           \
            short_k ? chain_launch_one<NT, E, MT_, true, true>(P, G, st) : chain_launch_one<NT, E, MT_, true, false>(P, G, st);             \
        else                                                                                                                                \
            short_k ? chain_launch_one<NT, E, MT_, false, true>(P, G, st) : chain_launch_one<NT, E, MT_, false, false>(P, G, st);           \
        return CSD_OK;                                                                                                                      \
    }
    if constexpr (EPI == EPI_GU) {
        CH_FOR_GU(CH_LAUNCH, MT)
    } else if constexpr (EPI == EPI_QKV && MT == 2) {
        CH_FOR_QKV_TALL(CH_LAUNCH, MT)
    } else {
        CH_FOR_ALL_NT(CH_LAUNCH, EPI, MT)
    }
#undef CH_LAUNCH
    return CSD_ESHAPE;
}

template <int EPI>
static int32_t chain_launch(ChainGemm &P, int n_tiles, hipStream_t st) {
    constexpr int UT = EPI == EPI_GU ? 2 : 1;
    P.n_units = n_tiles / UT;
    const int G = chain_groups(P.n_units, UT);
    const int per = (P.n_units + G - 1) / G * UT;            // most tiles of a workgroup
    const int mt = (P.M + 15) / 16;
    if (mt == 1) return chain_launch_mt<EPI, 1>(P, G, per, st);
    if (mt == 2) return chain_launch_mt<EPI, 2>(P, G, per, st);
    return CSD_ESHAPE;
}

bool csd_planes_fit(const csd_model *mod) {
    size_t most = mod->q_plane;
    for (size_t p : mod->x_plane) most = p > most ? p : most;
    return 2 * 2 * most < (size_t)1 << 31;
}

bool csd_chain_eligible(const csd_model *mod, int32_t B, int32_t m) {
    if (!csd_planes_fit(mod)) return false;
    // (the cache appends address a layer's keys, or values, through one 32-bit offset)
    const size_t layer_kv = (size_t)mod->cfg.max_batch * mod->cfg.n_heads * mod->seq_pad * mod->cfg.head_dim * 2;
    if (B * m > 16 && 3 * mod->hd / 16 > 6 * 256) return false;
    return mod->chain_on && B * m <= 16 * CH_MT_MAX && mod->seq_pad <= CA_KEYS * CA_MAX_CHUNKS && layer_kv < (1ull << 31);
}

int32_t csd_attn_mfma_enqueue(csd_model *mod, const KvGeom &geo, const void *kv, const int32_t *cache_len, int B, int m,
                              int layer, float scale, const AttnMode &mode, hipStream_t st, bf16_t *out,
                              size_t out_plane);   // csd_attention.hip

int32_t csd_chain_enqueue(csd_model *mod, void *kv, const int32_t *tokens, const int32_t *cache_len, int32_t B, int32_t m,
                          float *logits, hipStream_t st) {
    const csd_model_cfg &c = mod->cfg;
    const int M = B * m, d = c.d_model, F = c.d_ffn, hd = mod->hd, V = c.vocab, L = c.n_layers;
    const bool t5 = c.arch == 1;     // T5-style decoder: no rotary embedding, biased unscaled scores, a cross-attention sub-layer
    const KvGeom geo{c.max_batch, c.n_heads, c.head_dim, mod->seq_pad, L, mod->kperm ? 1 : 0};
    const int mtp = mod->act_mtp;
    const int pb_d = (int)(mod->x_plane[0] * 2), pb_hd = (int)(mod->x_plane[1] * 2), pb_F = (int)(mod->x_plane[3] * 2);
    bf16_t *X1 = (bf16_t *)mod->x[0], *X2 = (bf16_t *)mod->x[1], *X3 = (bf16_t *)mod->x[2], *X4 = (bf16_t *)mod->x[3];
    float *ssq1 = mod->ssq[0], *ssq3 = mod->ssq[1];
    const float scale = t5 ? 1.0f : 1.0f / sqrtf((float)c.head_dim);
    const int ssq_rows = (M + 15) / 16 * 16;
    {
        ProfScope ps(mod, st, CSD_PROF_OTHER);
        hipLaunchKernelGGL(kc_embed, dim3(M), dim3(CE_ROW + 64), 0, st, tokens, (const bf16_t *)mod->embed, V, d, mod->layers[0].attn_norm,
                           mod->h, X1, pb_d, mtp, ssq1, ssq_rows, cache_len, m, c.head_dim, t5 ? 0.f : c.rope_theta, mod->rope,
                           mod->tree_call ? mod->tree_depth : nullptr);
        CSD_LAUNCH_CHECK();
    }
    if (mod->trace) CSD_HIP(hipMemcpyAsync(mod->trace, mod->h, sizeof(float) * (size_t)M * d, hipMemcpyDeviceToDevice, st));
    ChainGemm base{};
    base.mtp = mtp;
    base.M = M;
    base.inv_d = 1.0f / (float)d;
    base.eps = c.rms_eps;
    base.h = mod->h;
    base.d = d;
    base.m = m;
    base.hd = hd;
    base.dh = c.head_dim;
    base.geo = geo;
    base.cache_len = cache_len;
    base.rope = (!t5 && c.rope_theta > 0.f) ? mod->rope : nullptr;
    base.q = (bf16_t *)mod->qbuf;
    base.q_plane_bytes = (int)(mod->q_plane * 2);
    base.kv = (bf16_t *)kv;
    base.live = mod->live;
    base.n_ssq = d / 16;
    base.ssq_rows = ssq_rows;
    auto gemm = [&](const GemmW &w, const bf16_t *a, int a_plane_bytes, const float *ssq_in) {
        ChainGemm P = base;
        P.Wp = (const u32x4 *)w.data;
        P.KS = w.K / 32;
        P.wbytes = (int)((size_t)w.K * w.N * 2);
        P.a = a;
        P.a_plane_bytes = a_plane_bytes;
        P.ssq_in = ssq_in;
        return P;
    };
    AttnArgs attn{};
    attn.q = (const bf16_t *)mod->qbuf;
    attn.q_plane = (int)mod->q_plane;
    attn.m = m;
    attn.cache_len = cache_len;
    attn.scale = scale;
    attn.part = mod->attn_part;
    attn.chunks_max = mod->attn_chunks_max;
    attn.counters = mod->attn_cnt;
    attn.anc = mod->tree_call ? mod->tree_anc : nullptr;
    attn.out = X2;
    attn.out_plane_bytes = pb_hd;
    attn.mtp = mtp;
    attn.live = mod->live;
    auto attn_of = [&](const KvGeom &g_, const void *kv_, int l) {
        AttnArgs A = attn;
        A.geo = g_;
        A.k = (const bf16_t *)kv_ + kv_k_off(g_, l, 0, 0);
        A.v = (const bf16_t *)kv_ + kv_v_off(g_, l, 0, 0);
        return A;
    };
    int32_t rc;
    for (int l = 0; l < L; l++) {
        const LayerW &lw = mod->layers[l];
        ChainGemm Pq = gemm(lw.qkv, X1, pb_d, ssq1);
        Pq.layer = l;
        ChainGemm Po = gemm(lw.o, X2, pb_hd, nullptr);
        Po.gain = lw.ffn_norm;
        Po.out = X3;
        Po.out_plane_bytes = pb_d;
        Po.ssq_out = ssq3;
        ChainGemm Pg = gemm(lw.gu, X3, pb_d, ssq3);
        Pg.out = X4;
        Pg.out_plane_bytes = pb_F;
        ChainGemm Pd = gemm(lw.down, X4, pb_F, nullptr);
        Pd.gain = (l + 1 < L) ? mod->layers[l + 1].attn_norm : mod->final_norm;
        Pd.out = X1;
        Pd.out_plane_bytes = pb_d;
        Pd.ssq_out = ssq1;
        if (t5) {
            // QKV -> self-attention (bias by relative position) -> O (+h) -> cross-q -> cross-attention over the projected
            // encoder rows -> cross-O (+h) -> gate|up (tanh-GELU) -> down (+h): eight launches, two of them attention
            AttnMode self_mode, cross_mode;
            self_mode.rel_bias = mod->rel_bias;
            self_mode.bucket = mod->rel_bucket;
            self_mode.bias_hd = mod->rel_bias_hd;
            cross_mode.fixed_nk = c.enc_len;
            const KvGeom cgeo{c.max_batch, c.n_heads, c.head_dim, mod->enc_pad, L, 0};
            const void *kv_cross = (const char *)kv + csd_self_kv_bytes(mod);
            Po.gain = lw.cross_norm;                           // the O projection feeds the cross-attention's norm
            ChainGemm Pcq = gemm(lw.cq, X3, pb_d, ssq3);       // queries only: the epilogue of QKV with one region
            Pcq.layer = l;
            ChainGemm Pco = gemm(lw.co, X2, pb_hd, nullptr);
            Pco.gain = lw.ffn_norm;
            Pco.out = X3;
            Pco.out_plane_bytes = pb_d;
            Pco.ssq_out = ssq3;
            Pg.gelu = 1;
#define CH_STEP(EPI_, P_, W_)                                                                   \
    {                                                                                           \
        ProfScope ps(mod, st, CSD_PROF_GEMM);                                                   \
        if ((rc = chain_launch<EPI_>(P_, (W_).N / 16, st)) != CSD_OK) return rc;               \
        CSD_LAUNCH_CHECK();                                                                     \
    }
            // either attention: the kernel whose last chunk merges, or (more than 16 rows per sequence, or so many chunks
            // that bandwidth rather than latency binds) the one with longer key runs and a merge kernel
            auto attention = [&](const KvGeom &g_, const void *kv_, int keys_pad, const AttnMode &mode, const GemmW *const *mats, int n_mats) -> int32_t {
                const int chunks = (keys_pad + CA_KEYS - 1) / CA_KEYS;
                if (m > 16 || (!attn_one_fits(mod, B, keys_pad) && ((long long)chunks * c.n_heads * B > 1024 || chunks > CA_MAX_CHUNKS)))
                    return csd_attn_mfma_enqueue(mod, g_, kv_, cache_len, B, m, l, scale, mode, st, X2, mod->x_plane[1]);
                ProfScope ps(mod, st, CSD_PROF_ATTN);
                AttnArgs A = attn_of(g_, kv_, l);
                A.bias_hd = mode.bias_hd;
                A.fixed_nk = mode.fixed_nk;
                return attn_launch_small(mod, A, mats, n_mats, keys_pad, B, st);
            };
            const GemmW *const after_self[] = {&lw.o}, *const after_cross[] = {&lw.co, &lw.gu, &lw.down};
            CH_STEP(EPI_QKV, Pq, lw.qkv)
            if ((rc = attention(geo, kv, mod->seq_pad, self_mode, after_self, 1)) != CSD_OK) return rc;
            CH_STEP(EPI_RESID, Po, lw.o)
            CH_STEP(EPI_QKV, Pcq, lw.cq)
            if ((rc = attention(cgeo, kv_cross, mod->enc_pad, cross_mode, after_cross, 3)) != CSD_OK) return rc;
            CH_STEP(EPI_RESID, Pco, lw.co)
            CH_STEP(EPI_GU, Pg, lw.gu)
            CH_STEP(EPI_RESID, Pd, lw.down)
#undef CH_STEP
            if (mod->trace)
                CSD_HIP(hipMemcpyAsync(mod->trace + (size_t)(l + 1) * M * d, mod->h, sizeof(float) * (size_t)M * d,
                                       hipMemcpyDeviceToDevice, st));
            continue;
        }
        const AttnArgs A = attn_of(geo, kv, l);
        const int chunks = (mod->seq_pad + CA_KEYS - 1) / CA_KEYS;           // chunk slots; those past a sequence's rows leave at once
        {
            {
                ProfScope ps(mod, st, CSD_PROF_GEMM);
                if ((rc = chain_launch<EPI_QKV>(Pq, lw.qkv.N / 16, st)) != CSD_OK) return rc;
                CSD_LAUNCH_CHECK();
            }
            if (m > 16 || (!attn_one_fits(mod, B, mod->seq_pad) && (long long)chunks * c.n_heads * B > 1024)) {
                // many sequences or long caches: the attention is bound by bandwidth, not by latency, and the kernel
                // with longer key runs per wave (and a merge kernel) moves the cache faster; it also takes the blocks of
                // more than 16 rows per sequence
                AttnMode am;
                if (mod->tree_call) am.anc = mod->tree_anc;
                if ((rc = csd_attn_mfma_enqueue(mod, geo, kv, cache_len, B, m, l, scale, am, st, X2, mod->x_plane[1])) != CSD_OK)
                    return rc;
            } else {
                ProfScope ps(mod, st, CSD_PROF_ATTN);
                const GemmW *const mats[] = {&lw.o, &lw.gu, &lw.down};
                if ((rc = attn_launch_small(mod, A, mats, 3, mod->seq_pad, B, st)) != CSD_OK) return rc;
            }
            {
                ProfScope ps(mod, st, CSD_PROF_GEMM);
                if ((rc = chain_launch<EPI_RESID>(Po, lw.o.N / 16, st)) != CSD_OK) return rc;
                CSD_LAUNCH_CHECK();
            }
            {
                ProfScope ps(mod, st, CSD_PROF_GEMM);
                if ((rc = chain_launch<EPI_GU>(Pg, lw.gu.N / 16, st)) != CSD_OK) return rc;
                CSD_LAUNCH_CHECK();
            }
            {
                ProfScope ps(mod, st, CSD_PROF_GEMM);
                if ((rc = chain_launch<EPI_RESID>(Pd, lw.down.N / 16, st)) != CSD_OK) return rc;
                CSD_LAUNCH_CHECK();
            }
        }
        if (mod->trace)
            CSD_HIP(hipMemcpyAsync(mod->trace + (size_t)(l + 1) * M * d, mod->h, sizeof(float) * (size_t)M * d,
                                   hipMemcpyDeviceToDevice, st));
    }
    {
        ProfScope ps(mod, st, CSD_PROF_GEMM);
        ChainGemm P = gemm(mod->lm, X1, pb_d, ssq1);
        P.logits = logits;
        P.V = V;
        if ((rc = chain_launch<EPI_LOGITS>(P, mod->lm.N / 16, st)) != CSD_OK) return rc;
        CSD_LAUNCH_CHECK();
    }
    (void)F;
    return CSD_OK;
}
