// GEMM for blocks of more rows than csd_chain.hip and k_gemm_rs take (a new prompt in large blocks, the encoder rows of
// an arch 1 prompt): tiles of up to 192 columns x 128 rows per workgroup, both operands through LDS.
//
// With hundreds of rows the matrix instructions bound a launch (two activation planes: 4 * M * N * K operations), so what
// counts is how little has to move per matrix instruction.  Four waves share a tile as a 2 x 2 grid; a wave owns CTW column
// tiles x RTW row tiles of 16 and reads each of its CTW + 2 * RTW operand fragments of a k-step once from LDS for
// 2 * CTW * RTW matrix instructions.  Fragments are 1 KB of consecutive memory on both sides (weights pre-tiled,
// activations in fragment order), so a stage is brought in by direct loads to LDS, one instruction per fragment, lanes
// placed in operand order; NST stages of one k-step are in flight or in use.  A wave holds the fragments of the running
// k-step in registers and reads the next one's between its matrix instructions; one workgroup barrier per k-step.
// Row blocks of one column group go to one compute die, which then fetches those weights once.
// A wave issues in order, and with one or two waves per SIMD whatever is issued in a bunch leaves the matrix pipe empty: operand reads and
// loads go between the matrix instructions one at a time (in a bunch per column tile: a prompt of 1000 rows of the 7B shape 27.6 ms against 26.5; in traces of
// whole calls, blocks of 512 and 488 rows, QKV 94.6 us against 89.8, O and down together 115 against 108, LM head 233 against 229, gate|up 147 against 149).
// 7B shape, 512 rows, against four launches of the row-split form over 128 rows each, every GEMM timed by itself before that: QKV 122 -> 81 us,
// gate|up 188 -> 146, down 111 -> 79, O 57 -> 34, LM head 254 -> 223.
// What bounds QKV now, by the counters: of 196000 cycles a SIMD's matrix pipe is busy for 98000, waves wait 30000 for barriers and loads,
// 28000 are launch and teardown; the rest is prologue, epilogue, and what does not fit between the matrix instructions.  Loads further ahead (four and five
// stages: 94.6 and 96.1 us against 94.9) and the 32x32x16 instruction (10 % slower in a loop of nothing else on random operands: 1.8 against 2.0
// PFLOP/s) gain nothing.
#include "csd_tall.h"

// EPI_CROSS: keys | values of the encoder rows into the cross-attention part of the cache
__device__ __forceinline__ void cross_epilogue(const TallArgs &A, const f32x4 &v, int row, int T, int g) {
    const ChainGemm &P = A.g;
    if (row >= P.M) return;
    const int r = A.row0 + row, b = r / A.enc_len, pos = r % A.enc_len;
    const bool is_v = T >= P.hd / 16;
    const int j = (is_v ? T - P.hd / 16 : T) * 16 + 4 * g, hh = j / P.dh, x = j % P.dh;
    if (!is_v) {
        u32x2 k;
        k[0] = pack_bf16x2(v[0], v[1]);
        k[1] = pack_bf16x2(v[2], v[3]);
        *reinterpret_cast<u32x2 *>(P.kv + kv_k_off(P.geo, P.layer, b, hh) + (size_t)pos * P.dh + x) = k;
    } else {
        bf16_t *vc = P.kv + kv_v_off(P.geo, P.layer, b, hh);
#pragma unroll
        for (int i = 0; i < 4; i++) vc[kv_v_idx(P.geo, x + i, pos)] = f32_to_bf16(v[i]);
    }
}

// Sums over K in chains, as many as the row-split form has K splits for the same matrix: one chain through all of K rounds at the
// size of the whole sum in every step (7B shape, two layers, 512 rows, against 64 bits with the K/V rows as stored: logits off by
// 5.52e-6 in one chain, 5.42e-6 in chains and with the row-split form; encoder rows through 4096 features: 2.7e-4 of the K/V
// elements rounded to the other side in one chain, 2.0e-4 with the split form, 1.5e-4 in chains).  At a chain's end the
// accumulators go into a second set of sums and start from zero.  Where two workgroups with 6 x 4 tiles per wave share a compute
// unit there are no registers for a second set (one workgroup per compute unit: gate|up at 512 rows 8 % slower; the sums in memory:
// 15 %): the upper 16 bits of the sum are set aside, packed in pairs, two thirds in registers and the rest in LDS, and the
// accumulators go on from what is left below them, which is exact and as good as zero.  Cost of either: 1 to 2 % of a call.
template <int CTW, int RTW, int NST>
static constexpr bool tall_sums() { return !(CTW == 6 && RTW == 4 && NST == 2); }
#define TALL_LEADS 16         /* tiles of a wave whose upper halves stay in registers */

template <int CTW, int RTW, int NST, int EPI>
__global__ __launch_bounds__(256, CTW == 6 && RTW == 4 && NST == 3 ? 1 : 2) void k_gemm_tall(TALL_PARAMS) {
    TALL_UNPACK(A)
    constexpr bool SUMS = tall_sums<CTW, RTW, NST>();
    extern __shared__ __align__(16) char tall_smem[];
    constexpr int WF = 2 * CTW, NF = WF + 4 * RTW;               // fragments of a stage: W tiles, then [plane][row tile]
    static_assert(WF % 4 == 0 && NF % 4 == 0, "every wave brings as many of either kind");
    constexpr int PW = NF / 4;                                   // per wave: fragments w, w + 4, ...
    constexpr int STB = NF * 1024;                               // bytes of a stage
    const ChainGemm &P = A.g;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // workgroups go to the eight compute dies round-robin: consecutive tiles to the workgroups of one die
    const int grid = (A.n_tiles + WF - 1) / WF * A.rblocks * A.S, per_die = grid >> 3, rest = grid & 7, die = blockIdx.x & 7;
    const int wg = die * per_die + (die < rest ? die : rest) + (blockIdx.x >> 3);
    const int rb = wg % A.rblocks, s = (wg / A.rblocks) % A.S, grp = wg / (A.rblocks * A.S);
    const int ks0 = (int)((long long)P.KS * s / A.S), ks1 = (int)((long long)P.KS * (s + 1) / A.S);
    const int tile0 = grp * WF, rt0 = rb * 2 * RTW;
    const __amdgpu_buffer_rsrc_t rw = ch_rsrc(P.Wp, (size_t)P.wbytes);
    // (both planes of the input may take up to 4 GiB: no load here counts on an offset beyond 2 GiB being outside)
    const __amdgpu_buffer_rsrc_t ra =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(P.a), 0, (int)(2u * (unsigned)P.a_plane_bytes), 0x00020000);
    // Tiles and row tiles past the end are read as the last one (their sums are not stored), k-steps past the slice likewise:
    // every address is inside the matrix, and every wave issues PW loads per stage, so the waits can count them.
    unsigned base[PW];
#pragma unroll
    for (int i = 0; i < PW; i++) {
        const int f = i * 4 + w, a = f - WF;
        base[i] = i < WF / 4 ? min(tile0 + f, A.n_tiles - 1) * P.KS * 1024
                             : a / (2 * RTW) * (unsigned)P.a_plane_bytes + min(rt0 + a % (2 * RTW), P.mtp - 1) * 1024;
    }
    // Activations: a fragment is 16 rows of 64 bytes.  Four lanes fetch a row's (lanes 64 bytes apart get 33 bytes per cycle into a compute unit,
    // neighbours 55), in an order that spreads the 16 bytes of a lane group's rows over all banks when they are read as operands.
    const int vw = lane * 16, va = (lane ^ (lane >> 4)) * 16;
    // load i of this wave for k-step ks, whose stage begins at byte `stage` (its place for this wave: + w KB)
    auto load_part = [&](int i, int ks, int stage) {
        const int k = min(ks, ks1 - 1);
        const lds_void d = (lds_void)(tall_smem + stage + w * 1024 + i * 4096);
        if (i < WF / 4)
            lds_load16<0>(rw, d, vw, (int)(base[i] + k * 1024));
        else
            lds_load16<0>(ra, d, va, (int)(base[i] + k * P.mtp * 1024));
    };
    const int wc = w & 1, wr = w >> 1;
    f32x4 acc[RTW][CTW];
#pragma unroll
    for (int r = 0; r < RTW; r++)
#pragma unroll
        for (int c = 0; c < CTW; c++) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < NST; p++)
#pragma unroll
        for (int i = 0; i < PW; i++) load_part(i, ks0 + p, p * STB);
    f32x4 sum[RTW][CTW];
    u32x2 lead[TALL_LEADS];
    u32x2 *lead_lds = reinterpret_cast<u32x2 *>(tall_smem + NST * NF * 1024) + threadIdx.x;
    auto set_lead = [&](int i, u32x2 v) {
        if (i < TALL_LEADS)
            lead[i] = v;
        else
            lead_lds[(i - TALL_LEADS) * 256] = v;
    };
    auto get_lead = [&](int i) { return i < TALL_LEADS ? lead[i < TALL_LEADS ? i : 0] : lead_lds[(i - TALL_LEADS) * 256]; };
#pragma unroll
    for (int r = 0; r < RTW; r++)
#pragma unroll
        for (int c = 0; c < CTW; c++) {
            sum[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (!SUMS) set_lead(r * CTW + c, u32x2{0u, 0u});
        }
    // this wave's operands of a stage: W tiles, (hi) row tiles
    const char *Lw = tall_smem + wc * CTW * 1024 + lane * 16;
    const char *La = tall_smem + (WF + wr * RTW) * 1024 + ((lane & 15) * 4 + ((lane >> 4) ^ ((lane >> 2) & 3))) * 16;
    u32x4 fa[2][2 * RTW], fw[2][CTW];                            // [k-step parity]
    // operand i of a k-step: W tile i, then hi and lo row tiles
    auto read_part = [&](int i, int set, int stage) {
        if (i < CTW)
            fw[set][i] = *reinterpret_cast<const u32x4 *>(Lw + stage + i * 1024);
        else
            fa[set][i - CTW] = *reinterpret_cast<const u32x4 *>(La + stage + ((i - CTW) / RTW * 2 * RTW + (i - CTW) % RTW) * 1024);
    };
    wait_loads<(NST - 1) * PW>();
    stage_barrier();
#pragma unroll
    for (int i = 0; i < CTW + 2 * RTW; i++) read_part(i, 0, 0);
    int cur = 0, nxt = STB;
    // k-step K with its fragments in set PAR: the stage behind it has arrived, its own stage is free for k-step K + NST.  A wave issues
    // in order, and a matrix instruction takes as long as four others: what else there is to issue (two operand reads, then a load with its two
    // address sums) goes between them one by one.  With two stages the loads come first, since all they have to arrive in is the rest of the k-step (512
    // rows, gate|up 161 -> 156 us, LM head 257 -> 238; all of them in front of the first matrix instruction: 166 and 245).
#define TALL_STEP(PAR, K)                                                                                             \
    {                                                                                                                 \
        wait_loads<(NST - 2) * PW>();                                                                                 \
        stage_barrier();                                                                                              \
        _Pragma("unroll") for (int n = 0; n < 2 * CTW * RTW; n++) {                                                   \
            const int c = n / (2 * RTW), a = n % (2 * RTW), r = a % RTW;                                              \
            acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[PAR][c]),               \
                                                                __builtin_bit_cast(bf16x8, fa[PAR][a]), acc[r][c], 0, 0, 0); \
            _Pragma("unroll") for (int j = 0; j < 3 * PW; j++) if (j * (2 * CTW * RTW - 4) / (3 * PW) == n) {         \
                if (NST == 2 ? j < PW : j % 3 == 2)                                                                   \
                    load_part(NST == 2 ? j : j / 3, (K) + NST, cur);                                                  \
                else                                                                                                  \
                    read_part(NST == 2 ? j - PW : j / 3 * 2 + j % 3, 1 - (PAR), nxt);                                 \
            }                                                                                                         \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
        }                                                                                                             \
        cur = nxt;                                                                                                    \
        nxt = nxt + STB == NST * STB ? 0 : nxt + STB;                                                                 \
    }
    const int t = lane & 15, g = lane >> 4;
    bool kept = false;                                           // uniform
    int k = ks0;
    for (;;) {
        const int ke = min(k + A.chain, ks1);
        for (; k + 1 < ke; k += 2) {
            TALL_STEP(0, k)
            TALL_STEP(1, k + 1)
        }
        if (k + 1 >= ks1) break;
        asm volatile("");                                        // (a branch, not a selection between both outcomes)
#pragma unroll
        for (int r = 0; r < RTW; r++)
#pragma unroll
            for (int c = 0; c < CTW; c++) {
                if constexpr (SUMS) {
                    sum[r][c] += acc[r][c];
                    acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
                } else {
                    u32x2 ld = get_lead(r * CTW + c);
#pragma unroll
                    for (int i = 0; i < 4; i++) {            // (a sum that is not finite stays one in the upper half)
                        const float old = __uint_as_float(i & 1 ? ld[i / 2] & 0xFFFF0000u : ld[i / 2] << 16);
                        const uint32_t top = __float_as_uint(old + acc[r][c][i]) & 0xFFFF0000u;
                        const float rest = acc[r][c][i] - (__uint_as_float(top) - old);
                        acc[r][c][i] = __builtin_isfinite(rest) ? rest : 0.f;
                        ld[i / 2] = i & 1 ? (ld[i / 2] & 0xFFFFu) | top : (ld[i / 2] & 0xFFFF0000u) | (top >> 16);
                    }
                    set_lead(r * CTW + c, ld);
                }
            }
        kept = true;
    }
    if (k < ks1) TALL_STEP(0, k)
#undef TALL_STEP
    wait_loads<0>();                                             // nothing may land in this LDS after the workgroup has ended
    if (kept) {
        asm volatile("");
#pragma unroll
        for (int r = 0; r < RTW; r++)
#pragma unroll
            for (int c = 0; c < CTW; c++) {
                if constexpr (SUMS) {
                    acc[r][c] += sum[r][c];
                } else {
                    const u32x2 ld = get_lead(r * CTW + c);
#pragma unroll
                    for (int h = 0; h < 2; h++) {
                        acc[r][c][2 * h] += __uint_as_float(ld[h] << 16);
                        acc[r][c][2 * h + 1] += __uint_as_float(ld[h] & 0xFFFF0000u);
                    }
                }
            }
    }

#pragma unroll
    for (int r = 0; r < RTW; r++) {
        const int row = (rt0 + wr * RTW + r) * 16 + t;
        const bool valid = row < P.M;
        float rs = 1.f;
        if (EPI != EPI_PART && EPI != EPI_CROSS) rs = valid ? A.rstd[row] : 0.f;
        EpiIn E;
        E.hcur = E.gcur = f32x4{0.f, 0.f, 0.f, 0.f};
        E.pos = EPI == EPI_QKV && valid ? P.cache_len[row / P.m] + row % P.m : -1;
        constexpr int UT = EPI == EPI_GU ? 2 : 1;
#pragma unroll
        for (int c = 0; c < CTW; c += UT) {
            const int T = tile0 + wc * CTW + c;
            if (T >= A.n_tiles) break;                           // uniform
            if constexpr (EPI == EPI_PART) {
                if (valid) *reinterpret_cast<f32x4 *>(A.part + (((size_t)s * P.M + row) * A.n_tiles + T) * 16 + 4 * g) = acc[r][c];
            } else if constexpr (EPI == EPI_CROSS) {
                cross_epilogue(A, acc[r][c], row, T, g);
            } else {
#pragma unroll
                for (int i = 0; i < 4; i++) E.cs[i] = float2{1.f, 0.f};
                if (EPI == EPI_QKV && P.rope && valid && T < 2 * (P.hd / 16)) {
                    const int ti = T % (P.hd / 16) % (P.dh / 16);
#pragma unroll
                    for (int i = 0; i < 4; i++) E.cs[i] = P.rope[(size_t)row * (P.dh / 2) + 8 * ti + 4 * (g & 1) + i];
                }
                f32x4 v[UT];
#pragma unroll
                for (int i = 0; i < UT; i++) v[i] = acc[r][c + i] * rs;
                // (plain stores: neighbouring lanes and tiles fill whole lines in L2; written through, QKV took 8 us more)
                gemm_epilogue<EPI, 0>(P, v, E, row, T, g);
            }
        }
    }
}

// ------------------------------------------------------------------------------- host driver

template <int CTW, int RTW, int NST>
static constexpr int tall_lds() {
    return NST * (2 * CTW + 4 * RTW) * 1024 + (tall_sums<CTW, RTW, NST>() ? 0 : (CTW * RTW - TALL_LEADS) * 256 * 8);
}

template <int CTW, int RTW, int NST, int EPI>
static hipError_t tall_allow_lds() {
    return hipFuncSetAttribute((const void *)k_gemm_tall<CTW, RTW, NST, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               tall_lds<CTW, RTW, NST>());
}

int32_t csd_tall_setup() {
#define TALL_ALLOW_R(RTW, EPI)                       \
    CSD_HIP((tall_allow_lds<4, RTW, 4, EPI>()));     \
    CSD_HIP((tall_allow_lds<6, RTW, 3, EPI>()));     \
    CSD_HIP((tall_allow_lds<6, RTW, 2, EPI>()));
#define TALL_ALLOW(EPI) TALL_ALLOW_R(2, EPI) TALL_ALLOW_R(3, EPI) TALL_ALLOW_R(4, EPI)
    TALL_ALLOW(EPI_PART)
    TALL_ALLOW(EPI_CROSS)
    TALL_ALLOW(EPI_QKV)
    TALL_ALLOW(EPI_GU)
    TALL_ALLOW(EPI_LOGITS)
#undef TALL_ALLOW
#undef TALL_ALLOW_R
    return CSD_OK;
}

// Column tiles per wave (6 or 4), row tiles per wave (4, 3 or 2: row blocks of 128, 96 or 64) and K splits: the triple with the
// shortest launch by a model whose constants were fitted to traces of the 7B and 160M shapes at 160 to 512 rows with operand reads and loads in
// bunches.  Traces of the present loop, the same shapes in all six forms with two and three stages: the form it picks for QKV, gate|up and the LM head is on average 0.6 % slower
// than the fastest one, 1.5 % at most at the 7B shape (LM head, 384 rows 160.6 us against 158.3) and 6 % at the 160M shape (LM head, 512 rows 54.0 against 50.8,
// three stages instead of two).  A k-step of one workgroup per compute unit takes `one` us; with 6
// column tiles and more workgroups than compute units two share one (two stages each) and 512 of them take `two`; 4 column tiles go in rounds of
// 256.  Beside it the prologue and the epilogue, 0.5 us per tile of a wave (once per round where only one workgroup fits a compute unit,
// else under the other's k-steps), and the splits' partial sums.
// Narrow tiles fill the chip where a matrix is small or its row blocks few (all figures of the present loop in traces of whole calls): 160M shape, 512 rows, QKV 29.4 us in 48
// workgroups of 6 x 4 tiles per wave, 13.5 in 144 of 4 x 2; 7B shape, 384 rows, QKV 87.4 us at 6 x 4 (192 workgroups), 77.7 at 6 x 3 (256); 512 rows, where 6 x 4
// makes 256 workgroups, 91.9 against 117.9 at 6 x 3.  max_splits = 1 where the epilogue runs in the kernel.
// Stages: four of the narrow tiles; with 6 column tiles and more workgroups than compute units two of them share one (two stages
// each), which evens out the last round: gate|up at 512 rows 151 us against 165 with three stages and one workgroup at a time; at 256
// workgroups (QKV) 124 against 92.
struct TallPlan {
    int ctw, rtw, stages, S, rblocks, grid, chain;
};
static TallPlan tall_plan(int n_tiles, int KS, int M, int max_splits, size_t part_floats) {
    static const struct {
        int ctw, rtw;
        double one, two;
    } forms[6] = {{6, 4, 0.60, 1.09}, {6, 3, 0.49, 0.885}, {6, 2, 0.43, 0.85}, {4, 4, 0.45, 0}, {4, 3, 0.37, 0}, {4, 2, 0.29, 0}};
    const int row_tiles = (M + 15) / 16;
    int ct = 0, chains = 1;                                      // as the row-split form over 128 rows, memory for its partial sums aside
    (void)csd_rs_plan_host(n_tiles * 16, KS * 32, 128, (size_t)1 << 60, &ct, &chains);
    const int chain = ((KS + chains - 1) / chains + 1) / 2 * 2;
    TallPlan best{};
    double best_us = 1e30;
    for (const auto &f : forms) {
        const int rblocks = (row_tiles + 2 * f.rtw - 1) / (2 * f.rtw), groups = (n_tiles + 2 * f.ctw - 1) / (2 * f.ctw);
        for (int S = 1; S <= max_splits; S++) {
            if (S > 1 && (KS / S < 6 || (size_t)S * M * n_tiles * 16 > part_floats)) break;
            const long long wgs = (long long)groups * rblocks * S;
            const bool pairs = f.ctw == 6 && wgs > 256;
            const double rounds = (double)(pairs ? (wgs + 511) / 512 : (wgs + 255) / 256);
            const double ends = 0.5 * f.ctw * f.rtw * (f.ctw == 4 && f.rtw == 4 ? rounds : 1.0);
            const double us = rounds * ((KS + S - 1) / S) * (pairs ? f.two : f.one) + ends +
                              (max_splits > 1 ? S * 4.0 * M * n_tiles * 16 / 4e6 : 0.0);
            if (us < best_us) best_us = us, best = TallPlan{f.ctw, f.rtw, f.ctw == 4 ? 4 : pairs ? 2 : 3, S, rblocks, (int)wgs, chain};
        }
    }
    return best;
}

int32_t csd_tall_plan_host(int32_t N, int32_t K, int32_t rows, int32_t max_splits, size_t part_floats, int32_t *ctw, int32_t *rtw,
                           int32_t *stages, int32_t *S) {
    if (!ctw || !rtw || !stages || !S) return CSD_ENULL;
    if (N <= 0 || K <= 0 || N % 16 || K % 32 || rows < 1 || max_splits < 1) return CSD_EINVAL;
    const TallPlan p = tall_plan(N / 16, K / 32, rows, max_splits, part_floats);
    *ctw = p.ctw, *rtw = p.rtw, *stages = p.stages, *S = p.S;
    return CSD_OK;
}

template <int EPI>
static int32_t tall_launch(const csd_model *mod, TallArgs &A, int max_splits, hipStream_t st) {
    const TallPlan p = tall_plan(A.n_tiles, A.g.KS, A.g.M, max_splits, mod->part_floats);
    A.S = p.S;
    A.rblocks = p.rblocks;
    A.chain = p.chain;
#define TALL_LAUNCH(CTW, RTW, NST) \
    hipLaunchKernelGGL((k_gemm_tall<CTW, RTW, NST, EPI>), dim3(p.grid), dim3(256), (tall_lds<CTW, RTW, NST>()), st, TALL_ARGS(A))
#define TALL_LAUNCH_R(RTW)                                \
    {                                                     \
        if (p.ctw == 4) TALL_LAUNCH(4, RTW, 4);           \
        else if (p.stages == 2) TALL_LAUNCH(6, RTW, 2);   \
        else TALL_LAUNCH(6, RTW, 3);                      \
    }
    if (p.rtw == 4) TALL_LAUNCH_R(4)
    else if (p.rtw == 3) TALL_LAUNCH_R(3)
    else TALL_LAUNCH_R(2)
#undef TALL_LAUNCH_R
#undef TALL_LAUNCH
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

int32_t csd_tall_part(csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int M, int *S_used, hipStream_t st) {
    TallArgs A = tall_args(mod, w, a, plane, mod->act_mtp, M);
    A.part = mod->part;
    const int32_t rc = tall_launch<EPI_PART>(mod, A, w.S < 8 ? w.S : 8, st);
    *S_used = A.S;
    return rc;
}

bool csd_tall_fused(const csd_model *mod, int M) {
    if (!csd_planes_fit(mod)) return false;
    // the cache appends of the epilogue address a layer's keys, or values, through one 32-bit offset
    const size_t layer_kv = (size_t)mod->cfg.max_batch * mod->cfg.n_heads * mod->seq_pad * mod->cfg.head_dim * 2;
    return mod->chain_on && M >= CSD_TALL_MIN_ROWS && layer_kv < (1ull << 31);
}

int32_t csd_tall_qkv(csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int M, int m, int layer, const KvGeom &geo,
                     void *kv, const int32_t *cache_len, const float2 *rope, hipStream_t st) {
    TallArgs A = tall_args(mod, w, a, plane, mod->act_mtp, M);
    A.g.m = m;
    A.g.layer = layer;
    A.g.geo = geo;
    A.g.kv = (bf16_t *)kv;
    A.g.cache_len = cache_len;
    A.g.rope = rope;
    A.g.q = (bf16_t *)mod->qbuf;
    A.g.q_plane_bytes = (int)(mod->q_plane * 2);
    return tall_launch<EPI_QKV>(mod, A, 1, st);
}

int32_t csd_tall_gu(csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int M, bf16_t *out, size_t out_plane, int gelu,
                    hipStream_t st) {
    TallArgs A = tall_args(mod, w, a, plane, mod->act_mtp, M);
    A.g.out = out;
    A.g.out_plane_bytes = (int)(out_plane * 2);
    A.g.gelu = gelu;
    return tall_launch<EPI_GU>(mod, A, 1, st);
}

int32_t csd_tall_logits(csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int M, float *logits, hipStream_t st) {
    TallArgs A = tall_args(mod, w, a, plane, mod->act_mtp, M);
    A.g.logits = logits;
    A.g.V = w.N;
    return tall_launch<EPI_LOGITS>(mod, A, 1, st);
}

int32_t csd_tall_cross(csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int mtp, int M, int row0, int layer,
                       const KvGeom &geo, void *kv_cross, hipStream_t st) {
    TallArgs A = tall_args(mod, w, a, plane, mtp, M);
    A.enc_len = mod->cfg.enc_len;
    A.row0 = row0;
    A.g.layer = layer;
    A.g.geo = geo;
    A.g.kv = (bf16_t *)kv_cross;
    return tall_launch<EPI_CROSS>(mod, A, 1, st);
}
