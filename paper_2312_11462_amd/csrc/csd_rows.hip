// GEMM for blocks of 33 to 144 rows (3 to 9 row tiles of 16), where the matrix cores and the traffic of a compute unit matter as
// much as HBM.
//
// The rows are split over the waves of a workgroup (RW row tiles each) and the weights are what is shared: CT column tiles come
// into LDS by direct loads, a k-step per stage, every wave bringing its share and reading every fragment once for 2 * RW
// matrix instructions; a wave's own activation fragments go straight to registers.  Both streams run NSET - 1 k-steps ahead
// (loads return in order, so a wait for the activations of a k-step is one for all weights issued before them: the weights
// cannot run further ahead than the activations).  One barrier per k-step, the loads of a k-step dealt between its matrix
// instructions, so that a wave that waits for a place in the memory pipeline has instructions in the matrix pipe meanwhile.
// K is split over workgroups (rs_plan), one chain of sums per split.
//
// Bound by what a compute unit moves (activations from L2: every workgroup reads all rows of its K slice) and, at 40 rows, by
// the weight stream.  Against the form before it, whose four extra waves carried the weights to LDS through registers
// and whose compute waves always owned two or three row tiles (33 to 48 rows kept two of four busy, 144 rows three), per launch of the 7B
// shape in traces of whole steps: 40 rows QKV 24.8 -> 22.6 us, gate|up 37.7 -> 33.8, O and down together 34.0 -> 31.5; 136 rows QKV and
// gate|up together 98.8 -> 94.4, O and down 53.9 -> 52.0.  (Today, with the arguments in registers and the last turn without
// loads: 20.8, 32.4, 29.8; 88.7, 51.2.)  The weights are read once, so they pass the caches by (non-temporal: 22.2
// -> 20.5 us for QKV at 40 rows by itself).  Measured and not taken: 6 to 12 k-steps ahead (no faster), the fragments of 5, 6 and 9 row
// tiles dealt to four waves, a tile in two halves (fewer matrix instructions per wave, more loads: 136 rows 7755 -> 8000 us per step), one fragment for both planes
// of a last tile of up to eight rows (40 rows 5119 -> 5109, 72 rows 4775 -> 4720, 136 rows 7760 -> 7820), all of K in one workgroup
// and the epilogue inside (40 rows, gate|up by itself 39 to 43 us against 33 and 5 for the epilogue kernel; 136 rows 68.8 against 58.0 and 7.8).
#include "csd_tall.h"

#include <type_traits>

#define RS_SETS 4             /* k-steps of activations in registers; as many stages of weights, and one in use, in LDS */

// A stage's weight tiles, with four waves also places for what the padding loads write.
template <int CT, int NW>
static constexpr int rs_tiles() { return NW == 4 ? (CT + 3) / 4 * 4 : CT; }
template <int CT, int NW>
static constexpr int rs_lds() { return (RS_SETS + 1) * rs_tiles<CT, NW>() * 1024; }

template <int CT, int RW, int NW>
__global__ __launch_bounds__(NW * 64, 1) void k_gemm_rs(TALL_PARAMS) {
    TALL_UNPACK(A)
    extern __shared__ __align__(16) char rs_smem[];
    constexpr int PW = (CT + NW - 1) / NW;                       // weight loads per wave and k-step
    constexpr int AL = 2 * RW, NA = RS_SETS - 1, NST = RS_SETS + 1;
    constexpr int RA = CT * RW < 48 ? 4 : 3;                     // weight fragments read ahead (48 sums a lane and four spill)
    // Every wave issues the same loads in every k-step that issues any, so the waits can count them, and some of them bring nothing that is used:
    // k-steps past the slice, and the waves' last tiles where CT is no multiple of the waves.  With four waves those are out of the buffer, where a
    // load reads no memory: re-reading the slice's last k-step, or the last tile into its own place, cost more (7B shape, whole steps, 128 rows 5667 us
    // against 5693).  With three waves the selects cost as much as that (160M shape, 136 rows 824 against 835; 40 rows 1010 against 1002), and
    // everything past an end is read as the last one.
    constexpr bool SKIP = NW == 4;
    constexpr int TILES = rs_tiles<CT, NW>();
    const ChainGemm &P = A.g;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // workgroups go to the eight compute dies round-robin: consecutive shares to the workgroups of one die
    const int grid = (A.n_tiles + CT - 1) / CT * A.S, per_die = grid >> 3, rest = grid & 7, die = blockIdx.x & 7;
    const int wg = die * per_die + (die < rest ? die : rest) + (blockIdx.x >> 3);
    const int s = wg % A.S, grp = wg / A.S;
    const int ks0 = (int)((long long)P.KS * s / A.S), ks1 = (int)((long long)P.KS * (s + 1) / A.S);
    const int tile0 = grp * CT, rt0 = w * RW;
    const __amdgpu_buffer_rsrc_t rw = ch_rsrc(P.Wp, (size_t)P.wbytes);
    const __amdgpu_buffer_rsrc_t ra =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(P.a), 0, (int)(2u * (unsigned)P.a_plane_bytes), 0x00020000);
    // Column tiles and row tiles past the end are read as the last one (their sums are not stored): every address is inside the matrix,
    // or outside the buffer.
    int wbase[PW];
#pragma unroll
    for (int i = 0; i < PW; i++) wbase[i] = min(tile0 + min(i * NW + w, CT - 1), A.n_tiles - 1) * P.KS * 1024;
    unsigned abase[RW];
#pragma unroll
    for (int r = 0; r < RW; r++) abase[r] = min(rt0 + r, (P.M - 1) >> 4) * 1024;
    const int vw = lane * 16, va = (4 * (lane & 15) + (lane >> 4)) * 16;     // see act_tiled_idx
    auto load_w = [&](int i, int k, int buf) {
        const int t = i * NW + w;
        const bool none = SKIP && (t >= CT || k >= ks1);         // (uniform)
        lds_load16<2>(rw, (lds_void)(rs_smem + (buf * TILES + (SKIP ? t : min(t, CT - 1))) * 1024), none ? CH_OOB : vw,
                      none ? 0 : wbase[i] + min(k, ks1 - 1) * 1024);
    };
    u32x4 fa[RS_SETS][RW][2];
    auto load_a = [&](int i, int k, int set) {
        const bool none = SKIP && k >= ks1;                      // (uniform; in planes of more than 2 GiB together it is read at 2 GiB)
        const unsigned off = none ? 0u : abase[i >> 1] + (unsigned)(min(k, ks1 - 1) * P.mtp) * 1024u + (i & 1 ? (unsigned)P.a_plane_bytes : 0u);
        fa[set][i >> 1][i & 1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, none ? CH_OOB : va, (int)off, 0));
    };
    f32x4 acc[RW][CT];
#pragma unroll
    for (int r = 0; r < RW; r++)
#pragma unroll
        for (int c = 0; c < CT; c++) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // order of issue: W(0), then A(k), W(k + 1) for k = 0 .. NA - 1; in k-step k: A(k + NA), W(k + NA + 1)
#pragma unroll
    for (int i = 0; i < PW; i++) load_w(i, ks0, 0);
#pragma unroll
    for (int p = 0; p < NA; p++) {
#pragma unroll
        for (int i = 0; i < AL; i++) load_a(i, ks0 + p, p);
#pragma unroll
        for (int i = 0; i < PW; i++) load_w(i, ks0 + p + 1, p + 1);
    }
    const u32x4 *L = reinterpret_cast<const u32x4 *>(rs_smem) + lane;
    u32x4 f[CT + RA];
    wait_loads<NA * (PW + AL)>();
    stage_barrier();
#pragma unroll
    for (int c = 0; c < RA; c++) f[c] = L[c * 64];
    int cur = 0, last = NST - 1, k = ks0;                        // the stages of W(k) and of W(k - 1), the latter free for W(k + NA + 1)
    // END: how many k-steps behind the last one that issued loads (0: this one issues its own).  The last k-steps of a slice issue none, also where the
    // slice is whole turns: a load costs its time in the memory pipeline whether its data is used or not (7B shape, whole steps, 40 rows 5196 ->
    // 5134 us, 136 rows 7983 -> 7755, 128 rows 5689 -> 5667; 160M shape, 136 rows 794 -> 779; T5 shape, 40 rows 3916 -> 3849).  The compiler takes
    // loads of activations that are not used out by itself, but not those to LDS, and the waits have to count what is issued.  A slice that ends one
    // or two k-steps after a turn still requests two or one too many: a tail for each remainder spilt registers, and no form of this kernel may spill
    // (accesses to scratch memory are counted by the same waits).
    auto step = [&](int set, auto END) __attribute__((always_inline)) {
        constexpr int E = decltype(END)::value;
        wait_loads<(E ? NA - E : NA - 1) * (PW + AL)>();         // W(k + 1), this wave's share
        stage_barrier();
        const u32x4 *Lc = L + cur * TILES * 64;
        const int nxt = cur + 1 == NST ? 0 : cur + 1;
        const u32x4 *Ln = L + nxt * TILES * 64;
#pragma unroll
        for (int c = 0; c < CT; c++) {
            f[c + RA] = c + RA < CT ? Lc[(c + RA) * 64] : Ln[(c + RA - CT) * 64];
#pragma unroll
            for (int i = 0; i < AL + PW; i++)
                if (E == 0 && i * CT / (AL + PW) == c) {
                    if (i < AL)
                        load_a(i, k + NA, (set + NA) % RS_SETS);
                    else
                        load_w(i - AL, k + NA + 1, last);
                }
#pragma unroll
            for (int p = 0; p < 2; p++)
#pragma unroll
                for (int r = 0; r < RW; r++)
                    acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[c]),
                                                                        __builtin_bit_cast(bf16x8, fa[set][r][p]), acc[r][c], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < RA; c++) f[c] = f[c + CT];
        last = cur;
        cur = nxt;
        k++;
    };
    while (k + RS_SETS < ks1) {
#pragma unroll
        for (int u = 0; u < RS_SETS; u++) step(u, std::integral_constant<int, 0>{});
    }
    static_assert(RS_SETS == 4, "a k-step of each remainder");
    if (k + RS_SETS == ks1) {                                    // uniform over the workgroup
        step(0, std::integral_constant<int, 0>{});
        step(1, std::integral_constant<int, 1>{});
        step(2, std::integral_constant<int, 2>{});
        step(3, std::integral_constant<int, 3>{});
    } else {
        step(0, std::integral_constant<int, 1>{});
        if (k < ks1) step(1, std::integral_constant<int, 2>{});
        if (k < ks1) step(2, std::integral_constant<int, 3>{});
    }
    wait_loads<0>();                                             // nothing may land in this LDS after the workgroup has ended

    const int t = lane & 15, g = lane >> 4;
#pragma unroll
    for (int r = 0; r < RW; r++) {
        const int row = (rt0 + r) * 16 + t;
        if (row < P.M) {
#pragma unroll
            for (int c = 0; c < CT; c++)
                if (tile0 + c < A.n_tiles)
                    *reinterpret_cast<f32x4 *>(A.part + (((size_t)s * P.M + row) * A.n_tiles + tile0 + c) * 16 + 4 * g) = acc[r][c];
        }
    }
}

// ------------------------------------------------------------------------------- host driver

// Waves and row tiles per wave for 3 to 9 row tiles: three or four waves of one, two or three.  5 and 7 row tiles (65 to 80, 97 to 112 rows) are
// 3 and 4 waves of two, the last one's second tile all padding.
#define RS_FOR_ALL_ROWS(X) X(1, 3) X(1, 4) X(2, 3) X(2, 4) X(3, 3)
#define RS_FOR_ALL_CT(X, RW, NW) X(16, RW, NW) X(12, RW, NW) X(11, RW, NW) X(8, RW, NW) X(6, RW, NW)

template <int CT, int RW, int NW>
static hipError_t rs_allow_lds() {
    return hipFuncSetAttribute((const void *)k_gemm_rs<CT, RW, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, (rs_lds<CT, NW>()));
}

int32_t csd_rows_setup() {
#define RS_ALLOW(CT, RW, NW) CSD_HIP((rs_allow_lds<CT, RW, NW>()));
#define RS_ALLOW_ALL(RW, NW) RS_FOR_ALL_CT(RS_ALLOW, RW, NW)
    RS_FOR_ALL_ROWS(RS_ALLOW_ALL)
#undef RS_ALLOW_ALL
#undef RS_ALLOW
    return CSD_OK;
}

// What matters is how many compute units have a workgroup: the column tiles per workgroup (CT) and the K splits (S, at most
// 8: the partial sums are traffic too) are chosen per matrix so that the launch comes as close to one workgroup per
// compute unit as the shape allows, the wider workgroup winning a tie (it reads the activation rows less often).
// 7B shape, 40 rows, against half the tiles and half the splits, which leaves half of the partial sums: QKV 20.5 us against 21.3, O 9.7
// against 12.3, down 19.9 against 27.4.  rows: 33 to 144; the partial-sum buffer holds S x rows x N floats.
// Nine row tiles take the same widths (QKV at 136 rows 34 us in 12 tiles and 4 splits, 36.9 in 6 and 2).
static void rs_plan(int N, int K, int rows, size_t part_floats, int *ct, int *S) {
    const int n_tiles = N / 16, KS = K / 32;
    double best = -1.0;
    for (const int w : {16, 12, 11, 8, 6}) {
        const int groups = (n_tiles + w - 1) / w;
        int s = 1;
        while (groups * (s + 1) <= 256 && s < 8 && KS / (s + 1) >= 8 && (size_t)(s + 1) * rows * N <= part_floats) s++;
        const int wgs = groups * s;
        const double fill = (double)wgs / (256.0 * ((wgs + 255) / 256));
        if (fill > best) best = fill, *ct = w, *S = s;
    }
}

int32_t csd_rs_plan_host(int32_t N, int32_t K, int32_t rows, size_t part_floats, int32_t *ct, int32_t *S) {
    if (!ct || !S) return CSD_ENULL;
    if (N <= 0 || K <= 0 || N % 16 || K % 32 || rows < 1 || rows > 144) return CSD_EINVAL;
    rs_plan(N, K, rows, part_floats, ct, S);
    return CSD_OK;
}

template <int CT, int RW, int NW>
static int32_t rs_launch_t(const TallArgs &A, hipStream_t st) {
    const int grid = (A.n_tiles + CT - 1) / CT * A.S;
    hipLaunchKernelGGL((k_gemm_rs<CT, RW, NW>), dim3(grid), dim3(NW * 64), (rs_lds<CT, NW>()), st, TALL_ARGS(A));
    CSD_LAUNCH_CHECK();
    return CSD_OK;
}

static int32_t rs_launch(const TallArgs &A, int ct, hipStream_t st) {
    const int mt = (A.g.M + 15) / 16;
    if (mt > 9) return CSD_ESHAPE;                               // taller blocks take csd_tall.hip
    const int rw = mt <= 4 ? 1 : mt <= 8 ? 2 : 3, nw = (mt + rw - 1) / rw < 4 ? 3 : 4;
#define RS_LAUNCH(CT, RW, NW) if (ct == CT && rw == RW && nw == NW) return rs_launch_t<CT, RW, NW>(A, st);
#define RS_LAUNCH_ALL(RW, NW) RS_FOR_ALL_CT(RS_LAUNCH, RW, NW)
    RS_FOR_ALL_ROWS(RS_LAUNCH_ALL)
#undef RS_LAUNCH_ALL
#undef RS_LAUNCH
    return CSD_ESHAPE;
}

int32_t csd_rows_part(csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int M, int *S_used, hipStream_t st) {
    TallArgs A = tall_args(mod, w, a, plane, mod->act_mtp, M);
    int ct = 0;
    rs_plan(w.N, w.K, M, mod->part_floats, &ct, &A.S);
    A.part = mod->part;
    *S_used = A.S;
    return rs_launch(A, ct, st);
}
