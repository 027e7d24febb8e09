// What the two GEMMs that bring operands to LDS by direct loads share (csd_rows.hip, csd_tall.hip): the arguments of a launch, the
// loads, and the waits that go with them.
#pragma once

#include "csd_epilogue.h"

enum { EPI_PART = 4, EPI_CROSS = 5 };       // besides the epilogues of csd_epilogue.h

struct TallArgs {
    ChainGemm g;
    int n_tiles, S, rblocks;
    int chain;                // k-steps (even) added up in the accumulators before these go into the sums kept beside them
    float *part;              // EPI_PART: partial sums [S][M][16 n_tiles]
    const float *rstd;        // [M] scale of the folded norm (EPI_QKV, EPI_GU, EPI_LOGITS)
    int enc_len, row0;        // EPI_CROSS: row r of the launch is encoder row (row0 + r) % enc_len of sequence (row0 + r) / enc_len
};

typedef __attribute__((address_space(3))) void *lds_void;

// 16 bytes per lane from a buffer straight to LDS: lane l's go to d + 16 l
template <int AUX>
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, lds_void d, int voff, int soff) {
#ifdef __HIP_DEVICE_COMPILE__                // (the host pass does not know the 16-byte form)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, d, 16, voff, soff, 0, AUX);
#endif
}
// 4 bytes per lane likewise
__device__ __forceinline__ void lds_load4(__amdgpu_buffer_rsrc_t r, lds_void d, int voff, int soff) {
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, d, 4, voff, soff, 0, 0);
#endif
}
// At most V vector memory operations still outstanding, and no LDS read.
template <int V>
__device__ __forceinline__ void wait_loads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((V & 15) | ((V >> 4) << 14) | 0x0070);
}
// The barrier alone: lds_sync()'s fences would wait for every direct load to LDS still in flight.  What makes it safe is the
// wait in front of it: every wave has seen its own loads of the stage that is read next arrive, and has the fragments
// it read from the stage that is overwritten next in registers.
__device__ __forceinline__ void stage_barrier() {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The arguments that the first loads need come ahead of the structure, in registers when a wave starts (see kc_gemm).
#define TALL_PARAMS const u32x4 *Wp, const bf16_t *a, int KS, int n_tiles, int S, int wbytes, int a_plane_bytes, int mtp, int M, int rblocks, const TallArgs args
#define TALL_ARGS(A) (A).g.Wp, (A).g.a, (A).g.KS, (A).n_tiles, (A).S, (A).g.wbytes, (A).g.a_plane_bytes, (A).g.mtp, (A).g.M, (A).rblocks, A
#define TALL_UNPACK(A)                     \
    TallArgs A = args;                     \
    A.g.Wp = Wp;                           \
    A.g.a = a;                             \
    A.g.KS = KS;                           \
    A.n_tiles = n_tiles;                   \
    A.S = S;                               \
    A.g.wbytes = wbytes;                   \
    A.g.a_plane_bytes = a_plane_bytes;     \
    A.g.mtp = mtp;                         \
    A.g.M = M;                             \
    A.rblocks = rblocks;

static inline TallArgs tall_args(const csd_model *mod, const GemmW &w, const bf16_t *a, size_t plane, int mtp, int M) {
    TallArgs A{};
    A.g.Wp = (const u32x4 *)w.data;
    A.g.KS = w.K / 32;
    A.g.wbytes = (int)((size_t)w.K * w.N * 2);
    A.g.a = a;
    A.g.a_plane_bytes = (int)(plane * 2);
    A.g.mtp = mtp;
    A.g.M = M;
    A.g.hd = mod->hd;
    A.g.dh = mod->cfg.head_dim;
    A.n_tiles = w.N / 16;
    A.rstd = mod->rstd;
    return A;
}
