// Weights of the launches to come, brought into the L2s ahead of them.
//
// A line that is in a die's L2 when a kernel ends is still there in the next one (32 MB read again by the next launch 2.9 us, fresh
// 7.2), and workgroup i of every launch on a queue runs on the same die as workgroup i + 8 n of any other.  The attention of a few
// rows is a chain of latencies that leaves compute units and the memory idle: workgroups added to its launch read, each for its
// own die, the weights that the next GEMMs will read there.  Only reads of memory that no kernel of a call writes: nothing depends on
// whether, when or in which L2 a line arrives.
//
// Per step: 160M shape 396 -> 375 us, T5 shape 2649 -> 2551 (7B shape, O 8 -> 6.4 us, but the attention 0.9 to 1.4 longer, whose own loads wait
// behind these).  Elsewhere it gained nothing: the last waves of a GEMM reading for the next one (the stream never idles: 7B shape 3169
// -> 3254), K/V rows ahead of the attention (3169 -> 3188), the epilogue kernels in front of the GEMM over 33 to 144 rows (40 rows
// 5330 -> 5439 to 5512).
#pragma once

#include "csd_tall.h"

#define L2_WARM_MATS 3
struct L2Warm {
    struct Mat {
        const void *w;        // pre-tiled weights [tiles][KS][1 KB]
        int wbytes, KS;
        int units, ut;        // units of ut tiles, an eighth of them to every die, as gemm_share (csd_chain.hip) deals them over a multiple of 8 workgroups
        int keep;             // k-steps wanted of each wave's eighth of K, from its first on; 0: no matrix
    } mat[L2_WARM_MATS];
    int groups;               // workgroups of the launch that read ahead; a multiple of 8, or 0
};
struct NoWarm {};             // the argument of the form without them (the larger one costs a launch 0.5 us by itself)

// Workgroup e of them, number lin in the launch: one dword of every 128-byte line of the die's share, to LDS, where nobody looks (a
// load to a register would have to be waited for, matrix by matrix: 160M shape 410 us against 398).  A wave takes 8 KB, or what is
// wanted of one (tile, eighth of K), per load.
__device__ __forceinline__ void l2_warm(const L2Warm &Wm, int e, int lin, void *lds) {
    const int die = lin & 7, per = Wm.groups >> 3, k = e >> 3, lane = threadIdx.x & 63;
    if (k >= per) return;
    const int wpg = blockDim.x >> 6, nw = per * wpg;
    const int wv = k * wpg + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int i = 0; i < L2_WARM_MATS; i++) {
        const L2Warm::Mat &m = Wm.mat[i];
        if (m.keep <= 0) continue;
        const int lo = (m.units * die >> 3) * m.ut, hi = (m.units * (die + 1) >> 3) * m.ut;
        const __amdgpu_buffer_rsrc_t r = ch_rsrc(m.w, (size_t)m.wbytes);
        const bool all = m.keep * 8 >= m.KS;
        const int kb = all ? 8 : m.keep, end = hi * m.KS * 1024, segs = all ? ((hi - lo) * m.KS + 7) / 8 : (hi - lo) * 8;
        for (int first = 0; first < kb * 8; first += 64) {
            const int line = first + lane;
            for (int s = wv; s < segs; s += nw) {
                const int off = all ? lo * m.KS * 1024 + s * 8192 : ((lo + (s >> 3)) * m.KS + ((m.KS * (s & 7)) >> 3)) * 1024;
                lds_load4(r, (lds_void)lds, line < kb * 8 && off + line * 128 < end ? line * 128 : CH_OOB, off);
            }
        }
    }
    wait_loads<0>();                                         // nothing may land in this LDS after the workgroup has ended
}
