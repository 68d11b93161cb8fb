// Matrix-core sweep of networks of 32 or 64 columns: the message passing of
// Section 2.2 step 2,
//   a_v = sum_{u in xi(v)} m_u,   s_v <- s_v + g(a_v),   m_v = f(s_v),
// for one or two layers per network.  The layer step is that of the sweep of 128 columns (kernels_mfma.hip): activations
// split exactly into three bf16 parts as three rows of A, weights (split likewise where they are fp32) as B operands in
// registers, a wave owns sixteen output columns from end to end, A rows cross waves through LDS, a barrier per layer; so
// are the chunk plan, the table of the last kRing chunks' messages, the sign bit that carries reachability, the spare
// rows, and the meaning of FF, WX, BW and TR.  A wave has one column tile here and registers to spare, and in the kernel
// that served all widths the sum of the next chunk's sources and the issue of its loads took longer than the matrix
// instructions.  Hence:
//   * No register that a load is still filling is ever copied: four sets of records and two of everything else keep
//     their places in a loop over four chunks, and all is requested two chunks ahead of its use, records four.
//   * A row with a list of sources (the attention of a translation model: 41 of them, 7400 cycles) forms the byte offsets of
//     sixteen entries at a time, an entry to a lane, so that an entry takes a shuffle, a load and an addition; the
//     entries are requested a chunk ahead, and so are the first eight messages.
//   * Raw features are read here, no kernel packs them first; ids are local to the graph, and an address is one register.
//   * The sum of a chunk with one row tile and one near source per row, the usual one, is code without a taken branch.
// Forward pass, 64 NMT-like graphs 665 -> 567 us, 128 Inception-like ones 318 -> 290 us; 512 of those 741 -> 690 us.
// What is left of a chunk is its four dependent layers (LDS, six matrix instructions, epilogue, barrier: 450 cycles each).
// Waves issue in 0.40 of their cycles, 0.20 are waits for memory or LDS, the matrix cores are busy in 0.08 of the chip's
// (SQ counters, 64 NMT-like graphs on a quarter of it).
#include "sweep_tiles.h"

namespace pl {

namespace {

// Waves per SIMD that a variant leaves room for: a chain is all latency, so a batch that fits on the chip at once takes the time of
// one chain and one that does not takes two.  Left alone, the compiler gives the variants with one bf16 part per weight, the
// later sweeps and the reverse pass a few registers more than that many waves can have (130 to 180 instead of 128 or
// 168), and batches just past the smaller limit paid for it (4-module Inception-like graphs, without / with the bound: gradient of
// 320 graphs, H = 64, bf16, 723 -> 645 us; 513 graphs, H = 32, fp32, 706 -> 643 us; forward, two sweeps, 512 graphs, H = 64, bf16, one
// layer, 328 -> 287 us).  On batches that fit either way it costs 2 % at most (256 -> 251 us
// without it: forward, two sweeps, 768 graphs, H = 32, bf16).  No variant spills.
constexpr int tile_residency(int H, int WS, int L, bool FF, bool BW)
{
    if (WS == 1) return L == 1 ? (FF ? 3 : 4) : (H == 32 && !FF && !BW ? 4 : 3);
    return FF || (H == 64 && L == 2) ? 2 : 3;
}

template <int H, int WS, int L, bool FF, bool WX, bool BW, bool TR>
__global__ __launch_bounds__(64 * tile_waves(H), tile_residency(H, WS, L, FF, BW)) void k_sweep_tiles(SweepParams P)
{
#include "sweep_tiles_body.h"
}

}  // namespace

#define PL_TILE_SHAPES(CASE) CASE(64, 3, 2) CASE(64, 1, 2) CASE(64, 3, 1) CASE(64, 1, 1) CASE(32, 3, 2) CASE(32, 1, 2) CASE(32, 3, 1) CASE(32, 1, 1)

void launch_sweep_tiles(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                       const ForwardArgs &fa, const uint4 *wfrag, const float *bias, int WS,
                       bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride, uint8_t *gates,
                       hipStream_t s)
{
    if (gv.B == 0) return;
    const bool tr = keep && gates && first_sweep && !more_sweeps;
    SweepParams P{gv, wfrag, bias, ws.emb, ws.xb, ws.msg, ws.reach, fa.cur_node,
                  fa.node_feats, fa.placement, first_sweep ? mv.blob + mv.proj.w : nullptr, mv.D, tr ? gates : nullptr,
                  tr ? keep : nullptr, tr ? keep_stride : 0};
    const dim3 grid(2 * gv.B);
#define PL_CASE(HH, WW, LL)                                                      \
    if (mv.H == HH && WS == WW && mv.L == LL) {                                  \
        const dim3 block(64 * tile_waves(HH));                                  \
        if (tr)                                                                  \
            hipLaunchKernelGGL((k_sweep_tiles<HH, WW, LL, true, false, false, true>), grid, block, 0, s, P); \
        else if (first_sweep && more_sweeps)                                     \
            hipLaunchKernelGGL((k_sweep_tiles<HH, WW, LL, true, true, false, false>), grid, block, 0, s, P);   \
        else if (first_sweep)                                                    \
            hipLaunchKernelGGL((k_sweep_tiles<HH, WW, LL, true, false, false, false>), grid, block, 0, s, P);  \
        else if (more_sweeps)                                                    \
            hipLaunchKernelGGL((k_sweep_tiles<HH, WW, LL, false, true, false, false>), grid, block, 0, s, P);  \
        else                                                                     \
            hipLaunchKernelGGL((k_sweep_tiles<HH, WW, LL, false, false, false, false>), grid, block, 0, s, P); \
        return;                                                                  \
    }
    PL_TILE_SHAPES(PL_CASE)
#undef PL_CASE
}

// The reverse pass of one sweep in both directions; arrays as at launch_sweep_mfma_bw.
void launch_sweep_tiles_bw(const GraphView &gv, const ModelView &mv, const uint4 *wfrag, const float *bias,
                          int WS, const int32_t *cur_node, float *demb, float *dagg, uint8_t *mask4,
                          float *delta, size_t delta_stride, hipStream_t s)
{
    if (gv.B == 0) return;
    SweepParams P{gv, wfrag, bias, demb, nullptr, dagg, nullptr, cur_node, nullptr, nullptr, nullptr, mv.D,
                  mask4, delta, delta_stride};
    const dim3 grid(2 * gv.B);
#define PL_CASE(HH, WW, LL)                                                                  \
    if (mv.H == HH && WS == WW && mv.L == LL) {                                              \
        hipLaunchKernelGGL((k_sweep_tiles<HH, WW, LL, false, false, true, false>), grid,     \
                           dim3(64 * tile_waves(HH)), 0, s, P);                             \
        return;                                                                              \
    }
    PL_TILE_SHAPES(PL_CASE)
#undef PL_CASE
}

}  // namespace pl
