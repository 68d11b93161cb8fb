// What the sweep kernels of one column tile to a wave share (kernels_tiles.hip, kernels_wide.hip).
#pragma once
#include <type_traits>

#include "internal.h"

namespace pl {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int CH = kChunkRows, RING = kRing;
constexpr int kTileNodes = 4;                 // nodes per 16-row MFMA tile (hi, mid, lo, zero rows)
constexpr int NT = CH / kTileNodes;           // row tiles per chunk

// Workgroup barrier that orders LDS traffic only: global loads and stores stay outstanding.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ float trunc_bf16(float x)
{
    return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
}

// Element at a 32-bit byte offset from a base that is the same for all lanes (one register of address per lane).
template <typename T>
__device__ __forceinline__ T &elem(T *base, uint32_t byte)
{
    using Byte = std::conditional_t<std::is_const_v<T>, const char, char>;
    return *reinterpret_cast<T *>(reinterpret_cast<Byte *>(base) + byte);
}

struct SweepParams {
    GraphView gv;
    const uint4 *wfrag;     // packed weight fragments, see pack_sweep_weights()
    const float *bias;      // [2 dir][2L layers][H]
    float *emb;             // [n_tot, 2H]   output s_v in node order ([td ; bu])
    float *xb;              // [2, n_tot, H] residual input in bucket order, per direction
    float *msg;             // [2, n_tot, H]
    uint8_t *reach;         // [2, n_tot]
    const int32_t *cur_node;
    // first sweep: the input x_v = relu(W_in^T phi_v + b_in) (Section 2.2 step 1) is computed here
    const float *feats;     // [n_tot, 3] run time, output size, is-visited
    const int32_t *placement;
    const float *proj;      // [(F + 1), H]: rows of W_in, then b_in; NULL when the input comes from xb
    int D;
    // ReLU gates of every node's layers, one byte per (sweep direction, node, column), node order:
    // bit 0 m_v > 0 (gates the gathered sum of the reverse pass), bit 1 output of f's layer 0 > 0
    // (L = 2), bit 2 output of g's last layer > 0, bit 3 output of g's layer 0 > 0 (L = 2).
    // Written by a sweep that keeps activations (TR), read by the reverse pass (BW); row 2 n_tot
    // takes the stores of a chunk's unused rows.
    uint8_t *mask4;         // [2 n_tot + 1, H]
    float *delta;           // per sweep direction: [2L][n_tot, H] (f's layers, then g's), then H
                            // floats that take the stores of a chunk's unused rows
    size_t delta_stride;    // floats between the two directions' blocks
};

constexpr int tile_waves(int H) { return H / 16; }   // wave w owns output columns [16 w, 16 w + 16)

}  // namespace

}  // namespace pl
