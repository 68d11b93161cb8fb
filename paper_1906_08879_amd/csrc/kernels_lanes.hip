// Sweep kernel of narrow networks for gfx950: the message passing of Section 2.2 step 2,
//   a_v = sum_{u in xi(v)} m_u,   s_v <- s_v + g(a_v),   m_v = f(s_v),
// where the layers of one direction fit in a wave's registers (2 L H <= 128 weights per lane: H = 8, 16, 32
// with one or two layers, H = 64 with one).
//
// What bounds a sweep is the chain of its layers, a thousand of them one after another on a deep graph.
// On matrix cores a layer of 32 or 64 columns is a few instructions between a split into bf16 parts, an
// exchange through LDS and a barrier: 400 ns a layer at H = 32.  Here a layer never leaves the registers:
//   * One lane per (row of the chunk, column), 64 / H rows to a wave; a lane keeps its column of every
//     weight matrix.
//   * The inputs of a layer are the outputs of the lanes of the same row.  v_fmac_f32 takes its first operand
//     through DPP from lane k of its row of sixteen (row_newbcast), so a layer is H multiply-adds in fp32 and
//     nothing else; the sixteen lanes of the other halves of a wider row come over by v_permlane16_swap /
//     v_permlane32_swap.  97 ns a layer at H = 32, 196 at H = 64, 53 at H = 8 (a wave per SIMD, micro-benchmark).
//     That is 0.4 of a chunk's 1 us (H = 32, L = 2): about 170 of the 280 instructions of a wave with rows are the
//     layers'.  Waves issue in 0.45 of their cycles and wait for memory or LDS in 0.09; the rest is barriers and
//     instructions that need the result before them (SQ counters).
//   * Two LDS barriers per chunk: one between the messages that a chunk leaves in the table and the sums of the
//     next chunk, one that keeps a wave from overwriting a table row which another wave still sums.
// The chunk plan (plan.cpp), the table of the last kRing chunks' messages, far messages, the reachability flag
// in a message's sign bit and the rows that take the stores of unused chunk rows are those of kernels_mfma.hip; but
// a wave owns rows here, not columns, so the far message that it reads is another wave's (message_barrier).
// Everything a chunk needs from HBM is requested two chunks ahead, records four.
//
// Forward sweep of 64 layered graphs of 200 nodes (H = 32, L = 2, 40 chunks): 66.9 us on matrix cores, 40 here;
// one random graph of 32 nodes (H = 8): 35.6 us by the generic kernel, 9.5 here (kernel traces).
#include <type_traits>

#include "internal.h"

namespace pl {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int CH = kChunkRows, RING = kRing;

constexpr int lane_waves(int H) { return CH * H / 64; }   // 64 / H rows of a chunk to a wave

// Workgroup barrier that orders LDS traffic only: global loads and stores stay outstanding.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Workgroup barrier behind which every wave can read what was stored before it, from LDS and from memory: a row's
// far message is read by another wave than the one that stored it.  (A workgroup's waves share an L1 that keeps their
// accesses in order, so this is the same code as lds_barrier.  Threadgroup-split mode, where they would not, is
// closed to a kernel that allocates LDS.)
__device__ __forceinline__ void message_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Sums of w[k] * (x of lane k of this lane's row of sixteen), k = 0 .. 15.  The compiler does not fold a DPP move into
// a multiply-add, so this is assembly.  A DPP read needs two wait states after the vector unit has written the
// register, and the compiler does not look for that inside assembly: all sums of a layer are one statement that begins
// with the wait states, so that whatever writes an input comes before them.  A plain vector instruction must read
// the results (an addition, in dense).
#define PL_MAC16(A, X, W0, W1, W2, W3, W4, W5, W6, W7, W8, W9, WA, WB, WC, WD, WE, WF) \
    "v_mul_f32_dpp %" #A ", %" #X ", %" #W0 " row_newbcast:0 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W1 " row_newbcast:1 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W2 " row_newbcast:2 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W3 " row_newbcast:3 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W4 " row_newbcast:4 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W5 " row_newbcast:5 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W6 " row_newbcast:6 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W7 " row_newbcast:7 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W8 " row_newbcast:8 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W9 " row_newbcast:9 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #WA " row_newbcast:10 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #WB " row_newbcast:11 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #WC " row_newbcast:12 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #WD " row_newbcast:13 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #WE " row_newbcast:14 row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #WF " row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
#define PL_W4(w) "v"((w)[0]), "v"((w)[1]), "v"((w)[2]), "v"((w)[3])
#define PL_W16(w) PL_W4(w), PL_W4((w) + 4), PL_W4((w) + 8), PL_W4((w) + 12)
__device__ __forceinline__ float mac16(float x, const float *w)
{
    float s;
    asm volatile("s_nop 1\n" PL_MAC16(0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17)
                 : "=&v"(s) : "v"(x), PL_W16(w));
    return s;
}
__device__ __forceinline__ void mac32(float x0, float x1, const float *w, float &s0, float &s1)
{
    asm volatile("s_nop 1\n" PL_MAC16(0, 2, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19)
                 PL_MAC16(1, 3, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33, 34, 35)
                 : "=&v"(s0), "=&v"(s1) : "v"(x0), "v"(x1), PL_W16(w), PL_W16(w + 16));
}
__device__ __forceinline__ void mac64(float x0, float x1, float x2, float x3, const float *w, float &s0, float &s1, float &s2,
                                      float &s3)
{
    asm volatile("s_nop 1\n" PL_MAC16(0, 4, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19, 20, 21, 22, 23)
                 PL_MAC16(1, 5, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33, 34, 35, 36, 37, 38, 39)
                 PL_MAC16(2, 6, 40, 41, 42, 43, 44, 45, 46, 47, 48, 49, 50, 51, 52, 53, 54, 55)
                 PL_MAC16(3, 7, 56, 57, 58, 59, 60, 61, 62, 63, 64, 65, 66, 67, 68, 69, 70, 71)
                 : "=&v"(s0), "=&v"(s1), "=&v"(s2), "=&v"(s3)
                 : "v"(x0), "v"(x1), "v"(x2), "v"(x3), PL_W16(w), PL_W16(w + 16), PL_W16(w + 32), PL_W16(w + 48));
}
#undef PL_MAC16

// The same over the lanes of this lane's group of four: s0 of x0, s1 of x1.
#define PL_MAC4(A, X, W0, W1, W2, W3) \
    "v_mul_f32_dpp %" #A ", %" #X ", %" #W0 " quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W1 " quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W2 " quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #A ", %" #X ", %" #W3 " quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n"
__device__ __forceinline__ void mac8(float x0, float x1, const float *w, float &s0, float &s1)
{
    asm volatile("s_nop 1\n" PL_MAC4(0, 2, 4, 5, 6, 7) PL_MAC4(1, 3, 8, 9, 10, 11)
                 : "=&v"(s0), "=&v"(s1) : "v"(x0), "v"(x1), PL_W4(w), PL_W4(w + 4));
}
#undef PL_MAC4
#undef PL_W16
#undef PL_W4

// rows of sixteen lanes (A, B, C, D) -> lo = (A, A, C, C), hi = (B, B, D, D)
__device__ __forceinline__ void swap16(float x, float &lo, float &hi)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    lo = __uint_as_float(r[0]);
    hi = __uint_as_float(r[1]);
}

// halves of the wave (P, Q) -> lo = (P, P), hi = (Q, Q)
__device__ __forceinline__ void swap32(float x, float &lo, float &hi)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    lo = __uint_as_float(r[0]);
    hi = __uint_as_float(r[1]);
}

// Which input of a layer the k-th weight of a lane belongs to (see dense): H = 8 takes its own four lanes first
// and then the other four in mirrored order.
template <int H>
__device__ __forceinline__ int input_of(int k, int col)
{
    if constexpr (H == 8) return k < 4 ? (col & 4) + k : 7 - (col & 4) - (k - 4);
    return k;
}

// One dense layer over the lanes of a row: sum_k w[k] x_{input_of(k)} + b.  Sixteen terms to a running sum: the
// partial sums are added at the end.
template <int H>
__device__ __forceinline__ float dense(float x, const float (&w)[H], float b)
{
    if constexpr (H == 8) {
        const float y = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, true));   // row_half_mirror
        float s0, s1;
        mac8(x, y, w, s0, s1);
        return (s0 + s1) + b;
    } else if constexpr (H == 16) {
        return mac16(x, w) + b;
    } else if constexpr (H == 32) {
        float lo, hi, s0, s1;
        swap16(x, lo, hi);
        mac32(lo, hi, w, s0, s1);
        return (s0 + s1) + b;
    } else {
        static_assert(H == 64, "a row has 8, 16, 32 or 64 lanes");
        float p, q, r0, r1, r2, r3;
        swap16(x, p, q);
        swap32(p, r0, r2);
        swap32(q, r1, r3);
        float s0, s1, s2, s3;
        mac64(r0, r1, r2, r3, w, s0, s1, s2, s3);
        return ((s0 + s1) + (s2 + s3)) + b;
    }
}

// Element at a 32-bit byte offset from a base that is the same for all lanes (one register of address per lane).
template <typename T>
__device__ __forceinline__ T &elem(T *base, uint32_t byte)
{
    using Byte = std::conditional_t<std::is_const_v<T>, const char, char>;
    return *reinterpret_cast<T *>(reinterpret_cast<Byte *>(base) + byte);
}

struct LaneParams {
    GraphView gv;
    const float *blob;      // weights; the transposed copy for a reverse pass
    int32_t w[2][4], b[2][4];   // [dir][layer of a chunk]: offsets of its matrix and bias
    float *emb;             // [n_tot, 2H]
    float *xb;              // [2, n_tot, H] residual input in bucket order (sweeps after the first)
    float *msg;             // [2, n_tot, H]
    uint8_t *reach;         // [2, n_tot]
    const int32_t *cur_node;
    const float *feats;     // [n_tot, 3] raw features, placement [n_tot] (first sweep)
    const int32_t *placement;
    const float *proj;      // [F + 1, H]: rows of W_in, then b_in
    int D;
    uint8_t *mask4;         // ReLU gates, as in kernels_mfma.hip
    float *delta;           // kept activations (TR) or deltas (BW) per sweep direction
    size_t delta_stride;
};

// FF, WX, BW, TR as at k_sweep_mfma: first sweep (input from the raw features), another sweep follows, reverse
// pass, activations kept.
template <int H, int L, bool FF, bool WX, bool BW, bool TR>
__global__ __launch_bounds__(64 * lane_waves(H), 2) void k_sweep_lanes(LaneParams P)
{
    static_assert(!BW || (!FF && !WX), "the reverse pass reads its input from emb and writes no xb");
    static_assert(!TR || (FF && !WX && !BW), "activations are kept for a single forward sweep");
    constexpr int NL = 2 * L;                  // layers per chunk: g then f
    constexpr int kThreads = 64 * lane_waves(H);
    constexpr int RPW = 64 / H;                // rows of a wave
    constexpr int kZeroSlot = kMsgSlots;
    constexpr int kPre = 8;                    // messages of a list that are requested ahead of its sum
    __shared__ float msgtab[(kMsgSlots + 1) * H];   // messages of the last kRing chunks, then a row of zeros
    __shared__ float proj_dev[(kMaxD + 1) * H];     // one-hot device rows of W_in, then a row of zeros

    const int b = blockIdx.x >> 1, dir = blockIdx.x & 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane % H;                                // this lane's column
    int r = wave * RPW + lane / H;                           // its row of the chunk
    // (At H = 64 a record is the same for all lanes of a wave.  The compiler must not know: it would move every record
    // into scalar registers as soon as it is requested, and wait for it there.)
    asm("" : "+v"(r));

    const GraphView &gv = P.gv;
    const SweepPlanView plan = gv.plan[dir];
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    // arrays from the graph's first node on: node ids below are local to the graph
    const size_t first_row = static_cast<size_t>(dir) * gv.n_tot + n0;
    float *msg = P.msg + first_row * H;
    float *xb = P.xb + first_row * H;
    uint8_t *reach = P.reach + first_row;
    float *emb = P.emb + static_cast<size_t>(n0) * 2 * H + (BW ? 1 - dir : dir) * H;
    const float *feats = P.feats + static_cast<size_t>(n0) * 3;
    const int32_t *placement = P.placement + n0;
    const uint32_t cur = static_cast<uint32_t>(P.cur_node[b]);   // (outside the graph: none of its nodes)
    const int tm = gv.tmpl[b];
    const int c_begin = plan.ck_off[tm], c_end = plan.ck_off[tm + 1];
    if (c_begin >= c_end) return;
    // rows past both directions' messages: one that reads as zero, one that takes stores of unused rows
    const uint32_t spare_row = static_cast<uint32_t>((2 - dir) * gv.n_tot - n0), sink_row = spare_row + 1u;
    const uint32_t emb_sink = static_cast<uint32_t>(gv.n_tot - n0);

    // ---- records: requested four chunks before they are processed
    auto load_rec = [&](int c) __attribute__((always_inline)) {
        return elem(reinterpret_cast<const u32x4 *>(plan.rec + static_cast<size_t>(c < c_end ? c : c_end - 1) * CH), 16u * static_cast<uint32_t>(r));
    };
    u32x4 rec0 = load_rec(c_begin), rec1 = load_rec(c_begin + 1), rec2 = load_rec(c_begin + 2), rec3 = load_rec(c_begin + 3);

    // ---- this lane's column of the weights of this direction
    float W[NL][H], bias[NL];
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        const float *w = P.blob + P.w[dir][n];
#pragma unroll
        for (int k = 0; k < H; ++k) W[n][k] = w[static_cast<uint32_t>(input_of<H>(k, col) * H + col)];
        bias[n] = BW ? 0.0f : P.blob[P.b[dir][n] + col];
    }
    const int D = P.D;
    float pw_time = 0.0f, pw_size = 0.0f, pw_cur = 0.0f, pw_vis = 0.0f, pw_b = 0.0f;
    if constexpr (FF) {
        pw_time = P.proj[col];
        pw_size = P.proj[H + col];
        pw_cur = P.proj[(2 + D) * H + col];
        pw_vis = P.proj[(3 + D) * H + col];
        pw_b = P.proj[(4 + D) * H + col];
        for (int i = tid; i < (kMaxD + 1) * H; i += kThreads) proj_dev[i] = i < D * H ? P.proj[2 * H + i] : 0.0f;
    }
    for (int i = tid; i < (kMsgSlots + 1) * H; i += kThreads) msgtab[i] = 0.0f;

    float *dlt = BW ? P.delta + static_cast<size_t>(1 - dir) * P.delta_stride
                    : (TR ? P.delta + static_cast<size_t>(dir) * P.delta_stride : nullptr);
    const uint8_t *gates_in = BW ? P.mask4 + (static_cast<size_t>(1 - dir) * gv.n_tot + n0) * H : nullptr;
    uint8_t *gates_out = TR ? P.mask4 + first_row * H : nullptr;

    auto node_of = [&](const u32x4 &rec) __attribute__((always_inline)) {   // (some node for unused rows)
        const uint32_t id = rec[3] & kRecNoNode, last = static_cast<uint32_t>(n_b - 1);
        return id < last ? id : last;
    };
    auto rows_of = [](uint32_t info) __attribute__((always_inline)) { return static_cast<int>((info >> kRecRowsShift) & 7u) + 1; };
    auto first = [](uint32_t x) __attribute__((always_inline)) {
        return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
    };
    // element (row, column of this lane) of an array of rows of H, and its byte offset among floats
    auto at = [&](uint32_t row) __attribute__((always_inline)) { return row * H + static_cast<uint32_t>(col); };
    auto at4 = [&](uint32_t row) __attribute__((always_inline)) { return 4u * at(row); };

    // What a chunk reads of a node besides its messages: raw features (FF), the outside gradient of its state and
    // its gates (BW), or the input of a later sweep.
    struct Inputs {
        float time, size, vis, x;
        int dev, gates;
    };
    auto load_inputs = [&](const u32x4 &rec, int rows, int p, Inputs &in) __attribute__((always_inline)) {
        if constexpr (FF) {
            const uint32_t v = node_of(rec);
            const float *f = &elem(feats, v * 12u);
            in.time = f[0];
            in.size = f[1];
            in.vis = f[2];
            in.dev = elem(placement, v * 4u);
        } else if constexpr (BW) {
            const uint32_t v = node_of(rec);
            in.x = elem(emb, 8u * H * v + 4u * col);
            in.gates = elem(gates_in, at(v));
        } else {
            in.x = elem(xb, at4(static_cast<uint32_t>(p + (r < rows ? r : 0))));
        }
    };
    // x_v = relu(W_in^T phi_v + b) (Section 2.2 step 1)
    auto project = [&](const Inputs &in, uint32_t v) __attribute__((always_inline)) {
        float o = fmaf(in.time, pw_time, pw_b);
        o = fmaf(in.size, pw_size, o);
        const uint32_t dev = static_cast<uint32_t>(in.dev), none = static_cast<uint32_t>(D);
        o += proj_dev[(dev < none ? dev : none) * H + col];
        o += v == cur ? pw_cur : 0.0f;
        return fmaxf(fmaf(in.vis, pw_vis, o), 0.0f);
    };
    // the row's far message (a row of zeros if it has none)
    auto load_far = [&](const u32x4 &rec) __attribute__((always_inline)) {
        static_assert(kRecListed == 1u << 30 && kNoFar == 0xFFFFFFFFu, "a listed row's second word becomes kNoFar");
        const uint32_t u = rec[1] | static_cast<uint32_t>(static_cast<int32_t>(rec[0] << 1) >> 31);
        return elem(msg, at4(u < spare_row ? u : spare_row));
    };

    // ---- gather of a chunk: a_v = sum of neighbour messages.  `signs` collects the sign bits.
    auto add = [&](float &s, uint32_t &signs, float x) __attribute__((always_inline)) {
        s += BW ? x : fabsf(x);
        if (!BW) signs |= __float_as_uint(x);
    };
    auto sum_slots = [&](auto kc, uint32_t slots, float &s, uint32_t &signs) __attribute__((always_inline)) {
        constexpr int K = decltype(kc)::value;
        float x[K];
#pragma unroll
        for (int k = 0; k < K; ++k) x[k] = msgtab[((slots >> (6 * k)) & 63u) * H + col];
#pragma unroll
        for (int k = 0; k < K; ++k) add(s, signs, x[k]);
    };
    // A row with more sources than its record holds: a list of table slots and node ids.  The lanes of the row load an
    // entry each (an entry past the end names the rows of zeros) and form its rows' byte offsets, once for H entries;
    // then an entry takes a shuffle, a load and an addition, and only lists that have near sources read the table.  Of
    // the first H entries the lanes hold the ids a chunk before the sum, and the messages of the first kPre are on
    // their way.
    auto entry = [&](const u32x4 &rec, int i) __attribute__((always_inline)) {
        const bool in = (rec[0] & kRecListed) && i < static_cast<int>(rec[0] & 0xFFFFFFu);
        return in ? elem(plan.ovf, 4u * (rec[1] + static_cast<uint32_t>(i))) : -1 - kZeroSlot;
    };
    auto from_lane = [&](uint32_t x, int k) __attribute__((always_inline)) {   // lane k of this row's
        if constexpr (H == 64) return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), k));
        return static_cast<uint32_t>(__shfl(static_cast<int>(x), (lane & ~(H - 1)) + k));
    };
    auto far_row = [&](int u) __attribute__((always_inline)) { return 4u * H * (u >= 0 ? static_cast<uint32_t>(u) : spare_row); };
    auto request = [&](uint32_t rows, int first_lane, auto &y) __attribute__((always_inline)) {
        constexpr int K = sizeof(y) / sizeof(y[0]);
#pragma unroll
        for (int k = 0; k < K; ++k) y[k] = elem(msg, from_lane(rows, first_lane + k) + 4u * static_cast<uint32_t>(col));
    };
    auto sum_list = [&](const u32x4 &rec, int ids, const float (&pre)[kPre], float &s, uint32_t &signs) __attribute__((always_inline)) {
        constexpr int PB = H < 16 ? H : 16;
        const int cnt = static_cast<int>(rec[0] & 0xFFFFFFu);
        auto take = [&](const auto &y) __attribute__((always_inline)) {
            constexpr int K = sizeof(y) / sizeof(y[0]);
#pragma unroll
            for (int k = 0; k < K; ++k) add(s, signs, y[k]);
        };
        auto take_near = [&]() __attribute__((always_inline)) {       // among the H entries: the few places that are near in some row
            unsigned long long near = __ballot(ids < 0 && ids != -1 - kZeroSlot);
            const uint32_t rows = H * static_cast<uint32_t>(ids < 0 ? -1 - ids : kZeroSlot);
#pragma unroll
            for (int w = 32; w >= H; w /= 2) near |= near >> w;
            if constexpr (H < 64) near &= (1ull << H) - 1ull;
#pragma unroll 1
            for (; near != 0ull; near &= near - 1ull) {
                const float x[1] = {msgtab[from_lane(rows, __builtin_ctzll(near)) + col]};
                take(x);
            }
        };
        static_assert(kPre == 8, "the first pass asks for the second half of its entries only");
        uint32_t rows = far_row(ids);
        if (PB > kPre && cnt > kPre) {
            float y[kPre];
            request(rows, PB > kPre ? kPre : 0, y);
            take(pre);
            take_near();
            take(y);
        } else {
            take(pre);
            take_near();
        }
#pragma unroll 1
        for (int p = PB; p < cnt; p += PB) {
            if (p % H == 0) {
                ids = entry(rec, p + col);
                rows = far_row(ids);
            }
            float y[PB];
            request(rows, p % H, y);
            if (p % H == 0) take_near();
            take(y);
        }
        // (nothing of this path is in flight where it joins the others: they would wait for it)
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    };
    // info = word 3 of a record of the chunk (its chunk-wide bits)
    auto gather = [&](uint32_t info, const u32x4 &rec, float far, int ids, const float (&pre)[kPre], int gates, bool valid,
                      uint32_t &signs) __attribute__((always_inline)) {
        float s = BW ? far : fabsf(far);
        signs = BW ? 0u : __float_as_uint(far);
        const int cls = static_cast<int>((info >> kRecNearShift) & 3u);
        if ((info >> kRecGeneralBit) & 1u) {
            if (rec[0] & kRecListed)
                sum_list(rec, ids, pre, s, signs);
            else
                sum_slots(std::integral_constant<int, kMaxNear>{}, rec[0], s, signs);
        } else if (cls == 0) {
            sum_slots(std::integral_constant<int, 1>{}, rec[0], s, signs);
        } else if (cls == 1) {
            sum_slots(std::integral_constant<int, 2>{}, rec[0], s, signs);
        } else {
            sum_slots(std::integral_constant<int, kMaxNear>{}, rec[0], s, signs);
        }
        if constexpr (BW) s = (gates & 1) ? s : 0.0f;
        if constexpr (TR) {
            const uint32_t id = rec[3] & kRecNoNode;
            dlt[id == kRecNoNode || !valid ? static_cast<uint32_t>(2 * L * gv.n_tot * H + col) : at(static_cast<uint32_t>(n0) + id)] = s;
        }
        return s;
    };

    // ---- state of the pipeline.  A register that a load is still filling is never copied: the chunk loop is unrolled
    // by four, and every set of registers keeps its place.
    //   rec0 .. rec3  record of chunk c, c + 1, ..; that of chunk c is the target of chunk c + 4's
    //   in0 / in1     inputs of chunk c / c + 1, then targets of c + 2 / c + 3
    //   far0 / far1   far message of chunk c + 1 / target for chunk c + 2
    Inputs in0{}, in1{};
    float far0 = 0.0f, far1 = 0.0f, a;           // (the first kRing + 1 chunks have no far sources)
    int ids0 = -1 - kZeroSlot, ids1 = ids0;      // entries of chunk c + 1's lists / target for chunk c + 2's
    float pre[kPre] = {};                        // first messages of chunk c + 1's lists
    int rows0, p0;
    uint32_t vg, sign;                           // node; its sources' sign bits (chunk c)
    {
        const uint32_t info0 = first(rec0[3]), info1 = first(rec1[3]);
        rows0 = rows_of(info0);
        p0 = static_cast<int>(first(rec0[2]));
        vg = node_of(rec0);
        load_inputs(rec0, rows0, p0, in0);
        load_inputs(rec1, rows_of(info1), static_cast<int>(first(rec1[2])), in1);
        __syncthreads();
        // (the first chunk has no sources)
        a = gather(info0, rec0, 0.0f, ids0, pre, in0.gates, true, sign);
        if ((info1 >> kRecGeneralBit) & 1u) ids0 = entry(rec1, col);
    }
    __syncthreads();

    // rT: target for the record of chunk c + 4; rA, rB: records of chunks c + 1, c + 2; in: inputs of chunk c, then
    // target of chunk c + 2's; farA / farB: far message of chunk c + 1 / target for chunk c + 2; inN: inputs of chunk c + 1;
    // idsA / idsB: list entries of chunk c + 1 / target for chunk c + 2's
    auto step = [&](auto ringc, int c, u32x4 &rT, const u32x4 &rA, const u32x4 &rB, Inputs &in, const Inputs &inN, float &farA,
                    float &farB, int &idsA, int &idsB) __attribute__((always_inline)) {
        constexpr int ring = decltype(ringc)::value;     // (c - c_begin) % kRing: where its messages go in the table
        const int rows = rows0;
        const uint32_t v = vg;
        const bool live = r < rows;
        const uint32_t info1 = first(rA[3]);
        const uint32_t v_emb = live ? v : emb_sink, v_msg = live ? v : sink_row;
        auto delta_at = [&](int slot) __attribute__((always_inline)) {   // (unused rows: the spare row)
            return live ? static_cast<uint32_t>(slot * gv.n_tot * H) + at(static_cast<uint32_t>(n0) + v) : static_cast<uint32_t>(2 * L * gv.n_tot * H + col);
        };
        if ((info1 >> kRecGeneralBit) & 1u) request(far_row(idsA), 0, pre);
        farB = load_far(rB);
        rT = load_rec(c + 4);
        if ((first(rB[3]) >> kRecGeneralBit) & 1u) idsB = entry(rB, col);
        float x = 0.0f;
        if constexpr (FF) x = project(in, v);
        const int gates = in.gates;
        // (once the inputs of this chunk are used up)
        auto next_inputs = [&]() __attribute__((always_inline)) {
            load_inputs(rB, rows_of(first(rB[3])), static_cast<int>(first(rB[2])), in);
        };

        float y = a;
        if constexpr (!BW) {
            const bool busy = wave * RPW < rows;    // (a wave without rows only keeps step)
            float y0 = 0.0f, ys = 0.0f, yf = 0.0f;
            if (busy) {
                y = fmaxf(dense<H>(y, W[0], bias[0]), 0.0f);
                y0 = y;
                if constexpr (L == 2) y = fmaxf(dense<H>(y, W[1], bias[1]), 0.0f);
            }
            if constexpr (TR && L == 2) dlt[delta_at(1)] = y0;
            lds_barrier();                          // every wave has summed this chunk's sources
            ys = y + (FF ? x : in.x);
            next_inputs();
            elem(emb, 8u * H * v_emb + 4u * col) = ys;
            if constexpr (WX) elem(xb, at4(live ? static_cast<uint32_t>(p0 + r) : spare_row)) = ys;
            int gb = 0;
            if constexpr (TR) gb = (L == 2 && y0 > 0.0f ? 8 : 0) | (y > 0.0f ? 4 : 0);
            y = ys;
            if (busy) {
                y = fmaxf(dense<H>(y, W[L], bias[L]), 0.0f);
                yf = y;
                if constexpr (L == 2) y = fmaxf(dense<H>(y, W[L + 1], bias[L + 1]), 0.0f);
            }
            if constexpr (TR) {
                if constexpr (L == 2) dlt[delta_at(1 + L)] = yf;
                gb |= (L == 2 && yf > 0.0f ? 2 : 0) | (y > 0.0f ? 1 : 0);
                elem(gates_out, at(live ? v : spare_row)) = static_cast<uint8_t>(gb);
            }
            // the message, with the reachability flag of its node
            const uint32_t flag = sign | (v == cur ? 0x80000000u : 0u);
            y = __uint_as_float((__float_as_uint(y) & 0x7FFFFFFFu) | (flag & 0x80000000u));
            msgtab[(ring * CH + r) * H + col] = y;
            elem(msg, at4(v_msg)) = y;
            elem(reach, col == 0 ? v_msg : sink_row) = static_cast<uint8_t>(sign >> 31);
        } else {
            // f transposed from its last layer to its first, the outside gradient, g transposed; every gated
            // layer input is that layer's delta
            const bool busy = wave * RPW < rows;
            dlt[delta_at(L - 1)] = y;
            float ds = 0.0f, t = y;
            if (busy) {
                if constexpr (L == 2) {
                    t = dense<H>(t, W[0], 0.0f);
                    t = (gates & 2) ? t : 0.0f;
                }
                ds = t;
                t = dense<H>(t, W[L - 1], 0.0f);
            }
            if constexpr (L == 2) dlt[delta_at(0)] = ds;
            lds_barrier();
            ds = t + in.x;
            next_inputs();
            elem(emb, 8u * H * v_emb + 4u * col) = ds;
            t = (gates & 4) ? ds : 0.0f;
            dlt[delta_at(2 * L - 1)] = t;
            float d0 = 0.0f;
            if (busy) {
                if constexpr (L == 2) {
                    t = dense<H>(t, W[L], 0.0f);
                    t = (gates & 8) ? t : 0.0f;
                }
                d0 = t;
                t = dense<H>(t, W[NL - 1], 0.0f);
            }
            if constexpr (L == 2) dlt[delta_at(L)] = d0;
            msgtab[(ring * CH + r) * H + col] = t;
            elem(msg, at4(v_msg)) = t;
        }
        message_barrier();                          // this chunk's messages are in the table, and in msg
        a = gather(info1, rA, farA, idsA, pre, inN.gates, c + 1 < c_end, sign);
        rows0 = c + 1 < c_end ? rows_of(info1) : 0;
        p0 = static_cast<int>(first(rA[2]));
        vg = node_of(rA);
        // (a word of the record that nothing reads would be given to another value while its load is in flight, and
        // that value would wait for the load)
        asm volatile("" : : "v"(rA[2]));
    };
    // (four chunks per turn without a test between them, which would cost copies of what is still being loaded: chunks
    // past the last have no rows and store to the spare rows only)
    __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0): the loop's waits are counted from its own loads
    static_assert(RING == 4, "a turn takes as many chunks as the table holds");
    for (int c = c_begin; c < c_end; c += 4) {
        step(std::integral_constant<int, 0>{}, c, rec0, rec1, rec2, in0, in1, far0, far1, ids0, ids1);
        step(std::integral_constant<int, 1>{}, c + 1, rec1, rec2, rec3, in1, in0, far1, far0, ids1, ids0);
        step(std::integral_constant<int, 2>{}, c + 2, rec2, rec3, rec0, in0, in1, far0, far1, ids0, ids1);
        step(std::integral_constant<int, 3>{}, c + 3, rec3, rec0, rec1, in1, in0, far1, far0, ids1, ids0);
    }
}

}  // namespace

// Where these kernels are the faster ones.  H = 8, 16: everywhere (the generic kernel: random graphs of 32 nodes, 1 graph
// 35.6 -> 9.5 us, a forward pass of 4096 graphs 497 -> 290 us).  H = 32 and 64 as long as all workgroups of a batch are
// on the chip at once, two of four waves or one of eight to each of 256 compute units (forward pass, against the
// matrix-core sweep, whose workgroups are smaller: Inception-like graphs, H = 32, 256 graphs 294 -> 250 us, 320 graphs
// 310 -> 386; NMT-like graphs, H = 64, one layer, 128 graphs 552 -> 458 us, 160 graphs 607 -> 832), and with fp32
// weights: bf16 weights take a third of the matrix instructions, and their sums round less often than these here (H = 64:
// states 1.1e-7 from float64 against 1.3e-7; with fp32 weights 1.5e-7 against 1.3e-7).  The two kernels take their sums in
// different orders, so at H = 32 and 64 the last bits of a graph's results depend on the size of its batch.
bool sweep_lanes_preferred(int H, int L, int B, int weight_dtype)
{
    if (L < 1 || L > 2) return false;
    if (H == 8 || H == 16) return true;
    return weight_dtype == PL_WEIGHTS_FP32 && ((H == 32 && B <= 256) || (H == 64 && L == 1 && B <= 128));
}

#define PL_LANE_SHAPES(CASE) CASE(8, 1) CASE(8, 2) CASE(16, 1) CASE(16, 2) CASE(32, 1) CASE(32, 2) CASE(64, 1)

void launch_sweep_lanes(const GraphView &gv, const ModelView &mv, const Workspace &ws, const ForwardArgs &fa,
                        bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride, uint8_t *gates, hipStream_t s)
{
    if (gv.B == 0) return;
    const bool tr = keep && gates && first_sweep && !more_sweeps;
    LaneParams P{gv, mv.blob, {}, {}, ws.emb, ws.xb, ws.msg, ws.reach, fa.cur_node, fa.node_feats, fa.placement,
                 mv.blob + mv.proj.w, mv.D, tr ? gates : nullptr, tr ? keep : nullptr, tr ? keep_stride : 0};
    const int L = mv.L;
    for (int dir = 0; dir < 2; ++dir)
        for (int n = 0; n < 2 * L && n < 4; ++n) {
            const LayerRef &ly = n < L ? mv.g[dir].layer[n] : mv.f[dir].layer[n - L];
            P.w[dir][n] = ly.w;
            P.b[dir][n] = ly.b;
        }
    const dim3 grid(2 * gv.B);
#define PL_CASE(HH, LL)                                                                                             \
    if (mv.H == HH && L == LL) {                                                                                    \
        const dim3 block(64 * lane_waves(HH));                                                                      \
        if (tr)                                                                                                     \
            hipLaunchKernelGGL((k_sweep_lanes<HH, LL, true, false, false, true>), grid, block, 0, s, P);            \
        else if (first_sweep && more_sweeps)                                                                        \
            hipLaunchKernelGGL((k_sweep_lanes<HH, LL, true, true, false, false>), grid, block, 0, s, P);            \
        else if (first_sweep)                                                                                       \
            hipLaunchKernelGGL((k_sweep_lanes<HH, LL, true, false, false, false>), grid, block, 0, s, P);           \
        else if (more_sweeps)                                                                                       \
            hipLaunchKernelGGL((k_sweep_lanes<HH, LL, false, true, false, false>), grid, block, 0, s, P);           \
        else                                                                                                        \
            hipLaunchKernelGGL((k_sweep_lanes<HH, LL, false, false, false, false>), grid, block, 0, s, P);          \
        return;                                                                                                     \
    }
    PL_LANE_SHAPES(PL_CASE)
#undef PL_CASE
}

// The reverse pass of one sweep in both directions; arrays as at launch_sweep_mfma_bw.  blob_t: the blob with every
// matrix transposed.
void launch_sweep_lanes_bw(const GraphView &gv, const ModelView &mv, const float *blob_t, const int32_t *cur_node,
                           float *demb, float *dagg, uint8_t *mask4, float *delta, size_t delta_stride, hipStream_t s)
{
    if (gv.B == 0) return;
    LaneParams P{gv, blob_t, {}, {}, demb, nullptr, dagg, nullptr, cur_node, nullptr, nullptr, nullptr, mv.D,
                 mask4, delta, delta_stride};
    const int L = mv.L;
    for (int dir = 0; dir < 2; ++dir)
        for (int n = 0; n < 2 * L && n < 4; ++n)
            P.w[dir][n] = (n < L ? mv.f[1 - dir].layer[L - 1 - n] : mv.g[1 - dir].layer[2 * L - 1 - n]).w;
    const dim3 grid(2 * gv.B);
#define PL_CASE(HH, LL)                                                                                             \
    if (mv.H == HH && L == LL) {                                                                                    \
        hipLaunchKernelGGL((k_sweep_lanes<HH, LL, false, false, true, false>), grid, dim3(64 * lane_waves(HH)), 0, s, P); \
        return;                                                                                                     \
    }
    PL_LANE_SHAPES(PL_CASE)
#undef PL_CASE
}

}  // namespace pl
