// Policy head (Section 2.2 step 3, Appendix A.7), forward and reverse: q[i][d] = h_i(P[i][d]) (also for
// empty groups); z = [e_{v*} ; q]; two-layer policy network with a softmax over devices.
//
// One workgroup per graph does all of it (at H >= 128 and few graphs three, one per node set: see HeadShape).  The
// head is small (2 MB of weights at the NASNet-like shape, 0.3 MB at H = 64) and a chain of dense layers, so its
// time is its launches, the latency of its weight loads and, with many graphs, the rate at which a CU reads weights
// from L2; three launches with a workgroup per (graph, set), per (16 graphs, slice of z) and per graph spent most of
// theirs starting and on sequential loops (the output layer took one thread per device).
//   * A layer of the three h networks is one phase: a unit (set, slice of sixteen inputs) is H / 4
//     threads with four columns and up to eight rows each, so a weight is loaded once, as part of a
//     16-byte load, and an input read from LDS feeds four columns.  The slices' sums meet in LDS.
//   * The first policy layer spreads its blocks of sixteen inputs over groups of H / 4 threads, 64
//     weights per thread in flight; the output layer has a wave per device.
// Sums are taken in float64 by blocks (sixteen fp32 terms, the blocks and the terms past the last whole one
// in float64, the output layer entirely in float64): z holds sums over thousands of nodes, so a logit is a
// difference of terms far larger than itself, and plain fp32 sums would be the largest single source of its
// error.
// Forward head of 256 NASNet-like graphs (H = 128, 8 devices): 81 us as three launches, 37 us now; of one: 52,
// now 18; of 64 graphs at H = 32: 19, now 8.  Reverse head of those 256 graphs: 63, now 41.
#include <type_traits>

#include "internal.h"

namespace pl {

namespace {

constexpr int kBlock = 16;            // fp32 terms per float64 block
constexpr int kComputeUnits = 256;

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// Launch shapes.  kPerGraph: a workgroup per graph with as many threads as a layer of the h networks can use.
// kPerSet (H >= 128): a workgroup per (graph, set).  kPacked (H <= 64): a workgroup of few threads per graph.
enum HeadShape { kPerGraph, kPerSet, kPacked };

// Instantiations: HT = H where it is known when the kernel is compiled (32, 64, 128), else 0; RT: rows of a
// set per pass; SHAPE.
constexpr int head_threads(int HT, HeadShape shape)
{
    return shape == kPacked ? (HT == 64 ? 256 : 128) : HT == 0 || (HT == 128 && shape == kPerGraph) ? 1024 : 512;
}
// Threads of a launch over B graphs.  Where H is not known the kernel takes any whole number of waves: 1024 while a
// graph has a CU to itself, else five groups of H threads, so that several graphs share a CU.  Forward head at H =
// 48, 4 devices: 256 graphs 17 us with 1024 threads, 21 with 384; 2048 graphs 101 us with 1024, 77 with 384, 54
// with 256; at H = 8, 2 devices, 4096 graphs: 130 us with 1024, 19 with 64.
constexpr int head_launch_threads(int H, int B, int HT, HeadShape shape)
{
    if (HT != 0 || B <= kComputeUnits || 5 * H >= 1024) return head_threads(HT, shape);
    return (5 * H + 63) / 64 * 64;
}
constexpr int head_cols(int HT) { return HT != 0 ? 4 : 1; }             // columns per thread
constexpr int head_sets(int H, HeadShape shape) { return shape != kPerSet && H <= 128 ? 3 : 1; }   // networks taken together

// What a kernel of a width that is not known keeps in dynamic LDS beside the rows: the biases of `layers` layers
// and the output layer's weights.
constexpr size_t head_small(int H, int D, int layers, int HT) { return HT != 0 ? 0 : static_cast<size_t>(layers + D) * H; }

constexpr size_t head_lds(int H, int G, int RT, int HT, HeadShape shape, int threads, size_t small = 0)
{
    const size_t groups = static_cast<size_t>(threads / (H / head_cols(HT)));
    const size_t part = HT == 0 ? groups * RT * H * sizeof(double)
                                : static_cast<size_t>(head_sets(H, shape)) * (H / kBlock) * RT * H * sizeof(float);
    const size_t red = groups * H * sizeof(double);
    return (part > red ? part : red) + sizeof(float) * (static_cast<size_t>(2 + (shape == kPerSet ? 1 : 3) * G) * H + small + 4);
}

// Sixteen rows of four columns, the weights of one unit.
template <int HT>
struct WeightBlock {
    static constexpr int CPT = head_cols(HT);
    float w[kBlock][CPT];
    // rows k0 .. k0 + 15 of a matrix with H columns, from column j on
    __device__ __forceinline__ void load(const float *__restrict__ W, int H)
    {
#pragma unroll
        for (int k = 0; k < kBlock; ++k) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(W + static_cast<size_t>(k) * H);
#pragma unroll
            for (int c = 0; c < CPT; ++c) w[k][c] = v[c];
        }
    }
    __device__ __forceinline__ void apply(const float *x, float (&s)[CPT]) const
    {
#pragma unroll
        for (int c = 0; c < CPT; ++c) s[c] = 0.0f;
#pragma unroll
        for (int k = 0; k < kBlock; ++k) {
            const float xv = x[k];
#pragma unroll
            for (int c = 0; c < CPT; ++c) s[c] = fmaf(xv, w[k][c], s[c]);
        }
    }
};

// Any width: acc[r] += one column's product with row r of x over the blocks first, first + step, ... of the
// n_in inputs.  The inputs past the last whole block are summed in float64 one by one (by the group whose
// turn that block is): at H < 16 those are all of a layer's terms.  VEC: rows of x start on 16-byte boundaries, and
// are read four entries at a time (LDS reads are what these loops wait for: 1024 graphs at H = 100: 110 -> 97 us).
template <int RT, bool VEC>
__device__ __forceinline__ void dot_rows(const float *__restrict__ W, int H, int n_in, int first, int step, const float *x,
                                         int ldx, int rows, double (&acc)[RT])
{
    const int whole = n_in / kBlock;
    int u = first;
    for (; u < whole; u += step) {
        float w[kBlock];
#pragma unroll
        for (int k = 0; k < kBlock; ++k) w[k] = W[static_cast<size_t>(u * kBlock + k) * H];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const float *xr = x + min(r, rows - 1) * ldx + u * kBlock;
            float xv[kBlock];
#pragma unroll
            for (int k = 0; k < kBlock; k += VEC ? 4 : 1) {
                if constexpr (VEC)
                    *reinterpret_cast<f32x4 *>(xv + k) = *reinterpret_cast<const f32x4 *>(xr + k);
                else
                    xv[k] = xr[k];
            }
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k < kBlock; ++k) s = fmaf(xv[k], w[k], s);
            acc[r] += static_cast<double>(s);
        }
    }
    if (u != whole) return;
    const int kn = n_in - whole * kBlock;
    float w[kBlock];
#pragma unroll
    for (int k = 0; k < kBlock; ++k) w[k] = k < kn ? W[static_cast<size_t>(whole * kBlock + k) * H] : 0.0f;
#pragma unroll
    for (int k = 0; k < kBlock; ++k) {
        if (k >= kn) break;
#pragma unroll
        for (int r = 0; r < RT; ++r)
            acc[r] = fma(static_cast<double>(x[min(r, rows - 1) * ldx + whole * kBlock + k]), static_cast<double>(w[k]), acc[r]);
    }
}

// The layers of the h networks (set0 .. set0 + sets - 1 of the three) on the rows x [sets][G][H] (LDS), in
// place.  Where H is known, a unit is (set, slice of sixteen inputs), H / 4 threads, and a thread has at most
// one; AHEAD: its weights of the next layer are requested before the current layer's slices are added up.
// Otherwise the groups of H threads are shared out among the sets, and a group takes every so manieth slice.
template <int HT, int RT, HeadShape SHAPE, bool AHEAD>
struct HeadLayers {
    static constexpr int CPT = head_cols(HT);
    WeightBlock<HT> wb;
    int H, G, T, slices, cols, sets, groups, grp, j;

    __device__ __forceinline__ HeadLayers(int H_, int G_)
    {
        H = HT ? HT : H_;
        G = G_;
        T = HT ? head_threads(HT, SHAPE) : blockDim.x;
        slices = H / kBlock;
        cols = H / CPT;
        sets = head_sets(H, SHAPE);
        groups = T / cols;
        grp = static_cast<int>(threadIdx.x) / cols;
        j = (static_cast<int>(threadIdx.x) - grp * cols) * CPT;
    }
    // w0: place in `blob` of the layer's matrix of the first set, ws: distance to the next set's
    __device__ __forceinline__ void request(const float *__restrict__ blob, int w0, int ws, int set0)
    {
        if constexpr (AHEAD) {
            if (grp < sets * slices) {
                const int set = set0 + grp / slices, k0 = (grp % slices) * kBlock;
                wb.load(blob + w0 + static_cast<ptrdiff_t>(set) * ws + static_cast<size_t>(k0) * H + j, H);
            }
        }
    }
    // next(): what to request while the sums settle; finish(set, row, column, sum): the new value, `sum` in
    // float64 over the inputs in blocks
    template <typename N, typename F>
    __device__ __forceinline__ void layer(const float *__restrict__ blob, int w0, int ws, int set_first, float *x,
                                          float *part, N next, F finish)
    {
        const int tid = threadIdx.x;
        // sums to add up for an entry, and their distance
        const int n_part = HT ? slices : min(groups / sets, (H + kBlock - 1) / kBlock), part_step = RT * H;
        double *part64 = reinterpret_cast<double *>(part);
        for (int set0 = 0; set0 < (SHAPE == kPerSet ? 1 : 3); set0 += sets)
            for (int r0 = 0; r0 < G; r0 += RT) {
                const int rows = min(RT, G - r0);
                if constexpr (HT != 0) {
                    if (grp < sets * slices) {
                        const int q = grp / slices, k0 = (grp - q * slices) * kBlock;
                        if constexpr (!AHEAD)
                            wb.load(blob + w0 + static_cast<ptrdiff_t>(set_first + set0 + q) * ws + static_cast<size_t>(k0) * H + j, H);
#pragma unroll
                        for (int r = 0; r < RT; ++r) {
                            float s[CPT];
                            wb.apply(x + ((set0 + q) * G + r0 + min(r, rows - 1)) * H + k0, s);
#pragma unroll
                            for (int c = 0; c < CPT; ++c) part[(grp * RT + r) * H + j + c] = s[c];
                        }
                    }
                } else if (grp < sets * n_part) {
                    const int q = grp / n_part;
                    double acc[RT];
#pragma unroll
                    for (int r = 0; r < RT; ++r) acc[r] = 0.0;
                    const float *W = blob + w0 + static_cast<ptrdiff_t>(set_first + set0 + q) * ws + j, *xq = x + ((set0 + q) * G + r0) * H;
                    if (H % 4 == 0)
                        dot_rows<RT, true>(W, H, H, grp - q * n_part, n_part, xq, H, rows, acc);
                    else
                        dot_rows<RT, false>(W, H, H, grp - q * n_part, n_part, xq, H, rows, acc);
#pragma unroll
                    for (int r = 0; r < RT; ++r) part64[(grp * RT + r) * H + j] = acc[r];
                }
                if (AHEAD && r0 + RT >= G) next();
                __syncthreads();
                for (int i = tid; i < sets * rows * H; i += T) {
                    const int sr = i / H, c = i - sr * H, q = sr / rows, r = sr - q * rows;
                    const int at = q * n_part * part_step + r * H + c;
                    double s = 0.0;
                    for (int k = 0; k < n_part; ++k) s += HT ? static_cast<double>(part[at + k * part_step]) : part64[at + k * part_step];
                    x[((set0 + q) * G + r0 + r) * H + c] = finish(set_first + set0 + q, r0 + r, c, s);
                }
                __syncthreads();
            }
    }
};

struct HeadOut {
    // kept for the reverse pass, or null
    float *zbuf;          // [B, Z] policy inputs
    double *hid;          // [B, H] hidden layer of the policy network
    float *logit;         // [B, D] logits, also where out_logits gets NaN

    float *out_logits, *out_probs, *out_pooled;
    float *hin, *hact;    // kept for the reverse pass (or null): inputs [3, B G, H] and layer outputs [3, L, B G, H] of h
    double *hidp;         // (SPLIT) [B, 3, H] the sets' parts of the first policy layer
    uint32_t *done;       // (SPLIT) [B] workgroups of a graph that have written theirs; cleared by the pooling kernels
};

// Pooling of small graphs of narrow networks within the head's workgroup (pool_in_head): reachability and placement, and
// where its LDS begins.  reach is null where a kernel of its own has left partial sums.
struct PoolHere {
    const uint8_t *reach;
    const int32_t *placement;
    int lds_at;
};
constexpr int kHerePoolNodes = kPoolChunk / 2;   // graphs of one slice (pool_slices)
// floats of the three l networks, of embedding rows, of two layers' outputs; keys
constexpr int here_ld(int H) { return 2 * H + 1; }
constexpr size_t here_lds(int H, int L, int n)
{
    return sizeof(float) * (static_cast<size_t>(3) * ((L + 1) * H * H + L * H) + static_cast<size_t>(n) * (here_ld(H) + 2 * (H + 1)) + n);
}

template <int HT, int RT, HeadShape SHAPE>
__global__ __launch_bounds__(head_threads(HT, SHAPE)) void k_head(GraphView gv, ModelView mv, const float *__restrict__ emb,
                                                              const float *__restrict__ partial,
                                                              const int32_t *__restrict__ cur_node, int max_chunks,
                                                              HeadOut o, PoolHere here)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ double hid[kMaxH];
    __shared__ float logit[kMaxD], bias2[kMaxD], bias_s[HT ? (3 * kMaxLayers + 1) * HT : 1], w2_s[HT ? HT * kMaxD : 1];
    __shared__ uint32_t order;
    constexpr int CPT = head_cols(HT);
    constexpr bool SPLIT = SHAPE == kPerSet;
    const int H = HT ? HT : mv.H, G = mv.G, L = mv.L, D = mv.D, Z = mv.Z, T = HT ? head_threads(HT, SHAPE) : blockDim.x;
    const int b = SPLIT ? blockIdx.x / 3 : blockIdx.x, set_first = SPLIT ? blockIdx.x - 3 * b : 0;
    constexpr int n_sets = SPLIT ? 1 : 3;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (weights ahead take registers that 1024 threads do not have beside the float64 sums, and that many small
    // workgroups on a CU need for themselves)
    constexpr bool AHEAD = HT != 0 && head_threads(HT, SHAPE) == 512;
    HeadLayers<HT, RT, SHAPE, AHEAD> hl(mv.H, G);
    // h's weights and everything small that later phases need: requested before the graph's own data
    hl.request(mv.blob, mv.h[0].layer[0].w, mv.h[1].layer[0].w - mv.h[0].layer[0].w, set_first);
    // (places by distance between sets and layers: an index of a thread's own into the kernel's arguments
    // would be a load of its own ahead of each)
    float *z = reinterpret_cast<float *>(lds);              // e_{v*}, then the rows of the sets
    float *small = z + (2 + n_sets * G) * H;
    float *bias = HT ? bias_s : small, *w2 = HT ? w2_s : small + (n_sets * L + 1) * H;
    const int b_set = mv.h[1].layer[0].b - mv.h[0].layer[0].b, b_layer = L > 1 ? mv.h[0].layer[1].b - mv.h[0].layer[0].b : 0;
    const float *b_first = mv.blob + mv.h[0].layer[0].b;
    for (int i = tid; i < n_sets * L * H; i += T) {
        const int set = i / (L * H), r = i - set * L * H, l = r / H;
        bias[i] = b_first[(set_first + set) * b_set + l * b_layer + r - l * H];
    }
    if (tid < D) bias2[tid] = mv.blob[mv.pol2.b + tid];
    float *bias1 = bias + n_sets * L * H;
    for (int i = tid; i < H; i += T) bias1[i] = mv.blob[mv.pol1.b + i];
    for (int i = tid; i < H * D; i += T) w2[i] = mv.blob[mv.pol2.w + i];
    float *x = z + 2 * H, *part = z + (((2 + n_sets * G) * H + static_cast<int>(head_small(H, D, n_sets * L + 1, HT)) + 3) & ~3);
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int cl = cur_node[b];
    const bool cur_ok = cl >= 0 && cl < n_b;
    const int chunks = pool_slices(n_b, max_chunks);
    const size_t BG = static_cast<size_t>(gv.B) * G;
    // place of element i of a set's rows in the arrays kept for the reverse pass
    auto kept = [&](int set, int l, int layers, int i) {
        return ((static_cast<size_t>(set) * layers + l) * BG + static_cast<size_t>(b) * G) * H + i;
    };

    // ---- P[set][group] = sum of the pooling partials in slice order
    const int first = set_first * G * H;
    const float *src = partial + static_cast<size_t>(b) * max_chunks * 3 * G * H + first;
    auto pooled = [&](int i, float s) {
        x[i] = s;
        if (o.out_pooled) o.out_pooled[static_cast<size_t>(b) * 3 * G * H + first + i] = s;
        if (o.hin) {
            const int set = i / (G * H);
            o.hin[kept(set_first + set, 0, 1, i - set * G * H)] = s;
        }
    };
    bool here_pooled = false;
    if constexpr (HT == 0 && SHAPE == kPerGraph) {
        // Or, for a small graph: l of its nodes, a thread to an output, and their sums, in the order of the kernel that
        // otherwise does it (bias first, then the inputs; nodes ascending).
        here_pooled = here.reach != nullptr;
        if (here_pooled) {
            float *wl = reinterpret_cast<float *>(lds + here.lds_at);          // per set: matrices and biases as in the blob
            const int per_set = (L + 1) * H * H + L * H, ld = here_ld(H), la = H + 1;
            float *rows = wl + 3 * per_set, *act = rows + n_b * ld;
            int *key = reinterpret_cast<int *>(act + 2 * n_b * la);
            for (int i = tid; i < 3 * per_set; i += T) {
                const int set = i / per_set;
                wl[i] = mv.blob[mv.l[0].layer[0].w + set * (mv.l[1].layer[0].w - mv.l[0].layer[0].w) + i - set * per_set];
            }
            for (int i = tid; i < n_b * 2 * H; i += T) {
                const int v = i / (2 * H);
                rows[v * ld + i - v * 2 * H] = emb[static_cast<size_t>(n0) * 2 * H + i];
            }
            for (int v = tid; v < n_b; v += T) {
                const int dev = here.placement[n0 + v];
                const int set = mv.single_set ? 0 : (here.reach[static_cast<size_t>(gv.n_tot) + n0 + v] ? 0 : (here.reach[n0 + v] ? 1 : 2));
                key[v] = v == cl ? -1 : set * G + (dev < 0 || dev >= D ? -3 * G : (G == 1 ? 0 : dev));   // (negative: in no sum)
            }
            __syncthreads();
            const float *in = rows;
            for (int l = 0, n_in = 2 * H, ldi = ld; l < L; ++l, n_in = H, ldi = la) {
                float *out = act + l % 2 * n_b * la;
                for (int i = tid; i < n_b * H; i += T) {
                    const int v = i / H, j = i - v * H, k = key[v];
                    if (k < 0) continue;
                    const float *w = wl + k / G * per_set + (l == 0 ? 0 : 2 * H * H + H + (l - 1) * (H * H + H));
                    float s = w[n_in * H + j];
#pragma unroll 8
                    for (int q = 0; q < n_in; ++q) s = fmaf(in[v * ldi + q], w[q * H + j], s);
                    out[v * la + j] = fmaxf(s, 0.0f);
                }
                __syncthreads();
                in = out;
            }
            for (int i = tid; i < 3 * G * H; i += T) {
                const int k = i / H, j = i - k * H;
                float s = 0.0f;
#pragma unroll 8
                for (int v = 0; v < n_b; ++v) s += key[v] == k ? in[v * la + j] : 0.0f;
                pooled(i, s);
            }
        }
    }
    // From three slices on all of them are requested at once (past the last one, it again): one after the other, each waited
    // for, a graph of 200 nodes and four slices took 14.7 us (H = 64, one graph) and 8.6 (H = 32, 64 graphs), now 13.2 and 7.7.
    // With one or two, eight requests (each behind a branch) cost a batch of 4096 small graphs 1 %.
    for (int i = tid; i < n_sets * G * H && !here_pooled; i += T) {
        float s = 0.0f;
        if (chunks <= 2) {
            for (int c = 0; c < chunks; ++c) s += src[static_cast<size_t>(c) * 3 * G * H + i];
        } else {
            for (int c0 = 0; c0 < chunks; c0 += kPoolSlices) {
                float y[kPoolSlices];
#pragma unroll
                for (int c = 0; c < kPoolSlices; ++c) y[c] = src[static_cast<size_t>(min(c0 + c, chunks - 1)) * 3 * G * H + i];
#pragma unroll
                for (int c = 0; c < kPoolSlices; ++c) s += c0 + c < chunks ? y[c] : 0.0f;
            }
        }
        pooled(i, s);
    }
    for (int i = tid; i < 2 * H && set_first == 0; i += T)
        z[i] = cur_ok ? emb[static_cast<size_t>(n0 + cl) * 2 * H + i] : 0.0f;
    __syncthreads();

    // ---- first policy layer: group g takes the blocks g, g + groups, ... of this workgroup's part of z (the
    // first set's comes with e_{v*}); place of its first weight
    const int p_cols = H / CPT, p_groups = T / p_cols, p_grp = tid / p_cols, p_j = (tid - p_grp * p_cols) * CPT;
    const float *zp = set_first == 0 ? z : x;
    const int z_at = set_first == 0 ? 0 : (2 + set_first * G) * H;
    const int z_n = SPLIT ? (G + (set_first == 0 ? 2 : 0)) * H : Z;
    const int blocks = (z_n + kBlock - 1) / kBlock, used = min(p_groups, blocks);
    const float *W1 = mv.blob + mv.pol1.w + static_cast<size_t>(z_at) * H + p_j;

    // ---- h of the sets
    for (int l = 0; l < L; ++l) {
        const LayerRef &l0 = mv.h[0].layer[l];
        hl.layer(
            mv.blob, l0.w, mv.h[1].layer[l].w - l0.w, set_first, x, part,
            [&]() {
                if (l + 1 < L)
                    hl.request(mv.blob, mv.h[0].layer[l + 1].w, mv.h[1].layer[l + 1].w - mv.h[0].layer[l + 1].w, set_first);
                else if (p_grp < used)
                    hl.wb.load(W1 + static_cast<size_t>(p_grp) * kBlock * H, H);
            },
            [&](int set, int r, int c, double s) {
                const float y = fmaxf(static_cast<float>(s + static_cast<double>(bias[((set - set_first) * L + l) * H + c])), 0.0f);
                if (o.hact) o.hact[kept(set, l, L, r * H + c)] = y;
                return y;
            });
    }
    if (o.zbuf)
        for (int i = tid; i < z_n; i += T) o.zbuf[static_cast<size_t>(b) * Z + z_at + i] = zp[i];

    double *red = reinterpret_cast<double *>(part);         // [used][H]
    if (p_grp < used) {
        double acc[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) acc[c] = 0.0;
        if constexpr (HT == 0) {
            if (!SPLIT || H % 4 == 0)
                dot_rows<1, true>(W1, H, z_n, p_grp, p_groups, zp, 0, 1, acc);
            else
                dot_rows<1, false>(W1, H, z_n, p_grp, p_groups, zp, 0, 1, acc);
        } else {
            for (int q = p_grp; q < blocks; q += p_groups) {
                if (!AHEAD || q != p_grp) hl.wb.load(W1 + static_cast<size_t>(q) * kBlock * H, H);
                float s[CPT];
                hl.wb.apply(zp + q * kBlock, s);
#pragma unroll
                for (int c = 0; c < CPT; ++c) acc[c] += static_cast<double>(s[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) red[p_grp * H + p_j + c] = acc[c];
    }
    __syncthreads();
    for (int c = tid; c < H; c += T) {
        double s = 0.0;
        for (int g = 0; g < used; ++g) s += red[g * H + c];
        hid[c] = s;
        // (stored past the caches that workgroups on other dies do not share)
        if constexpr (SPLIT)
            __hip_atomic_store(o.hidp + (static_cast<size_t>(b) * 3 + set_first) * H + c, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if constexpr (SPLIT) {
        // The workgroup that finishes a graph last adds the sets' parts up and goes on.  Every thread's stores have
        // arrived where all dies see them before the one atomic that announces them: they are agent-scope stores, each
        // thread waits for its own, and the barrier is behind all of them; the loads are agent-scope loads and come
        // after the barrier that hands the atomic's result round.  An acquire-release atomic would order them too, but
        // writes the die's whole L2 back first (85 graphs: 22 -> 25.7 us).
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
        if (tid == 0) order = __hip_atomic_fetch_add(o.done + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (order != 2u) return;
        for (int c = tid; c < H; c += T) {
            double s = 0.0;
            for (int set = 0; set < 3; ++set)
                s += __hip_atomic_load(o.hidp + (static_cast<size_t>(b) * 3 + set) * H + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            hid[c] = s;
        }
    }
    for (int c = tid; c < H; c += T) {                      // (a column's sum is its own thread's)
        const double s = hid[c] + static_cast<double>(bias1[c]);
        hid[c] = s > 0.0 ? s : 0.0;
        if (o.hid) o.hid[static_cast<size_t>(b) * H + c] = hid[c];
    }
    __syncthreads();

    // ---- output layer (a wave per device), softmax
    for (int d = wave; d < D; d += T / 64) {
        double s = 0.0;
        for (int k = lane; k < H; k += 64)
            s = fma(hid[k], static_cast<double>(w2[k * D + d]), s);
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) s += __shfl_xor(s, step);
        if (lane == 0) logit[d] = static_cast<float>(s + static_cast<double>(bias2[d]));
    }
    __syncthreads();
    if (tid < D) {
        const float bad = __builtin_nanf("");               // no valid current node: nothing to decide
        const size_t at = static_cast<size_t>(b) * D + tid;
        if (o.logit) o.logit[at] = logit[tid];
        o.out_logits[at] = cur_ok ? logit[tid] : bad;
        if (o.out_probs) {
            float mx = logit[0], tot = 0.0f;
            for (int d = 1; d < D; ++d) mx = fmaxf(mx, logit[d]);
            for (int d = 0; d < D; ++d) tot += expf(logit[d] - mx);
            o.out_probs[at] = cur_ok ? expf(logit[tid] - mx) / tot : bad;
        }
    }
}

// ------------------------------------------------------------------ reverse
// d logits = c (one-hot(a) - softmax) + entropy term, back to the hidden layer, to the policy input z
// (dz; its first 2H entries are the gradient of e_{v*}) and through the h networks to dP[set][group].
// A graph whose current node or action is out of range gets a zero gradient and logp = NaN.
template <int HT, int RT, HeadShape SHAPE>
__global__ __launch_bounds__(head_threads(HT, SHAPE)) void k_head_bw(GraphView gv, ModelView mv, const float *__restrict__ blob_t,
                                                          const int32_t *__restrict__ cur_node, HeadBwArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float dpre[kMaxH];
    __shared__ float dlog[kMaxD];
    const int H = HT ? HT : mv.H, G = mv.G, L = mv.L, D = mv.D, Z = mv.Z, T = HT ? head_threads(HT, SHAPE) : blockDim.x;
    const int b = blockIdx.x, tid = threadIdx.x;
    // (weights ahead also with 1024 threads: no float64 sums are held here, 110 registers)
    HeadLayers<HT, RT, SHAPE, HT != 0 && SHAPE != kPacked> hl(mv.H, G);
    auto request = [&](int l) { hl.request(blob_t, mv.h[0].layer[l].w, mv.h[1].layer[l].w - mv.h[0].layer[l].w, 0); };
    request(L - 1);
    float *z = reinterpret_cast<float *>(lds);              // [Z]: dz
    float *part = z + ((Z + 3) & ~3), *x = z + 2 * H;
    const int n_b = gv.node_off[b + 1] - gv.node_off[b];
    const int cl = cur_node[b];
    const bool cur_ok = cl >= 0 && cl < n_b;
    const size_t BG = static_cast<size_t>(gv.B) * G;
    auto kept = [&](int set, int l, int i) {
        return ((static_cast<size_t>(set) * L + l) * BG + static_cast<size_t>(b) * G) * H + i;
    };
    if (tid < D) {
        const float *logit = a.logit + static_cast<size_t>(b) * D;
        float mx = logit[0], tot = 0.0f, ent = 0.0f;
        for (int d = 1; d < D; ++d) mx = fmaxf(mx, logit[d]);
        for (int d = 0; d < D; ++d) tot += expf(logit[d] - mx);
        const int act = a.actions[b];
        const bool ok = cur_ok && act >= 0 && act < D;
        const float c = ok ? a.coeff[b] : 0.0f;
        // entropy term (Appendix A.7): H = - sum p log p, dH / d logit_d = - p_d (log p_d + H), with
        // log p_d = logit_d - max - log(sum), which stays finite where p_d underflows to 0
        const float beta = (ok && a.entropy_coeff) ? a.entropy_coeff[b] : 0.0f;
        const float lse = logf(tot);
        for (int d = 0; d < D; ++d) ent -= expf(logit[d] - mx) / tot * ((logit[d] - mx) - lse);
        const float p = expf(logit[tid] - mx) / tot;
        const float g = c * ((tid == act ? 1.0f : 0.0f) - p) - beta * p * (((logit[tid] - mx) - lse) + ent);
        dlog[tid] = g;
        a.dlogit[static_cast<size_t>(b) * D + tid] = g;
        if (tid == 0) {
            if (a.out_logp) a.out_logp[b] = ok ? (logit[act] - mx) - lse : __builtin_nanf("");
            if (a.out_entropy) a.out_entropy[b] = cur_ok ? ent : __builtin_nanf("");
        }
    }
    __syncthreads();
    for (int j = tid; j < H; j += T) {
        const float *W = mv.blob + mv.pol2.w + static_cast<size_t>(j) * D;
        const float h = static_cast<float>(a.hid64[static_cast<size_t>(b) * H + j]);
        float s = 0.0f;
        for (int d = 0; d < D; ++d) s = fmaf(W[d], dlog[d], s);
        const float dp = h > 0.0f ? s : 0.0f;
        dpre[j] = dp;
        a.hid[static_cast<size_t>(b) * H + j] = h;
        a.dpre[static_cast<size_t>(b) * H + j] = dp;
    }
    __syncthreads();
    // dz[k] = sum_j W1[k][j] dpre[j], from the transposed layer [H, Z]; the rows of h's outputs gated
    {
        const float *W1t = blob_t + mv.pol1.w;
        for (int k = tid; k < Z; k += T) {
            float s = 0.0f;
            int j = 0;
            for (; j + kBlock <= H; j += kBlock) {
                float w[kBlock];
#pragma unroll
                for (int u = 0; u < kBlock; ++u) w[u] = W1t[static_cast<size_t>(j + u) * Z + k];
#pragma unroll
                for (int u = 0; u < kBlock; ++u) s = fmaf(w[u], dpre[j + u], s);
            }
            for (; j < H; ++j) s = fmaf(W1t[static_cast<size_t>(j) * Z + k], dpre[j], s);
            a.dz[static_cast<size_t>(b) * Z + k] = s;
            if (k >= 2 * H) {                               // delta of h's last layer
                const int i = k - 2 * H, set = i / (G * H);
                const size_t at = kept(set, L - 1, i - set * G * H);
                s = a.hact[at] > 0.0f ? s : 0.0f;
                a.dh[at] = s;
            }
            z[k] = s;
        }
    }
    __syncthreads();
    for (int l = L - 1; l >= 0; --l) {
        const LayerRef &l0 = mv.h[0].layer[l];
        hl.layer(blob_t, l0.w, mv.h[1].layer[l].w - l0.w, 0, x, part, [&]() { if (l > 0) request(l - 1); },
                 [&](int set, int r, int c, double s) {
            float y = static_cast<float>(s);
            if (l > 0) {
                const size_t at = kept(set, l - 1, r * H + c);
                y = a.hact[at] > 0.0f ? y : 0.0f;
                a.dh[at] = y;
            } else {
                a.dP[((static_cast<size_t>(b) * 3 + set) * G + r) * H + c] = y;
            }
            return y;
        });
    }
}

// Calls go(HT, RT, SHAPE) with the instantiation for width H, G rows per set and B graphs.
//   * H >= 128, forward: one CU reads a graph's weights longer than three; with more workgroups than CUs the hand-over
//     between them costs more than it gives.  Together / split at H = 128, 8 device groups: 1 graph 35 / 22 us, 85
//     graphs 32 / 22, 100 graphs 32 / 34, 256 graphs 35 / 53; one group: 15 / 13 at 85, 15 / 19 at 100; at H = 256, 4
//     groups: 78 / 41 at 85, 79 / 68 at 100 (the pass 1.807 / 1.792 ms), 98 / 115 at 256.
//   * H = 32 and 64: 512 threads with weights ahead have a CU to themselves, so a second graph per CU waits for the
//     first.  Above one graph per CU: small workgroups without (forward head at H = 64, 8 devices: 256 graphs 19 us,
//     small 22, 1024 graphs 60 and 40; at H = 32, 4 devices: 12 and 14, 30 and 16).  The reverse head at H = 64
//     takes fewer registers and changes over later (512 graphs of 8 devices: 27 us, small 30; 1024: 50 and 46).
template <typename F>
void head_dispatch(int H, int G, int B, bool forward, F go)
{
    auto rows = [&](auto ht, auto shape) {
        if (G == 1) go(ht, std::integral_constant<int, 1>{}, shape);
        else if (G == 2) go(ht, std::integral_constant<int, 2>{}, shape);
        else if (G <= 4) go(ht, std::integral_constant<int, 4>{}, shape);
        else go(ht, std::integral_constant<int, 8>{}, shape);
    };
    const std::integral_constant<HeadShape, kPerGraph> per_graph;
    const std::integral_constant<HeadShape, kPerSet> per_set;
    const std::integral_constant<HeadShape, kPacked> packed;
    const std::integral_constant<int, 128> h128;
    const std::integral_constant<int, 64> h64;
    const std::integral_constant<int, 32> h32;
    const std::integral_constant<int, 0> any;
    const bool split = forward && H >= 128 && 3 * B <= kComputeUnits;
    if (H == 128 && split) rows(h128, per_set);
    else if (H == 128) rows(h128, per_graph);
    else if (H == 64 && B <= (forward ? 1 : 2) * kComputeUnits) rows(h64, per_graph);
    else if (H == 64) rows(h64, packed);
    else if (H == 32 && B <= kComputeUnits) rows(h32, per_graph);
    else if (H == 32) rows(h32, packed);
    else if (split) rows(any, per_set);
    else rows(any, per_graph);
}

template <typename K>
void allow_lds(K kernel, size_t bytes)
{
    if (bytes > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(bytes));
}

}  // namespace

// Narrow networks on batches that leave a compute unit to every graph: the launch between costs more than the sums (forward
// pass with a pooling kernel and without: one graph of 32 nodes, H = 8, 26.3 / 22.0 us; 64 graphs of 64 nodes 46 / 30; 256
// graphs of 64 nodes and 8 devices 67 / 33; 128 graphs of 64 nodes, H = 16, 16 devices 58 / 40).  With more graphs than
// compute units the head has fewer threads.  Graphs of one slice: here a sum takes a graph's nodes in one go, and with more
// slices it would have other bits than in a larger batch, which another kernel pools (it would be faster still: one graph of
// 72 / 128 nodes, H = 8, 30.3 / 42.0 us as it is, 27.4 / 36.6 here; from 160 nodes on, H = 16, slower).
bool pool_in_head(int H, int L, int B, int n_max)
{
    return (H == 8 || H == 16) && L <= 2 && B <= kComputeUnits && n_max <= kHerePoolNodes;
}

// n_max: nodes of the largest graph, where the head pools (0: a kernel of its own has)
void launch_head(const GraphView &gv, const ModelView &mv, const Workspace &ws, const ForwardArgs &fa, int max_chunks,
                 int n_max, hipStream_t s)
{
    if (gv.B == 0) return;
    const HeadOut o{ws.zbuf,      ws.hid,       ws.logit, fa.out_logits, fa.out_probs, fa.out_pooled,
                    fa.keep_hin,  fa.keep_hact, ws.hidp,  ws.head_done};
    head_dispatch(mv.H, mv.G, gv.B, true, [&](auto ht, auto rt, auto shape) {
        constexpr int HT = decltype(ht)::value, RT = decltype(rt)::value;
        constexpr HeadShape SHAPE = decltype(shape)::value;
        const int threads = head_launch_threads(mv.H, gv.B, HT, SHAPE), sets = SHAPE == kPerSet ? 1 : 3;
        size_t lds = head_lds(mv.H, mv.G, RT, HT, SHAPE, threads, head_small(mv.H, mv.D, sets * mv.L + 1, HT));
        PoolHere here{nullptr, nullptr, 0};
        if (n_max > 0) {
            here = {ws.reach, fa.placement, static_cast<int>((lds + 15) / 16 * 16)};
            lds = here.lds_at + here_lds(mv.H, mv.L, n_max);
        }
        allow_lds(k_head<HT, RT, SHAPE>, lds);
        hipLaunchKernelGGL((k_head<HT, RT, SHAPE>), dim3(SHAPE == kPerSet ? 3 * gv.B : gv.B), dim3(threads), lds, s, gv, mv,
                           ws.emb, ws.partial, fa.cur_node, max_chunks, o, here);
    });
}

void launch_head_bw(const GraphView &gv, const ModelView &mv, const float *blob_t, const int32_t *cur_node,
                    const HeadBwArgs &a, hipStream_t s)
{
    if (gv.B == 0) return;
    head_dispatch(mv.H, mv.G, gv.B, false, [&](auto ht, auto rt, auto shape) {
        constexpr int HT = decltype(ht)::value, RT = decltype(rt)::value;
        constexpr HeadShape SHAPE = decltype(shape)::value;
        const int threads = head_launch_threads(mv.H, gv.B, HT, SHAPE);
        const size_t lds = head_lds(mv.H, mv.G, RT, HT, SHAPE, threads);
        if constexpr (SHAPE != kPerSet) {
            allow_lds(k_head_bw<HT, RT, SHAPE>, lds);
            hipLaunchKernelGGL((k_head_bw<HT, RT, SHAPE>), dim3(gv.B), dim3(threads), lds, s, gv, mv, blob_t, cur_node, a);
        }
    });
}

}  // namespace pl
