// Policy head (Section 2.2 step 3, Appendix A.7), forward and reverse: q[i][d] = h_i(P[i][d]) (also for
// empty groups); z = [e_{v*} ; q]; two-layer policy network with a softmax over devices.
//
// One workgroup of 1024 threads per graph does all of it.  The head is small (2 MB of weights at the
// NASNet-like shape, 0.3 MB at H = 64) and a chain of dense layers, so its time is its launches, the
// latency of its weight loads and, with many graphs, the rate at which a CU reads weights from L2; three
// launches with a workgroup per (graph, set), per (16 graphs, slice of z) and per graph spent most of
// theirs starting and on sequential loops (the output layer took one thread per device).
//   * A layer of the three h networks is one phase: a unit (set, slice of sixteen inputs) is H / 4
//     threads with four columns and up to eight rows each, so a weight is loaded once, as part of a
//     16-byte load, and an input read from LDS feeds four columns.  The slices' sums meet in LDS.
//   * The first policy layer spreads its blocks of sixteen inputs over groups of H / 4 threads, 64
//     weights per thread in flight; the output layer has a wave per device.
// Sums are taken in float64 by blocks (sixteen fp32 terms, the blocks in float64, the output layer
// entirely in float64): z holds sums over thousands of nodes, so a logit is a difference of terms far
// larger than itself, and plain fp32 sums would be the largest single source of its error.
// HEAD_FIG
#include <type_traits>

#include "internal.h"

namespace pl {

namespace {

constexpr int kHeadThreads = 1024;
constexpr int kBlock = 16;       // fp32 terms per float64 block

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// columns per thread, rows per pass, and whether the three networks are taken together, for width H
// (HT = H where it is known when the kernel is compiled, else 0)
constexpr int head_cols(int HT) { return HT >= 32 ? 4 : 1; }
constexpr bool head_sets_together(int H) { return H <= 128; }
constexpr int head_rows_max(int H) { return H <= 128 ? 8 : 4; }

constexpr size_t head_lds(int H, int G, int RT, int HT)
{
    const size_t units = static_cast<size_t>(head_sets_together(H) ? 3 : 1) * ((H + kBlock - 1) / kBlock);
    const size_t part = units * RT * H * sizeof(float);
    const size_t red = static_cast<size_t>(kHeadThreads / (H / head_cols(HT))) * H * sizeof(double);
    return (part > red ? part : red) + sizeof(float) * (static_cast<size_t>(2 + 3 * G) * H + 4);
}

// One layer of the three h networks on the rows x [3][G][H] (LDS), in place: finish(set, row, column,
// sum) gives the new value, `sum` in float64 over the inputs in blocks.  w0: place in `blob` of the
// layer's [H, H] matrix of the first set, ws: distance to the next set's.  part: LDS scratch.
template <int HT, int RT, typename F>
__device__ __forceinline__ void head_layer(const float *__restrict__ blob, int w0, int ws, float *x, float *part,
                                           int H_, int G, F finish)
{
    constexpr int CPT = head_cols(HT);
    const int H = HT ? HT : H_;
    const int slices = (H + kBlock - 1) / kBlock, cols = H / CPT;
    const int sets = head_sets_together(H) ? 3 : 1;
    const int tid = threadIdx.x, groups = kHeadThreads / cols, grp = tid / cols, j = (tid - grp * cols) * CPT;
    for (int set0 = 0; set0 < 3; set0 += sets)
        for (int r0 = 0; r0 < G; r0 += RT) {
            const int rows = min(RT, G - r0);
            for (int u = grp; u < sets * slices && grp < groups; u += groups) {
                const int set = set0 + u / slices, k0 = (u - (u / slices) * slices) * kBlock;
                const float *W = blob + w0 + static_cast<ptrdiff_t>(set) * ws + static_cast<size_t>(k0) * H + j;
                const int kn = min(kBlock, H - k0);
                float w[kBlock][CPT];
#pragma unroll
                for (int k = 0; k < kBlock; ++k) {
                    if constexpr (CPT == 4) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(W + static_cast<size_t>(k) * H);
#pragma unroll
                        for (int c = 0; c < CPT; ++c) w[k][c] = v[c];
                    } else {
                        w[k][0] = k < kn ? W[static_cast<size_t>(k) * H] : 0.0f;
                    }
                }
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const float *xr = x + (set * G + r0 + min(r, rows - 1)) * H + k0;
                    float s[CPT];
#pragma unroll
                    for (int c = 0; c < CPT; ++c) s[c] = 0.0f;
#pragma unroll
                    for (int k = 0; k < kBlock; ++k) {
                        const float xv = (CPT == 4 || k < kn) ? xr[k] : 0.0f;
#pragma unroll
                        for (int c = 0; c < CPT; ++c) s[c] = fmaf(xv, w[k][c], s[c]);
                    }
#pragma unroll
                    for (int c = 0; c < CPT; ++c) part[(u * RT + r) * H + j + c] = s[c];
                }
            }
            __syncthreads();
            for (int i = tid; i < sets * rows * H; i += kHeadThreads) {
                const int sr = i / H, c = i - sr * H, q = sr / rows, r = sr - q * rows;
                double s = 0.0;
                for (int sl = 0; sl < slices; ++sl) s += static_cast<double>(part[((q * slices + sl) * RT + r) * H + c]);
                x[((set0 + q) * G + r0 + r) * H + c] = finish(set0 + q, r0 + r, c, s);
            }
            __syncthreads();
        }
}

struct HeadOut {
    float *zbuf;          // [B, Z] policy inputs
    double *hid;          // [B, H] hidden layer of the policy network
    float *logit;         // [B, D] logits, also where out_logits gets NaN
    float *out_logits, *out_probs, *out_pooled;
    float *hin, *hact;    // kept for the reverse pass (or null): inputs [3, B G, H] and layer outputs [3, L, B G, H] of h
};

template <int HT, int RT>
__global__ __launch_bounds__(kHeadThreads) void k_head(GraphView gv, ModelView mv, const float *__restrict__ emb,
                                                       const float *__restrict__ partial,
                                                       const int32_t *__restrict__ cur_node, int max_chunks, HeadOut o)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ double hid[kMaxH];
    __shared__ float logit[kMaxD];
    constexpr int CPT = head_cols(HT);
    const int H = HT ? HT : mv.H, G = mv.G, L = mv.L, D = mv.D, Z = mv.Z;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float *z = reinterpret_cast<float *>(lds);              // [Z]: e_{v*}, then the rows of the three sets
    float *part = z + ((Z + 3) & ~3), *x = z + 2 * H;
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int cl = cur_node[b];
    const bool cur_ok = cl >= 0 && cl < n_b;
    const int chunks = min((n_b + kPoolChunk - 1) / kPoolChunk, max_chunks);
    const size_t BG = static_cast<size_t>(gv.B) * G;
    // place of element i of a set's rows in the arrays kept for the reverse pass
    auto kept = [&](int set, int l, int layers, int i) {
        return ((static_cast<size_t>(set) * layers + l) * BG + static_cast<size_t>(b) * G) * H + i;
    };

    // ---- P[set][group] = sum of the pooling partials in slice order
    const float *src = partial + static_cast<size_t>(b) * max_chunks * 3 * G * H;
    for (int i = tid; i < 3 * G * H; i += kHeadThreads) {
        float s = 0.0f;
#pragma unroll 4
        for (int c = 0; c < chunks; ++c) s += src[static_cast<size_t>(c) * 3 * G * H + i];
        x[i] = s;
        if (o.out_pooled) o.out_pooled[static_cast<size_t>(b) * 3 * G * H + i] = s;
        if (o.hin) {
            const int set = i / (G * H);
            o.hin[kept(set, 0, 1, i - set * G * H)] = s;
        }
    }
    for (int i = tid; i < 2 * H; i += kHeadThreads) z[i] = cur_ok ? emb[static_cast<size_t>(n0 + cl) * 2 * H + i] : 0.0f;
    __syncthreads();

    // ---- h of the three sets
    for (int l = 0; l < L; ++l) {
        const LayerRef &l0 = mv.h[0].layer[l];
        const int ws = mv.h[1].layer[l].w - l0.w;
        head_layer<HT, RT>(mv.blob, l0.w, ws, x, part, H, G, [&](int set, int r, int c, double s) {
            const float y = fmaxf(static_cast<float>(s + static_cast<double>(mv.blob[l0.b + set * ws + c])), 0.0f);
            if (o.hact) o.hact[kept(set, l, L, r * H + c)] = y;
            return y;
        });
    }
    if (o.zbuf)
        for (int i = tid; i < Z; i += kHeadThreads) o.zbuf[static_cast<size_t>(b) * Z + i] = z[i];

    // ---- first policy layer: group g takes the blocks g, g + groups, ... of z
    {
        const int cols = H / CPT, groups = kHeadThreads / cols, grp = tid / cols, j = (tid - grp * cols) * CPT;
        const int blocks = (Z + kBlock - 1) / kBlock, used = min(groups, blocks);
        double *red = reinterpret_cast<double *>(part);     // [used][H]
        if (grp < used) {
            double acc[CPT];
#pragma unroll
            for (int c = 0; c < CPT; ++c) acc[c] = 0.0;
            const float *W1 = mv.blob + mv.pol1.w + j;
#pragma unroll 2
            for (int q = grp; q < blocks; q += groups) {
                const int k0 = q * kBlock;
                float w[kBlock][CPT], s[CPT];
#pragma unroll
                for (int k = 0; k < kBlock; ++k) {
                    if constexpr (CPT == 4) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(W1 + static_cast<size_t>(k0 + k) * H);
#pragma unroll
                        for (int c = 0; c < CPT; ++c) w[k][c] = v[c];
                    } else {
                        w[k][0] = k0 + k < Z ? W1[static_cast<size_t>(k0 + k) * H] : 0.0f;
                    }
                }
#pragma unroll
                for (int c = 0; c < CPT; ++c) s[c] = 0.0f;
#pragma unroll
                for (int k = 0; k < kBlock; ++k) {
                    const float xv = (CPT == 4 || k0 + k < Z) ? z[k0 + k] : 0.0f;
#pragma unroll
                    for (int c = 0; c < CPT; ++c) s[c] = fmaf(xv, w[k][c], s[c]);
                }
#pragma unroll
                for (int c = 0; c < CPT; ++c) acc[c] += static_cast<double>(s[c]);
            }
#pragma unroll
            for (int c = 0; c < CPT; ++c) red[grp * H + j + c] = acc[c];
        }
        __syncthreads();
        for (int c = tid; c < H; c += kHeadThreads) {
            double s = static_cast<double>(mv.blob[mv.pol1.b + c]);
            for (int g = 0; g < used; ++g) s += red[g * H + c];
            hid[c] = s > 0.0 ? s : 0.0;
            o.hid[static_cast<size_t>(b) * H + c] = hid[c];
        }
    }
    __syncthreads();

    // ---- output layer (a wave per device), softmax
    for (int d = wave; d < D; d += kHeadThreads / 64) {
        double s = 0.0;
        for (int k = lane; k < H; k += 64) s = fma(hid[k], static_cast<double>(mv.blob[mv.pol2.w + k * D + d]), s);
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) s += __shfl_xor(s, step);
        if (lane == 0) logit[d] = static_cast<float>(s + static_cast<double>(mv.blob[mv.pol2.b + d]));
    }
    __syncthreads();
    if (tid < D) {
        const float bad = __builtin_nanf("");               // no valid current node: nothing to decide
        const size_t at = static_cast<size_t>(b) * D + tid;
        o.logit[at] = logit[tid];
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
template <int HT, int RT>
__global__ __launch_bounds__(kHeadThreads) void k_head_bw(GraphView gv, ModelView mv, const float *__restrict__ blob_t,
                                                          const int32_t *__restrict__ cur_node, HeadBwArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float dpre[kMaxH];
    __shared__ float dlog[kMaxD];
    const int H = HT ? HT : mv.H, G = mv.G, L = mv.L, D = mv.D, Z = mv.Z;
    const int b = blockIdx.x, tid = threadIdx.x;
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
    for (int j = tid; j < H; j += kHeadThreads) {
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
        for (int k = tid; k < Z; k += kHeadThreads) {
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
        head_layer<HT, RT>(blob_t, l0.w, mv.h[1].layer[l].w - l0.w, x, part, H, G, [&](int set, int r, int c, double s) {
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

// Calls run(kernel, dynamic LDS bytes) with the instantiation for width H and G rows per set.
template <typename Pick, typename Run>
void head_dispatch(int H, int G, Pick pick, Run run)
{
    const int most = head_rows_max(H);
    auto rows = [&](auto ht) {
        constexpr int HT = decltype(ht)::value;
        auto go = [&](auto rt) { run(pick(ht, rt), head_lds(H, G, decltype(rt)::value, HT)); };
        if (G == 1) go(std::integral_constant<int, 1>{});
        else if (G <= 4 || most == 4) go(std::integral_constant<int, 4>{});
        else go(std::integral_constant<int, 8>{});
    };
    if (H == 128) rows(std::integral_constant<int, 128>{});
    else if (H == 64) rows(std::integral_constant<int, 64>{});
    else if (H == 32) rows(std::integral_constant<int, 32>{});
    else rows(std::integral_constant<int, 0>{});
}

template <typename K>
void allow_lds(K kernel, size_t bytes)
{
    if (bytes > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(bytes));
}

}  // namespace

void launch_head(const GraphView &gv, const ModelView &mv, const Workspace &ws, const ForwardArgs &fa, int max_chunks,
                 hipStream_t s)
{
    if (gv.B == 0) return;
    const HeadOut o{ws.zbuf, ws.hid, ws.logit, fa.out_logits, fa.out_probs, fa.out_pooled, fa.keep_hin, fa.keep_hact};
    head_dispatch(
        mv.H, mv.G, [](auto ht, auto rt) { return k_head<decltype(ht)::value, decltype(rt)::value>; },
        [&](auto kernel, size_t lds) {
            allow_lds(kernel, lds);
            hipLaunchKernelGGL(kernel, dim3(gv.B), dim3(kHeadThreads), lds, s, gv, mv, ws.emb, ws.partial, fa.cur_node,
                               max_chunks, o);
        });
}

void launch_head_bw(const GraphView &gv, const ModelView &mv, const float *blob_t, const int32_t *cur_node,
                    const HeadBwArgs &a, hipStream_t s)
{
    if (gv.B == 0) return;
    head_dispatch(
        mv.H, mv.G, [](auto ht, auto rt) { return k_head_bw<decltype(ht)::value, decltype(rt)::value>; },
        [&](auto kernel, size_t lds) {
            allow_lds(kernel, lds);
            hipLaunchKernelGGL(kernel, dim3(gv.B), dim3(kHeadThreads), lds, s, gv, mv, blob_t, cur_node, a);
        });
}

}  // namespace pl
