// Reverse-mode pass of the policy network: the gradient of log pi(a | s) with respect to every
// parameter, summed over a batch with one scalar per state.  This is the term
// grad_theta log pi_theta(a_i | s_i) * (return - baseline) of the REINFORCE update (appendix
// "REINFORCE Algorithm", Eq. 1) for the network of Section 2.2 / Appendix A.7.
//
// The forward pass leaves the node embeddings e_v = [td_v ; bu_v], the pooled sums and the
// policy inputs in the batch's buffers.  From them:
//   1. head:   d logits = c (one-hot(a) - pi); back through the policy layers and h_i to the
//              pooled sums P[i][d] and to e_{v*};
//   2. pool:   every node u of set i on device d receives dP[i][d]; back through l_i to e_u;
//   3. sweeps: activations of f and g are recomputed for all nodes at once (they depend only
//              on the final states), then one workgroup per (graph, direction) walks the levels
//              in REVERSE order: a node's state gradient needs the gradients of all the sums it
//              was gathered into, which belong to later levels;
//   4. projection: both directions start from x_v, so its gradient is the sum of the two;
//   5. every weight gradient is a contraction over rows (nodes, pooled groups or graphs) of
//              layer input x layer delta, done in slabs with a fixed summation order (no
//              atomics).
// Two sets of kernels: generic fp32 vector kernels for any H <= 256, D <= 16, 1..4 layers; and,
// for H in {32, 64, 128}, the parallel parts (per-node layers, weight gradients) on the fp32
// matrix cores (v_mfma_f32_32x32x2_f32) and the dependent chain of step 3 in the matrix-core sweep
// kernel run in reverse.  Several sweeps are differentiated from the last to the first.
#include <algorithm>

#include "internal.h"

namespace pl {

namespace {

constexpr int kThreads = 256;
constexpr int kTile = 16;      // rows pushed through a layer together
constexpr int kWgI = 16;       // weight-matrix rows per workgroup of the contraction kernel
constexpr int kWgRB = 32;      // contraction rows staged at a time
constexpr int kPoolSub = 256;  // nodes classified at a time

// y[r][j] = bias[j] + sum_k x[r][k] * W[k * ldw + j] for r < rows (<= kTile), j < n_out, optional
// ReLU.  x and y in LDS.  Thread (grp, j) owns rows grp, grp + groups, ...  Requires
// n_out <= kThreads and min(kThreads / n_out, kTile) * RPT >= rows.  bias may be null.
template <int RPT>
__device__ __forceinline__ void dense_rows(const float *__restrict__ W, int ldw,
                                           const float *__restrict__ bias, int n_in, int n_out,
                                           const float *x, int ldx, float *y, int ldy, int rows,
                                           bool relu)
{
    const int tid = threadIdx.x;
    int groups = kThreads / n_out;
    if (groups > kTile) groups = kTile;
    const int grp = tid / n_out, j = tid - grp * n_out;
    if (grp >= groups || grp >= rows) return;
    float acc[RPT];
    const float bj = bias ? bias[j] : 0.0f;
#pragma unroll
    for (int i = 0; i < RPT; ++i) acc[i] = bj;
    int xoff[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) xoff[i] = min(grp + i * groups, rows - 1) * ldx;
    constexpr int KB = 16;
    int k = 0;
    for (; k + KB <= n_in; k += KB) {
        float w[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) w[u] = W[static_cast<size_t>(k + u) * ldw + j];
#pragma unroll
        for (int u = 0; u < KB; ++u)
#pragma unroll
            for (int i = 0; i < RPT; ++i) acc[i] = fmaf(x[xoff[i] + k + u], w[u], acc[i]);
    }
    for (; k < n_in; ++k) {
        const float w = W[static_cast<size_t>(k) * ldw + j];
#pragma unroll
        for (int i = 0; i < RPT; ++i) acc[i] = fmaf(x[xoff[i] + k], w, acc[i]);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = grp + i * groups;
        if (r < rows) y[r * ldy + j] = relu ? fmaxf(acc[i], 0.0f) : acc[i];
    }
}

// Position of activation / delta array (dir, layer) inside a [2][L][n_tot][H] buffer.
__device__ __forceinline__ size_t slab(int dir, int l, int L, int n_tot, int H)
{
    return (static_cast<size_t>(dir) * L + l) * static_cast<size_t>(n_tot) * H;
}

// Section 2.2 step 3: 0 = v*, 1 = can reach v*, 2 = reachable from v*, 3 = neither.
__device__ __forceinline__ int node_class_bw(int v, int cur, const uint8_t *reach, int n_tot, int single)
{
    if (v == cur) return 0;
    if (single) return 1;                  // every node other than v* is in the first set
    if (reach[static_cast<size_t>(n_tot) + v]) return 1;
    if (reach[v]) return 2;
    return 3;
}

// ------------------------------------------------------------------ 2. pooling
// Workgroup (chunk, graph) over a contiguous slice of the graph's nodes, bucketed by set as in
// the forward pass.  A tile of nodes of one set goes forward through l_set (outputs kept in
// lact), takes dP[set][device] as the gradient of its last output, and goes back to d e_u.
// The current node takes its gradient from the policy input; a node with a device id outside
// [0, D) was pooled nowhere and gets zero.
template <int RPT>
__global__ __launch_bounds__(kThreads) void k_bw_pool(GraphView gv, ModelView mv,
                                                      const float *__restrict__ blob_t,
                                                      const float *__restrict__ emb,
                                                      const uint8_t *__restrict__ reach,
                                                      const int32_t *__restrict__ placement,
                                                      const int32_t *__restrict__ cur_node,
                                                      const float *__restrict__ dP,
                                                      const float *__restrict__ dz,
                                                      uint8_t *__restrict__ cls_out,
                                                      float *__restrict__ lact,
                                                      float *__restrict__ dl,
                                                      float *__restrict__ demb, int max_chunks)
{
    extern __shared__ float lds[];
    __shared__ int16_t s_list[3][kPoolSub];
    __shared__ int8_t s_cls[kPoolSub];
    __shared__ int s_count[3];
    __shared__ int s_dev[kTile];
    __shared__ int s_node[kTile];
    const int H = mv.H, G = mv.G, D = mv.D, L = mv.L, Z = mv.Z;
    const int b = blockIdx.y, c = blockIdx.x, tid = threadIdx.x;
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    int chunks = (n_b + kPoolChunk - 1) / kPoolChunk;
    if (chunks > max_chunks) chunks = max_chunks;
    if (c >= chunks) return;
    const int per = (n_b + chunks - 1) / chunks;
    const int lo = n0 + c * per, hi = min(n0 + n_b, lo + per);
    const int cl = cur_node[b];
    const int cur = (cl >= 0 && cl < n_b) ? n0 + cl : -1;
    const size_t NH = static_cast<size_t>(gv.n_tot) * H;

    float *buf_x = lds;                    // [kTile][2H]
    float *buf_a = buf_x + kTile * 2 * H;  // [kTile][H]
    float *buf_b = buf_a + kTile * H;      // [kTile][H]

    for (int s0 = lo; s0 < hi; s0 += kPoolSub) {
        const int cnt = min(kPoolSub, hi - s0);
        if (tid < cnt) {
            const int k = node_class_bw(s0 + tid, cur, reach, gv.n_tot, mv.single_set);
            s_cls[tid] = static_cast<int8_t>(k);
            cls_out[s0 + tid] = static_cast<uint8_t>(k);
        }
        __syncthreads();
        if (tid < 3) {
            int m = 0;
            for (int i = 0; i < cnt; ++i)
                if (s_cls[i] == tid + 1) s_list[tid][m++] = static_cast<int16_t>(i);
            s_count[tid] = m;
        }
        // the current node: d e = first 2H entries of dz; its l rows are never used
        if (cur >= s0 && cur < s0 + cnt)
            for (int i = tid; i < 2 * H; i += kThreads)
                demb[static_cast<size_t>(cur) * 2 * H + i] = dz[static_cast<size_t>(b) * Z + i];
        __syncthreads();
        for (int set = 0; set < 3; ++set) {
            const int m = s_count[set];
            const MlpRef &ln = mv.l[set];
            for (int t0 = 0; t0 < m; t0 += kTile) {
                const int rows = min(kTile, m - t0);
                for (int i = tid; i < rows * 2 * H; i += kThreads) {
                    const int r = i / (2 * H), k = i - r * 2 * H;
                    buf_x[i] = emb[static_cast<size_t>(s0 + s_list[set][t0 + r]) * 2 * H + k];
                }
                if (tid < rows) {
                    const int v = s0 + s_list[set][t0 + tid];
                    const int dev = placement[v];
                    s_node[tid] = v;
                    s_dev[tid] = (dev >= 0 && dev < D) ? (G == 1 ? 0 : dev) : -1;
                }
                __syncthreads();
                // forward through l_set, every layer's output kept
                const float *in = buf_x;
                int n_in = 2 * H;
                float *out = buf_a;
                for (int l = 0; l < L; ++l) {
                    dense_rows<RPT>(mv.blob + ln.layer[l].w, H, mv.blob + ln.layer[l].b, n_in, H, in, n_in,
                                    out, H, rows, true);
                    __syncthreads();
                    for (int i = tid; i < rows * H; i += kThreads) {
                        const int r = i / H, h = i - r * H;
                        lact[static_cast<size_t>(l) * NH + static_cast<size_t>(s_node[r]) * H + h] = out[i];
                    }
                    in = out;
                    n_in = H;
                    out = (out == buf_a) ? buf_b : buf_a;
                }
                // `in` holds the last layer's output; delta of the last layer into `out`
                float *dcur = out, *dnext = const_cast<float *>(in);
                for (int i = tid; i < rows * H; i += kThreads) {
                    const int r = i / H, h = i - r * H;
                    const int dev = s_dev[r];
                    const float g = dev >= 0 ? dP[((static_cast<size_t>(b) * 3 + set) * G + dev) * H + h] : 0.0f;
                    dcur[i] = in[i] > 0.0f ? g : 0.0f;
                }
                __threadfence_block();
                __syncthreads();
                for (int l = L - 1; l >= 0; --l) {
                    for (int i = tid; i < rows * H; i += kThreads) {
                        const int r = i / H, h = i - r * H;
                        dl[static_cast<size_t>(l) * NH + static_cast<size_t>(s_node[r]) * H + h] = dcur[i];
                    }
                    if (l > 0) {
                        dense_rows<RPT>(blob_t + ln.layer[l].w, H, nullptr, H, H, dcur, H, dnext, H, rows, false);
                        __syncthreads();
                        for (int i = tid; i < rows * H; i += kThreads) {
                            const int r = i / H, h = i - r * H;
                            const float a = lact[static_cast<size_t>(l - 1) * NH + static_cast<size_t>(s_node[r]) * H + h];
                            dnext[i] = a > 0.0f ? dnext[i] : 0.0f;
                        }
                        __syncthreads();
                        float *t = dcur; dcur = dnext; dnext = t;
                    } else {
                        // first layer: [2H, H] stored transposed as [H][2H]; the two halves of d e
                        dense_rows<RPT>(blob_t + ln.layer[0].w, 2 * H, nullptr, H, H, dcur, H, buf_x, 2 * H, rows, false);
                        dense_rows<RPT>(blob_t + ln.layer[0].w + H, 2 * H, nullptr, H, H, dcur, H, buf_x + H, 2 * H, rows, false);
                        __syncthreads();
                        for (int i = tid; i < rows * 2 * H; i += kThreads) {
                            const int r = i / (2 * H), k = i - r * 2 * H;
                            demb[static_cast<size_t>(s_node[r]) * 2 * H + k] = buf_x[i];
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
}

// ------------------------------------------------------------------ 3. sweeps
// (a) f at the final state of every node: tile of 16 nodes x direction.
template <int RPT>
__global__ __launch_bounds__(kThreads) void k_bw_f_acts(GraphView gv, ModelView mv,
                                                        const float *__restrict__ emb,
                                                        float *__restrict__ fact)
{
    extern __shared__ float lds[];
    const int H = mv.H, L = mv.L, tid = threadIdx.x, dir = blockIdx.y;
    const int v0 = blockIdx.x * kTile, rows = min(kTile, gv.n_tot - v0);
    float *buf_a = lds, *buf_b = lds + kTile * H;
    for (int i = tid; i < rows * H; i += kThreads) {
        const int r = i / H, h = i - r * H;
        buf_a[i] = emb[static_cast<size_t>(v0 + r) * 2 * H + dir * H + h];
    }
    __syncthreads();
    float *in = buf_a, *out = buf_b;
    for (int l = 0; l < L; ++l) {
        const LayerRef &ly = mv.f[dir].layer[l];
        dense_rows<RPT>(mv.blob + ly.w, H, mv.blob + ly.b, H, H, in, H, out, H, rows, true);
        __syncthreads();
        float *dst = fact + slab(dir, l, L, gv.n_tot, H) + static_cast<size_t>(v0) * H;
        for (int i = tid; i < rows * H; i += kThreads) dst[i] = out[i];
        float *t = in; in = out; out = t;
    }
}

// (b) the gathered sums a_v = sum of the neighbours' messages, and g at them.
template <int RPT>
__global__ __launch_bounds__(kThreads) void k_bw_g_acts(GraphView gv, ModelView mv,
                                                        const float *__restrict__ fact,
                                                        float *__restrict__ agg,
                                                        float *__restrict__ gact)
{
    extern __shared__ float lds[];
    const int H = mv.H, L = mv.L, tid = threadIdx.x, dir = blockIdx.y;
    const int v0 = blockIdx.x * kTile, rows = min(kTile, gv.n_tot - v0);
    float *buf_a = lds, *buf_b = lds + kTile * H;
    const float *msg = fact + slab(dir, L - 1, L, gv.n_tot, H);
    const int32_t *nbr_ptr = gv.nbr_ptr[dir], *nbr_idx = gv.nbr_idx[dir];
    for (int i = tid; i < rows * H; i += kThreads) {
        const int r = i / H, h = i - r * H;
        const int v = v0 + r;
        float a = 0.0f;
        for (int p = nbr_ptr[v]; p < nbr_ptr[v + 1]; ++p) a += msg[static_cast<size_t>(nbr_idx[p]) * H + h];
        buf_a[i] = a;
        agg[(static_cast<size_t>(dir) * gv.n_tot + v) * H + h] = a;
    }
    __syncthreads();
    float *in = buf_a, *out = buf_b;
    for (int l = 0; l < L; ++l) {
        const LayerRef &ly = mv.g[dir].layer[l];
        dense_rows<RPT>(mv.blob + ly.w, H, mv.blob + ly.b, H, H, in, H, out, H, rows, true);
        __syncthreads();
        float *dst = gact + slab(dir, l, L, gv.n_tot, H) + static_cast<size_t>(v0) * H;
        for (int i = tid; i < rows * H; i += kThreads) dst[i] = out[i];
        float *t = in; in = out; out = t;
    }
}

// (c) the dependent chain.  s_v <- s_v + g(a_v), m_v = f(s_v), a_w = sum of m over xi(w).
// With dE/ds_v given from outside (pooling, head) in demb, for v in reverse level order:
//   dm_v   = sum over the nodes w that gathered m_v (v's neighbours in the OTHER direction) of da_w
//   ds_v  += f'(s_v)^T dm_v          (back through the layers of f)
//   da_v   = g'(a_v)^T ds_v          (back through the layers of g)
// demb becomes the gradient of the sweep's input (the residual passes ds_v through unchanged).
template <int RPT>
__global__ __launch_bounds__(kThreads) void k_bw_sweep_generic(GraphView gv, ModelView mv,
                                                               const float *__restrict__ blob_t,
                                                               const float *__restrict__ fact,
                                                               const float *__restrict__ gact,
                                                               float *__restrict__ demb,
                                                               float *__restrict__ dagg_base,
                                                               float *__restrict__ dfg, size_t dfg_stride)
{
    extern __shared__ float lds[];
    const int H = mv.H, L = mv.L;
    const int b = blockIdx.x, dir = blockIdx.y, tid = threadIdx.x;
    float *buf_a = lds, *buf_b = lds + kTile * H;
    float *dagg = dagg_base + static_cast<size_t>(dir) * gv.n_tot * H;
    const int32_t *order = gv.order[dir];
    const int32_t *suc_ptr = gv.nbr_ptr[1 - dir], *suc_idx = gv.nbr_idx[1 - dir];
    const int32_t *lvl = gv.lvl_ptr[dir] + gv.lvl_off[b];
    const int depth = gv.lvl_off[b + 1] - gv.lvl_off[b] - 1;
    const MlpRef &fn = mv.f[dir], &gn = mv.g[dir];
    const size_t NH = static_cast<size_t>(gv.n_tot) * H;
    float *df = dfg + dir * dfg_stride, *dg = df + L * NH;

    for (int level = depth - 1; level >= 0; --level) {
        const int beg = lvl[level], end = lvl[level + 1];
        for (int t0 = beg; t0 < end; t0 += kTile) {
            const int rows = min(kTile, end - t0);
            // dm_v, masked by the last layer of f
            for (int i = tid; i < rows * H; i += kThreads) {
                const int r = i / H, h = i - r * H;
                const int v = order[t0 + r];
                float a = 0.0f;
                for (int p = suc_ptr[v]; p < suc_ptr[v + 1]; ++p)
                    a += dagg[static_cast<size_t>(suc_idx[p]) * H + h];
                const float m = fact[slab(dir, L - 1, L, gv.n_tot, H) + static_cast<size_t>(v) * H + h];
                buf_a[i] = m > 0.0f ? a : 0.0f;
            }
            __syncthreads();
            float *dcur = buf_a, *dnext = buf_b;
            for (int l = L - 1; l >= 0; --l) {
                for (int i = tid; i < rows * H; i += kThreads) {
                    const int r = i / H, h = i - r * H;
                    df[l * NH + static_cast<size_t>(order[t0 + r]) * H + h] = dcur[i];
                }
                dense_rows<RPT>(blob_t + fn.layer[l].w, H, nullptr, H, H, dcur, H, dnext, H, rows, false);
                __syncthreads();
                if (l > 0) {
                    for (int i = tid; i < rows * H; i += kThreads) {
                        const int r = i / H, h = i - r * H;
                        const float a = fact[slab(dir, l - 1, L, gv.n_tot, H) + static_cast<size_t>(order[t0 + r]) * H + h];
                        dnext[i] = a > 0.0f ? dnext[i] : 0.0f;
                    }
                    __syncthreads();
                }
                float *t = dcur; dcur = dnext; dnext = t;
            }
            // ds_v = outside gradient + f-path; then the delta of g's last layer
            for (int i = tid; i < rows * H; i += kThreads) {
                const int r = i / H, h = i - r * H;
                const int v = order[t0 + r];
                const size_t at = static_cast<size_t>(v) * 2 * H + dir * H + h;
                const float ds = demb[at] + dcur[i];
                demb[at] = ds;
                const float u = gact[slab(dir, L - 1, L, gv.n_tot, H) + static_cast<size_t>(v) * H + h];
                dcur[i] = u > 0.0f ? ds : 0.0f;
            }
            __syncthreads();
            for (int l = L - 1; l >= 0; --l) {
                for (int i = tid; i < rows * H; i += kThreads) {
                    const int r = i / H, h = i - r * H;
                    dg[l * NH + static_cast<size_t>(order[t0 + r]) * H + h] = dcur[i];
                }
                dense_rows<RPT>(blob_t + gn.layer[l].w, H, nullptr, H, H, dcur, H, dnext, H, rows, false);
                __syncthreads();
                if (l > 0) {
                    for (int i = tid; i < rows * H; i += kThreads) {
                        const int r = i / H, h = i - r * H;
                        const float a = gact[slab(dir, l - 1, L, gv.n_tot, H) + static_cast<size_t>(order[t0 + r]) * H + h];
                        dnext[i] = a > 0.0f ? dnext[i] : 0.0f;
                    }
                    __syncthreads();
                }
                float *t = dcur; dcur = dnext; dnext = t;
            }
            for (int i = tid; i < rows * H; i += kThreads) {
                const int r = i / H, h = i - r * H;
                dagg[static_cast<size_t>(order[t0 + r]) * H + h] = dcur[i];
            }
            __syncthreads();
        }
        // da of this level is read by earlier levels of this same workgroup
        __threadfence_block();
        __syncthreads();
    }
}

// (d) inputs of the matrix-core chain kernel, in the bucket order of the direction whose chunks
// it walks (pd; the sweep being differentiated is sd = 1 - pd): the outside gradient of s_v and
// the ReLU gates of the node's layers, one byte per (node, column): bit 0 m_v > 0, bit 1 output
// of f's layer 0 > 0 (L = 2), bit 2 output of g's last layer > 0, bit 3 output of g's layer 0 > 0
// (L = 2).
struct GateSrc {
    const float *m;        // [n_tot, H] messages (output of f's last layer)
    const float *f0;       // output of f's layer 0 (L = 2)
    const float *g_last;   // output of g's last layer
    const float *g0;       // output of g's layer 0 (L = 2)
};

__global__ __launch_bounds__(kThreads) void k_bw_gates(GraphView gv, int H, int L, GateSrc src0, GateSrc src1,
                                                       uint8_t *__restrict__ mask4)
{
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (idx >= static_cast<size_t>(gv.n_tot) * H) return;
    for (int sd = 0; sd < 2; ++sd) {
        const GateSrc &gs = sd ? src1 : src0;
        int bits = fabsf(gs.m[idx]) > 0.0f ? 1 : 0;     // messages may carry a flag in their sign bit
        bits |= gs.g_last[idx] > 0.0f ? 4 : 0;
        if (L == 2) {
            bits |= gs.f0[idx] > 0.0f ? 2 : 0;
            bits |= gs.g0[idx] > 0.0f ? 8 : 0;
        }
        mask4[static_cast<size_t>(sd) * gv.n_tot * H + idx] = static_cast<uint8_t>(bits);
    }
}

// ------------------------------------------------------------------ 4. projection
// x_v = relu(W^T phi_v + b) feeds both directions: dx_v = (ds_td + ds_bu) masked by x_v > 0.
// Also writes phi_v, the input rows of the projection's weight gradient.
__global__ __launch_bounds__(kThreads) void k_bw_proj(GraphView gv, ModelView mv,
                                                      const float *__restrict__ feats,
                                                      const int32_t *__restrict__ placement,
                                                      const int32_t *__restrict__ cur_node,
                                                      const float *__restrict__ demb,
                                                      float *__restrict__ dx,
                                                      float *__restrict__ phi, int phi_ld)
{
    const int H = mv.H, D = mv.D;
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (idx >= static_cast<size_t>(gv.n_tot) * H) return;
    const int v = static_cast<int>(idx / H), h = static_cast<int>(idx - static_cast<size_t>(v) * H);
    const int b = gv.node_graph[v];
    const float *W = mv.blob + mv.proj.w;
    float s = mv.blob[mv.proj.b + h];
    s = fmaf(feats[v * 3 + 0], W[0 * H + h], s);
    s = fmaf(feats[v * 3 + 1], W[1 * H + h], s);
    const int dev = placement[v];
    if (dev >= 0 && dev < D) s += W[(2 + dev) * H + h];
    const bool is_cur = v - gv.node_off[b] == cur_node[b];
    if (is_cur) s += W[(2 + D) * H + h];
    s = fmaf(feats[v * 3 + 2], W[(3 + D) * H + h], s);
    const float g = demb[static_cast<size_t>(v) * 2 * H + h] + demb[static_cast<size_t>(v) * 2 * H + H + h];
    dx[idx] = s > 0.0f ? g : 0.0f;
    if (h < phi_ld) {                       // phi_ld >= F: columns past F are zero
        float p;
        if (h == 0) p = feats[v * 3 + 0];
        else if (h == 1) p = feats[v * 3 + 1];
        else if (h < 2 + D) p = (dev == h - 2) ? 1.0f : 0.0f;
        else if (h == 2 + D) p = is_cur ? 1.0f : 0.0f;
        else if (h == 3 + D) p = feats[v * 3 + 2];
        else p = 0.0f;
        phi[static_cast<size_t>(v) * phi_ld + h] = p;
    }
}

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4p;

// The same with four columns per thread, for H a multiple of four (vector loads and stores; the
// per-node values are read once per four columns; 300 layered graphs, H = 64, 16 devices: 22 us with k_bw_proj, 14).  The
// sum takes its terms in the order of k_bw_proj, which is the forward pass's.
__global__ __launch_bounds__(kThreads) void k_bw_proj_rows(GraphView gv, ModelView mv,
                                                           const float *__restrict__ feats,
                                                           const int32_t *__restrict__ placement,
                                                           const int32_t *__restrict__ cur_node,
                                                           const float *__restrict__ demb,
                                                           float *__restrict__ dx,
                                                           float *__restrict__ phi, int phi_ld)
{
    const int H = mv.H, D = mv.D, q = H / 4;
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (idx >= static_cast<size_t>(gv.n_tot) * q) return;
    const int v = static_cast<int>(idx / q), h = 4 * static_cast<int>(idx - static_cast<size_t>(v) * q);
    const int b = gv.node_graph[v];
    const float *W = mv.blob + mv.proj.w;
    auto row = [&](int r) { return *reinterpret_cast<const f32x4p *>(W + static_cast<size_t>(r) * H + h); };
    const float f_time = feats[v * 3 + 0], f_size = feats[v * 3 + 1], f_vis = feats[v * 3 + 2];
    const int dev = placement[v];
    const bool on_dev = dev >= 0 && dev < D;
    const bool is_cur = v - gv.node_off[b] == cur_node[b];
    const f32x4p bias = *reinterpret_cast<const f32x4p *>(mv.blob + mv.proj.b + h);
    const f32x4p w0 = row(0), w1 = row(1), wd = row(2 + (on_dev ? dev : 0)), wc = row(2 + D), wv = row(3 + D);
    const float *de = demb + static_cast<size_t>(v) * 2 * H + h;
    const f32x4p g0 = *reinterpret_cast<const f32x4p *>(de), g1 = *reinterpret_cast<const f32x4p *>(de + H);
    f32x4p out;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float s = bias[k];
        s = fmaf(f_time, w0[k], s);
        s = fmaf(f_size, w1[k], s);
        if (on_dev) s += wd[k];
        if (is_cur) s += wc[k];
        s = fmaf(f_vis, wv[k], s);
        out[k] = s > 0.0f ? g0[k] + g1[k] : 0.0f;
    }
    *reinterpret_cast<f32x4p *>(dx + static_cast<size_t>(v) * H + h) = out;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int c = h + k;
        if (c < phi_ld) {                   // phi_ld >= F: columns past F are zero
            float p;
            if (c == 0) p = f_time;
            else if (c == 1) p = f_size;
            else if (c < 2 + D) p = (dev == c - 2) ? 1.0f : 0.0f;
            else if (c == 2 + D) p = is_cur ? 1.0f : 0.0f;
            else if (c == 3 + D) p = f_vis;
            else p = 0.0f;
            phi[static_cast<size_t>(v) * phi_ld + c] = p;
        }
    }
}

// Gradient of the input projection, H a multiple of four, large batches: per slab of nodes, phi^T dx and the column sums of dx, with
// dx_v = (de_td + de_bu) [x_v > 0] formed on the way; neither dx nor phi exists in memory.  One read of d e bounds it (819 MB
// of 256 NASNet-like graphs).  A thread takes four columns of every so manieth node of the slab.  A row of phi is three
// numbers and two ones, so a node is five multiply-adds a column; its device's row of the sum is picked by comparison,
// with five to eight devices in LDS (a thread's own entries: a read and a write instead of sixteen instructions a column,
// 351 -> 160 us).  The pre-activation takes its terms in the forward pass's order.  Sums: a thread's nodes in order, the
// threads of a column in a fixed order, then the slabs (k_wgrad_reduce).  proj_fused says from which size on.
template <int DM>                              // most devices
__global__ __launch_bounds__(kThreads) void k_bw_proj4(GraphView gv, ModelView mv,
                                                       const float *__restrict__ feats,
                                                       const int32_t *__restrict__ placement,
                                                       const int32_t *__restrict__ cur_node,
                                                       const float *__restrict__ demb, int rows_per_slab,
                                                       float *__restrict__ partial)
{
    constexpr bool kLds = DM == 8;             // (of sixteen they would not fit)
    constexpr int DR = kLds ? 0 : DM;
    __shared__ f32x4p red[2][kThreads];
    __shared__ f32x4p w_dev[(DM + 1) * (kMaxH / 4)];      // one-hot device rows of W_in, then a row of zeros
    __shared__ f32x4p s_dev[kLds ? DM * kThreads : 1];
    const int H = mv.H, D = mv.D, q = H / 4, groups = kThreads / q;
    const int tid = threadIdx.x, grp = tid / q, c = tid - grp * q, h = 4 * c;
    const int r_beg = blockIdx.x * rows_per_slab, r_end = min(gv.n_tot, r_beg + rows_per_slab);
    const float *W = mv.blob + mv.proj.w;
    const f32x4p zero{0.f, 0.f, 0.f, 0.f};
    auto row = [&](int r) { return *reinterpret_cast<const f32x4p *>(W + static_cast<size_t>(r) * H + h); };
    for (int i = tid; i < (DM + 1) * q; i += kThreads)
        w_dev[i] = i < D * q ? *reinterpret_cast<const f32x4p *>(W + 2 * static_cast<size_t>(H) + 4 * i) : zero;
    if constexpr (kLds)
        for (int d = 0; d < DM; ++d) s_dev[d * kThreads + tid] = zero;
    __syncthreads();
    f32x4p s_time = zero, s_size = zero, s_cur = zero, s_vis = zero, s_one = zero, s_reg[DR + 1];
#pragma unroll
    for (int d = 0; d <= DR; ++d) s_reg[d] = zero;
    if (grp < groups) {
        const f32x4p bias = *reinterpret_cast<const f32x4p *>(mv.blob + mv.proj.b + h);
        const f32x4p w0 = row(0), w1 = row(1), wc = row(2 + D), wv = row(3 + D);
        struct Node {
            float time, size, vis;
            int dev;
            f32x4p g0, g1;
        };
        auto load = [&](int v) __attribute__((always_inline)) {
            Node x;
            x.time = feats[v * 3 + 0];
            x.size = feats[v * 3 + 1];
            x.vis = feats[v * 3 + 2];
            x.dev = placement[v];
            const float *de = demb + static_cast<size_t>(v) * 2 * H + h;
            x.g0 = *reinterpret_cast<const f32x4p *>(de);
            x.g1 = *reinterpret_cast<const f32x4p *>(de + H);
            return x;
        };
        int cur = -1, graph_end = -1;          // of the graph that the last node was in
        auto take = [&](int v, const Node &x) __attribute__((always_inline)) {
            if (v >= graph_end) {
                const int b = gv.node_graph[v], n0 = gv.node_off[b], cl = cur_node[b];
                graph_end = gv.node_off[b + 1];
                cur = cl >= 0 && cl < graph_end - n0 ? n0 + cl : -1;
            }
            const bool on_dev = x.dev >= 0 && x.dev < D, is_cur = v == cur;
            const f32x4p wd = w_dev[(on_dev ? x.dev : DM) * q + c];
            f32x4p dx;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float s = bias[k];
                s = fmaf(x.time, w0[k], s);
                s = fmaf(x.size, w1[k], s);
                s += wd[k];
                s += is_cur ? wc[k] : 0.0f;
                s = fmaf(x.vis, wv[k], s);
                dx[k] = s > 0.0f ? x.g0[k] + x.g1[k] : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s_time[k] = fmaf(x.time, dx[k], s_time[k]);
                s_size[k] = fmaf(x.size, dx[k], s_size[k]);
                s_vis[k] = fmaf(x.vis, dx[k], s_vis[k]);
                s_one[k] += dx[k];
                s_cur[k] += is_cur ? dx[k] : 0.0f;
#pragma unroll
                for (int d = 0; d < DR; ++d) s_reg[d][k] += x.dev == d ? dx[k] : 0.0f;
            }
            if constexpr (kLds) {
                const int at = (on_dev ? x.dev : 0) * kThreads + tid;
                f32x4p t = s_dev[at];
#pragma unroll
                for (int k = 0; k < 4; ++k) t[k] += on_dev ? dx[k] : 0.0f;
                s_dev[at] = t;
            }
        };
        int v = r_beg + grp;
        for (; v + 3 * groups < r_end; v += 4 * groups) {
            Node x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = load(v + u * groups);
#pragma unroll
            for (int u = 0; u < 4; ++u) take(v + u * groups, x[u]);
        }
        for (; v < r_end; v += groups) take(v, load(v));
    }
    // the threads of a column: those of a wave by shuffles where a wave holds whole groups, the rest through LDS
    const bool whole = 64 % q == 0;
    const int terms = whole ? kThreads / 64 : groups, step = whole ? 64 : q;
    float *dst = partial + static_cast<size_t>(blockIdx.x) * static_cast<size_t>(mv.F + 1) * H + h;
    int turn = 0;
    auto put = [&](int r, f32x4p t) __attribute__((always_inline)) {
        if (whole)
            for (int lanes = q; lanes < 64; lanes *= 2)
#pragma unroll
                for (int k = 0; k < 4; ++k) t[k] += __shfl_xor(t[k], lanes);
        f32x4p *buf = red[turn ^= 1];          // (a barrier lies between two uses of one)
        buf[tid] = t;
        __syncthreads();
        if (grp == 0) {
            t = buf[tid];
            for (int k = 1; k < terms; ++k) t += buf[tid + k * step];
            *reinterpret_cast<f32x4p *>(dst + static_cast<size_t>(r) * H) = t;
        }
    };
    put(0, s_time);
    put(1, s_size);
#pragma unroll
    for (int d = 0; d < DM; ++d)
        if (d < D) put(2 + d, kLds ? s_dev[d * kThreads + tid] : s_reg[kLds ? 0 : d]);
    put(2 + D, s_cur);
    put(3 + D, s_vis);
    put(4 + D, s_one);
}

// phi rows when H < F (more raw features than embedding columns): one thread per (node, feature).
__global__ __launch_bounds__(kThreads) void k_bw_phi(GraphView gv, ModelView mv,
                                                     const float *__restrict__ feats,
                                                     const int32_t *__restrict__ placement,
                                                     const int32_t *__restrict__ cur_node,
                                                     float *__restrict__ phi)
{
    const int D = mv.D, F = mv.F;
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (idx >= static_cast<size_t>(gv.n_tot) * F) return;
    const int v = static_cast<int>(idx / F), h = static_cast<int>(idx - static_cast<size_t>(v) * F);
    const int b = gv.node_graph[v];
    const int dev = placement[v];
    float p;
    if (h == 0) p = feats[v * 3 + 0];
    else if (h == 1) p = feats[v * 3 + 1];
    else if (h < 2 + D) p = (dev == h - 2) ? 1.0f : 0.0f;
    else if (h == 2 + D) p = (v - gv.node_off[b] == cur_node[b]) ? 1.0f : 0.0f;
    else p = feats[v * 3 + 2];
    phi[idx] = p;
}

// ------------------------------------------------------------------ dense layers on the matrix cores
// Y[row][j] = epi(bias[j] + sum_k X[row][k] Wt[j][k]) for a list of rows, H in {32, 64, 128} output
// columns (NJ tiles of 32) and K a multiple of 32.  A workgroup of four waves takes 128 rows; wave
// w multiplies rows 32 w .. 32 w + 31 by all columns; X and Wt go through LDS in chunks of 32 k.
// epi: optional ReLU, optional gate (Y = 0 where M[row][j] <= 0).  rows / n_rows_dev: optional row
// list and its length in device memory (the grid covers R rows; workgroups past the length exit).
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8w;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4v;

constexpr int kDenseKC = 32;                  // k per chunk
constexpr int kDenseRows = 128;               // rows per workgroup

// On the bf16 matrix cores at fp32 accuracy (operands split into three bf16 parts, six products
// kept: see k_wgrad_split).  The weights come in the transposed layout
// Wt[j][k] (row j holds the K inputs of output column j), so that both operands are contiguous
// along k: a 16-byte LDS cell holds the eight bf16 of one row (or output column) for eight
// consecutive k, and a fragment of v_mfma_f32_32x32x16_bf16 (lane = row, eight k) is one
// ds_read_b128.  A thread stages half cells: a float4 (coalesced along k: 128-byte row pieces),
// split in registers, three 8-byte stores; the row-group stride of 136 cells puts the two groups
// a store instruction touches on different halves of the banks.  One LDS buffer, the next chunk
// in registers meanwhile, two barriers per chunk; grid.z walks several row lists (z-th list,
// count, weights and bias: strides given) in one launch.
constexpr int kDsGS = 136;                    // cells between the row groups of the X parts
constexpr size_t dense_split_lds_bytes(int NJ) { return static_cast<size_t>(16) * 3 * 4 * (kDsGS + 32 * NJ + 8); }

template <int NJ>
__global__ __launch_bounds__(kThreads, 3) void k_dense_split(const float *__restrict__ X, int ldx,
                                                             const int32_t *__restrict__ rows,
                                                             const int32_t *__restrict__ n_rows_dev, int R, int K,
                                                             const float *__restrict__ Wt, int ldwt,
                                                             const float *__restrict__ bias, int relu,
                                                             const float *__restrict__ M, int ldm,
                                                             float *__restrict__ Y, int ldy, size_t list_stride,
                                                             size_t w_stride, size_t b_stride, size_t wt_half, int y_half)
{
    constexpr int Hc = 32 * NJ, GSW = Hc + 8;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint2 *half_x = reinterpret_cast<uint2 *>(lds_raw);                 // [3][4][kDsGS] cells of two halves
    uint2 *half_w = half_x + 2 * 3 * 4 * kDsGS;                         // [3][4][GSW]
    const uint4 *cell_x = reinterpret_cast<const uint4 *>(half_x);
    const uint4 *cell_w = reinterpret_cast<const uint4 *>(half_w);
    rows += blockIdx.z * list_stride;
    if (n_rows_dev) R = min(R, n_rows_dev[blockIdx.z]);
    Wt += blockIdx.z * w_stride + blockIdx.y * wt_half;
    Y += blockIdx.y * y_half;
    if (bias) bias += blockIdx.z * b_stride;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 31, lk = lane >> 5;
    const int tile0 = blockIdx.x * kDenseRows;
    if (tile0 >= R) return;                                // the whole workgroup, before any barrier

    // this thread's share of a chunk: float4 number (tid & 7) of the 32 k, of rows xr + 32 q and of
    // output columns xr + 32 q
    const int xr = tid >> 3, xc = (tid & 7) * 4;
    const int grp = xc >> 3, hf = (xc >> 2) & 1;
    const float *xsrc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = min(tile0 + xr + 32 * q, R - 1);
        xsrc[q] = X + static_cast<size_t>(rows ? rows[r] : r) * ldx + xc;
    }
    f32x4v xreg[4], wreg[NJ];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) xreg[q] = *reinterpret_cast<const f32x4v *>(xsrc[q] + k0);
#pragma unroll
        for (int q = 0; q < NJ; ++q)
            wreg[q] = *reinterpret_cast<const f32x4v *>(Wt + static_cast<size_t>(xr + 32 * q) * ldwt + k0 + xc);
    };
    auto put_half = [&](uint2 *cells, int stride, int c, const f32x4v &v) {
        auto top = [](float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); };
        auto pack = [](float lo, float hi) {
            return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
        };
        float r[4], l[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r[i] = v[i] - top(v[i]);
            l[i] = r[i] - top(r[i]);
        }
        cells[2 * ((0 * 4 + grp) * stride + c) + hf] = uint2{pack(v[0], v[1]), pack(v[2], v[3])};
        cells[2 * ((1 * 4 + grp) * stride + c) + hf] = uint2{pack(r[0], r[1]), pack(r[2], r[3])};
        cells[2 * ((2 * 4 + grp) * stride + c) + hf] = uint2{pack(l[0], l[1]), pack(l[2], l[3])};
    };
    auto stash = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q) put_half(half_x, kDsGS, xr + 32 * q, xreg[q]);
#pragma unroll
        for (int q = 0; q < NJ; ++q) put_half(half_w, GSW, xr + 32 * q, wreg[q]);
    };

    f32x16 acc[NJ];
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[jb][v] = 0.0f;

    const int n_chunks = K / kDenseKC;
    fetch(0);
    for (int c = 0; c < n_chunks; ++c) {
        stash();
        __syncthreads();
        if (c + 1 < n_chunks) fetch((c + 1) * kDenseKC);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int g = 2 * ks + lk;
            bf16x8w a[3];
#pragma unroll
            for (int p = 0; p < 3; ++p)
                a[p] = *reinterpret_cast<const bf16x8w *>(&cell_x[(p * 4 + g) * kDsGS + 32 * wave + li]);
            constexpr int JP = NJ > 1 ? 2 : 1;
            constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};   // small products first
#pragma unroll
            for (int j0 = 0; j0 < NJ; j0 += JP) {
                bf16x8w b[JP][3];
#pragma unroll
                for (int u = 0; u < JP; ++u)
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        b[u][p] = *reinterpret_cast<const bf16x8w *>(&cell_w[(p * 4 + g) * GSW + 32 * (j0 + u) + li]);
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int u = 0; u < JP; ++u)
                        acc[j0 + u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[t]], b[u][pb[t]], acc[j0 + u], 0, 0, 0);
            }
        }
        __syncthreads();
    }

    float bj[NJ];
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) bj[jb] = bias ? bias[32 * jb + li] : 0.0f;
    int orow[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int rc = min(tile0 + 32 * wave + 8 * (v / 4) + 4 * lk + (v % 4), R - 1);
        orow[v] = rows ? rows[rc] : rc;
    }
    auto finish = [&](auto gated) {
        // with gates: all gate values of a column tile are loaded before its first store (loads
        // and stores retire in order: a load behind a store would wait for it)
#pragma unroll
        for (int jb = 0; jb < NJ; ++jb) {
            float gate[16];
            if constexpr (decltype(gated)::value) {
#pragma unroll
                for (int v = 0; v < 16; ++v) gate[v] = M[static_cast<size_t>(orow[v]) * ldm + 32 * jb + li];
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = tile0 + 32 * wave + 8 * (v / 4) + 4 * lk + (v % 4);
                float y = acc[jb][v] + bj[jb];
                if (relu) y = fmaxf(y, 0.0f);
                if constexpr (decltype(gated)::value) y = gate[v] > 0.0f ? y : 0.0f;
                if (r < R) Y[static_cast<size_t>(orow[v]) * ldy + 32 * jb + li] = y;
            }
        }
    };
    if (M)
        finish(std::true_type{});
    else
        finish(std::false_type{});
}

// a_v = sum of the neighbours' messages, for every node and both directions (grid.y).
// Four columns per thread (H is a multiple of 32 on this path).
__global__ __launch_bounds__(kThreads) void k_bw_agg(GraphView gv, int H,
                                                     const float *__restrict__ msgs,
                                                     float *__restrict__ agg)
{
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    const int q = H / 4;
    if (idx >= static_cast<size_t>(gv.n_tot) * q) return;
    const int dir = blockIdx.y;
    const int v = static_cast<int>(idx / q), h = 4 * static_cast<int>(idx - static_cast<size_t>(v) * q);
    const float *msg = msgs + static_cast<size_t>(dir) * gv.n_tot * H;   // [2, n_tot, H] from the forward pass
    const int32_t *nbr_ptr = gv.nbr_ptr[dir], *nbr_idx = gv.nbr_idx[dir];
    f32x4v a{0.f, 0.f, 0.f, 0.f};
    for (int p = nbr_ptr[v]; p < nbr_ptr[v + 1]; ++p) {
        // messages are ReLU outputs; the matrix-core sweep keeps a flag in their sign bit
        const f32x4v m = *reinterpret_cast<const f32x4v *>(msg + static_cast<size_t>(nbr_idx[p]) * H + h);
        a += f32x4v{fabsf(m[0]), fabsf(m[1]), fabsf(m[2]), fabsf(m[3])};
    }
    *reinterpret_cast<f32x4v *>(agg + (static_cast<size_t>(dir) * gv.n_tot + v) * H + h) = a;
}

// Node set of every node and the three sets as row lists in ascending node order, in three
// steps with no atomics (the lists fix the summation order of l's weight gradients): per block
// of 256 nodes the number of nodes of each set; an exclusive scan over the blocks; the fill.
// The first step also copies the gradient of e_{v*} from dz.
__device__ __forceinline__ int node_class_of(const GraphView &gv, int v, const uint8_t *reach,
                                             const int32_t *cur_node, int single, int *graph)
{
    const int b = gv.node_graph[v];
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int cl = cur_node[b];
    const int cur = (cl >= 0 && cl < n_b) ? n0 + cl : -1;
    *graph = b;
    return node_class_bw(v, cur, reach, gv.n_tot, single);
}

__global__ __launch_bounds__(kThreads) void k_bw_cls_count(GraphView gv, int H, int Z, int single,
                                                           const uint8_t *__restrict__ reach,
                                                           const int32_t *__restrict__ cur_node,
                                                           const float *__restrict__ dz,
                                                           uint8_t *__restrict__ cls,
                                                           int32_t *__restrict__ blk_cnt,
                                                           float *__restrict__ demb)
{
    __shared__ int wcnt[4][3];
    const int v = blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int k = -1, b = 0;
    if (v < gv.n_tot) {
        k = node_class_of(gv, v, reach, cur_node, single, &b);
        cls[v] = static_cast<uint8_t>(k);
    }
    for (int c = 1; c <= 3; ++c) {
        const unsigned long long m = __ballot(k == c);
        if (lane == 0) wcnt[wave][c - 1] = __popcll(m);
    }
    __syncthreads();
    if (threadIdx.x < 3)
        blk_cnt[blockIdx.x * 3 + threadIdx.x] = wcnt[0][threadIdx.x] + wcnt[1][threadIdx.x] +
                                                wcnt[2][threadIdx.x] + wcnt[3][threadIdx.x];
    if (k == 0)
        for (int i = 0; i < 2 * H; ++i) demb[static_cast<size_t>(v) * 2 * H + i] = dz[static_cast<size_t>(b) * Z + i];
}

// One workgroup: blk_cnt[blk][c] becomes the position of the block's first node of set c in
// list c; counts[c] = size of set c.
__global__ __launch_bounds__(kThreads) void k_bw_cls_scan(int n_blocks, int32_t *__restrict__ blk_cnt,
                                                          int32_t *__restrict__ counts)
{
    __shared__ int part[kThreads][3];
    const int tid = threadIdx.x;
    const int per = (n_blocks + kThreads - 1) / kThreads;
    const int lo = min(n_blocks, tid * per), hi = min(n_blocks, lo + per);
    int sum[3] = {0, 0, 0};
    for (int i = lo; i < hi; ++i)
        for (int c = 0; c < 3; ++c) sum[c] += blk_cnt[i * 3 + c];
    for (int c = 0; c < 3; ++c) part[tid][c] = sum[c];
    __syncthreads();
    if (tid < 3) {
        int run = 0;
        for (int t = 0; t < kThreads; ++t) {
            const int x = part[t][tid];
            part[t][tid] = run;
            run += x;
        }
        counts[tid] = run;
    }
    __syncthreads();
    int run[3] = {part[tid][0], part[tid][1], part[tid][2]};
    for (int i = lo; i < hi; ++i)
        for (int c = 0; c < 3; ++c) {
            const int x = blk_cnt[i * 3 + c];
            blk_cnt[i * 3 + c] = run[c];
            run[c] += x;
        }
}

__global__ __launch_bounds__(kThreads) void k_bw_cls_fill(GraphView gv, const uint8_t *__restrict__ cls,
                                                          const int32_t *__restrict__ blk_off,
                                                          int32_t *__restrict__ lists)
{
    __shared__ int wcnt[4][3];
    const int v = blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = v < gv.n_tot ? cls[v] : -1;
    int before = 0;
    for (int c = 1; c <= 3; ++c) {
        const unsigned long long m = __ballot(k == c);
        if (lane == 0) wcnt[wave][c - 1] = __popcll(m);
        if (k == c) before = __popcll(m & ((1ull << lane) - 1));
    }
    __syncthreads();
    if (k >= 1) {
        int pos = blk_off[blockIdx.x * 3 + k - 1] + before;
        for (int w = 0; w < wave; ++w) pos += wcnt[w][k - 1];
        lists[static_cast<size_t>(k - 1) * gv.n_tot + pos] = v;
    }
}

// The same lists where the matrix-core pooling of this pass has sorted the nodes (klist: grouped by set and device, per
// graph): a workgroup per graph finds where its graph's part of every list begins, from the sets' sizes in the graphs
// before it, and copies it.  A list is then in the order (graph, device, node).  Also the class of every node, the gradient
// of e_{v*} from dz, and zero for that of nodes pooled nowhere (device id out of range), whose rows are in no list.
// One launch for the three above and one that cleared the rows: 64 layered graphs 20 -> 5.6 us, 48 NMT-like ones 28 -> 6.8,
// 256 NASNet-like ones 57 -> 12.6.
constexpr int kSetThreads = 1024;   // most: graphs of more than 512 nodes; 256 for smaller ones
// Up to this many graphs every workgroup adds the sets' sizes in all graphs before its own.  In larger batches, where that
// grows with the square of their number, a launch of its own (k_bw_set_begins) does it for a thousand graphs at a time.
// Gradient of 1536 / 2048 / 4096 / 16384 graphs of 8 nodes, H = 32: alone 225 / 270 / 487 / 2173 us, with that launch
// 227 / 267 / 448 / 1469 (three kernels without the sort's offsets: 250 / 286 / 462 / 1444).
constexpr int kSetsAlone = 1536;
constexpr int kSetGraphs = kSetThreads;   // graphs to a workgroup of k_bw_set_begins

// begins[c][b]: nodes of set c in those graphs before b that the same workgroup takes; sums[w][c]: of all that workgroup w takes.
__global__ __launch_bounds__(kSetThreads) void k_bw_set_begins(int B, int G, int koff_ld, const int32_t *__restrict__ koff,
                                                               int32_t *__restrict__ begins, int32_t *__restrict__ sums)
{
    __shared__ int before[kSetThreads / 64][3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x * kSetGraphs + tid;
    int size[3], run[3];
    for (int c = 0; c < 3; ++c) {
        const int32_t *k = koff + static_cast<size_t>(min(b, B - 1)) * koff_ld + c * G;
        size[c] = b < B ? k[G] - k[0] : 0;
    }
    for (int c = 0; c < 3; ++c) {
        run[c] = size[c];
        for (int step = 1; step < 64; step *= 2) {
            const int below = __shfl_up(run[c], step);
            run[c] += lane >= step ? below : 0;
        }
        if (lane == 63) before[wave][c] = run[c];
    }
    __syncthreads();
    for (int c = 0; c < 3; ++c) {
        for (int w = 0; w < wave; ++w) run[c] += before[w][c];
        if (b < B) begins[static_cast<size_t>(c) * B + b] = run[c] - size[c];
        if (tid == kSetThreads - 1) sums[3 * blockIdx.x + c] = run[c];
    }
}

__global__ __launch_bounds__(kSetThreads) void k_bw_sets(GraphView gv, int H, int Z, int G, int D, int single, int koff_ld,
                                                      const uint8_t *__restrict__ reach,
                                                      const int32_t *__restrict__ placement,
                                                      const int32_t *__restrict__ cur_node,
                                                      const int32_t *__restrict__ klist,
                                                      const int32_t *__restrict__ koff,
                                                      const float *__restrict__ dz, const int32_t *__restrict__ begins,
                                                      uint8_t *__restrict__ cls, int32_t *__restrict__ counts,
                                                      int32_t *__restrict__ lists, float *__restrict__ demb)
{
    __shared__ int before[kSetThreads / 64][3];
    const int b = blockIdx.x, threads = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int cl = cur_node[b];
    const int cur = (cl >= 0 && cl < n_b) ? n0 + cl : -1;
    auto first = [&](int g, int set) { return koff[static_cast<size_t>(g) * koff_ld + set * G]; };
    int sum[3] = {0, 0, 0};
    if (begins) {
        const int32_t *sums = begins + 3 * static_cast<size_t>(gv.B);
        for (int w = tid; w < b / kSetGraphs; w += threads)
            for (int c = 0; c < 3; ++c) sum[c] += sums[3 * w + c];
    } else {
        for (int g = tid; g < b; g += threads)
            for (int c = 0; c < 3; ++c) sum[c] += first(g, c + 1) - first(g, c);
    }
    for (int c = 0; c < 3; ++c) {
        for (int step = 32; step > 0; step /= 2) sum[c] += __shfl_xor(sum[c], step);
        if (lane == 0) before[wave][c] = sum[c];
    }
    // (node by node meanwhile)
    for (int v = n0 + tid; v < n0 + n_b; v += threads) {
        const int k = node_class_bw(v, cur, reach, gv.n_tot, single), dev = placement[v];
        cls[v] = static_cast<uint8_t>(k);
        if (k != 0 && (dev < 0 || dev >= D))
            for (int i = 0; i < 2 * H; ++i) demb[static_cast<size_t>(v) * 2 * H + i] = 0.0f;
    }
    if (cur >= 0)
        for (int i = tid; i < 2 * H; i += threads) demb[static_cast<size_t>(cur) * 2 * H + i] = dz[static_cast<size_t>(b) * Z + i];
    __syncthreads();
    for (int c = 0; c < 3; ++c) {
        int base = begins ? begins[static_cast<size_t>(c) * gv.B + b] : 0;
        for (int w = 0; w < threads / 64; ++w) base += before[w][c];
        const int lo = first(b, c), n = first(b, c + 1) - lo;
        if (b == gv.B - 1 && tid == 0) counts[c] = base + n;
        for (int i = tid; i < n; i += threads) lists[static_cast<size_t>(c) * gv.n_tot + base + i] = klist[n0 + lo + i];
    }
}

// Delta of l's last layer for every node: dP[set of the node][device of the node], gated by the
// layer's output; zero for a node whose device id is out of range (it was pooled nowhere).  Four
// columns per thread.
__global__ __launch_bounds__(kThreads) void k_bw_pool_seed(GraphView gv, int H, int G, int D,
                                                           const uint8_t *__restrict__ cls,
                                                           const int32_t *__restrict__ placement,
                                                           const float *__restrict__ dP,
                                                           const float *__restrict__ act,
                                                           float *__restrict__ dl)
{
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    const int q = H / 4;
    if (idx >= static_cast<size_t>(gv.n_tot) * q) return;
    const int v = static_cast<int>(idx / q), h = 4 * static_cast<int>(idx - static_cast<size_t>(v) * q);
    const int k = cls[v];
    if (k == 0) return;                       // the current node is in no set
    const int b = gv.node_graph[v];
    const int dev = placement[v];
    const bool ok = dev >= 0 && dev < D;
    const size_t at = static_cast<size_t>(v) * H + h;
    const f32x4v a = *reinterpret_cast<const f32x4v *>(act + at);
    f32x4v g{0.f, 0.f, 0.f, 0.f};
    if (ok) g = *reinterpret_cast<const f32x4v *>(dP + ((static_cast<size_t>(b) * 3 + (k - 1)) * G + (G == 1 ? 0 : dev)) * H + h);
    f32x4v o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = a[i] > 0.0f ? g[i] : 0.0f;
    *reinterpret_cast<f32x4v *>(dl + at) = o;
}

// ------------------------------------------------------------------ 5. weight gradients
// The weight gradients of a pass are up to 10 L + 3 contractions over rows that do not depend on
// each other, each followed by the sum of its slabs.  They are taken as a table of jobs, in one
// launch per kernel: on batches of a few thousand nodes a contraction of its own fills the chip for
// less time than its launch takes, and on large ones every launch ends in a wave of workgroups that
// does not fill it.  Gradient of 64 layered graphs (12800 nodes, H = 32): 442 -> 280 us, of 48 NMT-like
// ones (H = 64) 1376 -> 1263 us, of 256 NASNet-like ones (H = 128) 8.00 -> 7.76 ms; same bits, since a
// contraction keeps its slabs.  The workgroups of job k are first[k] .. first[k + 1] - 1 of the kernel that takes it.
struct WgradJob {
    const float *A, *Dl;            // inputs [.., lda] and deltas [.., ldd] by row
    const int32_t *rows;            // row list; null: rows 0 .. R - 1
    const int32_t *n_rows_dev;      // its length, at most R; null: R
    const uint8_t *row_cls;         // (k_wgrad) rows whose byte is not `want` are left out; null: none is
    float *partial, *out;           // slab sums [slabs][I J + J]; destination [n_in J + J], added to
    int32_t lda, ldd, want, R, I, J, n_in, rows_per_slab, slabs;
    // list lengths of the jobs before this one whose slab sums lie before its own in the same place (n_rows_dev's neighbours)
    int32_t n_prior;
    int32_t store;                  // the sum is stored instead of added to what is there
};
constexpr int kWgradJobs = 32;      // (a table travels in the 4 KB of kernel arguments)
struct WgradBatch {
    WgradJob job[kWgradJobs];
    int32_t first[kWgradJobs], first_sum[kWgradJobs];   // first workgroup of the contraction / of the slab sums
};
static_assert(sizeof(WgradBatch) <= 3840, "kernel arguments are at most 4 KB");

// First slab of a job in its place: behind the slabs that the lists before it fill.
__device__ __forceinline__ int wgrad_first_slab(const WgradJob &w)
{
    int at = 0;
    for (int k = 1; k <= w.n_prior; ++k) at += (min(w.R, w.n_rows_dev[-k]) + w.rows_per_slab - 1) / w.rows_per_slab;
    return at;
}

// Job in [lo, hi) that workgroup blk belongs to (first[lo] = 0).
__device__ __forceinline__ int wgrad_job_of(const int32_t (&first)[kWgradJobs], int lo, int hi, int blk)
{
    int k = lo;
#pragma unroll
    for (int i = 1; i < kWgradJobs; ++i) k += (i > lo && i < hi && blk >= first[i]) ? 1 : 0;
    return __builtin_amdgcn_readfirstlane(k);
}

// partial[slab][i * J + j] = sum over the slab's rows r of A[r][i] * Dl[r][j]  (i in this
// workgroup's block of kWgI), partial[slab][I * J + j] = sum of Dl[r][j] (the bias).  Rows whose
// class byte differs from `want` are skipped when row_cls is given.  Thread (grp, j): column j,
// rows grp, grp + groups, ... of every staged batch; groups are added in order at the end.
__global__ __launch_bounds__(kThreads) void k_wgrad(WgradBatch wb, int lo, int hi)
{
    const int k_job = wgrad_job_of(wb.first, lo, hi, blockIdx.x);
    const WgradJob &w = wb.job[k_job];
    const float *A = w.A, *Dl = w.Dl;
    const uint8_t *row_cls = w.row_cls;
    const int lda = w.lda, ldd = w.ldd, want = w.want, R = w.R, I = w.I, J = w.J, rows_per_slab = w.rows_per_slab;
    const int n_ib = (I + kWgI - 1) / kWgI, ib = (blockIdx.x - wb.first[k_job]) % n_ib;
    // (the matrix-core version below takes a row list instead of the class filter)
    __shared__ float a_s[kWgRB][kWgI];
    __shared__ int ok_s[kWgRB];
    __shared__ float red[kThreads * (kWgI + 1)];
    const int tid = threadIdx.x;
    const int i0 = ib * kWgI, sl = (blockIdx.x - wb.first[k_job]) / n_ib;
    const int r_beg = sl * rows_per_slab, r_end = min(R, r_beg + rows_per_slab);
    const int groups = kThreads / J;
    const int grp = tid / J, j = tid - grp * J;
    const bool active = grp < groups;
    float acc[kWgI];
#pragma unroll
    for (int ii = 0; ii < kWgI; ++ii) acc[ii] = 0.0f;
    float accb = 0.0f;
    for (int r0 = r_beg; r0 < r_end; r0 += kWgRB) {
        for (int idx = tid; idx < kWgRB * kWgI; idx += kThreads) {
            const int rr = idx / kWgI, ii = idx - rr * kWgI;
            const int row = r0 + rr;
            const bool ok = row < r_end && (!row_cls || row_cls[row] == want);
            a_s[rr][ii] = (ok && i0 + ii < I) ? A[static_cast<size_t>(row) * lda + i0 + ii] : 0.0f;
            if (ii == 0) ok_s[rr] = ok ? 1 : 0;
        }
        __syncthreads();
        if (active) {
            for (int rr = grp; rr < kWgRB; rr += groups) {
                if (!ok_s[rr]) continue;
                const float d = Dl[static_cast<size_t>(r0 + rr) * ldd + j];
#pragma unroll
                for (int ii = 0; ii < kWgI; ++ii) acc[ii] = fmaf(a_s[rr][ii], d, acc[ii]);
                accb += d;
            }
        }
        __syncthreads();
    }
    if (active) {
#pragma unroll
        for (int ii = 0; ii < kWgI; ++ii) red[(grp * (kWgI + 1) + ii) * J + j] = acc[ii];
        red[(grp * (kWgI + 1) + kWgI) * J + j] = accb;
    }
    __syncthreads();
    // (an entry to a thread: where J is small, few threads have a column, and they would add all groups of every row)
    float *dst = w.partial + static_cast<size_t>(sl) * (static_cast<size_t>(I) * J + J);
    for (int e = tid; e < (kWgI + 1) * J; e += kThreads) {
        const int ii = e / J;
        float s = 0.0f;
        for (int gq = 0; gq < groups; ++gq) s += red[gq * (kWgI + 1) * J + e];
        if (ii < kWgI) {
            if (i0 + ii < I) dst[static_cast<size_t>(i0) * J + e] = s;
        } else if (ib == 0) {
            dst[static_cast<size_t>(I) * J + (e - kWgI * J)] = s;
        }
    }
}

// The same contraction on the matrix cores, for I a multiple of 32 and J in {32, 64, 128}:
// v_mfma_f32_32x32x2_f32 multiplies a 32 x 2 block of A^T by a 2 x 32 block of Dl in fp32, so two
// contraction rows are consumed per instruction (lanes 0-31 take the even row, lanes 32-63 the odd
// one; no split into bf16 parts).  A workgroup owns rows [128 blockIdx.x, +128) of the weight
// matrix (wave w: 32 of them) and all J columns, for one slab of contraction rows.  The rows of A
// and Dl go through LDS in chunks of 16, double buffered: every element is read from global
// memory once per workgroup (coalesced float4), the loads of chunk c + 1 travel during the 32
// matrix instructions of chunk c, and the ids of a row list are read one chunk further ahead.
// Row strides in LDS keep the two halves of a wave on different banks.
constexpr int kWgRC = 32;

constexpr int wgrad_ldd(int J) { return J == 128 ? 160 : 96; }
constexpr size_t wgrad_lds_bytes(int NJ) { return sizeof(float) * 2 * kWgRC * (160 + wgrad_ldd(32 * NJ)); }

template <int NJ>
__global__ __launch_bounds__(kThreads) void k_wgrad_mfma(const float *__restrict__ A, int lda,
                                                         const float *__restrict__ Dl, int ldd,
                                                         const int32_t *__restrict__ rows,
                                                         const int32_t *__restrict__ n_rows_dev,
                                                         int R, int I, int rows_per_slab,
                                                         float *__restrict__ partial)
{
    constexpr int J = 32 * NJ, LDA_S = 160, LDD_S = wgrad_ldd(J);
    constexpr int DT = kWgRC * J / 4;                      // float4 of a Dl chunk: 512, 256, 128
    constexpr int DQ = (DT + kThreads - 1) / kThreads;     // per thread: 2, 1, 1
    extern __shared__ float lds[];
    float *as = lds;                                       // [2][kWgRC][LDA_S]
    float *dsm = lds + 2 * kWgRC * LDA_S;                  // [2][kWgRC][LDD_S]
    if (n_rows_dev) R = min(R, *n_rows_dev);               // slabs past the list's end write zeros
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 31, lk = lane >> 5;
    const int iw = blockIdx.x * 128, sl = blockIdx.y;
    const bool wave_on = iw + 32 * wave < I;
    const int r_beg = min(R, sl * rows_per_slab), r_end = min(R, r_beg + rows_per_slab);
    const int n_chunks = (r_end - r_beg + kWgRC - 1) / kWgRC;

    // this thread's pieces of a chunk: A rows ar + 8 q, floats ac .. ac + 3; Dl element 4 (tid + 256 q)
    const int ar = tid >> 5, ac = (tid & 31) * 4;
    const bool a_col_ok = iw + ac < I;
    constexpr int AQ = kWgRC / 8;                          // A pieces per thread and chunk
    int ida[AQ], idd[DQ];
    auto load_ids = [&](int r0) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int row = r0 + ar + 8 * q;
            ida[q] = row < r_end ? (rows ? rows[row] : row) : -1;
        }
#pragma unroll
        for (int q = 0; q < DQ; ++q) {
            const int e = (tid + kThreads * q) * 4;
            const int row = r0 + e / J;
            idd[q] = (e < kWgRC * J && row < r_end) ? (rows ? rows[row] : row) : -1;
        }
    };
    f32x4v areg[AQ], dreg[DQ];
    auto fetch = [&]() {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const f32x4v v = *reinterpret_cast<const f32x4v *>(
                A + static_cast<size_t>(max(ida[q], 0)) * lda + (a_col_ok ? iw + ac : 0));
            areg[q] = (ida[q] >= 0 && a_col_ok) ? v : f32x4v{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < DQ; ++q) {
            const int e = (tid + kThreads * q) * 4, c = e % J;
            const f32x4v v = *reinterpret_cast<const f32x4v *>(Dl + static_cast<size_t>(max(idd[q], 0)) * ldd + c);
            dreg[q] = idd[q] >= 0 ? v : f32x4v{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AQ; ++q)
            *reinterpret_cast<f32x4v *>(as + (buf * kWgRC + ar + 8 * q) * LDA_S + ac) = areg[q];
#pragma unroll
        for (int q = 0; q < DQ; ++q) {
            const int e = (tid + kThreads * q) * 4;
            if (e < kWgRC * J)
                *reinterpret_cast<f32x4v *>(dsm + (buf * kWgRC + e / J) * LDD_S + e % J) = dreg[q];
        }
    };

    f32x16 acc[NJ];
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[jb][v] = 0.0f;
    float bsum[NJ];
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) bsum[jb] = 0.0f;

    if (n_chunks > 0) {
        load_ids(r_beg);
        fetch();
        load_ids(r_beg + kWgRC);
        stash(0);
    }
    __syncthreads();
    for (int c = 0; c < n_chunks; ++c) {
        const int buf = c & 1;
        if (c + 1 < n_chunks) {
            fetch();                                       // chunk c + 1, ids read during chunk c - 1
            load_ids(r_beg + (c + 2) * kWgRC);
        }
        const float *ap = as + buf * kWgRC * LDA_S + lk * LDA_S + 32 * wave + li;
        const float *dp = dsm + buf * kWgRC * LDD_S + lk * LDD_S + li;
#pragma unroll
        for (int st = 0; st < kWgRC / 2; ++st) {
            const float a = ap[2 * st * LDA_S];
#pragma unroll
            for (int jb = 0; jb < NJ; ++jb) {
                const float b = dp[2 * st * LDD_S + 32 * jb];
                if (wave_on) acc[jb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[jb], 0, 0, 0);
                bsum[jb] += b;
            }
        }
        if (c + 1 < n_chunks) stash(buf ^ 1);
        __syncthreads();
    }
    if (!wave_on) return;
    float *dst = partial + static_cast<size_t>(sl) * (static_cast<size_t>(I) * J + J);
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int i = iw + 32 * wave + 8 * (v / 4) + 4 * lk + (v % 4);
            dst[static_cast<size_t>(i) * J + 32 * jb + li] = acc[jb][v];
        }
        const float other = __shfl_xor(bsum[jb], 32);
        if (blockIdx.x == 0 && wave == 0 && lk == 0) dst[static_cast<size_t>(I) * J + 32 * jb + li] = bsum[jb] + other;
    }
}

// The same contraction on the bf16 matrix cores at fp32 accuracy.  Every fp32 operand is split
// exactly into three bf16 parts by truncation (x = hi + mid + lo, 8 + 8 + 8 mantissa bits) and six
// of the nine products of parts are accumulated in fp32: hi hi, hi mid, mid hi, hi lo, lo hi,
// mid mid; the three left out are below 2^-24 of the product.  On v_mfma_f32_32x32x16_bf16 that
// is 2.7 times the rate of the fp32 instruction.
// A chunk is 32 contraction rows.  LDS holds the parts fragment-major: a 16-byte cell is the eight
// bf16 of one column for eight consecutive rows and the cells of consecutive columns are
// adjacent, so a fragment (lane = column, eight rows) is one conflict-free ds_read_b128.  A
// thread stages whole cells: eight rows of one column (the lanes of a wave on consecutive
// columns, 256-byte row segments), split in registers, three 16-byte stores.  The rows of chunk
// c + 1 are in flight in registers while chunk c is multiplied; the ids of a row list are staged
// in LDS one chunk further ahead.  Column sums of Dl (the bias gradient) are taken in fp32 from
// the staged values, by the thread that stages the column.

constexpr size_t wgrad_split_lds_bytes(int NJ)
{
    return static_cast<size_t>(16) * 3 * 4 * (128 + 32 * NJ) + sizeof(int32_t) * 2 * kWgRC + sizeof(float) * kThreads;
}

template <int NJ>
__global__ __launch_bounds__(kThreads, 3) void k_wgrad_split(WgradBatch wb, int n_jobs)
{
    constexpr int J = 32 * NJ;
    constexpr int NDC = (4 * J + kThreads - 1) / kThreads;     // Dl cells per thread: 2, 1, 1
    const int k_job = wgrad_job_of(wb.first, 0, n_jobs, blockIdx.x);
    const WgradJob &w = wb.job[k_job];
    const float *__restrict__ A = w.A, *__restrict__ Dl = w.Dl;
    const int32_t *__restrict__ rows = w.rows;
    const int lda = w.lda, ldd = w.ldd, I = w.I, rows_per_slab = w.rows_per_slab;
    const int R = w.n_rows_dev ? min(w.R, *w.n_rows_dev) : w.R;
    const int n_ib = (I + 127) / 128, local = blockIdx.x - wb.first[k_job];
    const int iw = (local % n_ib) * 128, sl = local / n_ib;
    if (static_cast<int64_t>(sl) * rows_per_slab >= R) return;   // past the list's end: the slab is not summed
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint4 *cell_a = reinterpret_cast<uint4 *>(lds_raw);                       // [3 parts][4 row groups][128 columns]
    uint4 *cell_d = cell_a + 3 * 4 * 128;                                      // [3 parts][4 row groups][J columns]
    int32_t *tab = reinterpret_cast<int32_t *>(cell_d + 3 * 4 * J);           // [2][32] row ids of a chunk
    float *bsh = reinterpret_cast<float *>(tab + 2 * kWgRC);                  // [256] column sums at the end
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 31, lk = lane >> 5;
    const bool wave_on = iw + 32 * wave < I;
    const int r_beg = sl * rows_per_slab, r_end = min(R, r_beg + rows_per_slab);
    const int n_chunks = (r_end - r_beg + kWgRC - 1) / kWgRC;

    // this thread's cells: A column ca, row groups ga and ga + 2; Dl column cd, row groups of cell tid + 256 q
    const int ca = tid & 127, ga = tid >> 7;
    const bool a_col_ok = iw + ca < I;
    const int cd = tid % J;
    float av[2][8], dv[NDC][8];       // the values of the chunk in flight, unmasked
    uint32_t amask = 0, dmask = 0;    // bit 8 q + k: value [q][k] belongs to the slab
    // ids of rows 8 grp .. 8 grp + 7 of the chunk at r0: from the staged list, or the row numbers
    // themselves; -1 past the slab's end.  Straight-line code: the loads that follow are all
    // issued before the first of them is used.
    auto row_ids = [&](int r0, int slot, int grp, int (&ids)[8]) {
        const int4 t0 = *reinterpret_cast<const int4 *>(tab + slot * kWgRC + 8 * grp);
        const int4 t1 = *reinterpret_cast<const int4 *>(tab + slot * kWgRC + 8 * grp + 4);
        const int listed[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int r = r0 + 8 * grp + k;
            ids[k] = rows ? listed[k] : (r < r_end ? r : -1);
        }
    };
    auto fetch = [&](int r0, int slot) {
        int ida[2][8], idd[NDC][8];
#pragma unroll
        for (int q = 0; q < 2; ++q) row_ids(r0, slot, ga + 2 * q, ida[q]);
#pragma unroll
        for (int q = 0; q < NDC; ++q) {
            const int cell = tid + kThreads * q;
            row_ids(r0, slot, cell < 4 * J ? cell / J : 0, idd[q]);
        }
        const int col_a = a_col_ok ? iw + ca : 0;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k)    // (the launcher checks that 32-bit element offsets suffice)
                av[q][k] = A[static_cast<uint32_t>(max(ida[q][k], 0)) * static_cast<uint32_t>(lda) + static_cast<uint32_t>(col_a)];
#pragma unroll
        for (int q = 0; q < NDC; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k)
                dv[q][k] = Dl[static_cast<uint32_t>(max(idd[q][k], 0)) * static_cast<uint32_t>(ldd) + static_cast<uint32_t>(cd)];
        // which of them count: one bit per value
        amask = 0;
        dmask = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) amask |= (ida[q][k] >= 0 && a_col_ok) ? 1u << (8 * q + k) : 0u;
#pragma unroll
        for (int q = 0; q < NDC; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k)
                dmask |= (idd[q][k] >= 0 && tid + kThreads * q < 4 * J) ? 1u << (8 * q + k) : 0u;
    };
    // the three bf16 parts of eight values, eight to a 16-byte cell (masked: the values whose bit
    // of ok is clear count as zero)
    auto put_cells = [&](auto masked, uint4 *cells, int C, int grp, int c, const float (&v)[8], uint32_t ok) {
        uint32_t h[4], m[4], l[4];
        auto top = [](float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); };
        auto pack = [](float lo, float hi) {       // the upper halves of two floats in one word
            return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float x0 = v[2 * k], x1 = v[2 * k + 1];
            if constexpr (decltype(masked)::value) {
                x0 = (ok >> (2 * k)) & 1u ? x0 : 0.0f;
                x1 = (ok >> (2 * k + 1)) & 1u ? x1 : 0.0f;
            }
            const float r0 = x0 - top(x0), r1 = x1 - top(x1);
            const float l0 = r0 - top(r0), l1 = r1 - top(r1);
            h[k] = pack(x0, x1);
            m[k] = pack(r0, r1);
            l[k] = pack(l0, l1);
        }
        cells[(0 * 4 + grp) * C + c] = uint4{h[0], h[1], h[2], h[3]};
        cells[(1 * 4 + grp) * C + c] = uint4{m[0], m[1], m[2], m[3]};
        cells[(2 * 4 + grp) * C + c] = uint4{l[0], l[1], l[2], l[3]};
    };
    float bsum = 0.0f;
    bool whole = false;               // the chunk in flight came in with fetch_whole(): nothing to mask
    auto stash = [&]() {
        if (whole) {
#pragma unroll
            for (int q = 0; q < 2; ++q) put_cells(std::false_type{}, cell_a, 128, ga + 2 * q, ca, av[q], 0u);
#pragma unroll
            for (int q = 0; q < NDC; ++q) {
                put_cells(std::false_type{}, cell_d, J, (tid + kThreads * q) / J, cd, dv[q], 0u);
#pragma unroll
                for (int k = 0; k < 8; ++k) bsum += dv[q][k];
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) put_cells(std::true_type{}, cell_a, 128, ga + 2 * q, ca, av[q], amask >> (8 * q));
#pragma unroll
        for (int q = 0; q < NDC; ++q) {
            const int cell = tid + kThreads * q;
            if (cell < 4 * J) {
                put_cells(std::true_type{}, cell_d, J, cell / J, cd, dv[q], dmask >> (8 * q));
#pragma unroll
                for (int k = 0; k < 8; ++k) bsum += (dmask >> (8 * q + k)) & 1u ? dv[q][k] : 0.0f;
            }
        }
    };
    // A chunk that lies wholly inside the slab, for J >= 64: the row group of each of a thread's
    // cells is the same over its wave, so row ids and row addresses are scalars and a load costs no
    // vector arithmetic; nothing is masked (columns past I load column 0 and are zeroed here).
    auto fetch_whole = [&](auto listed, int r0, int slot) {
        constexpr bool kListed = decltype(listed)::value;
        // ids of the eight rows of a group, as scalars (all reads of the list first, then the loads)
        auto group_ids = [&](int grp, int (&ids)[8]) {
            if constexpr (kListed) {
                const int4 t0 = *reinterpret_cast<const int4 *>(tab + slot * kWgRC + 8 * grp);
                const int4 t1 = *reinterpret_cast<const int4 *>(tab + slot * kWgRC + 8 * grp + 4);
                const int v[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
#pragma unroll
                for (int k = 0; k < 8; ++k) ids[k] = __builtin_amdgcn_readfirstlane(v[k]);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) ids[k] = r0 + 8 * grp + k;
            }
        };
        int ida[2][8], idd[NDC][8];
#pragma unroll
        for (int q = 0; q < 2; ++q) group_ids(__builtin_amdgcn_readfirstlane(ga + 2 * q), ida[q]);
#pragma unroll
        for (int q = 0; q < NDC; ++q) group_ids(__builtin_amdgcn_readfirstlane((tid + kThreads * q) / J), idd[q]);
        const uint32_t col_a = a_col_ok ? iw + ca : 0;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) av[q][k] = (A + static_cast<size_t>(ida[q][k]) * lda)[col_a];
#pragma unroll
        for (int q = 0; q < NDC; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) dv[q][k] = (Dl + static_cast<size_t>(idd[q][k]) * ldd)[static_cast<uint32_t>(cd)];
        if (!a_col_ok) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int k = 0; k < 8; ++k) av[q][k] = 0.0f;
        }
    };
    auto fetch_chunk = [&](int r0, int slot) {
        whole = J >= 64 && r0 + kWgRC <= r_end;
        if (!whole)
            fetch(r0, slot);
        else if (rows)
            fetch_whole(std::true_type{}, r0, slot);
        else
            fetch_whole(std::false_type{}, r0, slot);
    };
    auto list_id = [&](int r0) {                           // thread k < 32: id of row k of the chunk at r0
        return (rows && tid < kWgRC && r0 + tid < r_end) ? rows[r0 + tid] : -1;
    };

    f32x16 acc[NJ];
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[jb][v] = 0.0f;

    if (tid < kWgRC) {
        tab[tid] = list_id(r_beg);
        tab[kWgRC + tid] = list_id(r_beg + kWgRC);
    }
    __syncthreads();
    if (n_chunks > 0) fetch_chunk(r_beg, 0);
    for (int c = 0; c < n_chunks; ++c) {
        const int next_id = list_id(r_beg + (c + 2) * kWgRC);      // in flight until the end of the iteration
        stash();                                                   // chunk c: registers -> cells
        __syncthreads();
        if (c + 1 < n_chunks) fetch_chunk(r_beg + (c + 1) * kWgRC, (c + 1) & 1);
        if (wave_on) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int grp = 2 * ks + lk;
                bf16x8w a[3];
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    a[p] = *reinterpret_cast<const bf16x8w *>(&cell_a[(p * 4 + grp) * 128 + 32 * wave + li]);
                // two column tiles at a time, so that consecutive matrix instructions do not
                // wait for each other's accumulator
                constexpr int JP = NJ > 1 ? 2 : 1;
                constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};   // small products first
#pragma unroll
                for (int j0 = 0; j0 < NJ; j0 += JP) {
                    bf16x8w b[JP][3];
#pragma unroll
                    for (int u = 0; u < JP; ++u)
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            b[u][p] = *reinterpret_cast<const bf16x8w *>(&cell_d[(p * 4 + grp) * J + 32 * (j0 + u) + li]);
#pragma unroll
                    for (int t = 0; t < 6; ++t)
#pragma unroll
                        for (int u = 0; u < JP; ++u)
                            acc[j0 + u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[t]], b[u][pb[t]], acc[j0 + u], 0, 0, 0);
                }
            }
        }
        __syncthreads();
        if (tid < kWgRC) tab[(c & 1) * kWgRC + tid] = next_id;     // chunk c + 2; this half was last read for chunk c
    }
    // column sums of Dl: the threads that staged column j are tid = j, j + J, ...
    bsh[tid] = bsum;
    __syncthreads();
    float *dst = w.partial + static_cast<size_t>(wgrad_first_slab(w) + sl) * (static_cast<size_t>(I) * J + J);
    if (iw == 0 && tid < J) {
        float t = bsh[tid];
        for (int k = tid + J; k < kThreads && k < 4 * J; k += J) t += bsh[k];
        dst[static_cast<size_t>(I) * J + tid] = t;
    }
    if (!wave_on) return;
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int i = iw + 32 * wave + 8 * (v / 4) + 4 * lk + (v % 4);
            dst[static_cast<size_t>(i) * J + 32 * jb + li] = acc[jb][v];
        }
}

// out[idx] += sum over slabs, for every job of the table.  A workgroup takes 32 consecutive entries;
// its eight thread rows each add the slabs q, q + 8, ... in order, and the eight sums are added in
// order: a fixed summation order with enough loads in flight.
// A slab holds I J + J floats; entry idx of the output comes from entry idx of the slab, or, past the
// n_in J weights, from the bias row (the slab's matrix may be padded to more rows).
__global__ __launch_bounds__(kThreads) void k_wgrad_reduce(WgradBatch wb, int n_jobs)
{
    __shared__ float part[8][32];
    const int k_job = wgrad_job_of(wb.first_sum, 0, n_jobs, blockIdx.x);
    const WgradJob &w = wb.job[k_job];
    const int R = w.n_rows_dev ? min(w.R, *w.n_rows_dev) : w.R;
    const int n_slabs = (R + w.rows_per_slab - 1) / w.rows_per_slab;
    const size_t J = w.J, n_main = static_cast<size_t>(w.n_in) * J, count = n_main + J;
    const size_t src_count = static_cast<size_t>(w.I) * J + J, src_skip = src_count - count;
    const float *__restrict__ partial = w.partial + wgrad_first_slab(w) * src_count;
    const int c = threadIdx.x & 31, q = threadIdx.x >> 5;
    const size_t idx = static_cast<size_t>(blockIdx.x - wb.first_sum[k_job]) * 32 + c;
    const size_t src = idx < n_main ? idx : idx + src_skip;
    // four running sums per thread row (slabs q, q + 8, q + 16, q + 24, then again), added in order
    // at the end: still one fixed order, with four loads in flight
    float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (idx < count) {
        int sl = q;
        for (; sl + 24 < n_slabs; sl += 32) {
#pragma unroll
            for (int u = 0; u < 4; ++u) s4[u] += partial[static_cast<size_t>(sl + 8 * u) * src_count + src];
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)     // at most three slabs are left
            if (sl + 8 * u < n_slabs) s4[u] += partial[static_cast<size_t>(sl + 8 * u) * src_count + src];
    }
    part[q][c] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    __syncthreads();
    if (q == 0 && idx < count) {
        float t = part[0][c];
        for (int k = 1; k < 8; ++k) t += part[k][c];
        w.out[idx] = w.store ? t : w.out[idx] + t;
    }
}

__global__ __launch_bounds__(kThreads) void k_fill_zero(float *__restrict__ p, size_t n)
{
    const size_t idx = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (idx < n) p[idx] = 0.0f;
}

int pick_rpt_bw(int H)
{
    int groups = kThreads / H;
    if (groups > kTile) groups = kTile;
    int rpt = 1;
    while (groups * rpt < kTile) rpt *= 2;
    return rpt;
}

template <typename K>
void allow_lds_bw(K kernel, size_t bytes)
{
    if (bytes > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
}

#define PL_DISPATCH_RPT(rpt, CALL) \
    switch (rpt) {                 \
        case 1: { CALL(1); break; }  \
        case 2: { CALL(2); break; }  \
        case 4: { CALL(4); break; }  \
        case 8: { CALL(8); break; }  \
        default: { CALL(16); break; } \
    }

// about two slabs per CU (768, one for each of the three workgroups a CU holds, was slower: the
// slab sums grow with the slab count)
int wgrad_rows_per_slab_cores(int64_t R)
{
    int64_t per = (R + 511) / 512;
    if (per < 64) per = 64;
    return static_cast<int>((per + 7) / 8 * 8);
}

int wgrad_rows_per_slab(int64_t R)
{
    int64_t per = (R + 383) / 384;
    if (per < 256) per = 256;
    return static_cast<int>((per + kWgRB - 1) / kWgRB * kWgRB);
}

// Whether the projection's gradient is formed in one pass over d e: k_bw_proj4 saves a write and a read of dx and phi, and costs
// a thousand slab sums and, with every device, an entry of the sum per node.  Gradient of layered graphs, with
// k_bw_proj_rows / with it (us), by millions of elements of dx:
//   H = 32, 4 devices   1.5 261 / 264, 2.5 387 / 379, 4.5 590 / 578     16 devices   4.5 682 / 692, 9.6 1204 / 1194
//   H = 64, 4 devices   3.8 474 / 485, 5.1 647 / 644, 11 1131 / 1114    16 devices   7.7 946 / 957, 26 2575 / 2540
//   H = 128, 4 devices  3.3 573 / 578, 5.1 736 / 732, 11 1280 / 1271    16 devices   7.7 1420 / 1434, 26 3049 / 3025
// (256 NASNet-like graphs, 102 million, 8 devices: 2.65 / 2.35 ms for projection, contractions and slab sums.)
bool proj_fused(int64_t R, int H, int D)
{
    return H % 4 == 0 && R * H >= (D > 8 ? 12000000 : H <= 32 ? 2000000 : 4300000);
}

// Four nodes in flight to a thread, and about four workgroups to a compute unit.
int proj_rows_per_slab(int64_t R, int H)
{
    const int64_t batch = 4 * (kThreads / (H / 4));
    const int64_t per = (R + 1023) / 1024;
    return static_cast<int>((per + batch - 1) / batch * batch);
}

}  // namespace

// Room for the slab sums of the contractions that one launch takes: of all of a pass, or, on large
// batches, 128 MB (half of the last-level cache, so that the sums are read back from there), or of the
// largest one.  (Gradient step of 256 NASNet-like graphs with 32 / 64 / 128 / 256 / 512 MB: 8.06 / 8.07 / 7.93 / 7.84 /
// 7.91 ms; of 48 NMT-like ones 1.284 / 1.262 / 1.250 / 1.248 / 1.248 ms.)
size_t wgrad_workspace_floats(int64_t n, int64_t B, const ModelView &mv)
{
    size_t all = 0, largest = 0;
    auto need = [&](int64_t R, int I, int J, int times) {
        if (R <= 0) return;
        const int per_a = wgrad_rows_per_slab(R), per_b = wgrad_rows_per_slab_cores(R);
        const int64_t slabs = std::max((R + per_a - 1) / per_a, (R + per_b - 1) / per_b);
        const size_t one = (static_cast<size_t>(slabs + 2) * (static_cast<size_t>(I) * J + J) + 63) / 64 * 64;   // (of three lists)
        all += times * one;
        largest = std::max(largest, one);
    };
    const int H = mv.H, L = mv.L;
    need(n, std::max(32, mv.F), H, 1);
    if (proj_fused(n, H, mv.D)) largest = std::max(largest, static_cast<size_t>(1025) * (mv.F + 1) * H);   // (slabs of the projection's)
    need(n, H, H, 4 * L + 3 * (L - 1));
    need(n, 2 * H, H, 3);
    need(B * mv.G, H, H, 3 * L);
    need(B, mv.Z, H, 1);
    need(B, H, mv.D, 1);
    return std::max(largest, std::min(all, static_cast<size_t>(32) << 20));
}

void launch_fill_zero(float *p, size_t n, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill_zero, dim3(static_cast<unsigned>((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       s, p, n);
}

namespace {

// Weight gradients waiting to be launched.  add() launches what is waiting when the slab sums of one
// more contraction have no room (wgrad_workspace_floats); the caller launches the rest with flush(),
// before anything that a waiting contraction reads is overwritten.
class WgradQueue {
public:
    WgradQueue(float *grad, float *partial, size_t capacity, int H, int generic, hipStream_t s)
        : grad_(grad), partial_(partial), capacity_(capacity), H_(H), generic_(generic), s_(s) {}

    // I_pad: A has I_pad >= n_in columns, the extra ones zero (lets a narrow layer use the matrix cores).
    // With a row list (the nodes of one set, ascending) the class filter is not needed.
    // share, n_share: this is list `share` of n_share whose lengths stand side by side and sum up to at most R, added one
    // after the other: their slab sums take the room of one list of R rows (three sets of 256 NASNet-like graphs in one
    // launch instead of one each, none of which filled the chip: gradient 7.68 -> 7.49 ms).
    void add(const float *A, int lda, const float *Dl, int ldd, int64_t R, const LayerRef &ly, int I_pad = 0,
             const uint8_t *row_cls = nullptr, int want = 0, const int32_t *list = nullptr,
             const int32_t *list_count = nullptr, int share = 0, int n_share = 1)
    {
        if (R <= 0) return;
        const int I = I_pad ? I_pad : ly.n_in, J = ly.n_out;
        const bool cores = generic_ == 0 && I % 32 == 0 && J == H_ && (J == 32 || J == 64 || J == 128);
        const int per = cores ? wgrad_rows_per_slab_cores(R) : wgrad_rows_per_slab(R);
        const int slabs = static_cast<int>((R + per - 1) / per);
        // the bf16-split kernel addresses its operands with 32-bit element offsets
        const int kind = !cores ? 1 : static_cast<double>(R) * std::max(lda, ldd) < 4.0e9 ? 0 : 2;
        if (kind != 0 || !list) share = 0, n_share = 1;
        if (share == 0) {
            // (every list may end in a slab that is not full)
            const size_t floats = (static_cast<size_t>(slabs + n_share - 1) * (static_cast<size_t>(I) * J + J) + 63) / 64 * 64;
            if (n_[0] + n_[1] + n_[2] + n_[3] + n_share > kWgradJobs || used_ + floats > capacity_) flush();
            place_ = partial_ + used_;
            used_ += floats;
        }
        jobs_[kind][n_[kind]++] = {A, Dl, list, list_count, row_cls, place_, grad_ + ly.w, lda, ldd, want,
                                   static_cast<int32_t>(R), I, J, ly.n_in, per, slabs, share, store_};
    }

    // Slab sums [slabs][n_in J + J] that another kernel takes: their place, and their sum with the next flush.
    float *add_sums(int R, int per, const LayerRef &ly)
    {
        const int slabs = (R + per - 1) / per;
        const size_t floats = (static_cast<size_t>(slabs) * (static_cast<size_t>(ly.n_in) * ly.n_out + ly.n_out) + 63) / 64 * 64;
        if (n_[0] + n_[1] + n_[2] + n_[3] == kWgradJobs || used_ + floats > capacity_) flush();
        float *at = partial_ + used_;
        jobs_[3][n_[3]++] = {nullptr, nullptr, nullptr, nullptr, nullptr, at, grad_ + ly.w, 0, 0, 0, R, ly.n_in, ly.n_out, ly.n_in, per,
                             slabs, 0, store_};
        used_ += floats;
        return at;
    }

    // Contractions added from now on are the first of their layers' in this pass, and their sums go in place of what is there.
    void store_sums(bool yes) { store_ = yes; }

    void flush()
    {
        WgradBatch wb{};
        int n = 0, blocks[2] = {0, 0}, sum_blocks = 0;
        for (int kind = 0; kind < 4; ++kind)
            for (int k = 0; k < n_[kind]; ++k, ++n) {
                const WgradJob &j = jobs_[kind][k];
                wb.job[n] = j;
                if (kind < 2) {
                    wb.first[n] = blocks[kind];
                    blocks[kind] += j.slabs * (kind == 0 ? (j.I + 127) / 128 : (j.I + kWgI - 1) / kWgI);
                }
                wb.first_sum[n] = sum_blocks;
                sum_blocks += (j.n_in * j.J + j.J + 31) / 32;
            }
        if (n == 0) return;
#define CALL(NJ)                                                                                                  \
    if (n_[0]) {                                                                                                  \
        allow_lds_bw(k_wgrad_split<NJ>, wgrad_split_lds_bytes(NJ));                                               \
        hipLaunchKernelGGL(k_wgrad_split<NJ>, dim3(blocks[0]), dim3(kThreads), wgrad_split_lds_bytes(NJ), s_, wb, n_[0]); \
    }                                                                                                             \
    for (int k = 0; k < n_[2]; ++k) {                                                                             \
        const WgradJob &j = jobs_[2][k];                                                                          \
        allow_lds_bw(k_wgrad_mfma<NJ>, wgrad_lds_bytes(NJ));                                                      \
        hipLaunchKernelGGL(k_wgrad_mfma<NJ>, dim3((j.I + 127) / 128, j.slabs), dim3(kThreads), wgrad_lds_bytes(NJ), s_, \
                           j.A, j.lda, j.Dl, j.ldd, j.rows, j.n_rows_dev, j.R, j.I, j.rows_per_slab, j.partial);  \
    }
        if (H_ == 32) { CALL(1) } else if (H_ == 64) { CALL(2) } else if (H_ == 128) { CALL(4) }
#undef CALL
        if (n_[1])
            hipLaunchKernelGGL(k_wgrad, dim3(blocks[1]), dim3(kThreads), 0, s_, wb, n_[0], n_[0] + n_[1]);
        hipLaunchKernelGGL(k_wgrad_reduce, dim3(sum_blocks), dim3(kThreads), 0, s_, wb, n);
        n_[0] = n_[1] = n_[2] = n_[3] = 0;
        used_ = 0;
    }

private:
    float *grad_, *partial_, *place_ = nullptr;
    int32_t store_ = 0;
    size_t capacity_, used_ = 0;
    int H_, generic_, n_[4] = {0, 0, 0, 0};
    hipStream_t s_;
    WgradJob jobs_[4][kWgradJobs];   // by kernel: k_wgrad_split, k_wgrad, k_wgrad_mfma; slab sums taken elsewhere
};

struct DenseCall {
    const float *X; int ldx;
    const int32_t *rows; const int32_t *n_rows_dev; int R; int K;
    const float *Wt; int ldwt;     // row j = the K inputs of output column j
    const float *bias; int relu;
    const float *M; int ldm;
    float *Y; int ldy;
    // n_lists row lists in one launch: z-th list at rows + z list_stride with count n_rows_dev[z],
    // weights at Wt + z w_stride, bias + z b_stride
    int n_lists = 1; size_t list_stride = 0, w_stride = 0, b_stride = 0;
    // n_halves blocks of output columns: block k has its weights at Wt + k wt_half and goes to Y + k y_half
    int n_halves = 1; size_t wt_half = 0; int y_half = 0;
};

void launch_dense(const DenseCall &c, int H, hipStream_t s)
{
    if (c.R <= 0) return;
    const dim3 grid((c.R + kDenseRows - 1) / kDenseRows, c.n_halves, c.n_lists);
#define CALL(NJ)                                                                                                 \
    allow_lds_bw(k_dense_split<NJ>, dense_split_lds_bytes(NJ));                                                  \
    hipLaunchKernelGGL(k_dense_split<NJ>, grid, dim3(kThreads), dense_split_lds_bytes(NJ), s, c.X, c.ldx, c.rows, \
                       c.n_rows_dev, c.R, c.K, c.Wt, c.ldwt, c.bias, c.relu, c.M, c.ldm, c.Y, c.ldy, c.list_stride, \
                       c.w_stride, c.b_stride, c.wt_half, c.y_half)
    if (H == 32) { CALL(1); } else if (H == 64) { CALL(2); } else { CALL(4); }
#undef CALL
}

}  // namespace

void launch_backward(const GraphView &gv, const ModelView &mv, const float *blob_t, const Workspace &ws,
                     const GradWorkspace &gw, const ForwardArgs &fa, const BackwardArgs &ba, int k_sweeps,
                     int pool_chunks, int generic, bool lanes, const uint4 *wfrag_bw, const float *sweep_bias, int sweep_ws,
                     const float *keep, bool pool_kept, const StageMarks *marks, hipStream_t s)
{
    if (gv.B == 0) return;
    float *grad = ba.grad;
    const int H = mv.H, L = mv.L, G = mv.G, B = gv.B, n = gv.n_tot;
    const int rpt = pick_rpt_bw(H);
    const size_t NH = static_cast<size_t>(n) * H;
    const size_t BG = static_cast<size_t>(B) * G;

    auto mark = [&](int stage, bool begin) {
        if (marks && marks->mark) marks->mark(marks->ctx, stage, begin, s);
    };
    WgradQueue wq(grad, gw.partial, gw.partial_floats, H, generic, s);
    // Unless the call adds to grad, the sums of a layer's first contraction are stored: every layer has one, but f and g
    // without a sweep.
    if (!ba.accumulate && k_sweeps == 0) launch_fill_zero(grad, ba.n_grad, s);
    const bool fresh = !ba.accumulate && k_sweeps > 0;
    // 1. head
    mark(PL_STAGE_BW_HEAD, true);
    launch_head_bw(gv, mv, blob_t, fa.cur_node,
                   {ws.hid, ws.logit, ba.actions, ba.coeff, ba.entropy_coeff, gw.hact, gw.hid, gw.dpre, gw.dlogit, gw.dz,
                    gw.dh, gw.dP, ba.out_logp, ba.out_entropy},
                   s);
    mark(PL_STAGE_BW_HEAD, false);
    mark(PL_STAGE_BW_POOL, true);
    // matrix-core dense layers: every output width of the embedding networks is H
    const bool dense = generic == 0 && (H == 32 || H == 64 || H == 128);
    // a chain that reads gate bytes and, with one sweep, activations that the forward pass kept
    const bool chain = lanes || wfrag_bw;
    // 2. pooling
    if (dense) {
        if (pool_kept) {
            constexpr int koff_ld = 3 * kMaxD + 1;
            int32_t *begins = B > kSetsAlone ? gw.blk_cnt : nullptr;
            if (begins)
                hipLaunchKernelGGL(k_bw_set_begins, dim3((B + kSetGraphs - 1) / kSetGraphs), dim3(kSetThreads), 0, s, B, G, koff_ld,
                                   ws.koff, begins, begins + 3 * static_cast<size_t>(B));
            const int threads = n > 512 * static_cast<int64_t>(B) ? kSetThreads : begins && n <= 64 * static_cast<int64_t>(B) ? 64 : kThreads;
            hipLaunchKernelGGL(k_bw_sets, dim3(B), dim3(threads), 0, s, gv, H,
                               mv.Z, G, mv.D, mv.single_set, koff_ld, ws.reach, fa.placement, fa.cur_node, ws.klist, ws.koff,
                               gw.dz, begins, gw.cls, gw.counts, gw.lists, gw.demb);
        } else {
            const int n_blocks = (n + kThreads - 1) / kThreads;
            hipLaunchKernelGGL(k_bw_cls_count, dim3(n_blocks), dim3(kThreads), 0, s, gv, H, mv.Z, mv.single_set, ws.reach,
                               fa.cur_node, gw.dz, gw.cls, gw.blk_cnt, gw.demb);
            hipLaunchKernelGGL(k_bw_cls_scan, dim3(1), dim3(kThreads), 0, s, n_blocks, gw.blk_cnt, gw.counts);
            hipLaunchKernelGGL(k_bw_cls_fill, dim3(n_blocks), dim3(kThreads), 0, s, gv, gw.cls, gw.blk_cnt, gw.lists);
        }
        for (int set = 0; set < 3; ++set) {
            const int32_t *list = gw.lists + static_cast<size_t>(set) * n, *cnt = gw.counts + set;
            const MlpRef &ln = mv.l[set];
            for (int l = 0; l < L && !pool_kept; ++l)     // kept: the forward pooling kernel wrote lact
                launch_dense({l == 0 ? ws.emb : gw.lact + static_cast<size_t>(l - 1) * NH, l == 0 ? 2 * H : H, list,
                              cnt, n, l == 0 ? 2 * H : H, blob_t + ln.layer[l].w, l == 0 ? 2 * H : H,
                              mv.blob + ln.layer[l].b, 1, nullptr, 0, gw.lact + static_cast<size_t>(l) * NH, H}, H, s);
        }
        // Where the forward pooling kernel kept l's layer outputs and its reverse is built, one pass
        // over the same tiles gives the deltas of l's layers and d e; else the dense-layer kernels.
        const bool stream_bw = pool_kept && ba.pool_bw_frag != nullptr;
        if (stream_bw) {
            launch_pool_stream_bw(gv, mv, ws, ba.pool_bw_frag, gw.lact, gw.dP, gw.dl, gw.demb, s);
        } else {
        hipLaunchKernelGGL(k_bw_pool_seed, dim3(static_cast<unsigned>((NH / 4 + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, s, gv, H, G, mv.D, gw.cls, fa.placement, gw.dP,
                           gw.lact + static_cast<size_t>(L - 1) * NH, gw.dl + static_cast<size_t>(L - 1) * NH);
        {
            // back through l's layers, the three sets' row lists in one launch each.  The weights go
            // in as they are stored (row i of a layer = the outputs fed by input i), which is the
            // transposed layout of this contraction; the three networks are equally far apart.
            const MlpRef &l0 = mv.l[0];
            const size_t w_stride = static_cast<size_t>(mv.l[1].layer[0].w - l0.layer[0].w);
            for (int l = L - 1; l >= 1; --l) {
                DenseCall c{gw.dl + static_cast<size_t>(l) * NH, H, gw.lists, gw.counts, n, H, mv.blob + l0.layer[l].w, H,
                            nullptr, 0, gw.lact + static_cast<size_t>(l - 1) * NH, H,
                            gw.dl + static_cast<size_t>(l - 1) * NH, H};
                c.n_lists = 3;
                c.list_stride = static_cast<size_t>(n);
                c.w_stride = w_stride;
                launch_dense(c, H, s);
            }
            // the first layer is [2H, H]: inputs half H .. half H + H - 1
            DenseCall c{gw.dl, H, gw.lists, gw.counts, n, H, mv.blob + l0.layer[0].w, H, nullptr, 0, nullptr, 0, gw.demb, 2 * H};
            c.n_lists = 3;
            c.list_stride = static_cast<size_t>(n);
            c.w_stride = w_stride;
            c.n_halves = 2;
            c.wt_half = static_cast<size_t>(H) * H;
            c.y_half = H;
            launch_dense(c, H, s);
        }
        }
    } else {
        const size_t lds = sizeof(float) * kTile * 4 * H;
#define CALL(R)                                                                                             \
    allow_lds_bw(k_bw_pool<R>, lds);                                                                        \
    hipLaunchKernelGGL(k_bw_pool<R>, dim3(pool_chunks, B), dim3(kThreads), lds, s, gv, mv, blob_t, ws.emb,  \
                       ws.reach, fa.placement, fa.cur_node, gw.dP, gw.dz, gw.cls, gw.lact, gw.dl, gw.demb, \
                       pool_chunks)
        PL_DISPATCH_RPT(rpt, CALL)
#undef CALL
    }
    mark(PL_STAGE_BW_POOL, false);
    // 3. sweeps.  Where the layer outputs live: kept by the forward sweep (keep: slot 0 a_v, slots
    // 1 .. L g's layers, then f's layers but the last), or recomputed into fact / gact / agg.
    auto agg_of = [&](int dir) {
        return keep ? keep + dir * gw.dfg_stride : gw.agg + static_cast<size_t>(dir) * NH;
    };
    auto gact_of = [&](int dir, int l) {
        return keep ? keep + dir * gw.dfg_stride + static_cast<size_t>(1 + l) * NH
                    : gw.gact + (static_cast<size_t>(dir) * L + l) * NH;
    };
    auto fact_of = [&](int dir, int l) {       // l < L - 1 on the keep path (the last layer is ws.msg)
        return keep ? keep + dir * gw.dfg_stride + static_cast<size_t>(1 + L + l) * NH
                    : gw.fact + (static_cast<size_t>(dir) * L + l) * NH;
    };
    // one sweep at a time, from the last to the first: demb holds the outside gradient of the sweep's
    // output on entry and the gradient of its input on exit; the states and messages of an earlier
    // sweep come from the snapshots taken during the forward pass
    for (int j = k_sweeps - 1; j >= 0; --j) {
    const float *emb_j = j == k_sweeps - 1 ? ws.emb : ba.snap_emb + static_cast<size_t>(j) * 2 * NH;
    const float *msg_j = j == k_sweeps - 1 ? ws.msg : ba.snap_msg + static_cast<size_t>(j) * 2 * NH;
    mark(PL_STAGE_BW_ACTS, true);
    if (dense && !keep) {
        // the last layer of f is the message itself, which the forward pass left in msg_j (the
        // generic chain kernel reads it from fact, so there it is computed again)
        for (int dir = 0; dir < 2; ++dir)
            for (int l = 0; l + 1 < L || (l < L && !chain); ++l) {
                const LayerRef &ly = mv.f[dir].layer[l];
                launch_dense({l == 0 ? emb_j + dir * H : gw.fact + (static_cast<size_t>(dir) * L + l - 1) * NH,
                              l == 0 ? 2 * H : H, nullptr, nullptr, n, H, blob_t + ly.w, H, mv.blob + ly.b, 1,
                              nullptr, 0, gw.fact + (static_cast<size_t>(dir) * L + l) * NH, H}, H, s);
            }
        hipLaunchKernelGGL(k_bw_agg, dim3(static_cast<unsigned>((NH / 4 + kThreads - 1) / kThreads), 2), dim3(kThreads),
                           0, s, gv, H, msg_j, gw.agg);
        for (int dir = 0; dir < 2; ++dir)
            for (int l = 0; l < L; ++l) {
                const LayerRef &ly = mv.g[dir].layer[l];
                launch_dense({l == 0 ? gw.agg + static_cast<size_t>(dir) * NH
                                     : gw.gact + (static_cast<size_t>(dir) * L + l - 1) * NH,
                              H, nullptr, nullptr, n, H, blob_t + ly.w, H, mv.blob + ly.b, 1, nullptr, 0,
                              gw.gact + (static_cast<size_t>(dir) * L + l) * NH, H}, H, s);
            }
    }
    {
        const size_t lds = sizeof(float) * 2 * kTile * H;
        const unsigned tiles = static_cast<unsigned>((n + kTile - 1) / kTile);
        if (!dense && !keep) {
#define CALL(R)                                                                                              \
    allow_lds_bw(k_bw_f_acts<R>, lds);                                                                       \
    allow_lds_bw(k_bw_g_acts<R>, lds);                                                                       \
    hipLaunchKernelGGL(k_bw_f_acts<R>, dim3(tiles, 2), dim3(kThreads), lds, s, gv, mv, emb_j, gw.fact);     \
    hipLaunchKernelGGL(k_bw_g_acts<R>, dim3(tiles, 2), dim3(kThreads), lds, s, gv, mv, gw.fact, gw.agg, gw.gact)
            PL_DISPATCH_RPT(rpt, CALL)
#undef CALL
        }
        if (chain && !keep) {
            // the forward sweep that keeps activations also writes the gate bytes; otherwise they
            // are taken from the recomputed layer outputs here
            GateSrc src[2];
            for (int sd = 0; sd < 2; ++sd) {
                src[sd].m = dense ? msg_j + static_cast<size_t>(sd) * NH : fact_of(sd, L - 1);
                src[sd].f0 = L == 2 ? fact_of(sd, 0) : nullptr;
                src[sd].g_last = gact_of(sd, L - 1);
                src[sd].g0 = L == 2 ? gact_of(sd, 0) : nullptr;
            }
            hipLaunchKernelGGL(k_bw_gates, dim3(static_cast<unsigned>((NH + kThreads - 1) / kThreads)),
                               dim3(kThreads), 0, s, gv, H, L, src[0], src[1], gw.mask4);
        }
        mark(PL_STAGE_BW_ACTS, false);
        mark(PL_STAGE_BW_CHAIN, true);
        if (lanes) {
            launch_sweep_lanes_bw(gv, mv, blob_t, fa.cur_node, gw.demb, gw.dagg, gw.mask4, gw.dfg, gw.dfg_stride, s);
        } else if (wfrag_bw) {
            launch_sweep_mfma_bw(gv, mv, wfrag_bw, sweep_bias, sweep_ws, fa.cur_node, gw.demb, gw.dagg, gw.mask4,
                                 gw.dfg, gw.dfg_stride, s);
        } else {
#define CALL(R)                                                                                            \
    allow_lds_bw(k_bw_sweep_generic<R>, lds);                                                              \
    hipLaunchKernelGGL(k_bw_sweep_generic<R>, dim3(B, 2), dim3(kThreads), lds, s, gv, mv, blob_t, gw.fact, \
                       gw.gact, gw.demb, gw.dagg, gw.dfg, gw.dfg_stride)
            PL_DISPATCH_RPT(rpt, CALL)
#undef CALL
        }
        mark(PL_STAGE_BW_CHAIN, false);
    }
    {
        mark(PL_STAGE_BW_WGRAD, true);
        wq.store_sums(fresh && j == k_sweeps - 1);
        for (int dir = 0; dir < 2; ++dir)
            for (int l = 0; l < L; ++l) {
                const float *dfl = gw.dfg + dir * gw.dfg_stride + static_cast<size_t>(l) * NH;
                const float *dgl = dfl + static_cast<size_t>(L) * NH;
                const float *fin = l == 0 ? emb_j + dir * H : fact_of(dir, l - 1);
                wq.add(fin, l == 0 ? 2 * H : H, dfl, H, n, mv.f[dir].layer[l]);
                const float *gin = l == 0 ? agg_of(dir) : gact_of(dir, l - 1);
                wq.add(gin, H, dgl, H, n, mv.g[dir].layer[l]);
            }
        if (j > 0) wq.flush();    // the sweep before this one overwrites the deltas and layer outputs
        mark(PL_STAGE_BW_WGRAD, false);
    }
    }
    // 4. projection
    mark(PL_STAGE_BW_PROJ, true);
    wq.store_sums(fresh);
    {
        if (proj_fused(n, H, mv.D)) {
            const int per = proj_rows_per_slab(n, H);
            float *sums = wq.add_sums(n, per, mv.proj);
#define CALL(DM)                                                                                                       \
    hipLaunchKernelGGL(k_bw_proj4<DM>, dim3((n + per - 1) / per), dim3(kThreads), 0, s, gv, mv, fa.node_feats, fa.placement, \
                       fa.cur_node, gw.demb, per, sums)
            if (mv.D <= 4) { CALL(4); } else if (mv.D <= 8) { CALL(8); } else { CALL(kMaxD); }
#undef CALL
        } else {
            const auto rows = H % 4 == 0 ? k_bw_proj_rows : k_bw_proj;
            const size_t threads = H % 4 == 0 ? NH / 4 : NH;
            hipLaunchKernelGGL(rows, dim3(static_cast<unsigned>((threads + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                               gv, mv, fa.node_feats, fa.placement, fa.cur_node, gw.demb, gw.dx, gw.phi, dense ? 32 : mv.F);   // (raw features padded to 32 columns)
            if (H < mv.F) {
                const size_t tf = static_cast<size_t>(n) * mv.F;
                hipLaunchKernelGGL(k_bw_phi, dim3(static_cast<unsigned>((tf + kThreads - 1) / kThreads)),
                                   dim3(kThreads), 0, s, gv, mv, fa.node_feats, fa.placement, fa.cur_node, gw.phi);
            }
            wq.add(gw.phi, dense ? 32 : mv.F, gw.dx, H, n, mv.proj, dense ? 32 : 0);
        }
    }
    mark(PL_STAGE_BW_PROJ, false);
    // 5. weight gradients
    mark(PL_STAGE_BW_WGRAD, true);
    for (int l = 0; l < L; ++l)
        for (int set = 0; set < 3; ++set)
            wq.add(l == 0 ? ws.emb : gw.lact + static_cast<size_t>(l - 1) * NH, l == 0 ? 2 * H : H,
                   gw.dl + static_cast<size_t>(l) * NH, H, n, mv.l[set].layer[l], 0, gw.cls, set + 1,
                   dense ? gw.lists + static_cast<size_t>(set) * n : nullptr, dense ? gw.counts + set : nullptr, set, 3);
    for (int set = 0; set < 3; ++set)
        for (int l = 0; l < L; ++l)
            wq.add(l == 0 ? gw.hin + static_cast<size_t>(set) * BG * H
                          : gw.hact + (static_cast<size_t>(set) * L + l - 1) * BG * H,
                   H, gw.dh + (static_cast<size_t>(set) * L + l) * BG * H, H, static_cast<int64_t>(BG), mv.h[set].layer[l]);
    wq.add(ws.zbuf, mv.Z, gw.dpre, H, B, mv.pol1);
    wq.add(gw.hid, H, gw.dlogit, mv.D, B, mv.pol2);
    wq.flush();
    mark(PL_STAGE_BW_WGRAD, false);
}

}  // namespace pl
