// One MDP transition (Section 2.1) for every graph of a batch, on the device: the sampled
// action updates the current node's placement, the node is marked visited, and the next node
// of the visiting order becomes current.  One thread per graph: the work is B x D numbers.
#include <algorithm>

#include "internal.h"

namespace pl {

namespace {

// softmax over a graph's D logits (Appendix A.7) and inverse CDF over devices 0 .. D-1: the first device whose
// cumulative weight exceeds u x total.  Returns the action, its log-probability in logp.
__device__ __forceinline__ int sample_action(const float *__restrict__ logits, int D, float u, float &logp)
{
    float e[kMaxD];
    float m = -INFINITY;
    for (int d = 0; d < D; ++d) m = fmaxf(m, logits[d]);
    float total = 0.0f;
    for (int d = 0; d < D; ++d) {
        e[d] = expf(logits[d] - m);
        total += e[d];
    }
    const float thr = u * total;
    int a = D - 1;
    float c = 0.0f;
    for (int d = 0; d < D; ++d) {
        c += e[d];
        if (c > thr) {
            a = d;
            break;
        }
    }
    logp = logits[a] - m - logf(total);
    return a;
}

__global__ __launch_bounds__(256) void k_episode_step(GraphView gv, int D, const float *__restrict__ logits,
                                                      const float *__restrict__ uniforms,
                                                      const int32_t *__restrict__ order, int t,
                                                      float *__restrict__ node_feats,
                                                      int32_t *__restrict__ placement,
                                                      int32_t *__restrict__ cur_node,
                                                      int32_t *__restrict__ out_action,
                                                      float *__restrict__ out_logp)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= gv.B) return;
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int cl = cur_node[b];
    if (cl < 0 || cl >= n_b) {             // the graph's episode is over (or the state is invalid)
        cur_node[b] = -1;
        if (out_action) out_action[b] = -1;
        if (out_logp) out_logp[b] = 0.0f;
        return;
    }
    float logp;
    const int a = sample_action(logits + static_cast<size_t>(b) * D, D, uniforms[b], logp);
    if (out_action) out_action[b] = a;
    if (out_logp) out_logp[b] = logp;
    placement[n0 + cl] = a;
    node_feats[static_cast<size_t>(n0 + cl) * 3 + 2] = 1.0f;
    cur_node[b] = (t + 1 < n_b) ? order[n0 + t + 1] : -1;
}

// ---- steps taken ahead: every state that the next steps of an episode can reach
// A pass over a few graphs is one chain of levels, two workgroups of it a graph, and leaves the rest of the chip idle: a
// batch of 73 NASNet-like graphs takes 1.41 ms, one graph 1.32.  So where a batch is that small, the states that its
// graphs are in after 0, 1, .. steps, one for every sequence of actions, go through the forward pass together as copies
// of the batch, and the actions are drawn afterwards, a step after the other, each from the logits of the state that the
// ones before it led to.  The logits of a state do not depend on the batch that it is in, so nothing else changes.
// Copies are numbered by depth: copy 0 is the state as it stands, the copies of the states reached by actions
// a_0 .. a_{i-1} are those from (D^i - 1) / (D - 1) on, in the order of the actions as digits of base D.

// Offsets of the copies' graphs; which plan they use and the graph of every node (nothing else of the graph is read
// on the paths that take copies).
__global__ __launch_bounds__(256) void k_copies_index(GraphView gv, int copies, int32_t *__restrict__ node_off,
                                                      int32_t *__restrict__ tmpl, int32_t *__restrict__ node_graph)
{
    const int i = blockIdx.x * 256 + threadIdx.x, graphs = copies * gv.B;
    if (i <= graphs) node_off[i] = i == graphs ? copies * gv.n_tot : i / gv.B * gv.n_tot + gv.node_off[i % gv.B];
    if (i < graphs) tmpl[i] = gv.tmpl[i % gv.B];
    if (i < gv.n_tot) {
        const int b = gv.node_graph[i];
        for (int j = 0; j < copies; ++j) node_graph[static_cast<size_t>(j) * gv.n_tot + i] = j * gv.B + b;
    }
}

// States of the copies: a workgroup takes 256 nodes of one graph of one copy.  The first one also clears what the pass
// reads as zero without writing it (workspace.cpp), whose place depends on the number of copies.
__global__ __launch_bounds__(256) void k_copies_state(GraphView gv, int D, const int32_t *__restrict__ order, int t,
                                                      const float *__restrict__ feats,
                                                      const int32_t *__restrict__ placement,
                                                      const int32_t *__restrict__ cur_node,
                                                      float *__restrict__ out_feats,
                                                      int32_t *__restrict__ out_placement,
                                                      int32_t *__restrict__ out_cur, float *__restrict__ zero_msg,
                                                      int n_zero_msg, uint32_t *__restrict__ zero_reach)
{
    const int b = blockIdx.y, j = blockIdx.z;
    if (blockIdx.x == 0 && b == 0 && j == 0) {
        for (int i = threadIdx.x; i < n_zero_msg; i += 256) zero_msg[i] = 0.0f;
        if (threadIdx.x < 5) zero_reach[threadIdx.x] = 0u;
    }
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int v = blockIdx.x * 256 + threadIdx.x;
    int depth = 0, index = j;
    for (int states = 1; index >= states; states *= D, ++depth) index -= states;
    int scale = 1;
    for (int i = 1; i < depth; ++i) scale *= D;
    const bool in = v < n_b;
    const size_t from = static_cast<size_t>(n0) + (in ? v : 0);
    float vis = feats[from * 3 + 2];
    int device = placement[from];
    int cur = cur_node[b];
    for (int i = 0; i < depth; ++i, scale = scale > D ? scale / D : 1) {
        if (cur < 0 || cur >= n_b) {
            cur = -1;
            break;
        }
        if (v == cur) {
            vis = 1.0f;
            device = index / scale % D;
        }
        cur = t + i + 1 < n_b ? order[n0 + t + i + 1] : -1;
    }
    if (in) {
        const size_t to = static_cast<size_t>(j) * gv.n_tot + from;
        out_feats[to * 3] = feats[from * 3];
        out_feats[to * 3 + 1] = feats[from * 3 + 1];
        out_feats[to * 3 + 2] = vis;
        out_placement[to] = device;
    }
    if (v == 0) out_cur[static_cast<size_t>(j) * gv.B + b] = cur;
}

// The steps themselves, a thread to a graph, on the logits of the copies.  logits_stride: floats between the steps of
// out_logits (0: the last step's are kept).
__global__ __launch_bounds__(256) void k_copies_steps(GraphView gv, int D, int steps,
                                                      const float *__restrict__ copy_logits,
                                                      const float *__restrict__ uniforms,
                                                      const int32_t *__restrict__ order, int t,
                                                      float *__restrict__ node_feats,
                                                      int32_t *__restrict__ placement,
                                                      int32_t *__restrict__ cur_node,
                                                      float *__restrict__ out_logits, size_t logits_stride,
                                                      int32_t *__restrict__ out_action,
                                                      float *__restrict__ out_logp)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= gv.B) return;
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    int cl = cur_node[b];
    int first = 0, states = 1, index = 0;
    for (int i = 0; i < steps; ++i) {
        const float *l = copy_logits + (static_cast<size_t>(first + index) * gv.B + b) * D;
        const size_t at = static_cast<size_t>(i) * gv.B + b;
        float *keep = out_logits + i * logits_stride + static_cast<size_t>(b) * D;
        for (int d = 0; d < D; ++d) keep[d] = l[d];
        int a = -1;
        float logp = 0.0f;
        if (cl < 0 || cl >= n_b) {
            cl = -1;
        } else {
            a = sample_action(l, D, uniforms[at], logp);
            placement[n0 + cl] = a;
            node_feats[static_cast<size_t>(n0 + cl) * 3 + 2] = 1.0f;
            cl = (t + i + 1 < n_b) ? order[n0 + t + i + 1] : -1;
        }
        if (out_action) out_action[at] = a;
        if (out_logp) out_logp[at] = logp;
        first += states;
        states *= D;
        index = index * D + (a < 0 ? 0 : a);
    }
    cur_node[b] = cl;
}

// The same transition with a given action (replay of a recorded episode): nothing is sampled.
// A graph whose episode is over, or whose action is outside [0, D), only has its current node
// set to -1.
__global__ __launch_bounds__(256) void k_episode_apply(GraphView gv, int D, const int32_t *__restrict__ actions,
                                                       const int32_t *__restrict__ order, int t,
                                                       float *__restrict__ node_feats,
                                                       int32_t *__restrict__ placement,
                                                       int32_t *__restrict__ cur_node)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= gv.B) return;
    const int n0 = gv.node_off[b], n_b = gv.node_off[b + 1] - n0;
    const int cl = cur_node[b];
    const int a = actions[b];
    if (cl < 0 || cl >= n_b || a < 0 || a >= D) {
        cur_node[b] = -1;
        return;
    }
    placement[n0 + cl] = a;
    node_feats[static_cast<size_t>(n0 + cl) * 3 + 2] = 1.0f;
    cur_node[b] = (t + 1 < n_b) ? order[n0 + t + 1] : -1;
}

// Weights of the REINFORCE sum (appendix "REINFORCE Algorithm", Eq. 1): the return that follows
// every decision, G[t][b] = sum_{t' >= t} r[t'][b] (one thread per rollout, from the last step
// backwards), the per-step baseline of every group of rollouts (mean of G[t][.] over the group,
// members added in ascending order), and their difference.
__global__ __launch_bounds__(256) void k_returns(int T, int B, const float *__restrict__ rewards,
                                                 float *__restrict__ coeff)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    float g = 0.0f;
    for (int t = T - 1; t >= 0; --t) {
        g += rewards[static_cast<size_t>(t) * B + b];
        coeff[static_cast<size_t>(t) * B + b] = g;
    }
}

__global__ __launch_bounds__(256) void k_baseline(int T, int B, int n_groups, const float *__restrict__ G,
                                                  const int32_t *__restrict__ group,
                                                  float *__restrict__ baseline)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= T * n_groups) return;
    const int t = idx / n_groups, g = idx - t * n_groups;
    float sum = 0.0f;
    int cnt = 0;
    for (int b = 0; b < B; ++b)
        if (group[b] == g) {
            sum += G[static_cast<size_t>(t) * B + b];
            ++cnt;
        }
    baseline[idx] = cnt ? sum / static_cast<float>(cnt) : 0.0f;
}

__global__ __launch_bounds__(256) void k_advantage(int T, int B, int n_groups, const int32_t *__restrict__ group,
                                                   const float *__restrict__ baseline,
                                                   float *__restrict__ coeff)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= T * B) return;
    const int t = idx / B, b = idx - t * B;
    const int g = group[b];
    if (g >= 0 && g < n_groups) coeff[idx] -= baseline[static_cast<size_t>(t) * n_groups + g];
}

}  // namespace

void launch_episode_apply(const GraphView &gv, int D, const int32_t *actions, const int32_t *order, int t,
                          float *node_feats, int32_t *placement, int32_t *cur_node, hipStream_t s)
{
    if (gv.B == 0) return;
    hipLaunchKernelGGL(k_episode_apply, dim3((gv.B + 255) / 256), dim3(256), 0, s, gv, D, actions, order, t,
                       node_feats, placement, cur_node);
}

void launch_reinforce_coeff(int T, int B, int n_groups, const float *rewards, const int32_t *group,
                            float *coeff, float *baseline, hipStream_t s)
{
    if (T <= 0 || B <= 0) return;
    hipLaunchKernelGGL(k_returns, dim3((B + 255) / 256), dim3(256), 0, s, T, B, rewards, coeff);
    if (n_groups <= 0) return;
    hipLaunchKernelGGL(k_baseline, dim3((T * n_groups + 255) / 256), dim3(256), 0, s, T, B, n_groups, coeff, group,
                       baseline);
    hipLaunchKernelGGL(k_advantage, dim3((T * B + 255) / 256), dim3(256), 0, s, T, B, n_groups, group, baseline,
                       coeff);
}

void launch_copies_index(const GraphView &gv, int copies, int32_t *node_off, int32_t *tmpl, int32_t *node_graph,
                         hipStream_t s)
{
    const int n = std::max(gv.n_tot, copies * gv.B + 1);
    hipLaunchKernelGGL(k_copies_index, dim3((n + 255) / 256), dim3(256), 0, s, gv, copies, node_off, tmpl, node_graph);
}

void launch_copies_state(const GraphView &gv, int D, int copies, int n_max, const int32_t *order, int t, const float *feats,
                         const int32_t *placement, const int32_t *cur_node, const EpisodeCopies &c, hipStream_t s)
{
    const size_t spare = 2 * static_cast<size_t>(c.view.n_tot);
    hipLaunchKernelGGL(k_copies_state, dim3((n_max + 255) / 256, gv.B, copies), dim3(256), 0, s, gv, D, order, t, feats,
                       placement, cur_node, c.feats, c.placement, c.cur_node, c.ws.msg + spare * c.ws.H, 2 * c.ws.H,
                       reinterpret_cast<uint32_t *>(c.ws.reach + spare / 4 * 4));
}

void launch_copies_steps(const GraphView &gv, int D, int steps, const float *copy_logits, const float *uniforms,
                         const int32_t *order, int t, float *node_feats, int32_t *placement, int32_t *cur_node,
                         float *out_logits, size_t logits_stride, int32_t *out_action, float *out_logp, hipStream_t s)
{
    hipLaunchKernelGGL(k_copies_steps, dim3((gv.B + 255) / 256), dim3(256), 0, s, gv, D, steps, copy_logits, uniforms,
                       order, t, node_feats, placement, cur_node, out_logits, logits_stride, out_action, out_logp);
}

void launch_episode_step(const GraphView &gv, int D, const float *logits, const float *uniforms,
                         const int32_t *order, int t, float *node_feats, int32_t *placement,
                         int32_t *cur_node, int32_t *out_action, float *out_logp, hipStream_t s)
{
    if (gv.B == 0) return;
    hipLaunchKernelGGL(k_episode_step, dim3((gv.B + 255) / 256), dim3(256), 0, s, gv, D, logits, uniforms, order,
                       t, node_feats, placement, cur_node, out_action, out_logp);
}

}  // namespace pl
