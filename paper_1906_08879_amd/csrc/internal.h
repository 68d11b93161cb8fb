// Internal declarations shared by the host layout builder, the C ABI and the kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

#include "placeto.h"
#include "sweep_plan.h"

namespace pl {

constexpr int kMaxD = 16;
constexpr int kMaxH = 256;
constexpr int kMaxLayers = 4;
constexpr int kMaxSweeps = 8;

void set_error(const std::string &msg);
int fail(int code, const std::string &msg);
int hip_fail(hipError_t e, const char *what);

#define PL_HIP(call)                                             \
    do {                                                         \
        hipError_t e__ = (call);                                 \
        if (e__ != hipSuccess) return ::pl::hip_fail(e__, #call); \
    } while (0)

// ---- host-side layout of a batch (Section 2.2 step 2 needs parents and children of every
// node and an order in which all of a node's neighbours are final before the node).
struct HostLayout {
    int32_t B = 0;
    int64_t n_tot = 0, e_tot = 0;
    int32_t max_depth = 0;
    std::vector<int64_t> node_off;   // [B+1]
    std::vector<int64_t> edge_off;   // [B+1]
    std::vector<int64_t> par_ptr;    // [n_tot+1] into par_idx
    std::vector<int64_t> chi_ptr;    // [n_tot+1]
    std::vector<int32_t> par_idx;    // [e_tot] graph-local ids, ascending per node
    std::vector<int32_t> chi_idx;    // [e_tot]
    std::vector<int32_t> td_level;   // [n_tot]
    std::vector<int32_t> bu_level;   // [n_tot]
    std::vector<int32_t> td_order;   // [n_tot] graph-local ids by (level, id)
    std::vector<int32_t> bu_order;   // [n_tot]
    std::vector<int32_t> depth;      // [B] number of levels (same in both directions)
    std::vector<int64_t> lvl_off;    // [B+1] offset of graph b's level pointers
    std::vector<int32_t> td_lvl_ptr; // [lvl_off[B]] per graph depth+1 positions into its order
    std::vector<int32_t> bu_lvl_ptr; // same for bottom-up
    // graphs of the same topology (the rollouts of one graph) share what depends on the
    // topology alone: graph b uses the plan of template tmpl[b]; tmpl_graph[t] is a graph with it
    int32_t n_templates = 0;
    std::vector<int32_t> tmpl;       // [B]
    std::vector<int32_t> tmpl_graph; // [n_templates]
};

int build_layout(int32_t B, const int32_t *n_nodes, const int32_t *n_edges,
                 const int32_t *edge_src, const int32_t *edge_dst, HostLayout *out);
// The layout of R copies of the one graph of `one`, equal to what build_layout gives for the
// graph repeated R times, with all copies sharing one template.
int replicate_layout(const HostLayout &one, int32_t R, HostLayout *out);

// ---- device-side view of a batch, passed to kernels by value
struct GraphView {
    int32_t B;
    int32_t n_tot;
    const int32_t *node_off;   // [B+1]
    const int32_t *lvl_off;    // [B+1]
    // index 0 = top-down (neighbours = parents), 1 = bottom-up (neighbours = children)
    const int32_t *nbr_ptr[2]; // [n_tot+1]
    const int32_t *nbr_idx[2]; // [e_tot] GLOBAL node ids
    const int32_t *order[2];   // [n_tot] GLOBAL node ids by (graph, level, id)
    const int32_t *lvl_ptr[2]; // per graph depth+1 GLOBAL positions into order
    const int32_t *node_graph; // [n_tot] graph of each node
    const int32_t *pos[2];     // [n_tot] bucket position of each node (inverse of order)
    const int32_t *tmpl;       // [B] which plan (distinct topology) graph b uses
    SweepPlanView plan[2];     // per direction
};

// ---- parameters: offsets (in floats) of every layer inside the fp32 device blob
struct LayerRef {
    int32_t w;      // offset of the [in,out] matrix
    int32_t b;      // offset of the bias
    int32_t n_in;
    int32_t n_out;
};

struct MlpRef {
    LayerRef layer[kMaxLayers];
};

struct ModelView {
    int32_t D, H, L, G, Z, F;
    int32_t single_set;      // 1: every node other than v* belongs to the first node set
    const float *blob;       // fp32 (bf16-rounded values when the model stores bf16)
    LayerRef proj;
    MlpRef f[2], g[2];       // [direction]
    MlpRef l[3], h[3];       // [set]: parents, children, parallel
    LayerRef pol1, pol2;
};

// ---- scratch owned by a batch for one (H, G)
struct Workspace {
    unsigned char *base = nullptr;  // the one allocation that holds every buffer but reach (null: not owned)
    float *emb = nullptr;       // [n_tot, 2H]  [td ; bu]
    float *msg = nullptr;       // [2, n_tot, H]
    float *xb = nullptr;        // [2, n_tot, H]  input of sweeps after the first, in bucket order (not on the generic path)
    float4 *featb = nullptr;    // [n_tot] raw-feature records in node order (sweep of 128 columns)
    uint8_t *reach = nullptr;   // [2, n_tot]   0: descendant-of-v* bit, 1: ancestor-of-v* bit
    float *partial = nullptr;   // [B, n_chunks_max, 3G, H] pooling partial sums
    // for the reverse pass (null: not kept)
    float *zbuf = nullptr;      // [B, Z] policy inputs
    double *hid = nullptr;      // [B, H] hidden layer of the policy network
    float *logit = nullptr;     // [B, D] (room for kMaxD) logits, also of graphs that have no valid current node
    double *hidp = nullptr;     // [B, 3, H] the node sets' parts of the first policy layer (H >= 128)
    uint32_t *head_done = nullptr;   // [B] workgroups of a graph that have written theirs; cleared by the pooling kernels
    int32_t *klist = nullptr;   // [n_tot] node ids grouped by (set, device group), per graph (matrix-core pooling)
    int32_t *koff = nullptr;    // [B][3 kMaxD + 1] first position of every key within its graph
    int32_t n_chunks = 0;
    int32_t H = 0, G = 0;
};

// ---- copies of a batch, one for every state that the next steps of an episode can reach (kernels_episode.hip)
// Room for them, kept by the batch: tables of the copies' graphs for `most` copies, of which fewer copies read the
// beginning, and behind them what a pass writes.  The tables depend on the batch alone and are written once, when the
// room is made; everything behind them is laid out, and cleared where it has to read as zero, by every pass for itself.
// So passes of any networks and numbers of copies, replayed captured ones among them, can follow each other in any order,
// as long as a room stays where it is: it is never moved and lives as long as the batch.
struct CopiesRoom {
    unsigned char *base;
    size_t bytes;
    int32_t most;
};
constexpr int kCopiesRooms = 8;
struct EpisodeRooms {
    CopiesRoom room[kCopiesRooms] = {};
    int32_t n = 0;
    size_t bytes = 0;                                     // of all rooms
    size_t refused = std::numeric_limits<size_t>::max();  // smallest size that there was no memory for
};

// What one pass finds in a room.
struct EpisodeCopies {
    float *feats = nullptr, *logits = nullptr;       // [copies, n_tot, 3], [copies, B, D]
    int32_t *placement = nullptr, *cur_node = nullptr;
    Workspace ws;
    GraphView view{};
};

// (workspace.cpp)
bool workspace_fits(const Workspace &ws, const ModelView &mv);
size_t carve_workspace(unsigned char *base, size_t n, size_t B, const ModelView &mv, bool with_reach, Workspace *ws);
size_t carve_copies(unsigned char *base, size_t n, size_t B, int most, int copies, const ModelView &mv, EpisodeCopies *c);
const CopiesRoom *find_room(const EpisodeRooms &rooms, size_t n, size_t B, int copies, const ModelView &mv);
size_t new_room_bytes(const EpisodeRooms &rooms, size_t n, size_t B, int most, const ModelView &mv);
const CopiesRoom *add_room(EpisodeRooms *rooms, unsigned char *base, size_t bytes, int most);

// ---- kernel launchers (kernels_generic.hip)
struct ForwardArgs {
    const float *node_feats;
    const int32_t *placement;
    const int32_t *cur_node;
    float *out_logits;
    float *out_probs;
    float *out_pooled;
    // inputs [3, B G, H] and layer outputs [3, L, B G, H] of h, kept for the reverse pass, or null
    float *keep_hin = nullptr;
    float *keep_hact = nullptr;
};

constexpr int kPoolChunk = 128;   // nodes per slice of a graph's pooling
// Slices of a graph of n nodes: one for every 128 nodes, in small graphs for every 64 up to six (pooling of 64 layered
// graphs of 200 nodes, H = 32, with two and with four: 13.8 / 10.8 us; forward pass of 256 of them at H = 48 582 / 499 us, at
// H = 128 189 / 170; of one of 300 nodes at H = 32 with four and with five 75.6 / 74.5 us; of 128 Inception-like graphs of 590
// nodes with five and with six 275.5 / 277).
__host__ __device__ inline int pool_slices(int n, int most)
{
    const int by_chunk = (n + kPoolChunk - 1) / kPoolChunk, by_half = (2 * n + kPoolChunk - 1) / kPoolChunk;
    const int want = by_chunk > 6 ? by_chunk : (by_half < 6 ? by_half : 6);
    return want < most ? want : most;
}

void launch_project(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                    const ForwardArgs &fa, bool to_emb, bool to_xb, hipStream_t s);
void launch_sweep_generic(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                          const ForwardArgs &fa, bool write_reach, hipStream_t s);
void launch_reach_only(const GraphView &gv, const int32_t *cur_node, uint8_t *reach, int n_max, int e_max,
                       int depth_max, hipStream_t s);
void launch_classes(const GraphView &gv, const int32_t *cur_node, const uint8_t *reach,
                    uint8_t *out_class, hipStream_t s);
void launch_pool_generic(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                         const ForwardArgs &fa, hipStream_t s);

// ---- policy head (kernels_head.hip)
bool pool_in_head(int H, int L, int B, int n_max);
void launch_head(const GraphView &gv, const ModelView &mv, const Workspace &ws, const ForwardArgs &fa, int max_chunks,
                 int n_max, hipStream_t s);
struct HeadBwArgs {
    const double *hid64;          // [B, H], logit [B, D]: left by the forward pass
    const float *logit;
    const int32_t *actions;
    const float *coeff, *entropy_coeff;
    const float *hact;            // [3, L, B G, H] layer outputs of h
    float *hid, *dpre, *dlogit;   // [B, H], [B, H], [B, D]
    float *dz;                    // [B, Z]
    float *dh;                    // [3, L, B G, H] deltas of h's layers
    float *dP;                    // [B, 3, G, H]
    float *out_logp, *out_entropy;
};
void launch_head_bw(const GraphView &gv, const ModelView &mv, const float *blob_t, const int32_t *cur_node,
                    const HeadBwArgs &a, hipStream_t s);

// ---- MDP transition (kernels_episode.hip)
void launch_episode_step(const GraphView &gv, int D, const float *logits, const float *uniforms,
                         const int32_t *order, int t, float *node_feats, int32_t *placement,
                         int32_t *cur_node, int32_t *out_action, float *out_logp, hipStream_t s);

// steps taken ahead: copies of the batch, one for every state that its next steps can reach
void launch_copies_index(const GraphView &gv, int copies, int32_t *node_off, int32_t *tmpl, int32_t *node_graph,
                         hipStream_t s);
void launch_copies_state(const GraphView &gv, int D, int copies, int n_max, const int32_t *order, int t, const float *feats,
                         const int32_t *placement, const int32_t *cur_node, const EpisodeCopies &c, hipStream_t s);
void launch_copies_steps(const GraphView &gv, int D, int steps, const float *copy_logits, const float *uniforms,
                         const int32_t *order, int t, float *node_feats, int32_t *placement, int32_t *cur_node,
                         float *out_logits, size_t logits_stride, int32_t *out_action, float *out_logp, hipStream_t s);

void launch_episode_apply(const GraphView &gv, int D, const int32_t *actions, const int32_t *order, int t,
                          float *node_feats, int32_t *placement, int32_t *cur_node, hipStream_t s);
void launch_reinforce_coeff(int T, int B, int n_groups, const float *rewards, const int32_t *group,
                            float *coeff, float *baseline, hipStream_t s);

// ---- run-time simulator of a placement (kernels_simulator.hip); n_max / e_max: largest graph
size_t simulator_lds_bytes(int n_max, int e_max);
int launch_simulate(const GraphView &gv, int D, int n_max, int e_max, const float *node_feats,
                    const int32_t *placement, float inv_bw, bool per_child, float *out_runtime,
                    int32_t *out_events, hipStream_t s);

int launch_simulate_reward(const GraphView &gv, int D, int n_max, int e_max, const float *node_feats,
                           const int32_t *placement, float inv_bw, bool per_child, float mem_limit, float penalty,
                           float *op_start, float *op_end, float *arrival, float *arrival_last, double *peaks,
                           uint32_t *done, float *runtime, float *out_peak, float *out_reward, int32_t *out_events,
                           hipStream_t s);

// ---- matrix-core pooling (kernels_pool_mfma.hip); writes ws.partial as [B, kPoolSlices, 3G, H]
constexpr int kPoolSlices = 8;
bool pool_mfma_supported(int H, int L, int weight_dtype);
void pack_pool_weights(const ModelView &mv, const float *blob, int WS, std::vector<uint16_t> *frag,
                       std::vector<float> *bias);
// fragments of the streaming pooling kernel (weights as A operands); bf16 weights at H = 128
bool pool_stream_supported(int H, int L, int weight_dtype);
void pack_pool_stream_weights(const ModelView &mv, const float *blob, std::vector<uint16_t> *frag);
// the reverse of the streaming pooling kernel (two-layer l): deltas of l's layers and d e of every
// pooled node from the kept layer outputs; reads the sort (ws.klist, ws.koff) of the forward pass
bool pool_stream_bw_supported(int H, int L, int weight_dtype);
void pack_pool_stream_bw_weights(const ModelView &mv, const float *blob, std::vector<uint16_t> *frag);
void launch_pool_stream_bw(const GraphView &gv, const ModelView &mv, const Workspace &ws, const uint4 *frag, const float *lact,
                           const float *dP, float *dl, float *demb, hipStream_t s);
// n_max: nodes of the largest graph, needed where pool_sort_asks(); returns the number of slices per graph that ws.partial
// holds afterwards
inline bool pool_sort_asks(int G) { return 3 * G > 24; }
int launch_pool_mfma(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                     const ForwardArgs &fa, const uint4 *wfrag, const uint4 *afrag, const float *bias, int WS,
                     float *keep, int n_max, hipStream_t s);

// ---- policy gradient (kernels_backward.hip): buffers owned by a batch for one (D, H, L)
struct GradWorkspace {
    float *fact = nullptr, *gact = nullptr;   // [2, L, n_tot, H] layer outputs of f and g
    float *agg = nullptr, *dagg = nullptr;    // [2, n_tot, H] gathered sums and their gradients
    float *dfg = nullptr;                     // per direction [2L, n_tot, H] layer deltas of f, then of g,
                                              // then H spare floats; dfg_stride floats per direction
    size_t dfg_stride = 0;
    float *keep = nullptr;                    // per direction [2L, n_tot, H]: a_v and layer outputs stored by
                                              // the forward sweep (same stride as dfg)
    float *snap_emb = nullptr, *snap_msg = nullptr;   // k >= 2 sweeps: states and messages after every
                                              // sweep but the last, [k - 1][2 n_tot H] each
    int32_t snap_sweeps = 0;
    uint8_t *mask4 = nullptr;                 // [2 n_tot + 1, H] ReLU gates per (sweep direction, node, column)
    float *lact = nullptr, *dl = nullptr;     // [L, n_tot, H] layer outputs / deltas of l (own set)
    float *demb = nullptr;                    // [n_tot, 2H] gradient of the embeddings
    float *dx = nullptr;                      // [n_tot, H] delta of the projection
    float *phi = nullptr;                     // [n_tot, F] raw feature rows
    uint8_t *cls = nullptr;                   // [n_tot] node set of every node
    int32_t *counts = nullptr;                // [4] sizes of the three node sets
    int32_t *blk_cnt = nullptr;               // [ceil(n_tot / 256), 3] per-block counts, then offsets; or where graphs' parts of lists begin (k_bw_set_begins)
    int32_t *lists = nullptr;                 // [3, n_tot] nodes of each set
    float *dP = nullptr;                      // [B, 3, G, H]
    float *hin = nullptr;                     // [3, B G, H] inputs of h per set
    float *hact = nullptr, *dh = nullptr;     // [3, L, B G, H]
    float *dz = nullptr;                      // [B, Z]
    float *hid = nullptr, *dpre = nullptr;    // [B, H] policy hidden layer and its delta
    float *dlogit = nullptr;                  // [B, D]
    float *partial = nullptr;                 // slab sums of the weight-gradient contractions
    size_t partial_floats = 0;
    int32_t H = 0, G = 0, L = 0, D = 0;
};

// Optional per-stage timing hook: called at the beginning and the end of every stage of a pass.
struct StageMarks {
    void *ctx;
    void (*mark)(void *ctx, int stage, bool begin, hipStream_t s);
};

size_t wgrad_workspace_floats(int64_t n, int64_t B, const ModelView &mv);
void launch_fill_zero(float *p, size_t n, hipStream_t s);
// what a reverse pass is asked for (device arrays; the last three may be null)
struct BackwardArgs {
    const int32_t *actions;
    const float *coeff;
    const float *entropy_coeff;
    float *grad;
    float *out_logp;
    float *out_entropy;
    // states [k - 1][n_tot, 2H] and messages [k - 1][2, n_tot, H] after every sweep but the last
    const float *snap_emb;
    const float *snap_msg;
    // fragments of the reverse streaming pooling kernel, or null (then the dense-layer kernels do it)
    const uint4 *pool_bw_frag = nullptr;
    bool accumulate = false;      // add to grad instead of replacing it
    size_t n_grad = 0;            // its entries
};

void launch_backward(const GraphView &gv, const ModelView &mv, const float *blob_t, const Workspace &ws,
                     const GradWorkspace &gw, const ForwardArgs &fa, const BackwardArgs &ba, int k_sweeps,
                     int pool_chunks, int generic, bool lanes, const uint4 *wfrag_bw, const float *sweep_bias, int sweep_ws,
                     const float *keep, bool pool_kept, const StageMarks *marks, hipStream_t s);

// ---- sweep of narrow networks (kernels_lanes.hip)
bool sweep_lanes_preferred(int H, int L, int B, int weight_dtype);
void launch_sweep_lanes(const GraphView &gv, const ModelView &mv, const Workspace &ws, const ForwardArgs &fa,
                        bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride, uint8_t *gates,
                        hipStream_t s);
void launch_sweep_lanes_bw(const GraphView &gv, const ModelView &mv, const float *blob_t, const int32_t *cur_node,
                           float *demb, float *dagg, uint8_t *mask4, float *delta, size_t delta_stride, hipStream_t s);

// ---- matrix-core sweep of 32 or 64 columns (kernels_tiles.hip); called by the launchers of kernels_mfma.hip
void launch_sweep_tiles(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                       const ForwardArgs &fa, const uint4 *wfrag, const float *bias, int WS,
                       bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride, uint8_t *gates,
                       hipStream_t s);
void launch_sweep_tiles_bw(const GraphView &gv, const ModelView &mv, const uint4 *wfrag, const float *bias,
                          int WS, const int32_t *cur_node, float *demb, float *dagg, uint8_t *mask4,
                          float *delta, size_t delta_stride, hipStream_t s);

// ---- matrix-core sweep of 128 columns, few graphs (kernels_wide.hip)
void launch_sweep_wide(const GraphView &gv, const ModelView &mv, const Workspace &ws, const ForwardArgs &fa, const uint4 *wfrag,
                       const float *bias, bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride,
                       uint8_t *gates, hipStream_t s);
void launch_sweep_wide_bw(const GraphView &gv, const ModelView &mv, const uint4 *wfrag, const float *bias,
                          const int32_t *cur_node, float *demb, float *dagg, uint8_t *mask4, float *delta,
                          size_t delta_stride, hipStream_t s);

// ---- matrix-core sweep (kernels_mfma.hip: 128 columns; hands 32 and 64, and few graphs, on)
bool sweep_mfma_supported(int H, int L, int weight_dtype);
void pack_sweep_weights(const ModelView &mv, const float *blob, int WS, std::vector<uint16_t> *frag,
                        std::vector<float> *bias, bool reverse = false);
void launch_sweep_mfma_bw(const GraphView &gv, const ModelView &mv, const uint4 *wfrag, const float *bias,
                          int WS, const int32_t *cur_node, float *demb, float *dagg, uint8_t *mask4,
                          float *delta, size_t delta_stride, hipStream_t s);
void launch_sweep_mfma(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                       const ForwardArgs &fa, const uint4 *wfrag, const float *bias, int WS,
                       bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride, uint8_t *gates,
                       hipStream_t s);

}  // namespace pl
