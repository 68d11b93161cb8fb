// Host-side layout of a forward pass's intermediate buffers.
#include <cstddef>

#include "internal.h"

namespace pl {

// A block that was laid out for one network serves every other one of the same width and the same number
// of device groups.  Hence no buffer's size may depend on anything else of the network: without
// grouping by device, networks of any number of devices have one group.
bool workspace_fits(const Workspace &ws, const ModelView &mv) { return ws.H == mv.H && ws.G == mv.G; }

// Lays the intermediate buffers of one forward pass out in one block starting at `base` (which
// may be null: then only the size is computed) and returns the block's size in bytes.  Every
// buffer starts on a 256-byte boundary.  With `with_reach` the reachability bytes are part of
// the block, otherwise ws->reach is left alone.
// Rows past the data (the sweeps that walk chunks: all but the generic one): emb row n, msg row 2n + 1, xb row 2n and reach byte
// 2n + 1 take the stores of a chunk's unused rows; msg row 2n and reach byte 2n are never
// written, must read as zero, and are the target of dummy loads.
size_t carve_workspace(unsigned char *base, size_t n, size_t B, const ModelView &mv, bool with_reach, Workspace *ws)
{
    size_t at = 0;
    auto take = [&](size_t bytes) {
        unsigned char *p = base ? base + at : nullptr;
        at += (bytes + 255) / 256 * 256;
        return p;
    };
    const size_t H = mv.H;
    ws->n_chunks = 8;
    ws->emb = reinterpret_cast<float *>(take(sizeof(float) * ((n + 1) * 2 * H + 4)));
    ws->msg = reinterpret_cast<float *>(take(sizeof(float) * ((2 * n + 2) * H + 4)));
    ws->xb = reinterpret_cast<float *>(take(sizeof(float) * ((2 * n + 1) * H + 4)));
    ws->featb = reinterpret_cast<float4 *>(take(sizeof(float4) * (n + 1)));
    ws->partial = reinterpret_cast<float *>(take(sizeof(float) * (B * ws->n_chunks * 3 * mv.G * H + 4)));
    ws->zbuf = reinterpret_cast<float *>(take(sizeof(float) * (B * mv.Z + 4)));
    // (a split head has H >= 128 and Z >= 640: three parts of a graph's first policy layer fit)
    ws->hidp = reinterpret_cast<double *>(take(sizeof(double) * (static_cast<size_t>((mv.Z + 255) / 256) * B * H + 4)));
    if (with_reach) {
        // a block of fixed size, whose callers have no reverse pass: what only that reads is not kept,
        // so that the block takes every batch that it took before those arrays were there
        ws->head_done = reinterpret_cast<uint32_t *>(ws->zbuf);
        ws->zbuf = nullptr;
    } else {
        ws->hid = reinterpret_cast<double *>(take(sizeof(double) * (B * H + 4)));
        ws->logit = reinterpret_cast<float *>(take(sizeof(float) * (B * kMaxD + 4)));   // (for any D: see workspace_fits)
        ws->head_done = reinterpret_cast<uint32_t *>(take(sizeof(uint32_t) * (B + 4)));
    }
    ws->klist = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (n + 16)));
    ws->koff = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (B * (3 * kMaxD + 1) + 4)));
    if (with_reach) ws->reach = take(2 * n + 32);
    ws->H = mv.H;
    ws->G = mv.G;
    return at;
}

// ---- room for the copies of a batch's graphs (internal.h)
constexpr size_t kCopiesBytes = static_cast<size_t>(4) << 30;   // most memory that a batch's rooms take together

// Lays a pass of `copies` copies out in a room with tables for `most`, as carve_workspace does.
size_t carve_copies(unsigned char *base, size_t n, size_t B, int most, int copies, const ModelView &mv, EpisodeCopies *c)
{
    size_t at = 0;
    auto take = [&](size_t bytes) {
        unsigned char *p = base ? base + at : nullptr;
        at += (bytes + 255) / 256 * 256;
        return p;
    };
    const size_t M = static_cast<size_t>(most), N = n * copies, G = B * copies;
    c->view.node_off = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (B * M + 1)));
    c->view.tmpl = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * B * M));
    c->view.node_graph = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * n * M));
    c->feats = reinterpret_cast<float *>(take(sizeof(float) * N * 3));
    c->placement = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * N));
    c->cur_node = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * G));
    c->logits = reinterpret_cast<float *>(take(sizeof(float) * G * mv.D));
    c->view.B = static_cast<int32_t>(G);
    c->view.n_tot = static_cast<int32_t>(N);
    return at + carve_workspace(base ? base + at : nullptr, N, G, mv, true, &c->ws);
}

// A room that a pass fits in, or null.
const CopiesRoom *find_room(const EpisodeRooms &rooms, size_t n, size_t B, int copies, const ModelView &mv)
{
    EpisodeCopies sized;
    for (int i = 0; i < rooms.n; ++i) {
        const CopiesRoom &r = rooms.room[i];
        if (copies <= r.most && carve_copies(nullptr, n, B, r.most, copies, mv, &sized) <= r.bytes) return &r;
    }
    return nullptr;
}

// Size of another room, for a network's largest pass; 0 where the batch may not have it, or asked for as much in vain.
size_t new_room_bytes(const EpisodeRooms &rooms, size_t n, size_t B, int most, const ModelView &mv)
{
    EpisodeCopies sized;
    const size_t bytes = carve_copies(nullptr, n, B, most, most, mv, &sized);
    return rooms.n < kCopiesRooms && rooms.bytes + bytes <= kCopiesBytes && bytes < rooms.refused ? bytes : 0;
}

// base: the memory, or null if there was none.
const CopiesRoom *add_room(EpisodeRooms *rooms, unsigned char *base, size_t bytes, int most)
{
    if (!base) {
        rooms->refused = bytes;
        return nullptr;
    }
    rooms->room[rooms->n] = {base, bytes, most};
    rooms->bytes += bytes;
    return &rooms->room[rooms->n++];
}

}  // namespace pl
