// Test driver: the room that a batch keeps for the copies of its graphs (workspace.cpp), over sequences of episode calls
// that run at once or are captured and replayed later.  Memory is the host's: a room's tables are written when it is made, a pass
// checks those that it reads and overwrites everything that it may write.  Prints what fails; exits with 1 if anything
// does.  Test infrastructure only.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "internal.h"

namespace {

constexpr size_t kNodes = 7;

int bad = 0;
void check(bool ok, const char *what, int where)
{
    if (ok) return;
    ++bad;
    std::printf("%s (sequence %d)\n", what, where);
}

pl::ModelView network(int D, int H, int by_device)
{
    pl::ModelView mv{};
    mv.D = D;
    mv.H = H;
    mv.L = 2;
    mv.G = by_device ? D : 1;
    mv.Z = (2 + 3 * mv.G) * H;
    mv.F = D + 4;
    return mv;
}

int states(int D, int steps)
{
    int all = 0, at = 1;
    for (int i = 0; i < steps; ++i, at *= D) all += at;
    return all;
}

struct Pass {
    const unsigned char *base = nullptr;   // of its room; null: step by step
    size_t bytes = 0;
    int copies = 0;
    pl::EpisodeCopies c;
};

class Batch {
public:
    Batch(size_t B, int where) : B_(B), n_(B * kNodes), where_(where) {}
    ~Batch()
    {
        for (int i = 0; i < rooms.n; ++i) std::free(rooms.room[i].base);
    }
    // what pl_episode_run decides for a call, and the pass that it launches or records
    Pass call(const pl::ModelView &mv, int steps, bool captured, bool memory = true)
    {
        int longest = 1;
        while (static_cast<size_t>(states(mv.D, longest + 1)) * B_ <= 256) ++longest;
        const int copies = states(mv.D, steps < longest ? steps : longest), most = states(mv.D, longest);
        const pl::CopiesRoom *room = copies > 1 ? pl::find_room(rooms, n_, B_, copies, mv) : nullptr;
        if (copies > 1 && !room && !captured) {
            const size_t bytes = pl::new_room_bytes(rooms, n_, B_, most, mv);
            if (bytes) {
                ++asked;
                unsigned char *base = memory ? static_cast<unsigned char *>(std::malloc(bytes)) : nullptr;
                room = pl::add_room(&rooms, base, bytes, most);
                check((room != nullptr) == memory, "a room is there with its memory and only then", where_);
                if (room) {
                    std::memset(base, 0xCD, bytes);
                    pl::EpisodeCopies c;
                    pl::carve_copies(base, n_, B_, most, most, mv, &c);
                    tables(c, most, true);
                }
            }
        }
        Pass p;
        p.copies = copies;
        if (room) {
            p.base = room->base;
            p.bytes = pl::carve_copies(room->base, n_, B_, room->most, copies, mv, &p.c);
            check(p.bytes <= room->bytes, "a pass ends in its room", where_);
        }
        if (!captured) run(p);
        return p;
    }
    void run(const Pass &p)
    {
        if (!p.base) return;
        check(tables(p.c, p.copies, false), "the tables that a pass reads are those of its copies", where_);
        // all that is laid out behind the tables, the first of it the features
        unsigned char *from = reinterpret_cast<unsigned char *>(p.c.feats);
        std::memset(from, 0xAB, p.bytes - static_cast<size_t>(from - p.base));
    }
    pl::EpisodeRooms rooms;
    int asked = 0;

private:
    bool tables(const pl::EpisodeCopies &c, int copies, bool write)
    {
        auto *off = const_cast<int32_t *>(c.view.node_off), *tmpl = const_cast<int32_t *>(c.view.tmpl);
        auto *graph = const_cast<int32_t *>(c.view.node_graph);
        const int graphs = copies * static_cast<int>(B_), nodes = copies * static_cast<int>(n_);
        bool same = c.view.B == graphs && c.view.n_tot == nodes;
        auto entry = [&](int32_t *at, int want) {
            if (write) *at = want;
            same = same && *at == want;
        };
        for (int i = 0; i <= graphs; ++i) entry(off + i, i * static_cast<int>(kNodes));
        for (int i = 0; i < graphs; ++i) entry(tmpl + i, i % static_cast<int>(B_));
        for (int i = 0; i < nodes; ++i) entry(graph + i, i / static_cast<int>(kNodes));
        return same;
    }
    size_t B_, n_;
    int where_;
};

}  // namespace

int main()
{
    const pl::ModelView net = network(8, 64, 1), wide = network(8, 128, 1), few = network(3, 64, 1), many = network(16, 64, 1),
                        plain = network(4, 64, 0), narrow = network(8, 8, 1);
    {   // fewer steps captured where more have run, then run before the first replay
        Batch b(1, 1);
        b.call(net, 8, false);
        const Pass p = b.call(net, 2, true);
        check(p.base != nullptr, "a captured call uses a room that is there", 1);
        b.call(net, 2, false);
        for (int i = 0; i < 3; ++i) b.run(p), b.call(net, 2, false), b.call(net, 8, false);
    }
    {   // as many steps captured as have run, then fewer run before the replay
        Batch b(1, 2);
        b.call(net, 8, false);
        const Pass p = b.call(net, 8, true);
        for (int i = 0; i < 3; ++i) b.call(net, 2, false), b.run(p);
    }
    {   // captured with few, then more steps and other networks: what the capture uses stays where it is
        Batch b(1, 3);
        b.call(net, 2, false);
        const Pass p = b.call(net, 2, true);
        b.call(net, 8, false);
        check(b.asked == 1, "one room serves every number of steps", 3);
        b.run(p);
        const pl::ModelView *others[] = {&wide, &few, &many, &plain, &narrow};
        for (const pl::ModelView *mv : others)
            for (int steps : {3, 2, 8}) b.call(*mv, steps, false), b.run(p);
        const Pass q = b.call(wide, 8, true);
        for (const pl::ModelView *mv : others) b.call(*mv, 8, false), b.run(q), b.run(p);
    }
    {   // a capture makes no room and changes nothing
        Batch b(2, 4);
        pl::EpisodeRooms before;
        std::memcpy(&before, &b.rooms, sizeof(before));
        check(b.call(net, 8, true).base == nullptr && std::memcmp(&before, &b.rooms, sizeof(before)) == 0, "no room: step by step", 4);
        b.call(few, 8, false);
        std::memcpy(&before, &b.rooms, sizeof(before));
        check(b.call(wide, 8, true).base == nullptr && std::memcmp(&before, &b.rooms, sizeof(before)) == 0, "too small: step by step", 4);
    }
    {   // no memory: asked for once, a smaller room may still be had
        Batch b(1, 5);
        for (int i = 0; i < 3; ++i) check(b.call(wide, 8, false, false).base == nullptr, "no memory: step by step", 5);
        check(b.asked == 1, "asked for once", 5);
        check(b.call(narrow, 8, false).base != nullptr && b.asked == 2, "a smaller room", 5);
        check(b.call(wide, 8, false).base == nullptr && b.asked == 2, "not asked for again", 5);
    }
    {   // all rooms of a batch together have a limit
        pl::EpisodeRooms r;
        r.n = 1;
        r.bytes = static_cast<size_t>(4) << 30;
        check(pl::new_room_bytes(r, 64, 1, 73, net) == 0, "memory of all rooms", 6);
        r.bytes = 0;
        r.n = pl::kCopiesRooms;
        check(pl::new_room_bytes(r, 64, 1, 73, net) == 0, "number of rooms", 6);
        check(pl::new_room_bytes(pl::EpisodeRooms(), 1 << 20, 1, 73, wide) == 0, "one room", 6);
    }
    std::printf("%d faults\n", bad);
    return bad ? 1 : 0;
}
