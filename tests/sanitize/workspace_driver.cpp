// Test driver: the block of intermediate buffers that a batch keeps between calls (workspace.cpp).  For
// every pair of networks of which the second takes the block that was laid out for the first
// (workspace_fits), the extents that the kernels use for the second have to be inside the block and apart
// from each other.  Prints the pairs that fail; exits with 1 if there is one.  Test infrastructure only.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "internal.h"

namespace {

struct Extent {
    const char *name;
    const void *p;
    size_t bytes;
};

// What the kernels read or write for network mv, by buffer.
std::vector<Extent> extents(const pl::Workspace &ws, size_t n, size_t B, const pl::ModelView &mv, bool fixed)
{
    const size_t H = mv.H, G = mv.G, D = mv.D, Z = mv.Z;
    std::vector<Extent> e{{"emb", ws.emb, 4 * (n + 1) * 2 * H},
                          {"msg", ws.msg, 4 * (2 * n + 2) * H},
                          {"xb", ws.xb, 4 * (2 * n + 1) * H},
                          {"featb", ws.featb, 16 * (n + 1)},
                          {"partial", ws.partial, 4 * B * 8 * 3 * G * H},
                          {"head_done", ws.head_done, 4 * B},
                          {"klist", ws.klist, 4 * n},
                          {"koff", ws.koff, 4 * B * (3 * pl::kMaxD + 1)}};
    if (H >= 128) e.push_back({"hidp", ws.hidp, 8 * B * 3 * H});
    if (fixed) {
        e.push_back({"reach", ws.reach, 2 * n + 2});
    } else {
        e.push_back({"zbuf", ws.zbuf, 4 * B * Z});
        e.push_back({"hid", ws.hid, 8 * B * H});
        e.push_back({"logit", ws.logit, 4 * B * D});
    }
    return e;
}

pl::ModelView network(int D, int H, int L, int by_device)
{
    pl::ModelView mv{};
    mv.D = D;
    mv.H = H;
    mv.L = L;
    mv.G = by_device ? D : 1;
    mv.Z = (2 + 3 * mv.G) * H;
    mv.F = D + 4;
    return mv;
}

}  // namespace

int main()
{
    std::vector<pl::ModelView> nets;
    for (int D : {1, 2, 4, 9, 16})
        for (int H : {8, 17, 32, 64, 128, 256})
            for (int L : {1, 4})
                for (int by_device : {0, 1}) nets.push_back(network(D, H, L, by_device));
    int pairs = 0, bad = 0;
    for (const auto &size : {std::pair<size_t, size_t>{1, 1}, {64, 64}, {300, 100}, {3000, 256}})
        for (const auto &a : nets)
            for (const bool fixed : {false, true}) {
                const size_t n = size.first, B = size.second;
                pl::Workspace ws;
                const size_t bytes = pl::carve_workspace(nullptr, n, B, a, fixed, &ws);
                unsigned char *base = static_cast<unsigned char *>(std::malloc(bytes));
                if (!base) return 2;
                if (pl::carve_workspace(base, n, B, a, fixed, &ws) != bytes) ++bad;
                for (const auto &b : nets) {
                    // (the fixed block is laid out anew for every call)
                    if (fixed ? &a != &b : !pl::workspace_fits(ws, b)) continue;
                    ++pairs;
                    auto e = extents(ws, n, B, b, fixed);
                    std::sort(e.begin(), e.end(), [](const Extent &x, const Extent &y) { return x.p < y.p; });
                    for (size_t i = 0; i < e.size(); ++i) {
                        const unsigned char *p = static_cast<const unsigned char *>(e[i].p);
                        const unsigned char *next = i + 1 < e.size() ? static_cast<const unsigned char *>(e[i + 1].p) : base + bytes;
                        if (p >= base && e[i].bytes <= static_cast<size_t>(next - p)) continue;
                        ++bad;
                        std::printf("%s: %zu bytes used, %td to the next buffer; n %zu B %zu H %d, laid out for D %d G %d, used with D %d\n",
                                    e[i].name, e[i].bytes, p ? next - p : 0, n, B, a.H, a.D, a.G, b.D);
                    }
                }
                std::free(base);
            }
    std::printf("%d pairs, %d faults\n", pairs, bad);
    return bad ? 1 : 0;
}
