// Run-time simulator of a placement (Appendix, "Simulator"): per device a FIFO queue of
// runnable operations and a FIFO queue of output tensors waiting to leave the device; a device
// runs one operation at a time, its bus carries one tensor at a time, transfers overlap with
// compute; an event loop over op-done and transfer-done events; the run time is the timestamp
// of the last op-done event.
//
// A discrete-event simulation is one dependent chain, so a graph gets one wave, and the batch
// of graphs (rollouts) supplies the parallelism; the whole state of the graph sits in LDS.  At most
// 2 D events are pending (one per device, one per bus): lane d holds the queue ends and the pending
// event of device d, lane D + d those of bus d.  The next event is a wave-wide minimum over
// (timestamp, creation number).
//
// What bounds it: a single wave issues an instruction about every five cycles, so an event costs
// its instructions (and LDS round trips), not arithmetic.  Hence:
//   * An event concerns one device and one bus only (the device whose operation ended and its bus;
//     the bus whose transfer ended and the destination): the handler is scalar code that reads and
//     writes those two lanes' registers (v_readlane / v_writelane) and branches on the scalar unit,
//     no lane-masked code over all devices.
//   * A node's record (cost, transfer duration, children, queue link) is 16 bytes.  Every lane reads
//     the record of its queue's first item at the end of every event, whether or not it changed: the
//     read is off the chain, and no branch or copy makes anything wait for it.
//   * A record holds the ids of up to two children themselves (longer lists their place in cidx), so
//     the handler starts with the read of the children's states.
//   * A bus queues operations, not transfers: the transfers of an operation leave back to back.  Which devices an output
//     goes to follows from the placement: the lists are made by all threads while the graph is staged, not by the
//     handler of the operation's end, and two entries of them travel with the operation in 16 bits.
//   * An item that leaves its queue becomes the pending event of the same lane, whose registers hold its record: lane
//     selects, no way through scalar registers.
//   * A child that becomes runnable on an idle device starts from the registers that its record was
//     read into.
// About 80 instructions per event.  256 NASNet-like graphs (3124 nodes, 8 devices, about 7300 events
// each): 2.31 ms; 2.65 ms with the destinations found by the handler and items moved through scalar registers; 4.56 ms with
// lane-masked queues, a transfer record per transfer and every read on the chain.
//
// Timestamps are float32 with one rounding per operation (no fused multiply-add), and events
// are ordered by (timestamp, creation number): the order is the same as that of a scalar
// implementation of the same rules, event by event.
#include "internal.h"

namespace pl {

// v_writelane (clang has no builtin for it): v with lane l's value replaced by x
__device__ int write_lane(int x, int l, int v) __asm("llvm.amdgcn.writelane.i32");

namespace {

constexpr int kSimThreads = 256;   // they stage the graph into LDS; the first wave then runs the events

// Graph-local ids and places in cidx take 14 bits: a graph whose state fits in LDS has at most 9100
// nodes and 12600 edges.  Id n is the node that is not there: the absent second child of a node, the
// end of a queue; it has a record and a state of its own, on device kNoDev.
constexpr uint32_t kIdBits = 14, kIdMask = (1u << kIdBits) - 1, kList = 1u << 31;
// A node's state: its device in the low bits, inputs not yet available on that device above them.
constexpr uint32_t kDevBits = 5, kNoDev = (1u << kDevBits) - 1, kInput = 1u << kDevBits;
// Entry of an operation's transfer list: the destination device or, with one transfer per child, the
// child, with kFirst set where it is the first to its device.
constexpr uint32_t kFirst = 0x8000u;

// LDS: rec [n + 1] {cost; duration of a transfer; children: id | id << 14, or kList | place in cidx | number << 14;
// link | crossings << 16}, node [n + 1] states, cidx [e] children (ascending per node), xl [e] transfer lists of more
// than two entries, from the place of the operation's first child.  Crossings (one transfer per destination): number
// of destinations | first << 5 | second << 10; which they are follows from the placement alone, so they are found
// while the graph is staged, all operations at once.  (With one transfer per child the handler finds them, and an output
// that waits for the bus has transfers | first entry << 16 in place of its cost, its second entry in the crossings' place.)
//  States take 16 bits where 32 do not fit.
template <typename Word>
constexpr size_t sim_lds(size_t n, size_t e)
{
    return (16 + sizeof(Word)) * (n + 1) + 4 * e;
}

// Minimum of an unsigned value over lanes 0..15 (one DPP row) or 0..31, as a scalar.
template <bool TWO>
__device__ __forceinline__ uint32_t event_min(uint32_t v)
{
#define PL_ROW_MIN(ctrl)                                                                                       \
    {                                                                                                          \
        const uint32_t o = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(-1, static_cast<int>(v), ctrl, 0xF, 0xF, false)); \
        v = o < v ? o : v;                                                                                     \
    }
    PL_ROW_MIN(0xB1)     // quad_perm [1,0,3,2]
    PL_ROW_MIN(0x4E)     // quad_perm [2,3,0,1]
    PL_ROW_MIN(0x141)    // row_half_mirror
    PL_ROW_MIN(0x140)    // row_mirror
#undef PL_ROW_MIN
    const uint32_t r0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 0));
    if constexpr (!TWO) return r0;
    const uint32_t r1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 16));
    return r0 < r1 ? r0 : r1;
}

__device__ __forceinline__ uint32_t get(uint32_t v, uint32_t l)
{
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), static_cast<int>(l)));
}
__device__ __forceinline__ void put(uint32_t &v, uint32_t l, uint32_t x)
{
    v = static_cast<uint32_t>(write_lane(static_cast<int>(x), static_cast<int>(l), static_cast<int>(v)));
}
__device__ __forceinline__ uint32_t first_lane(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}

// TL: the timeline is written out as well (for the peak-memory model): start and end of every
// operation, and the time at which an output arrived on every device it was sent to.
// PC: the op-done handler as the appendix prints it: the output is enqueued once for EVERY child
// on another device and a transfer-done event releases that one child (so an output needed by
// several children on one remote device crosses the bus several times; the timeline then keeps
// the first and the last arrival per device).  Otherwise an output crosses once per destination
// device and its arrival releases every child waiting there.
// TWO: more than eight devices, so the pending events take two DPP rows.
template <bool TL, bool PC, bool TWO, typename Word>
__global__ __launch_bounds__(kSimThreads) void k_simulate(GraphView gv, int D, int n_max, int e_max,
                                                 const float *__restrict__ node_feats,
                                                 const int32_t *__restrict__ placement, float inv_bw,
                                                 float *__restrict__ out_runtime,
                                                 int32_t *__restrict__ out_events,
                                                 float *__restrict__ op_start, float *__restrict__ op_end,
                                                 float *__restrict__ arrival, float *__restrict__ arrival_last)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint4 *rec = reinterpret_cast<uint4 *>(lds_raw);
    Word *node = reinterpret_cast<Word *>(rec + n_max + 1);
    uint16_t *cidx = reinterpret_cast<uint16_t *>(node + n_max + 1), *xl = cidx + e_max;
    auto link_of = [&](uint32_t v) __attribute__((always_inline)) { return reinterpret_cast<uint16_t *>(rec + v) + 6; };
    const int b = blockIdx.x;
    const int n0 = gv.node_off[b], n = gv.node_off[b + 1] - n0;
    const int32_t *gptr = gv.nbr_ptr[1] + n0;            // children CSR (global offsets / ids)
    const int e0 = gptr[0], e = gptr[n] - e0;
    const uint32_t none = static_cast<uint32_t>(n);

    // ---- the graph's state into LDS.  rec[n].x: some device id is outside [0, D)
    if (threadIdx.x == 0) {
        rec[n] = uint4{0, 0, none | none << kIdBits, none};
        node[n] = static_cast<Word>(kNoDev);
    }
    __syncthreads();
#pragma unroll 4
    for (int v = threadIdx.x; v < n; v += kSimThreads) {
        const int d = placement[n0 + v];
        if (d < 0 || d >= D) rec[n].x = 1u;
        const int c0 = gptr[v], cnt = gptr[v + 1] - c0;
        uint32_t kids;
        if (cnt > 2) {
            kids = kList | static_cast<uint32_t>(c0 - e0) | static_cast<uint32_t>(cnt) << kIdBits;
        } else {
            const uint32_t k0 = cnt > 0 ? static_cast<uint32_t>(gv.nbr_idx[1][c0] - n0) : none;
            const uint32_t k1 = cnt > 1 ? static_cast<uint32_t>(gv.nbr_idx[1][c0 + 1] - n0) : none;
            kids = k0 | k1 << kIdBits;
        }
        rec[v] = uint4{__float_as_uint(node_feats[static_cast<size_t>(n0 + v) * 3 + 0]),
                       __float_as_uint(__fmul_rn(node_feats[static_cast<size_t>(n0 + v) * 3 + 1], inv_bw)), kids, none};
        const uint32_t parents = static_cast<uint32_t>(gv.nbr_ptr[0][n0 + v + 1] - gv.nbr_ptr[0][n0 + v]);
        node[v] = static_cast<Word>((static_cast<uint32_t>(d) & kNoDev) | parents << kDevBits);
    }
#pragma unroll 4
    for (int i = threadIdx.x; i < e; i += kSimThreads) cidx[i] = static_cast<uint16_t>(gv.nbr_idx[1][e0 + i] - n0);
    __syncthreads();
    if constexpr (!PC) {
        // A thread per operation, until every other device has been found.  A list of more than kWide children goes to the
        // whole wave, 64 children at a time: the walk of one thread is two dependent reads per child (a node of 5000 children:
        // 400 us of 2240, 8 now; of 130: 11 of 125).
        constexpr uint32_t kWide = 64;
        const uint32_t all = (1u << D) - 1u | 1u << kNoDev;    // (a child that is not there needs no transfer)
        const uint32_t lane = threadIdx.x & 63u;
        for (int v0 = static_cast<int>(threadIdx.x - lane); v0 < n; v0 += kSimThreads) {
            const uint32_t v = min(static_cast<uint32_t>(v0) + lane, none);
            const uint32_t kids = rec[v].z, listed = kids & kList;
            const uint32_t c0 = kids & kIdMask, cnt = listed ? (kids & ~kList) >> kIdBits : 2u;
            const uint32_t own = 1u << (node[v] & kNoDev) | 1u << kNoDev;
            if (cnt <= kWide) {
                uint32_t sent = own, m = 0, cross = 0;
                for (uint32_t i = 0; i < cnt && sent != all; ++i) {
                    const uint32_t c = listed ? cidx[c0 + i] : (i == 0 ? c0 : kids >> kIdBits), pd = node[c] & kNoDev;
                    if ((sent >> pd) & 1u) continue;
                    sent |= 1u << pd;
                    if (m < 2) cross |= pd << (5 + 5 * m);
                    if (listed) xl[c0 + m] = static_cast<uint16_t>(pd);
                    ++m;
                }
                link_of(v)[1] = static_cast<uint16_t>(cross | m);
            }
            for (unsigned long long wide = __ballot(cnt > kWide); wide != 0ull; wide &= wide - 1ull) {
                const uint32_t l = static_cast<uint32_t>(__builtin_ctzll(wide)), w = static_cast<uint32_t>(v0) + l;
                const uint32_t w0 = get(c0, l), w_cnt = get(cnt, l);
                uint32_t sent = get(own, l), m = 0, cross = 0;
                for (uint32_t base = 0; base < w_cnt && sent != all; base += 64) {
                    const uint32_t i = base + lane, pd = i < w_cnt ? node[cidx[w0 + i]] & kNoDev : kNoDev;
                    unsigned long long rest = __ballot(!((sent >> pd) & 1u));
                    while (rest != 0ull) {                    // destinations in the order of their first child
                        const uint32_t d = get(pd, static_cast<uint32_t>(__builtin_ctzll(rest)));
                        rest &= ~__ballot(pd == d);
                        sent |= 1u << d;
                        if (m < 2) cross |= d << (5 + 5 * m);
                        if (lane == 0) xl[w0 + m] = static_cast<uint16_t>(d);
                        ++m;
                    }
                }
                if (lane == 0) link_of(w)[1] = static_cast<uint16_t>(cross | m);
            }
        }
        __syncthreads();
    }
    if (rec[n].x != 0) {
        if (threadIdx.x == 0) {
            out_runtime[b] = __builtin_nanf("");
            if (out_events) out_events[b] = -1;
        }
        return;
    }
    if (threadIdx.x >= 64) return;
    const uint32_t lane = threadIdx.x, nd = static_cast<uint32_t>(D);

    // ---- lane-private state (lane d: device d, lane D + d: bus d)
    constexpr uint32_t kIdle = 0xFFFFFFFFu;
    uint32_t ev_t = kIdle, ev_key = 0;                    // pending event: time (bits); operation | creation number << 14
    uint32_t cur_dur = 0, cur_kids = 0;                   // its operation's transfer duration and children
    // Device: crossings of its operation.  Bus: destinations left, the one in progress with them | its device << 5 | the
    // next one << 10 | number of the entry after that << 15.  (One transfer per child: list entry in progress | the
    // next one << 16, and x_more: entries left | place in xl of the entry after the next << 14.)
    uint32_t x_cur = 0, x_more = 0;
    uint32_t head = none, tail = none;                    // queue
    uint4 hr = rec[none];                                 // record of the queue's first item
    uint32_t seq = 0, n_events = 0, last = 0;

    auto push = [&](uint32_t q, uint32_t v) __attribute__((always_inline)) {
        if (get(head, q) == none)
            put(head, q, v);
        else
            *link_of(get(tail, q)) = static_cast<uint16_t>(v);
        put(tail, q, v);
    };
    // lane q's pending event, for operation o: `duration` after `now` (both as bits).  (No more than n + e
    // events are ever created, and 18 n + 13 e bytes of at most 160 KB leave n + e below 12700: the creation number
    // fits beside the id.)
    auto schedule = [&](uint32_t q, uint32_t now, uint32_t duration, uint32_t o) __attribute__((always_inline)) {
        const float t = __fadd_rn(__uint_as_float(now), __uint_as_float(duration));
        ev_t = lane == q ? __float_as_uint(t) : ev_t;
        put(ev_key, q, o | seq << kIdBits);
        ++seq;
        return t;
    };
    // operation v starts on device q
    auto start_op = [&](uint32_t q, uint32_t v, uint32_t now, uint32_t cost, uint32_t dur, uint32_t kids, uint32_t w) __attribute__((always_inline)) {
        const float t = schedule(q, now, cost, v);
        put(cur_dur, q, dur);
        put(cur_kids, q, kids);
        if constexpr (!PC) put(x_cur, q, w >> 16);
        if constexpr (TL) {
            op_start[n0 + static_cast<int>(v)] = __uint_as_float(now);
            op_end[n0 + static_cast<int>(v)] = t;
        }
    };
    // bus q starts the m transfers of operation o, the first two to e1 and e2
    auto start_transfers = [&](uint32_t q, uint32_t now, uint32_t o, uint32_t dur, uint32_t kids, uint32_t m, uint32_t e1,
                               uint32_t e2) __attribute__((always_inline)) {
        schedule(q, now, dur, o);
        put(cur_dur, q, dur);
        put(cur_kids, q, kids);
        put(x_cur, q, e1 | e2 << 16);
        put(x_more, q, (m - 1) | ((kids & kIdMask) + 2) << kIdBits);
    };

    // bus q starts the transfers of operation o, whose crossings are x
    auto start_crossing = [&](uint32_t q, uint32_t now, uint32_t o, uint32_t dur, uint32_t kids, uint32_t x) __attribute__((always_inline)) {
        schedule(q, now, dur, o);
        put(cur_dur, q, dur);
        put(cur_kids, q, kids);
        put(x_cur, q, x | 2u << 15);
    };
    // The first item of queue q (whose record lane q holds) becomes lane q's pending event and leaves the queue: all of
    // it in the lane itself.  `after`: the lane's duration; x: its new x_cur.
    auto start_first = [&](uint32_t q, uint32_t now, uint32_t after, uint32_t x) __attribute__((always_inline)) {
        const bool it = lane == q;
        const float t = __fadd_rn(__uint_as_float(now), __uint_as_float(after));
        ev_t = it ? __float_as_uint(t) : ev_t;
        ev_key = it ? head | seq << kIdBits : ev_key;
        ++seq;
        cur_dur = it ? hr.y : cur_dur;
        cur_kids = it ? hr.z : cur_kids;
        x_cur = it ? x : x_cur;
        head = it ? hr.w & 0xFFFFu : head;
        return t;
    };

    for (int base = 0; base < n; base += 64) {            // operations without parents, ascending id
        const uint32_t v = static_cast<uint32_t>(base) + lane;
        const uint32_t word = node[v < none ? v : none];
        unsigned long long roots = __ballot(v < none && word < kInput);
        while (roots != 0ull) {
            const uint32_t l = static_cast<uint32_t>(__builtin_ctzll(roots));
            roots &= roots - 1;
            push(get(word, l), static_cast<uint32_t>(base) + l);
        }
    }
    for (uint32_t d = 0; d < nd; ++d) {
        const uint32_t v = get(head, d);
        if (v == none) continue;
        const uint4 r = rec[v];
        start_op(d, v, 0, first_lane(r.x), first_lane(r.y), first_lane(r.z), first_lane(r.w));
        put(head, d, first_lane(r.w) & 0xFFFFu);
    }
    hr = rec[head];

    const uint32_t max_events = static_cast<uint32_t>(n + e + 8);   // every operation and transfer ends once
    // The loop begins on a boundary of 32 bytes: a single wave waits for its instructions, and where the loop's branches lie
    // within the lines that it fetches moves the whole simulation by 5 % (256 NASNet-like graphs: 2.31 to 2.43 ms over the
    // eight places that four-byte instructions can have).
    asm volatile(".p2align 5");
    do {
        // ---- next event: smallest (timestamp, creation number).  Timestamps are >= 0, so their
        // bit patterns order like the values.
        const uint32_t now = event_min<TWO>(ev_t);
        if (now == kIdle) break;                          // nothing pending: the simulation is over
        // Usually one pending event carries the smallest timestamp; only ties need the second
        // reduction, over the creation numbers.
        uint32_t first = static_cast<uint32_t>(__ballot(ev_t == now));
        if (__builtin_expect(first & (first - 1), 0)) {
            const uint32_t s_bits = ev_t == now ? ev_key : kIdle;
            first = static_cast<uint32_t>(__ballot(s_bits == event_min<TWO>(s_bits)));
        }
        const uint32_t slot = static_cast<uint32_t>(__builtin_ctz(first));
        const uint32_t o = get(ev_key, slot) & kIdMask, kids = get(cur_kids, slot), dur = get(cur_dur, slot);
        ++n_events;
        put(ev_t, slot, kIdle);

        // The operation's children where its output now is (its own device after op-done, the
        // destination after transfer-done) have one input fewer to wait for, and join that device's
        // queue when it was the last one; after op-done the others make the output cross.  In
        // ascending child id throughout.  An idle device goes on with its queue before anything is
        // appended to it; if it has none, the first child that becomes runnable starts at once.
        uint32_t wait = 0;                                // 0: the device would start a runnable child at once
        auto next_op = [&](uint32_t dev) __attribute__((always_inline)) {
            const uint32_t v = get(head, dev);
            wait = v ^ none;
            if (v == none) return;
            const float t = start_first(dev, now, hr.x, hr.w >> 16);
            if constexpr (TL) {
                op_start[n0 + static_cast<int>(v)] = __uint_as_float(now);
                op_end[n0 + static_cast<int>(v)] = __uint_as_float(get(__float_as_uint(t), dev));
            }
        };
        auto runnable = [&](uint32_t dev, uint32_t v, const uint4 &r, uint32_t l) __attribute__((always_inline)) {
            if (__builtin_expect(wait == 0, 1)) {
                wait = 1;
                start_op(dev, v, now, get(r.x, l), get(r.y, l), get(r.z, l), PC ? 0u : get(r.w, l));
            } else {
                push(dev, v);
            }
        };
        // children 0 and 1 of an operation that has no more: their states, one in each of lanes 0 and 1
        auto two_kids = [&](uint32_t dev, uint4 &r) __attribute__((always_inline)) {
            uint32_t c = none;
            put(c, 0, kids & kIdMask);
            put(c, 1, kids >> kIdBits);
            const uint32_t word = node[c];
            r = rec[c];
            node[c] = static_cast<Word>((word & kNoDev) == dev ? word - kInput : word);
            return word;
        };
        // 64 children at a time of one that has more: lane's child (none past the end) and its state
        auto more_kids = [&](uint32_t dev, uint32_t at, uint32_t left, uint32_t &c, uint4 &r) __attribute__((always_inline)) {
            c = lane < left ? cidx[at + lane] : none;
            const uint32_t word = node[c];
            r = rec[c];
            node[c] = static_cast<Word>((word & kNoDev) == dev ? word - kInput : word);
            unsigned long long ready = __ballot(word == (kInput | dev));
            while (ready != 0ull) {
                const uint32_t l = static_cast<uint32_t>(__builtin_ctzll(ready));
                ready &= ready - 1;
                runnable(dev, get(c, l), r, l);
            }
            return word;
        };
        const uint32_t c0 = kids & kIdMask, cnt = (kids & ~kList) >> kIdBits;   // (of a longer list)

        if (slot < nd) {
            last = now;
            const uint32_t cross = PC ? 0u : get(x_cur, slot);   // (before the device goes on with its queue)
            uint32_t m = 0, e1 = 0, e2 = 0;               // (one per child) transfers of the output: number and first two entries
            uint4 r;
            if constexpr (!PC) {
                if (__builtin_expect(!(kids & kList), 1)) {
                    const uint32_t word = two_kids(slot, r);
                    next_op(slot);
                    const uint32_t w0 = get(word, 0), w1 = get(word, 1), want = kInput | slot;
                    if (__builtin_expect(w0 == want, 0)) runnable(slot, kids & kIdMask, r, 0);
                    if (__builtin_expect(w1 == want, 0)) runnable(slot, kids >> kIdBits, r, 1);
                } else {
                    next_op(slot);
                    for (uint32_t base = 0; base < cnt; base += 64) {
                        uint32_t c;
                        (void)more_kids(slot, c0 + base, cnt - base, c, r);
                    }
                }
            } else if (__builtin_expect(!(kids & kList), 1)) {
                const uint32_t word = two_kids(slot, r);
                next_op(slot);
                const uint32_t w0 = get(word, 0), w1 = get(word, 1), want = kInput | slot;
                if (__builtin_expect(w0 == want, 0)) runnable(slot, kids & kIdMask, r, 0);
                if (__builtin_expect(w1 == want, 0)) runnable(slot, kids >> kIdBits, r, 1);
                const uint32_t d0 = w0 & kNoDev, d1 = w1 & kNoDev;
                const uint32_t same_dev = d0 == d1 ? 1u : 0u;
                if (d0 != slot && d0 != kNoDev) {
                    e1 = (kids & kIdMask) | kFirst;
                    m = 1;
                }
                if (d1 != slot && d1 != kNoDev) {
                    e2 = kids >> kIdBits | (m == 0 || !same_dev ? kFirst : 0u);
                    e1 = m == 0 ? e2 : e1;
                    ++m;
                }
            } else {
                next_op(slot);
                uint32_t sent = 0;
                for (uint32_t base = 0; base < cnt; base += 64) {
                    uint32_t c;
                    const uint32_t pc = more_kids(slot, c0 + base, cnt - base, c, r) & kNoDev;
                    const unsigned long long cross = __ballot(pc != slot && pc != kNoDev);
                    unsigned long long rest = cross, firsts = 0ull;
                    while (rest != 0ull) {                // per destination: its first child in this round
                        const uint32_t l = static_cast<uint32_t>(__builtin_ctzll(rest));
                        const uint32_t pd = get(pc, l);
                        rest &= ~__ballot(pc == pd);
                        if ((sent >> pd) & 1u) continue;
                        sent |= 1u << pd;
                        firsts |= 1ull << l;
                    }
                    if (cross != 0ull) {
                        const uint32_t x = c | (((firsts >> lane) & 1ull) ? kFirst : 0u);
                        if ((cross >> lane) & 1ull)
                            xl[c0 + m + static_cast<uint32_t>(__popcll(cross & ((1ull << lane) - 1ull)))] = static_cast<uint16_t>(x);
                        const uint32_t k = static_cast<uint32_t>(__popcll(cross));
                        const uint32_t x1 = get(x, static_cast<uint32_t>(__builtin_ctzll(cross)));
                        if (k > 1 && m == 0) e2 = get(x, static_cast<uint32_t>(__builtin_ctzll(cross & (cross - 1))));
                        if (m == 1) e2 = x1;
                        if (m == 0) e1 = x1;
                        m += k;
                    }
                }
            }
            // the output joins the bus's queue, or starts to cross at once
            const uint32_t bus = nd + slot;
            if constexpr (!PC) {
                if (__builtin_expect((cross & kNoDev) != 0, 1)) {
                    if (get(ev_t, bus) == kIdle) {
                        start_crossing(bus, now, o, dur, kids, cross);
                    } else {
                        *link_of(o) = static_cast<uint16_t>(none);
                        push(bus, o);
                    }
                }
            } else if (__builtin_expect(m != 0, 1)) {
                if (get(ev_t, bus) == kIdle) {
                    start_transfers(bus, now, o, dur, kids, m, e1, e2);
                } else {
                    rec[o].x = m | e1 << 16;
                    rec[o].w = none | e2 << 16;
                    push(bus, o);
                }
            }
        } else {
            const uint32_t xc = get(x_cur, slot);
            uint4 r;
            if constexpr (PC) {
                // the transfer was made for one child: it alone has one input fewer to wait for
                const uint32_t c = xc & kIdMask;
                r = rec[c];
                const uint32_t word = first_lane(node[c]), dev = word & kNoDev;
                node[c] = static_cast<Word>(word - kInput);
                if constexpr (TL) {
                    const size_t at = static_cast<size_t>(n0 + static_cast<int>(o)) * D + dev;
                    if (xc & kFirst) arrival[at] = __uint_as_float(now);
                    arrival_last[at] = __uint_as_float(now);
                }
                wait = ~get(ev_t, dev);                   // (idle: its queue is empty)
                if ((word >> kDevBits) == 1u) runnable(dev, c, r, 0);
            } else {
                const uint32_t dev = xc >> 5 & kNoDev;
                if constexpr (TL) arrival[static_cast<size_t>(n0 + static_cast<int>(o)) * D + dev] = __uint_as_float(now);
                wait = ~get(ev_t, dev);                   // (idle: its queue is empty)
                if (__builtin_expect(!(kids & kList), 1)) {
                    const uint32_t word = two_kids(dev, r);
                    const uint32_t w0 = get(word, 0), w1 = get(word, 1), want = kInput | dev;
                    if (w0 == want) runnable(dev, kids & kIdMask, r, 0);
                    if (__builtin_expect(w1 == want, 0)) runnable(dev, kids >> kIdBits, r, 1);
                } else {
                    for (uint32_t base = 0; base < cnt; base += 64) {
                        uint32_t c;
                        (void)more_kids(dev, c0 + base, cnt - base, c, r);
                    }
                }
            }
            // the bus goes on with the operation's next transfer, or with its queue
            if constexpr (!PC) {
                const uint32_t left = (xc & kNoDev) - 1u;
                if (__builtin_expect(left != 0, 0)) {
                    uint32_t x = left | (xc >> 10 & kNoDev) << 5;
                    const uint32_t at = xc >> 15;
                    if (left > 1) x |= first_lane(xl[c0 + at]) << 10;
                    put(x_cur, slot, x | (at + 1u) << 15);
                    schedule(slot, now, dur, o);
                } else if (get(head, slot) != none) {
                    start_first(slot, now, hr.y, hr.w >> 16 | 2u << 15);
                }
            } else {
                const uint32_t more = get(x_more, slot), left = more & kIdMask;
                if (__builtin_expect(left != 0, 0)) {
                    uint32_t x = xc >> 16;
                    if (left > 1) x |= first_lane(xl[more >> kIdBits]) << 16;
                    put(x_cur, slot, x);
                    put(x_more, slot, more + (1u << kIdBits) - 1u);
                    schedule(slot, now, dur, o);
                } else {
                    const uint32_t q = get(head, slot);
                    if (q != none) {
                        const uint32_t a = get(hr.x, slot), w = get(hr.w, slot);
                        put(head, slot, w & 0xFFFFu);
                        start_transfers(slot, now, q, get(hr.y, slot), get(hr.z, slot), a & 0xFFFFu, a >> 16, w >> 16);
                    }
                }
            }
        }
        hr = rec[head];
    } while (n_events != max_events);
    if (lane == 0) {
        out_runtime[b] = __uint_as_float(last);
        if (out_events) out_events[b] = static_cast<int32_t>(n_events);
    }
}

// Launches k_simulate for D devices and graphs of at most n_max nodes and e_max edges: 16-bit states
// where 32-bit ones do not fit (then e_max < n_max / 4, and in-degrees fit 11 bits).
template <bool TL, bool PC>
int simulate(const GraphView &gv, int D, int n_max, int e_max, const float *node_feats, const int32_t *placement,
             float inv_bw, float *runtime, int32_t *events, float *op_start, float *op_end, float *arrival,
             float *arrival_last, hipStream_t s)
{
    auto run = [&](auto kernel, size_t lds) {
        if (lds > 64 * 1024)
            PL_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
        hipLaunchKernelGGL(kernel, dim3(gv.B), dim3(kSimThreads), lds, s, gv, D, n_max, e_max, node_feats, placement,
                           inv_bw, runtime, events, op_start, op_end, arrival, arrival_last);
        return static_cast<int>(PL_OK);
    };
    const size_t wide = sim_lds<uint32_t>(n_max, e_max), narrow = sim_lds<uint16_t>(n_max, e_max);
    if (wide <= 160 * 1024)
        return D > 8 ? run(k_simulate<TL, PC, true, uint32_t>, wide) : run(k_simulate<TL, PC, false, uint32_t>, wide);
    return D > 8 ? run(k_simulate<TL, PC, true, uint16_t>, narrow) : run(k_simulate<TL, PC, false, uint16_t>, narrow);
}

// ---- peak memory of every device from the timeline (appendix "Simulator": the start and end
// timestamps of the operations and the tensor sizes predict the peak memory).  The model: the
// output of v occupies v's device from v's start until the latest of v's end, the end of its last
// consumer there and the arrival of its last outgoing transfer; on another device that consumes
// it, a copy lives from the transfer's arrival until the end of its last consumer there.
// Intervals are half-open [alloc, free).  Then the memory-penalised run time R(p) = r if m <= M else
// r + c (m - M) (appendix, "Reward"), m the largest peak.
//
// T threads take a device: the copies that live on it are collected in LDS (alloc, free, size; node order), and for
// each of their allocation times (the live sum only grows there) the live sizes are summed in float64 in node
// order.  The pairs of copies bound it (six instructions each), so a thread takes two times per pass over the
// copies.  TOGETHER: a workgroup has all D devices of a graph, a wave each, and takes the maximum over them itself;
// otherwise it has one device, and the workgroup of a graph that finishes last takes the maximum.
// (64 NMT-like graphs, 4 devices: 86 us; 412 us with one workgroup per graph that took its devices in
// turn, after a kernel that wrote every interval to memory and one that cleared the arrivals.)
constexpr int kPeakTimes = 2;          // allocation times per thread and pass

constexpr int peak_capacity(int n_max) { return (n_max + 3) / 4 * 4; }
constexpr size_t peak_lds(int n_max) { return 4 * sizeof(float) * static_cast<size_t>(peak_capacity(n_max)); }   // per device

// arrival: first crossing of an output to a device (the copy there exists from then on); arrival_last:
// last crossing (the source is kept until then); the same array unless an output may cross twice.
// peaks [B, D] and done [B] (zero between launches): exchange between a graph's workgroups.
template <int T, bool TOGETHER>
__global__ __launch_bounds__(TOGETHER ? T * kMaxD : T) void k_peak_memory(GraphView gv, int D, int n_max,
                                                     const float *__restrict__ node_feats,
                                                     const int32_t *__restrict__ placement,
                                                     const float *__restrict__ op_start,
                                                     const float *__restrict__ op_end,
                                                     const float *__restrict__ arrival,
                                                     const float *__restrict__ arrival_last,
                                                     const float *__restrict__ runtime, float mem_limit,
                                                     float penalty, double *peaks, uint32_t *done,
                                                     float *__restrict__ out_peak,
                                                     float *__restrict__ out_reward)
{
    typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
    static_assert(T % 64 == 0 && (!TOGETHER || T == 64), "devices that share a workgroup have a wave each");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    constexpr int W = T / 64;
    __shared__ double red[TOGETHER ? kMaxD : W];
    __shared__ int wave_cnt[W];
    const int cap = peak_capacity(n_max);
    // (scalars: a device's threads are whole waves)
    const int seat = TOGETHER ? __builtin_amdgcn_readfirstlane(threadIdx.x / T) : 0, seats = TOGETHER ? D : 1;
    const int b = TOGETHER ? blockIdx.x : blockIdx.x / D, d = TOGETHER ? seat : blockIdx.x - b * D;
    const int tid = threadIdx.x - seat * T, lane = tid & 63, wave = tid >> 6, threads = TOGETHER ? blockDim.x : T;
    float *ca = reinterpret_cast<float *>(lds_raw) + seat * 3 * cap, *cf = ca + cap, *cs = cf + cap;
    // by seat: bits of the latest use on that device + 1, 0: none
    uint32_t *until = reinterpret_cast<uint32_t *>(lds_raw) + seats * 3 * cap;
    const int n0 = gv.node_off[b], n = gv.node_off[b + 1] - n0;
    const float r = runtime[b];
    if (!(r == r)) {                       // invalid placement: the simulator wrote NaN
        if (tid == 0) {
            if (out_peak) out_peak[static_cast<size_t>(b) * D + d] = r;
            if (d == 0) out_reward[b] = r;
        }
        return;
    }
    for (int v = threadIdx.x; v < (TOGETHER ? seats * cap : n); v += threads) until[v] = 0;
    __syncthreads();
    // eight lanes share a node's children
    for (int v = threadIdx.x >> 3; v < n; v += threads / 8) {
        const int pv = placement[n0 + v], end = gv.nbr_ptr[1][n0 + v + 1];
        for (int p = gv.nbr_ptr[1][n0 + v] + (lane & 7); p < end; p += 8) {
            const int c = gv.nbr_idx[1][p], pc = placement[c];
            auto use = [&](int dev, float t) { atomicMax(&until[(TOGETHER ? dev * cap : 0) + v], __float_as_uint(t) + 1u); };
            auto sent = [&]() { return arrival_last[static_cast<size_t>(n0 + v) * D + pc]; };
            if constexpr (TOGETHER) {
                use(pc, op_end[c]);
                if (pc != pv) use(pv, sent());
            } else if (pc == d) {
                use(d, op_end[c]);
            } else if (pv == d) {
                use(d, sent());
            }
        }
    }
    __syncthreads();
    int k = 0;                             // copies so far
    for (int base = 0; base < n; base += T) {
        const int v = base + tid;
        float al = 0.0f, fr = 0.0f, size = 0.0f;
        bool have = false;
        if (v < n) {
            const uint32_t u = until[seat * cap + v];
            const float last = u ? __uint_as_float(u - 1u) : 0.0f;
            const bool own = placement[n0 + v] == d;
            have = own || u != 0;
            if (have) {
                al = own ? op_start[n0 + v] : arrival[static_cast<size_t>(n0 + v) * D + d];
                fr = fmaxf(own ? op_end[n0 + v] : al, last);
                size = node_feats[static_cast<size_t>(n0 + v) * 3 + 1];
            }
        }
        const unsigned long long m = __ballot(have);
        int pos = k + __popcll(m & ((1ull << lane) - 1ull));
        if constexpr (W == 1) {
            k += __popcll(m);
        } else {
            if (lane == 0) wave_cnt[wave] = __popcll(m);
            __syncthreads();
            for (int w = 0; w < W; ++w) {
                pos += w < wave ? wave_cnt[w] : 0;
                k += wave_cnt[w];
            }
        }
        if (have) {
            ca[pos] = al;
            cf[pos] = fr;
            cs[pos] = size;
        }
        if constexpr (W > 1) __syncthreads();
    }
    const int k4 = (k + 3) / 4 * 4;
    if (tid < k4 - k) {                    // padding: allocated after every time, never live
        ca[k + tid] = __builtin_inff();
        cf[k + tid] = -1.0f;
        cs[k + tid] = 0.0f;
    }
    __syncthreads();
    double mx = 0.0;
    for (int i = tid; i < k; i += T * kPeakTimes) {
        float t[kPeakTimes];
        double live[kPeakTimes];
#pragma unroll
        for (int q = 0; q < kPeakTimes; ++q) {
            t[q] = ca[min(i + q * T, k - 1)];
            live[q] = 0.0;
        }
        for (int j = 0; j < k4; j += 4) {
            const f32x4 a4 = *reinterpret_cast<const f32x4 *>(ca + j);
            const f32x4 f4 = *reinterpret_cast<const f32x4 *>(cf + j);
            const f32x4 s4 = *reinterpret_cast<const f32x4 *>(cs + j);
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int q = 0; q < kPeakTimes; ++q)
                    live[q] += static_cast<double>((a4[x] <= t[q] && t[q] < f4[x]) ? s4[x] : 0.0f);
        }
#pragma unroll
        for (int q = 0; q < kPeakTimes; ++q) mx = live[q] > mx ? live[q] : mx;
    }
    for (int step = 32; step > 0; step >>= 1) {
        const double o = __shfl_xor(mx, step);
        mx = o > mx ? o : mx;
    }
    if (lane == 0) red[TOGETHER ? seat : wave] = mx;
    __syncthreads();
    if (tid != 0) return;
    if constexpr (!TOGETHER)
        for (int w = 1; w < W; ++w) mx = red[w] > mx ? red[w] : mx;
    if (out_peak) out_peak[static_cast<size_t>(b) * D + d] = static_cast<float>(mx);
    if constexpr (TOGETHER) {
        if (seat != 0) return;
        for (int o = 1; o < D; ++o) mx = red[o] > mx ? red[o] : mx;
    } else {
        // The peak has arrived where all dies see it (an agent-scope store, waited for) before the atomic that
        // announces it, and the loads come after the atomic's result.  An acquire-release atomic would order them
        // too, but writes the die's whole L2 back first, 20 ns per workgroup and one after the other; a kernel of
        // its own for the maximum takes up to 5 us.
        double *mine = peaks + static_cast<size_t>(b) * D;
        __hip_atomic_store(mine + d, mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        const uint32_t before = __hip_atomic_fetch_add(done + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (before != static_cast<uint32_t>(D) - 1u) return;
        for (int o = 0; o < D; ++o) {
            const double x = __hip_atomic_load(mine + o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            mx = x > mx ? x : mx;
        }
        __hip_atomic_store(done + b, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const double M = static_cast<double>(mem_limit);
    out_reward[b] = mx <= M ? r : static_cast<float>(static_cast<double>(r) + static_cast<double>(penalty) * (mx - M));
}

}  // namespace

// The size that the limit of include/placeto.h is stated in: 18 n + 13 e bytes and some padding (the
// kernel takes less).
size_t simulator_lds_bytes(int n_max, int e_max)
{
    return 18 * static_cast<size_t>(n_max) + 13 * static_cast<size_t>(e_max) + 24 + 2 * (n_max & 1) + 6 * (e_max & 1);
}

int launch_simulate(const GraphView &gv, int D, int n_max, int e_max, const float *node_feats,
                    const int32_t *placement, float inv_bw, bool per_child, float *out_runtime,
                    int32_t *out_events, hipStream_t s)
{
    if (gv.B == 0) return PL_OK;
    return (per_child ? simulate<false, true> : simulate<false, false>)(gv, D, n_max, e_max, node_feats, placement, inv_bw,
                                                                        out_runtime, out_events, nullptr, nullptr, nullptr,
                                                                        nullptr, s);
}

// Simulation with the timeline, then peaks and R(p).  scratch: op_start, op_end [n_tot]; arrival,
// arrival_last (used with per_child only) [n_tot, D]; peaks [B, D]; done [B].
int launch_simulate_reward(const GraphView &gv, int D, int n_max, int e_max, const float *node_feats,
                           const int32_t *placement, float inv_bw, bool per_child, float mem_limit, float penalty,
                           float *op_start, float *op_end, float *arrival, float *arrival_last, double *peaks,
                           uint32_t *done, float *runtime, float *out_peak, float *out_reward, int32_t *out_events,
                           hipStream_t s)
{
    if (gv.B == 0) return PL_OK;
    const int rc = (per_child ? simulate<true, true> : simulate<true, false>)(
        gv, D, n_max, e_max, node_feats, placement, inv_bw, runtime, out_events, op_start, op_end, arrival, arrival_last, s);
    if (rc) return rc;
    auto run = [&](auto kernel, int blocks, int threads, size_t lds) {
        if (lds > 48 * 1024)
            PL_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(lds)));
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), lds, s, gv, D, n_max, node_feats, placement, op_start, op_end,
                           arrival, per_child ? arrival_last : arrival, runtime, mem_limit, penalty, peaks, done, out_peak,
                           out_reward);
        return static_cast<int>(PL_OK);
    };
    // A wave per device in one workgroup: no hand-over and the children read once per graph.  On large
    // graphs 512 threads share a device's pairs; in between that pays while the chip is not full of workgroups.
    // (peaks and R(p), together / apart: 4096 graphs of 32 nodes, 16 devices: 48 and 269 us; 1024 of 400, 8 devices: 115
    // and 184; 64 of 250, 4 devices: 33 and 27; 512 of 1000, 2 devices: 307 and 186.)
    if (n_max <= 128 || (n_max <= 512 && gv.B * D >= 1024))
        return run(k_peak_memory<64, true>, gv.B, 64 * D, D * peak_lds(n_max));
    return run(k_peak_memory<512, false>, gv.B * D, 512, peak_lds(n_max));
}

}  // namespace pl
