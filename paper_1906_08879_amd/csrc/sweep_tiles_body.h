// Body of the sweep kernels of one column tile to a wave (kernels_tiles.hip says how it works): included in a kernel with
// parameters `SweepParams P` where H, WS, L, FF, WX, BW and TR are compile-time constants.  (As text: as a function that both
// kernels call, one variant of the narrow ones spills.)
    static_assert(!BW || (!FF && !WX), "the reverse pass reads its input from emb and writes no xb");
    static_assert(!TR || (FF && !WX && !BW), "activations are kept for a single forward sweep");
    constexpr int NTL = H / 16, KS = H / 32;   // output column tiles (a wave each), k-steps of a product
    constexpr int kThreads = 64 * NTL;
    constexpr int NL = 2 * L;                  // layers per chunk: g then f
    constexpr int LDA = H + 16;
    constexpr int kActTile = 16 * LDA;         // one 16-row tile
    constexpr int LDM = H + 16;
    constexpr int kZeroSlot = kMsgSlots;
    constexpr int kPre = 8;                    // messages of a list that are requested ahead of its sum
    constexpr bool kLdsFirst = !BW && !TR && !WX;   // what the next layer waits for goes to LDS ahead of the stores to HBM
    __shared__ __attribute__((aligned(16))) float msgtab[(kMsgSlots + 1) * LDM];
    __shared__ __attribute__((aligned(16))) __bf16 actbuf[2][NT * kActTile];
    __shared__ float proj_dev[(kMaxD + 1) * H];   // one-hot device rows of W_in, then a zero row
    auto act_at = [&](int buf, int r, int k) __attribute__((always_inline)) { return &actbuf[buf][r * LDA + k]; };

    const int b = blockIdx.x >> 1, dir = blockIdx.x & 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, kg = lane >> 4;    // MFMA result: column col, node kg of a tile
    const uint32_t mc = static_cast<uint32_t>(16 * wave + col);   // this lane's output column

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
    const uint32_t spare_row = static_cast<uint32_t>((2 - dir) * gv.n_tot - n0), sink_row = spare_row + 1u;
    const uint32_t emb_sink = static_cast<uint32_t>(gv.n_tot - n0);

    // ---- records: requested four chunks before they are processed
    auto load_rec = [&](int c, u32x4 (&rec)[NT]) __attribute__((always_inline)) {
        const u32x4 *base = reinterpret_cast<const u32x4 *>(plan.rec + static_cast<size_t>(c < c_end ? c : c_end - 1) * CH);
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) rec[ct] = elem(base, 16u * static_cast<uint32_t>(4 * ct + kg));
    };
    u32x4 rec0[NT], rec1[NT], rec2[NT], rec3[NT];
    load_rec(c_begin, rec0);
    load_rec(c_begin + 1, rec1);
    load_rec(c_begin + 2, rec2);
    load_rec(c_begin + 3, rec3);

    bf16x8 W[NL][KS][WS];
    float bias[NL];
#pragma unroll
    for (int n = 0; n < NL; ++n) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int ws = 0; ws < WS; ++ws) {
                const size_t at = ((((static_cast<size_t>(dir) * NL + n) * NTL + wave) * KS + ks) * WS + ws) * 64 + lane;
                const uint4 raw = P.wfrag[at];
                W[n][ks][ws] = *reinterpret_cast<const bf16x8 *>(&raw);
            }
        bias[n] = P.bias[(static_cast<size_t>(dir) * NL + n) * H + mc];
    }
    const int D = P.D;
    float pw_time = 0.0f, pw_size = 0.0f, pw_cur = 0.0f, pw_vis = 0.0f, pw_b = 0.0f;
    if constexpr (FF) {
        pw_time = P.proj[mc];
        pw_size = P.proj[H + mc];
        pw_cur = P.proj[(2 + D) * H + mc];
        pw_vis = P.proj[(3 + D) * H + mc];
        pw_b = P.proj[(4 + D) * H + mc];
        for (int i = tid; i < (kMaxD + 1) * H; i += kThreads) proj_dev[i] = (i < D * H) ? P.proj[2 * H + i] : 0.0f;
    }
    for (int i = tid; i < (kMsgSlots + 1) * LDM; i += kThreads) msgtab[i] = 0.0f;
    for (int i = tid; i < 2 * NT * kActTile; i += kThreads) (&actbuf[0][0])[i] = static_cast<__bf16>(0.0f);

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
    // byte offset of this lane's column of a row of floats
    auto at4 = [&](uint32_t row) __attribute__((always_inline)) { return 4u * (row * H + mc); };

    // What a chunk reads of a node besides its messages: raw features (FF), the outside gradient of its state and
    // its gates (BW), or the input of a later sweep.
    struct Inputs {
        float time, size, vis, x;
        int dev, gates;
    };
    auto load_inputs = [&](const u32x4 &rec, int ct, int rows, int p, Inputs &in) __attribute__((always_inline)) {
        if constexpr (FF) {
            const uint32_t v = node_of(rec);
            const float *f = &elem(feats, v * 12u);
            in.time = f[0];
            in.size = f[1];
            in.vis = f[2];
            in.dev = elem(placement, v * 4u);
        } else if constexpr (BW) {
            const uint32_t v = node_of(rec);
            in.x = elem(emb, 8u * H * v + 4u * mc);
            in.gates = elem(gates_in, v * H + mc);
        } else {
            const int r = 4 * ct + kg;
            in.x = elem(xb, at4(static_cast<uint32_t>(p + (r < rows ? r : 0))));
        }
    };
    // x_v = relu(W_in^T phi_v + b) (Section 2.2 step 1)
    auto project = [&](const Inputs &in, uint32_t v) __attribute__((always_inline)) {
        const uint32_t dev = static_cast<uint32_t>(in.dev), none = static_cast<uint32_t>(D);
        float o = fmaf(in.time, pw_time, pw_b);
        o = fmaf(in.size, pw_size, o);
        o += proj_dev[(dev < none ? dev : none) * H + mc];
        o += v == cur ? pw_cur : 0.0f;
        return fmaxf(fmaf(in.vis, pw_vis, o), 0.0f);
    };
    // the row's far message (a row of zeros if it has none)
    auto load_far = [&](const u32x4 &rec) __attribute__((always_inline)) {
        static_assert(kRecListed == 1u << 30 && kNoFar == 0xFFFFFFFFu, "a listed row's second word becomes kNoFar");
        const uint32_t u = rec[1] | static_cast<uint32_t>(static_cast<int32_t>(rec[0] << 1) >> 31);
        return elem(msg, at4(u < spare_row ? u : spare_row));
    };
    // Writes this lane's value of node row r, split exactly into three bf16 parts, as rows 4 r .. 4 r + 2 of an A operand.
    auto put_rows = [&](int buf, int r, float y) __attribute__((always_inline)) {
        const float rr = y - trunc_bf16(y), ll = rr - trunc_bf16(rr);
        unsigned short *dst = reinterpret_cast<unsigned short *>(act_at(buf, 4 * r, mc));
        dst[0] = static_cast<unsigned short>(__float_as_uint(y) >> 16);
        dst[LDA] = static_cast<unsigned short>(__float_as_uint(rr) >> 16);
        dst[2 * LDA] = static_cast<unsigned short>(__float_as_uint(ll) >> 16);
    };

    // ---- gather of a chunk: a_v = sum of neighbour messages, for rows kg and kg + 4 and this lane's column.  `signs` collects
    // the sign bits.
    auto add = [&](float &s, uint32_t &signs, float x) __attribute__((always_inline)) {
        s += BW ? x : fabsf(x);
        if (!BW) signs |= __float_as_uint(x);
    };
    auto start_sum = [&](float far, float &s, uint32_t &signs) __attribute__((always_inline)) {
        signs = BW ? 0u : __float_as_uint(far);
        s = BW ? far : fabsf(far);
    };
    // slots K0 .. K1 - 1 of a record
    auto add_slots = [&](auto k0c, auto k1c, uint32_t slots, float &s, uint32_t &signs) __attribute__((always_inline)) {
        constexpr int K0 = decltype(k0c)::value, K1 = decltype(k1c)::value;
        float x[K1 - K0];
#pragma unroll
        for (int k = K0; k < K1; ++k) x[k - K0] = elem(msgtab, ((slots >> (6 * k)) & 63u) * (4u * LDM) + 4u * mc);
#pragma unroll
        for (int k = K0; k < K1; ++k) add(s, signs, x[k - K0]);
    };
    using k0 = std::integral_constant<int, 0>;
    using k1 = std::integral_constant<int, 1>;
    using k2 = std::integral_constant<int, 2>;
    using kmax = std::integral_constant<int, kMaxNear>;
    // entry i of a listed row: a table slot (-1 - slot) or a node id; past the end, the table's row of zeros
    auto entry = [&](const u32x4 &rec, int i) __attribute__((always_inline)) {
        const bool in = (rec[0] & kRecListed) && i < static_cast<int>(rec[0] & 0xFFFFFFu);
        return in ? elem(plan.ovf, 4u * (rec[1] + static_cast<uint32_t>(i))) : -1 - kZeroSlot;
    };
    // Byte offsets of sixteen entries' rows, an entry to a lane: of the message of a far one (a row of zeros otherwise), and of
    // the table row of a near one.
    auto far_row = [&](int id) __attribute__((always_inline)) { return 4u * H * (id >= 0 ? static_cast<uint32_t>(id) : spare_row); };
    auto near_row = [&](int id) __attribute__((always_inline)) { return 4u * LDM * static_cast<uint32_t>(id < 0 ? -1 - id : kZeroSlot); };
    auto from_lane = [&](uint32_t x, int k) __attribute__((always_inline)) {
        return static_cast<uint32_t>(__shfl(static_cast<int>(x), (lane & 48) + k));
    };
    // far messages of entries K0 .. of sixteen
    auto request = [&](auto k0c, uint32_t rows, auto &y) __attribute__((always_inline)) {
        constexpr int K0 = decltype(k0c)::value, K = sizeof(y) / sizeof(y[0]);
#pragma unroll
        for (int k = 0; k < K; ++k) y[k] = elem(msg, from_lane(rows, K0 + k) + 4u * mc);
    };
    auto sum_list = [&](const u32x4 &rc, int ids, const float (&pre)[kPre], float &s, uint32_t &signs) __attribute__((always_inline)) {
        const int cnt = static_cast<int>(rc[0] & 0xFFFFFFu);
        auto take = [&](const auto &y) __attribute__((always_inline)) {
            constexpr int K = sizeof(y) / sizeof(y[0]);
#pragma unroll
            for (int k = 0; k < K; ++k) add(s, signs, y[k]);
        };
        // near sources among the sixteen entries: the few places that are near in some row
        auto take_near = [&](int id) __attribute__((always_inline)) {
            const unsigned long long all = __ballot(id < 0 && id != -1 - kZeroSlot);
            uint32_t near = static_cast<uint32_t>(all) | static_cast<uint32_t>(all >> 32);
            near = (near | near >> 16) & 0xFFFFu;
            const uint32_t rows = near_row(id);
#pragma unroll 1
            for (; near != 0u; near &= near - 1u) {
                const float x[1] = {elem(msgtab, from_lane(rows, __builtin_ctz(near)) + 4u * mc)};
                take(x);
            }
        };
        // Messages y of the entries K0 .. of sixteen, and their near ones, in list order: at 128 columns, where batches of
        // more graphs take another kernel (k_sweep_mfma), which sums that way: a graph's results are the same bits there.
        auto take_in_order = [&](auto k0c, int id, const auto &y) __attribute__((always_inline)) {
            constexpr int K0 = decltype(k0c)::value, K = sizeof(y) / sizeof(y[0]);
            const unsigned long long all = __ballot(id < 0 && id != -1 - kZeroSlot);
            const uint32_t near = static_cast<uint32_t>(all) | static_cast<uint32_t>(all >> 32);
            if ((((near | near >> 16) >> K0) & ((1u << K) - 1u)) == 0u) {
                take(y);
                return;
            }
            const uint32_t rows = near_row(id);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float x = elem(msgtab, from_lane(rows, K0 + k) + 4u * mc);
                s += BW ? x + y[k] : fabsf(x) + fabsf(y[k]);
                if (!BW) signs |= __float_as_uint(x) | __float_as_uint(y[k]);
            }
        };
        using i8 = std::integral_constant<int, 8>;
        using i0 = std::integral_constant<int, 0>;
        int id1 = entry(rc, 16 + col);
        if constexpr (H == 128) {
            float y8[8];
            if (cnt > 8) request(i8{}, far_row(ids), y8);
            take_in_order(i0{}, ids, pre);
            if (cnt > 8) take_in_order(i8{}, ids, y8);
        } else if (cnt > 8) {
            float y[8];
            request(i8{}, far_row(ids), y);
            take(pre);
            take_near(ids);
            take(y);
        } else {
            take(pre);
            take_near(ids);
        }
#pragma unroll 1
        for (int p = 16; p < cnt; p += 16) {
            float y[16];
            request(i0{}, far_row(id1), y);
            const int id2 = entry(rc, p + 16 + col);
            if constexpr (H == 128) {
                take_in_order(i0{}, id1, y);
            } else {
                take_near(id1);
                take(y);
            }
            id1 = id2;
        }
        // (nothing of this path is in flight where it joins the others: they would wait for it)
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    };
    auto finish_row = [&](int ct, float s, uint32_t w3, const Inputs (&in)[NT], bool valid, float (&gs)[NT]) __attribute__((always_inline)) {
        if constexpr (BW) {
            s = (in[ct].gates & 1) ? s : 0.0f;
            gs[ct] = s;
        }
        if constexpr (TR) {
            const uint32_t id = w3 & kRecNoNode;
            dlt[(id == kRecNoNode || !valid ? static_cast<size_t>(2 * L) * gv.n_tot : static_cast<size_t>(static_cast<uint32_t>(n0) + id)) * H + mc] = s;
        }
        put_rows(0, 4 * ct + kg, s);
    };
    // info = word 3 of a record of the chunk (its chunk-wide bits); valid: there is such a chunk
    auto gather = [&](uint32_t info, const u32x4 (&rec)[NT], const float (&far)[NT], const int (&ids)[NT],
                      const float (&pre)[NT][kPre], const Inputs (&in)[NT], bool valid, uint32_t (&signs)[NT],
                      float (&gs)[NT]) __attribute__((always_inline)) {
        const bool two = ((info >> kRecRowsShift) & 7u) >= kTileNodes;
        const int cls = static_cast<int>((info >> kRecNearShift) & 3u);
        float s[NT];
        start_sum(far[0], s[0], signs[0]);
        if (two) start_sum(far[1], s[1], signs[1]);
        if ((info >> kRecGeneralBit) & 1u) {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                if (ct > 0 && !two) break;
                if (rec[ct][0] & kRecListed)
                    sum_list(rec[ct], ids[ct], pre[ct], s[ct], signs[ct]);
                else
                    add_slots(k0{}, kmax{}, rec[ct][0], s[ct], signs[ct]);
            }
        } else if (!two) {
            add_slots(k0{}, k1{}, rec[0][0], s[0], signs[0]);
            if (cls != 0) {
                add_slots(k1{}, k2{}, rec[0][0], s[0], signs[0]);
                if (cls == 2) add_slots(k2{}, kmax{}, rec[0][0], s[0], signs[0]);
            }
        } else {
            add_slots(k0{}, k1{}, rec[0][0], s[0], signs[0]);
            add_slots(k0{}, k1{}, rec[1][0], s[1], signs[1]);
            if (cls != 0) {
                add_slots(k1{}, k2{}, rec[0][0], s[0], signs[0]);
                add_slots(k1{}, k2{}, rec[1][0], s[1], signs[1]);
                if (cls == 2) {
                    add_slots(k2{}, kmax{}, rec[0][0], s[0], signs[0]);
                    add_slots(k2{}, kmax{}, rec[1][0], s[1], signs[1]);
                }
            }
        }
        finish_row(0, s[0], rec[0][3], in, valid, gs);
        if (two) finish_row(1, s[1], rec[1][3], in, valid, gs);
    };

    // ---- state of the pipeline.  A register that a load is still filling is never copied: the chunk loop is unrolled
    // by four, and every set of registers keeps its place.
    //   rec0 .. rec3  records of chunk c, c + 1, ..; those of chunk c are the target of chunk c + 4's
    //   in0 / in1     inputs of chunk c / c + 1, then targets of c + 2 / c + 3
    //   far0 / far1, ids0 / ids1   far messages, list entries of chunk c + 1 / targets for chunk c + 2
    //   pre           first messages of chunk c + 1's lists;  gs: (BW) gated sums of chunk c
    Inputs in0[NT] = {}, in1[NT] = {};
    float far0[NT] = {}, far1[NT] = {};   // (the first kRing + 1 chunks have no far sources)
    int ids0[NT], ids1[NT];
    float pre[NT][kPre] = {};
    float gs[NT] = {};
    int rows0, p0;
    uint32_t vg[NT], sign[NT] = {};
    {
        const uint32_t info0 = first(rec0[0][3]), info1 = first(rec1[0][3]);
        rows0 = rows_of(info0);
        p0 = static_cast<int>(first(rec0[0][2]));
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            ids0[ct] = ids1[ct] = -1 - kZeroSlot;
            vg[ct] = node_of(rec0[ct]);
            load_inputs(rec0[ct], ct, rows0, p0, in0[ct]);
            load_inputs(rec1[ct], ct, rows_of(info1), static_cast<int>(first(rec1[0][2])), in1[ct]);
        }
        __syncthreads();
        gather(info0, rec0, far0, ids0, pre, in0, true, sign, gs);   // (the first chunk has no sources)
        if ((info1 >> kRecGeneralBit) & 1u) {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) ids0[ct] = entry(rec1[ct], col);
        }
    }
    __syncthreads();

    // rT: target for the records of chunk c + 4; rA, rB: records of chunks c + 1, c + 2; in: inputs of chunk c, then
    // target of chunk c + 2's; inN: of chunk c + 1; farA / farB, idsA / idsB: of chunk c + 1 / target for chunk c + 2
    auto step = [&](auto twoc, auto ringc, int c, u32x4 (&rT)[NT], const u32x4 (&rA)[NT], const u32x4 (&rB)[NT], Inputs (&in)[NT],
                    const Inputs (&inN)[NT], float (&farA)[NT], float (&farB)[NT], int (&idsA)[NT],
                    int (&idsB)[NT]) __attribute__((always_inline)) {
        constexpr bool two = decltype(twoc)::value != 0;   // the chunk fills a second row tile
        constexpr int T = two ? 2 : 1;
        constexpr uint32_t ring_row = decltype(ringc)::value * CH;   // where this chunk's messages go in the table
        const int rows = rows0;
        const uint32_t info1 = first(rA[0][3]), info2 = first(rB[0][3]);
        const bool two2 = rows_of(info2) > kTileNodes;
        f32x4 acc[T];
        int gate_bits[T];
        float x0[T];
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            bf16x8 a1[KS];
            if constexpr (!two) {     // (the loads and stores of the pipeline are issued while the fragments travel)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) a1[ks] = *reinterpret_cast<const bf16x8 *>(act_at(n & 1, col, 32 * ks + 8 * kg));
                __builtin_amdgcn_sched_barrier(0);
            }
            auto mid_block = [&]() __attribute__((always_inline)) {
                if (n == 0) {
                    farB[0] = load_far(rB[0]);
                    if (two2) farB[1] = load_far(rB[1]);
                    load_rec(c + 4, rT);
                    if ((info1 >> kRecGeneralBit) & 1u) {
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) request(std::integral_constant<int, 0>{}, far_row(idsA[ct]), pre[ct]);
                    }
                    if ((info2 >> kRecGeneralBit) & 1u) {
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) idsB[ct] = entry(rB[ct], col);
                    }
                }
                if (n == L - 1) {
                    if constexpr (FF) {
#pragma unroll
                        for (int ct = 0; ct < T; ++ct) x0[ct] = project(in[ct], vg[ct]);
                    }
                }
                if (n == (BW ? NL - 1 : L)) {
                    const int p2 = static_cast<int>(first(rB[0][2]));
                    load_inputs(rB[0], 0, rows_of(info2), p2, in[0]);
                    if (two2) load_inputs(rB[1], 1, rows_of(info2), p2, in[1]);
                }
                if (n == NL - 1) {
                    if constexpr (!BW) {
#pragma unroll
                        for (int ct = 0; ct < T; ++ct) {
                            const bool mine = wave == 0 && col == 0 && ct * kTileNodes + kg < rows;
                            elem(reach, mine ? vg[ct] : sink_row) = static_cast<uint8_t>(sign[ct] >> 31);
                        }
                    }
                }
            };
            auto mfma = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int ct = 0; ct < T; ++ct) {
                        const bf16x8 a = two ? *reinterpret_cast<const bf16x8 *>(act_at(n & 1, 16 * ct + col, 32 * ks + 8 * kg)) : a1[ks];
#pragma unroll
                        for (int ws = 0; ws < WS; ++ws) {
                            const f32x4 c_in = (ks == 0 && ws == 0) ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[ct];
                            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, W[n][ks][ws], c_in, 0, 0, 0);
                        }
                    }
            };
            // lane (col, kg) holds, for node 4 ct + kg and its output column, the three partial products in elements 0..2
            auto epilogue = [&](int ct) __attribute__((always_inline)) {
                const int r = ct * kTileNodes + kg;
                const bool live = r < rows;
                const uint32_t v = vg[ct];
                const uint32_t v_emb = live ? v : emb_sink, v_msg = live ? v : sink_row;
                auto delta_to = [&](int slot, float d) __attribute__((always_inline)) {   // (unused rows: the spare row)
                    dlt[(live ? static_cast<size_t>(slot) * gv.n_tot + (static_cast<uint32_t>(n0) + v) : static_cast<size_t>(2 * L) * gv.n_tot) * H + mc] = d;
                };
                float y = acc[ct][0] + acc[ct][1] + acc[ct][2];
                if constexpr (BW) {
                    // delta slot of this layer's gated output: f's layers L-2 .. 0, then g's layers L-1 .. 0
                    if (n == 0) delta_to(L - 1, gs[ct]);
                    const int gates = in[ct].gates;
                    if (n == L - 1) {                // end of f^T: ds_v = outside gradient + f path
                        y += in[ct].x;
                        elem(emb, 8u * H * v_emb + 4u * mc) = y;
                        y = (gates & 4) ? y : 0.0f;
                        delta_to(2 * L - 1, y);
                    } else if (n < L - 1) {
                        y = (gates & 2) ? y : 0.0f;
                        delta_to(L - 2 - n, y);
                    } else if (n < NL - 1) {
                        y = (gates & 8) ? y : 0.0f;
                        delta_to(L + NL - 2 - n, y);
                    }
                    if (n == NL - 1) {               // end of g^T: da_v
                        msgtab[(ring_row + r) * LDM + mc] = y;
                        elem(msg, at4(v_msg)) = y;
                    } else {
                        put_rows((n + 1) & 1, r, y);
                    }
                    return;
                }
                y = fmaxf(y + bias[n], 0.0f);
                if constexpr (TR) {
                    const int bit = n == NL - 1 ? 1 : (n == L - 1 ? 4 : (n == 0 ? 8 : 2));
                    gate_bits[ct] = (n == 0 ? 0 : gate_bits[ct]) | (y > 0.0f ? bit : 0);
                }
                const float out = y;
                if (n == L - 1) y += FF ? x0[ct] : in[ct].x;    // end of g: residual update of s_v
                if (n == NL - 1) {                   // end of f: the message of v, flagged
                    const uint32_t flag = sign[ct] | (v == cur ? 0x80000000u : 0u);
                    y = __uint_as_float((__float_as_uint(y) & 0x7FFFFFFFu) | (flag & 0x80000000u));
                }
                if (n < NL - 1)
                    put_rows((n + 1) & 1, r, y);
                else
                    msgtab[(ring_row + r) * LDM + mc] = y;
                if constexpr (kLdsFirst) __builtin_amdgcn_sched_barrier(0);
                if constexpr (TR) {
                    // (the output of g's last layer is only ever needed as a gate)
                    if (n < NL - 1 && n != L - 1) delta_to(1 + n, out);
                    if (n == NL - 1) elem(gates_out, (live ? v : spare_row) * H + mc) = static_cast<uint8_t>(gate_bits[ct]);
                }
                if (n == L - 1) {
                    elem(emb, 8u * H * v_emb + 4u * mc) = y;
                    if constexpr (WX) elem(xb, at4(live ? static_cast<uint32_t>(p0 + r) : spare_row)) = y;
                }
                if (n == NL - 1) elem(msg, at4(v_msg)) = y;
            };
            mid_block();
            __builtin_amdgcn_sched_barrier(0);
            mfma();
            epilogue(0);
            if constexpr (two) epilogue(1);
            if (n == NL - 1) gather(info1, rA, farA, idsA, pre, inN, c + 1 < c_end, sign, gs);
            lds_barrier();
        }
        rows0 = c + 1 < c_end ? rows_of(info1) : 0;
        p0 = static_cast<int>(first(rA[0][2]));
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            vg[ct] = node_of(rA[ct]);
            // (a word of the record that nothing reads would be given to another value while its load is in flight, and
            // that value would wait for the load)
            asm volatile("" : : "v"(rA[ct][2]));
        }
    };
    auto any_step = [&](auto ringc, int c, u32x4 (&rT)[NT], const u32x4 (&rA)[NT], const u32x4 (&rB)[NT], Inputs (&in)[NT],
                        const Inputs (&inN)[NT], float (&farA)[NT], float (&farB)[NT], int (&idsA)[NT],
                        int (&idsB)[NT]) __attribute__((always_inline)) {
        if (rows0 > kTileNodes)
            step(std::integral_constant<int, 1>{}, ringc, c, rT, rA, rB, in, inN, farA, farB, idsA, idsB);
        else
            step(std::integral_constant<int, 0>{}, ringc, c, rT, rA, rB, in, inN, farA, farB, idsA, idsB);
    };
    // Four chunks per turn; chunks past the last have no rows and store to the spare rows only.  One test, in the middle: a test
    // costs copies of what is still being loaded (one behind every chunk: 64 NMT-like graphs 566 -> 572 us), but a graph
    // of 13 chunks should not take the time of 16 (forward pass, 512 random graphs of 13 nodes, H = 64, fp32, without a
    // test / with it: 102 / 95 us; 8 nodes 77 / 73).  Where it would take the last registers of tile_residency there is none.
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the loop's waits are counted from its own loads
    static_assert(RING == 4, "a turn takes as many chunks as the table holds");
    constexpr bool kMiddleTest = !(H == 64 && WS == 1 && L == 1 && !FF);
    for (int c = c_begin; c < c_end; c += 4) {
        any_step(std::integral_constant<int, 0>{}, c, rec0, rec1, rec2, in0, in1, far0, far1, ids0, ids1);
        any_step(std::integral_constant<int, 1>{}, c + 1, rec1, rec2, rec3, in1, in0, far1, far0, ids1, ids0);
        if (kMiddleTest && c + 2 >= c_end) return;
        any_step(std::integral_constant<int, 2>{}, c + 2, rec2, rec3, rec0, in0, in1, far0, far1, ids0, ids1);
        any_step(std::integral_constant<int, 3>{}, c + 3, rec3, rec0, rec1, in1, in0, far1, far0, ids1, ids0);
    }
