// What the reductions over the vertices leave, and where an epoch keeps it: host arithmetic, free of HIP so that it can be tested by itself.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include "gcn.h"

namespace gcn {

// Compute units for which kernels are cut whose partial results lie in the caller's workspace: its size, asked before or under another device,
// and the order of the sums must not depend on the device that is current.
constexpr int SIZED_FOR_CUS = 256;

// A gradient over few rows, M x N, which is cut into shares of 64 of them: as many as a workgroup of the kernel of few and short rows makes, which then
// leaves the same partial results (see gradient_next).  In an epoch that saves a launch (17 K to 24 K rows: 0.87 to 0.96 of the time of an epoch with
// longer shares, 32 K 0.90 to 0.97), and a layer's own call is cut alike, for the same bits.  With more than 32 columns, not beyond
// 16 K rows: more workgroups than compute units.
inline bool few_rows(int64_t M, int64_t N, int64_t K) {
    const int64_t wide = M > N ? M : N, narrow = M > N ? N : M;
    return K >= 64 && narrow <= 16 && (wide <= 32 ? K <= 32768 : wide <= 64 && K <= 16384);
}

// The same for a product by itself, which has no rows to wait for: one trip of a workgroup is the faster only while there are few of them (16 x 16 over 1000
// rows 4.6 us and 5.3 with longer shares, 32 x 16 over 12 K 6.3 and 6.8, over 20 K 6.7 and 7.0, but 16 x 16 over 32 K 6.7 and 6.0; 64 x 16 over 8 K 5.9 and
// 6.2, alike from 12 K on).
inline bool few_rows_alone(int64_t M, int64_t N, int64_t K) {
    return few_rows(M, N, K) && K <= (M <= 32 && N <= 32 ? 20000 : 12000);
}

// Launch geometry of the A^T B product (K long): which operand goes on the 64-column groups, wavefronts per
// workgroup, split of K, partial buffers.  Any shape.
struct TnShape {
    bool swap, narrow;
    int64_t Mw, Nw, blocks, kpb;
    int NT, ny, nz, gw, rw, MG, fold;
    size_t scratch_bytes;
};

inline TnShape tn_shape(int64_t M, int64_t N, int64_t K, bool few) {
    TnShape g;
    // Put the wider of (M, N) on the 64-column groups: if N > M compute C^T = B^T A and let the
    // reduction write it back transposed.
    g.swap = N > M;
    g.Mw = g.swap ? N : M;
    g.Nw = g.swap ? M : N;
    const int nt = (int)((g.Nw + 15) / 16);
    g.ny = (nt + 3) / 4;                                  // up to 64 columns of B per wavefront, in equal shares
    g.NT = (nt + g.ny - 1) / g.ny;
    g.narrow = g.Mw <= 32;
    const int groups = (int)((g.Mw + 63) / 64);
    g.rw = 1; g.nz = 1; g.gw = 4;
    if (g.narrow) {
        g.MG = (int)((g.Mw + 15) / 16);
    } else {
        // column groups per wavefront: what two sets of accumulators and two trips leave room for (250 registers)
        const int mg_max = g.NT >= 2 ? 1 : 3;
        // wavefronts on different groups: one per group up to 8, else the count in 4..8 that leaves the fewest idle
        // slots (300 columns: 5 groups on 5 wavefronts instead of 2+1+1+1 on 4)
        g.gw = groups;
        if (groups > 8) {
            int best = 1 << 30;
            for (int w = 4; w <= 8; ++w) {
                const int idle = (groups + w - 1) / w * w - groups;
                if (idle < best) { best = idle; g.gw = w; }
            }
        }
        g.rw = g.gw >= 4 ? 1 : 4 / g.gw;                  // 1 group: 4 sets of rows, 2: 2, 3: 1
        g.MG = (groups + g.gw - 1) / g.gw;
        if (g.MG > mg_max) g.MG = mg_max;
        g.nz = (groups + g.gw * g.MG - 1) / (g.gw * g.MG);
    }
    // Workgroups over K: at least two trips of every wavefront each,
    const int64_t rows = g.narrow ? 64 : 16 * g.rw;       // rows per trip of a workgroup
    const int64_t count = g.Mw * g.Nw;
    // or one trip where the gradient is over few rows (see few_rows),
    int64_t blocks = few ? (K + 63) / 64 : K / (2 * rows);
    // but no more workgroups than run side by side: a workgroup loads its next trip while it multiplies, and the partial results
    // are written and read once more.  One per compute unit, two where the partial results are below 1/40 of the operands
    // (200 x 32 over 1 M rows 231 and 199 us; 256 x 64 over 120 K rows 52 and 64); four of the narrow kernel (16 x 16 over 4.4 M rows:
    // 105 us, two 150, eight 112), eight where a row of both has less than 32 floats, so that lanes are idle and less is on its
    // way (7 x 3 over 3.8 M rows: 62 us, four 67; 16 x 8 over 3.6 M 72 and 77).  With up to 8192, and partial results below an eighth of the operands: 300 x 16 over 14.2 M
    // rows 3.20 ms (now 2.86, 6.4 TB/s), 128 x 16 over 4.4 M 425 us (364), 256 x 64 over 120 K 89 (52), 602 x 64 over 100 K 255 (127).
    const int64_t cus = SIZED_FOR_CUS, operands = K * (g.Mw + g.Nw);
    int64_t most = (g.narrow ? (g.Mw + g.Nw < 32 ? 8 : 4) : (80 * cus * count <= operands ? 2 : 1)) * cus / ((int64_t)g.ny * g.nz);
    // partial results below a third of the operands, unless that leaves fewer than 64 workgroups over K (fewer still where
    // the result alone is large)
    const int64_t fair = operands / (3 * count);
    const int64_t least = count >= (1ll << 26) ? 1 : (count > (1ll << 20) ? (1ll << 26) / count : 64);
    if (most > fair) most = fair;
    if (most < least) most = least;
    if (few) most = blocks;
    if (blocks > most) blocks = most;
    if (blocks < 1) blocks = 1;
    int64_t kpb = (K + blocks - 1) / blocks;
    kpb = (kpb + rows - 1) / rows * rows;
    g.kpb = kpb;
    g.blocks = (K + kpb - 1) / kpb;
    g.fold = g.blocks > 512 ? 64 : 0;                     // two-stage reduction when there are many partials
    g.scratch_bytes = (size_t)(g.blocks + g.fold) * count * sizeof(float);
    return g;
}

// Workgroups of the loss kernel over n rows of C classes: up to 256 classes four to a lane, 256 lanes to a workgroup, else four rows to one.
constexpr int LOSS_BLOCKS_MAX = 2048;
inline int loss_lanes(int32_t C) {            // of a row; up to four classes a row is one lane's (two classes, 2 M rows: 12.9 us, two lanes 24.8)
    int lanes = 1;
    while (4 * lanes < C && lanes < 64) lanes <<= 1;
    return lanes;
}
inline int64_t loss_blocks(int64_t n, int32_t C) {
    const int64_t rows = 256 / loss_lanes(C), blocks = (n + rows - 1) / rows;
    return blocks > LOSS_BLOCKS_MAX ? LOSS_BLOCKS_MAX : blocks;
}
inline size_t loss_scratch_bytes() { return (size_t)LOSS_BLOCKS_MAX * sizeof(double); }
// What n rows need of it: a partial sum of each workgroup, or of every 16 rows where the product's kernel makes the loss (see loss_next).
inline size_t loss_part_bytes(int64_t n, int32_t C) {
    const int64_t blocks = loss_blocks(n, C), strips = (n + 15) / 16;
    return (size_t)(strips > blocks ? (strips < LOSS_BLOCKS_MAX ? strips : LOSS_BLOCKS_MAX) : blocks) * sizeof(double);
}

// The fused last layer: tiles of 16 classes, and its workgroups.
constexpr int FUSED_BLOCKS_MAX = 2048;
inline int fused_nt(int32_t C) {
    const int need = (C + 15) / 16;
    const int have[6] = {1, 2, 3, 4, 8, 16};
    for (int i = 0; i < 6; ++i)
        if (have[i] >= need) return have[i];
    return 0;
}

// Four strips and more per wavefront, which pay for its operands and for its partial result (233 K rows, 41 classes, whole layer: 26 us
// with 2048 workgroups, 21 with a thousand; 1.8 M, 24: 74 and 75), but as many workgroups as there are compute units before any takes a
// second strip: a strip is a chain of latencies, and beyond 64 classes a workgroup goes through its strips one by one (epochs of
// 982 rows, 183 classes 66.5 us with 4 workgroups, 36.0 with 62; 12 K, 166: 73.7 with 48, 49.9 with 256).
inline int64_t fused_blocks(int64_t n, int NT) {
    const int64_t strips = (n + 15) / 16, at_once = NT > 4 ? strips : (strips + 3) / 4;
    constexpr int64_t cus = SIZED_FOR_CUS;
    int64_t blocks = (strips + 15) / 16;
    if (blocks < cus) blocks = at_once < cus ? at_once : cus;
    return blocks > FUSED_BLOCKS_MAX ? FUSED_BLOCKS_MAX : (blocks < 1 ? 1 : blocks);
}

inline bool fused_last_supported(int32_t f_in, int32_t C) { return f_in == 16 && C >= 1 && fused_nt(C) != 0; }

inline size_t fused_last_scratch_bytes(int64_t n, int32_t C) {
    const int NT = fused_nt(C);
    if (!NT) return 0;
    const size_t per = (size_t)16 * 16 * NT * sizeof(float);
    return (size_t)fused_blocks(n, NT) * per + (size_t)FUSED_BLOCKS_MAX * sizeof(double);
}

inline int resolve_order(int order, int32_t f_in, int32_t f_out) {
    if (order == GCN_ORDER_GEMM_FIRST || order == GCN_ORDER_SPMM_FIRST) return order;
    // The SpMM costs in proportion to its width: run it at min(f_in, f_out).
    return f_out <= f_in ? GCN_ORDER_GEMM_FIRST : GCN_ORDER_SPMM_FIRST;
}

// ---- epoch workspace layout -------------------------------------------------------------------
struct EpochLayout {
    std::vector<size_t> Z, H, T, G;   // byte offsets per layer index 0..L_w-1 (layer l = index + 1)
    size_t S = 0, XS = 0, total = 0;  // XS: pre-scaled SpMM operand of the value-free product
    size_t scratch = 0;               // partial sums of the fused last layer, and the next where they do not fit XS
    std::vector<int> order;
};

inline size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

inline EpochLayout epoch_layout(int64_t n, int32_t L, const int32_t* dims, int order) {
    EpochLayout lay;
    size_t off = 0, smax = 0;
    auto take = [&](size_t elems) { size_t o = off; off += round256(elems * sizeof(float)); return o; };
    for (int l = 0; l < L; ++l) {
        const int32_t fi = dims[l], fo = dims[l + 1];
        const int ord = resolve_order(order, fi, fo);
        lay.order.push_back(ord);
        // Hidden layers keep only H = ReLU(Z): the ReLU is fused into the kernel that produces Z, and
        // sigma'(Z) = [Z > 0] = [H > 0], so backward never needs Z itself.  The last layer keeps Z.
        lay.Z.push_back(take((size_t)n * fo));
        lay.H.push_back(lay.Z.back());
        lay.T.push_back(take((size_t)n * (ord == GCN_ORDER_GEMM_FIRST ? fo : fi)));
        lay.G.push_back(take((size_t)n * fo));
        const size_t sneed = (size_t)n * (ord == GCN_ORDER_GEMM_FIRST ? fo : fi);
        if (sneed > smax) smax = sneed;
    }
    lay.S = take(smax);
    lay.XS = take(smax);
    // The partial sums of the reductions over n live in the caller's workspace too, so that an epoch never touches
    // library-owned scratch (which is per stream and would have to exist before a graph capture).  XS is idle outside
    // the sparse products: it holds the partial sums of the weight gradients and of the loss where it is large
    // enough, and a region of their own behind it holds what does not fit.
    size_t sc = loss_scratch_bytes(), tn = sc;
    for (int l = 0; l < L; ++l) {
        const size_t need = tn_shape(dims[l], dims[l + 1], n, false).scratch_bytes;
        if (need > tn) tn = need;
    }
    const size_t xs_bytes = smax * sizeof(float);
    if (tn > xs_bytes && tn > sc) sc = tn;
    // the fused last layer (SpMM-first order; a single layer can be put into that order by the pre-aggregated epoch)
    if ((lay.order[L - 1] == GCN_ORDER_SPMM_FIRST || L == 1) && fused_last_supported(dims[L - 1], dims[L])) {
        const size_t need = fused_last_scratch_bytes(n, dims[L]);
        if (need > sc) sc = need;
    }
    lay.scratch = take((sc + sizeof(float) - 1) / sizeof(float));
    lay.total = off;
    return lay;
}

// Where an epoch leaves the partial sums of all its reductions side by side, to be added up in one launch at its end (EpochEnd; the launches it
// saves are what a small epoch waits for: 4096 vertices, 64-16-8: 59 -> 50 us; 120 K vertices, 256-64-64-41: 1030 -> 1016).  In memory
// that is idle from the loss on, so that the workspace is not larger for it: the region of the scaled operand where the products need none, else the first
// layer's T, which forward has read by then or, with A^T H0 given, nobody does; and the scratch unless the fused last layer has it.
// The gradients over few rows, which have more partial results, lie in the T of their own layer where its forward product has read it and they fit: with more
// than 32 columns, a last share that is not whole may take up to 4 KB more than it.  What else fits nowhere: what those T leave, and, where the
// fused last layer does not store G, its T and G together.  All of them or none.
struct EpochRoom {
    static constexpr int MOST = 8;                // layers and one more
    static constexpr size_t NOWHERE = ~(size_t)0;
    size_t loss = NOWHERE;                        // offsets in the workspace
    size_t grad[MOST] = {NOWHERE, NOWHERE, NOWHERE, NOWHERE, NOWHERE, NOWHERE, NOWHERE, NOWHERE};
    bool few[MOST] = {};                          // the gradient's partial results are those of shares of 64 rows
    bool any = false;
};

// `value_free`: the products need the scaled operand; `p0`: A^T H0 is given; `fuse`: the last layer is fused, `keep`: its logits and gradient are stored.
inline EpochRoom epoch_room(const EpochLayout& lay, int64_t n, int32_t L, const int32_t* dims, bool value_free, bool p0, bool fuse, bool keep) {
    struct Piece { size_t at, left; };
    const int last = fuse ? L - 2 : L - 1;        // the last layer that has a gradient of its own launch
    auto gemm_first = [&](int l) { return lay.order[l] == GCN_ORDER_GEMM_FIRST && !(l == 0 && p0); };
    if (L >= EpochRoom::MOST) return EpochRoom();
    // Shares of 64 rows: of all gradients that can have them; of the GEMM-first layers', beside whose rows they may be made; of those that fit their own T; of
    // none, which finds room wherever the plain shares do in turn.
    for (int most = 3; most >= 0; --most) {
        EpochRoom room;
        Piece base[2], own[EpochRoom::MOST], behind = {0, 0};
        int pieces = 0;
        const bool first_t = value_free && (p0 || (gemm_first(0) && L >= 2));
        if (!value_free) base[pieces++] = {lay.XS, (fuse ? lay.scratch : lay.total) - lay.XS};
        if (first_t) base[pieces++] = {lay.T[0], lay.G[0] - lay.T[0]};
        if (value_free && !fuse) base[pieces++] = {lay.scratch, lay.total - lay.scratch};
        for (int l = 0; l < L; ++l) own[l] = {lay.T[l], gemm_first(l) || (l == 0 && p0) ? lay.G[l] - lay.T[l] : 0};
        if (first_t) own[0].left = 0;
        if (fuse && !keep) behind = {lay.T[L - 1], lay.S - lay.T[L - 1]};
        auto take = [](Piece& p, size_t bytes, size_t* at) {
            if (bytes > p.left) return false;
            *at = p.at;
            p.at += bytes;
            p.left -= bytes;
            return true;
        };
        bool placed[EpochRoom::MOST] = {}, all = true;
        auto bytes_of = [&](int l) { return round256(tn_shape(dims[l], dims[l + 1], n, room.few[l]).scratch_bytes); };
        for (int l = 0; l <= last; ++l) {
            room.few[l] = few_rows(dims[l], dims[l + 1], n) && (most == 3 || (most > 0 && gemm_first(l)));
            placed[l] = room.few[l] && gemm_first(l) && take(own[l], bytes_of(l), &room.grad[l]);
            if (most == 1) room.few[l] = placed[l];
        }
        auto first_fit = [&](size_t bytes, bool gradient, size_t* at) {
            for (int k = 0; k < pieces; ++k)
                if (take(base[k], bytes, at)) return true;
            if (!gradient || most == 0) return false;
            for (int l = 0; l < L; ++l)
                if (take(own[l], bytes, at)) return true;
            return take(behind, bytes, at);
        };
        if (!fuse) all = first_fit(round256(loss_part_bytes(n, dims[L])), false, &room.loss);
        for (int l = last; l >= 0 && all; --l)
            if (!placed[l]) all = first_fit(bytes_of(l), true, &room.grad[l]);
        room.any = all && (!fuse || pieces > 0);
        if (room.any) return room;
    }
    return EpochRoom();
}

}  // namespace gcn
