// How work is divided between workgroups, in whole numbers only: used on the host and in kernels, and
// compiled without HIP by the tests.
#ifndef TDT_SPLIT_H
#define TDT_SPLIT_H

#ifdef __HIPCC__
#define TDT_HD __host__ __device__
#else
#define TDT_HD
#endif

namespace tdt {

constexpr int kXcds = 8;             // accelerator dies of an MI355X; workgroups are dealt to them in turn
constexpr int kMaxWindow = 64;       // frames of one hypothesis per joint pass
constexpr int kMaxHypsPerCluster = 256;   // hypotheses one group of workgroups decodes
constexpr int kRowTile = 16;         // activation rows per tile

// ---- automatic number of hypothesis groups
// What the rules look at: column tiles of W_pred, of W_hh (4 units x 4 gates a tile) and of W_out.
struct SplitModel {
    bool lstm;
    int nt_a, nt_b, nt_out;
};
struct GroupSplit {
    int n_clusters;
    bool one_workgroup;   // a group each, and no more workgroups than groups
    int window_most;      // longest automatic window of a hypothesis
};
// An LSTM predictor.  A group runs as long as its longest hypothesis and the fewer hypotheses it
// holds the shorter its joint passes, so more groups pay -- until a group has too few workgroups
// to give each at most four column tiles of the predictor-side products (two weight batches per
// wavefront); that many groups are the rule from 16 hypotheses on.  Small batches: two groups
// also for a single hypothesis (half the workgroups synchronise faster), four from four hypotheses on
// (3 to 8 % faster than two at B = 4 ... 12; measured on the general kernel).
// Returned beside it: whether a larger batch takes yet more groups.
inline int lstm_groups(const SplitModel &m, int B, int max_grid, bool *may_grow)
{
    const int q4 = (m.nt_a + 3) / 4 + (m.nt_b + 3) / 4;
    int fit = (2 * max_grid + q4) / (2 * q4);   // max_grid / q4, rounded
    if (fit < 1) fit = 1;
    *may_grow = B >= 16 && fit < 8;
    if (B >= 16) return fit;
    const int n = B < 4 ? 2 : (fit < 4 ? fit : 4);
    return n < 2 ? 2 : n;
}
// A stateless predictor: no predictor-side phase, no matrix but the output layer's.  Groups of as many
// workgroups as its column tiles make items of k of them, k the smallest with about three hypotheses a
// group (items of eight tiles: five).  Measured with label_loop.hip on the stateless benchmark model
// (65 tiles), best of all group counts in brackets: B = 9, 7 groups, 1.31 ms (1.31); B = 32, 11 groups,
// 1.58 (1.58; 16 groups 1.71); B = 64, 23 groups, 1.85 (1.85; 32 groups 1.94); B = 128, 28 groups, 2.47
// (2.47); B = 256, 42 groups, 3.40 (3.40; 32 groups 3.57)
inline int stateless_groups(const SplitModel &m, int B, int max_grid)
{
    const int per_item[6] = {2, 3, 4, 6, 8, 12};
    int n = 2;
    for (const int k : per_item) {
        n = max_grid / ((m.nt_out + k - 1) / k);
        if (5 * B <= (k < 8 ? 16 : 25) * n) break;
    }
    return n > 64 ? 64 : n < 2 ? 2 : n;
}
// A streamed output layer (`least`: the fewest groups that form takes): every group streams the whole
// output matrix in every pass, and a pass lasts as long as its workgroups need for that, so groups are few
// while the batch is small (8198 outputs, T = 300: B = 4, four groups 1.47 ms, eight 1.71; B = 32, eight
// 2.69, four 2.93, sixteen 2.99; B = 130, sixteen 5.24, eight 5.67; B = 256, sixteen 7.8, eight 9.1, thirty-two 8.8)
inline int streaming_groups(int B, int least) { return least * (B < 12 ? 1 : B <= 96 ? 2 : 4); }   // (some may stay empty)

// ... but no group holds more than it can
inline int enough_groups(int n, int B)
{
    const int least = (B + kMaxHypsPerCluster - 1) / kMaxHypsPerCluster;
    return n < least ? least : n;
}
// Groups of a call of label_loop.hip's kernel.  Large LSTM batches, from about 14 hypotheses per group of
// eight on: groups of one full row tile (B = 160, ten groups: 3.04 ms, eight: 3.81 ms) while a group keeps
// about 20 workgroups, then 16 groups (B = 256: 4.59 ms, eight: 4.91 ms).  A stateless predictor with an
// output layer of up to four tiles, one round of the kernel: a workgroup for every hypothesis, which then
// needs no other (the smallest benchmark model, B = 4, T = 200: 454 us against 489 us in groups of 64
// workgroups; B = 60: 560 us and less against 675 us).
// (streaming_least: 0, or see streaming_groups)
inline GroupSplit label_split(const SplitModel &m, int B, int max_grid, int streaming_least)
{
    GroupSplit s{1, false, kMaxWindow};
    if (streaming_least > 0) {
        s.n_clusters = enough_groups(streaming_groups(B, streaming_least), B);
        return s;
    }
    s.one_workgroup = !m.lstm && m.nt_out <= 4;
    bool may_grow = false;
    int n = s.one_workgroup ? max_grid : m.lstm ? lstm_groups(m, B, max_grid, &may_grow) : stateless_groups(m, B, max_grid);
    if (may_grow && B >= 14 * 8) {
        const int full = (B + 15) / 16;
        n = full <= 8 ? 8 : full <= 13 ? full : 16;
    }
    if (n > B && (B > 1 || s.one_workgroup)) n = B;
    s.n_clusters = enough_groups(n, B);
    return s;
}
// Groups of a call of the general kernel (decode.hip), which never does without its group: one workgroup a
// hypothesis took 12.3 ms against 3.6 ms in groups of 64 (projections on the fly, 51 outputs, joint width
// 640, B = 4), 0.44 ms against 0.37 ms (the smallest benchmark model, the same) and 22.9 ms against
// 19.4 ms (float32, joint width 1024, 51 outputs, B = 32).
// Projections on the fly, an output layer of up to four tiles, a hypothesis or a few a group: of a pass's
// rows every one is projected, so a hypothesis gets at most one row tile of frames -- as many as it
// has with projections ahead of the loops, where its group is one workgroup (one hypothesis a group:
// B = 60, 1.26 ms against 1.58 ms with 64 frames; 51 outputs, joint width 640, B = 32, 5.3 ms against 9.4 ms).
inline GroupSplit general_split(const SplitModel &m, int B, int max_grid, int streaming_least, bool on_the_fly)
{
    GroupSplit s = label_split(m, B, max_grid, streaming_least);
    if (s.one_workgroup) {
        s.one_workgroup = false;
        s.n_clusters = stateless_groups(m, B, max_grid);
        if (s.n_clusters > B && B > 1) s.n_clusters = B;
        s.n_clusters = enough_groups(s.n_clusters, B);
        if (on_the_fly) s.window_most = kRowTile;
    }
    return s;
}

// What a workgroup of label_loop.hip owns of the predictor side: `na` column tiles of W_pred from `qt0` on,
// `nr` of W_hh from `r0` on, and with those the hidden units u0 .. u0 + U - 1 (of every layer).
struct PredShare {
    int qt0, na, r0, nr, u0, U;
};
// nt_a, nt_b: column tiles of W_pred and W_hh (none: no LSTM); C workgroups.  One round of one layer
// (deep false): a stretch of the [W_pred | W_hh] tiles, `per` a workgroup.  Else its share of each: a
// W_hh tile stands for three products of a deeper LSTM (its input, its recurrent product in every
// layer), a W_pred tile for one.  u0 is a unit of the model in every workgroup, also in one that is left
// without any (beyond the last tile): all of them request a row of the per-label table from there.
TDT_HD inline PredShare pred_share(bool deep, int nt_a, int nt_b, int h_pred, int C, int rank)
{
    PredShare s{0, 0, 0, 0, 0, 0};
    if (nt_b == 0) return s;
    if (deep) {
        s.qt0 = rank * nt_a / C;
        s.na = (rank + 1) * nt_a / C - s.qt0;
        s.r0 = rank * nt_b / C;
        s.nr = (rank + 1) * nt_b / C - s.r0;
    } else {
        const int per = (nt_a + nt_b + C - 1) / C, all = nt_a + nt_b - rank * per;   // tiles from its first one on
        s.qt0 = rank * per;
        s.na = nt_a - s.qt0 < 0 ? 0 : nt_a - s.qt0 < per ? nt_a - s.qt0 : per;
        s.r0 = s.qt0 < nt_a ? 0 : s.qt0 - nt_a;
        s.nr = (all < 0 ? 0 : all < per ? all : per) - s.na;
    }
    if (s.nr > 0) {
        s.u0 = s.r0 * 4;
        s.U = s.nr * 4 < h_pred - s.u0 ? s.nr * 4 : h_pred - s.u0;
    }
    return s;
}

}  // namespace tdt

#endif
