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
