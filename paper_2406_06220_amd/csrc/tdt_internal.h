// Internal declarations shared by the translation units of libtdt_decode.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "split.h"
#include "tdt_decode.h"

// 1: profiling build.  Thread 0 of workgroup 0 records (event id, device wall clock) pairs of a
// few label-loop iterations into a device array that tdt_debug_trace() copies out -- a time line
// of one workgroup through the phases, their exchanges and the steps of a work item.
#ifndef TDT_TRACE
#define TDT_TRACE 0
#endif

namespace tdt {

constexpr int kThreads = 512;                 // threads per workgroup of the decode kernel
constexpr int kWaves = kThreads / 64;         // 64-wide wavefronts per workgroup
constexpr int kMaxRowsPerPass = 1024;         // (hypothesis, frame) rows of one joint pass
constexpr int kMaxColGroups = 64;             // output-column slices of one joint pass
constexpr int kPartialEntries = kMaxRowsPerPass * kMaxGrid;  // per partial buffer
constexpr int kBarrierStride = 32;            // uint32 slots between two workgroups' barrier flags
constexpr int kMaxRankedBatch = 1024;          // largest batch whose hypotheses are dealt to the clusters by length
constexpr int kMaxDuration = 1 << 20;          // largest frame increment of a duration class
constexpr size_t kLdsBytes = 160 * 1024;      // LDS of a compute unit
// label_loop.hip: hypotheses a group can hold (one lane each)
constexpr int kLabelThreads = 256;
constexpr int kLabelMaxHyps = 64;

// Softmax-denominator share of one slice of label columns for one joint row.
struct __align__(8) LsePartial {
    float max_lab;   // largest label logit in the slice
    float sumexp;    // sum of exp(logit - max_lab) over the slice (0 if it has no label column)
};
static_assert(sizeof(LsePartial) == 8, "LsePartial must be 8 bytes");

struct DecodeParams {
    // sizes
    int B, T, d_enc, H, V, D, O;   // D: outputs of the duration head (0 for a multi-blank model)
    int VL;                // last output of the label head: V, or V + number of big blanks
    int multi_blank;       // the outputs V+1 .. VL are big blanks with the increments in durations[]
    int pred_kind, pred_layers, h_pred, emb_dim;
    int max_symbols, u_cap;
    int window;            // 0 = automatic
    int joint_tiles;       // column tiles per joint work item the automatic window aims at (0 = automatic: 4 to 12)
    int kseg_max;          // longest K segment staged at once (set by launch_decode)
    int lds_bytes;         // dynamic LDS of the launch, a multiple of 16 (set by launch_decode)
    int wide_part;         // label_loop.hip, eight wavefronts: floats per wavefront and row of the partial sums
    int n_clusters, hyps_per_cluster;
    int frame_loop;        // non-zero: batched frame-looping (Algorithm 2) instead of label-looping
    int selftest_stall;    // non-zero: rank 0 of cluster 0 withholds its first barrier arrival
    int durations[TDT_MAX_DURATIONS];
    // weights
    const void *w_enc;       // [H][d_enc]   (read by the kernel only when it projects on the fly)
    const float *b_enc;
    const void *emb;
    const void *w_ih[TDT_MAX_LSTM_LAYERS], *w_hh[TDT_MAX_LSTM_LAYERS];
    const float *b_lstm[TDT_MAX_LSTM_LAYERS];
    const void *w_pred;
    const float *b_pred;
    const void *w_out;
    const float *b_out;
    // inputs
    const void *enc;         // [B][T][d_enc]   (read by the kernel only when it projects on the fly)
    float *enc_proj;         // [B][T][H]; on the fly: written row by row as joint passes need them
    const float *emb_gates;  // [V+1][h_pred][4 gates]: w_ih[0] * emb[label] + b_lstm[0] (LSTM only)
    const float *pred_tab;   // [ctx][V+1][H]: projected predictor output per label and context position
                             // (stateless predictor with precomputed projections only, else null)
    const int32_t *enc_len;  // [B]
    // outputs
    int32_t *out_labels, *out_frames, *out_len, *out_status;
    float *out_score;
    long long *out_stats;    // may be null
    // state carried between the chunks of longer utterances; all null for whole utterances
    int32_t *st_started, *st_time, *st_last, *st_last2;   // [B] each
    float *st_h, *st_c;      // [layers][B][h_pred] (LSTM only)
    // workspace
    float *hbuf;             // [2][layers][B][h_pred]  ping-pong hidden state
    float *cbuf;             // [layers][B][h_pred]
    float *rgate;            // [B][h_pred][4]: W_hh[0] . h of the first layer, for its next step
    float *pred_proj;        // [B][H]
    LsePartial *partials;    // [2][kPartialEntries]
    unsigned long long *row_lab;  // [n_clusters][kRowBufs][rows_per_cluster] packed (logit, ~label)
    unsigned long long *row_dur;  // same shape, packed (logit, ~duration class)
    int rows_per_cluster;
    // label_loop.hip: row_lab and row_lse are [n_clusters][kRowBufs][cells_per_cluster], row_dur is
    // [n_clusters][kRowBufs][2][rows_per_cluster], present [n_clusters][kRowBufs + 1][C] (workgroups
    // without a work item)
    unsigned long long *row_lse, *present;
    int cells_per_cluster;
    const void *packed;    // all fragment-major copies, and where each starts (bytes)
    size_t packed_bytes;
    int off_w_pred, off_w_out, off_w_ih[TDT_MAX_LSTM_LAYERS], off_w_hh[TDT_MAX_LSTM_LAYERS];
    unsigned *barrier;       // one flag word per workgroup, a cluster's flags side by side
    int *abort_flag;
    long long timeout_ticks; // bound on one wait, in wall-clock ticks
    int window_most;         // longest automatic window (decode.hip)
};

struct WorkspaceLayout {
    size_t packed;                 // bfloat16: the matrices the decode kernel streams, fragment by fragment
    size_t enc_proj, emb_gates, pred_tab, hbuf, cbuf, rgate, pred_proj, partials, row_lab, row_dur, barrier, abort_flag, total;
    size_t need_general;           // what a call of decode.hip's kernel needs (total: what a caller is asked for)
    size_t row_entries;            // uint64 entries in each of row_lab / row_dur
    size_t zero_begin, zero_end;   // byte range the init kernel clears
};

WorkspaceLayout workspace_layout(const tdt_weights_t *w, int B, int T);

// What label_loop.hip exchanges, laid over the part of the workspace the general kernel uses
// from `partials` on (byte offsets from there).  [ones_begin, ones_end) is filled with ones,
// [zero_begin, zero_end) with zeros before the kernel starts.
struct LabelLayout {
    size_t ones_begin, hx, px, ones_end, zero_begin, row_lab, row_lse, row_dur, present, abort_flag, zero_end;
    int rows_per_cluster, cells_per_cluster;
};
LabelLayout label_layout(const tdt_weights_t *w, bool wide, int n_clusters, int hyps_per_cluster, int C);
// whether that kernel can decode groups of this many hypotheses on C workgroups each
bool label_kernel_takes(const tdt_weights_t *w, bool chunked, bool wide, int hyps_per_cluster, int C);

// the caller-held state of tdt_greedy_decode_chunk: byte offsets of its arrays
struct StateLayout {
    size_t started, time, last, last2, h, c, total;
};
StateLayout state_layout(const tdt_weights_t *w, int B);

// launches (each returns a hipError_t)
hipError_t launch_encoder_projection(const void *enc, int64_t rows, const tdt_weights_t *w,
                                     float *out, hipStream_t stream);
// the encoder projection of the valid frames of B utterances (any dtype)
hipError_t launch_encoder_projection_valid(const void *enc, const int32_t *enc_len, int B, int T,
                                           const tdt_weights_t *w, float *out, hipStream_t stream);
// Fragment-major copies of the weight matrices the decode kernels multiply by (float32 models:
// label_loop.hip only).  A matrix [N][K] (row-major) is cut into column tiles of 16 rows of it and
// steps of 32 inputs (float32: 16); fragment (tile, step) is 1 KiB, lane l's 16 bytes at l * 16: inputs
// step * 32 + (l / 16) * 8 .. + 7 (float32: step * 16 + (l / 16) * 4 .. + 3) of the tile's row l % 16 --
// what lane l feeds the matrix core -- zeros where the matrix ends.
// Fragments of a tile follow each other by step.  A wavefront's fragment load is then one
// contiguous KiB; from the row-major matrix it is 16 pieces of 64 bytes from 16 rows, which
// the texture addresser takes four times as long over.
// Row of a tile: plain tile*16 + j; for LSTM gate matrices (gate-major [4][h][K]) a tile is
// 4 hidden units x 4 gates: row (j % 4) * h + tile * 4 + j / 4.
struct PackedMatrix {
    size_t offset;   // bytes from the start of the packed region
    int tiles, steps;
};
struct PackedLayout {
    PackedMatrix w_enc, w_pred, w_out, w_ih[TDT_MAX_LSTM_LAYERS], w_hh[TDT_MAX_LSTM_LAYERS];
    size_t total;
};
PackedLayout packed_layout(const tdt_weights_t *w);
hipError_t launch_pack_weights(const tdt_weights_t *w, const PackedLayout &pl, bool on_the_fly, void *packed,
                               hipStream_t stream);
// what a call clears before its decode kernel: one range to zeros, one to ones (multiples of 16 bytes)
struct ClearRanges {
    void *zero, *ones;
    size_t zero_bytes, ones_bytes;
};
// Everything before the decode kernel in one launch (two where the encoder projection takes the
// 256 x 256 kernel): the encoder projection of frames t < enc_len[b] (B == 0: none), the predictor side's
// per-label tables (first LSTM layer's input product into emb_gates; a stateless predictor's projected
// output into pred_tab, which may be null: then none), the copies (pl.total == 0: none), the clearing
hipError_t launch_prepare(const void *enc, const int32_t *enc_len, int B, int T, const tdt_weights_t *w,
                          float *enc_proj, float *emb_gates, float *pred_tab, const PackedLayout &pl,
                          bool on_the_fly, void *packed, const ClearRanges &clear, long long *out_stats,
                          hipStream_t stream);
hipError_t launch_init(const ClearRanges &clear, long long *out_stats, hipStream_t stream);
// which compiled form of the decode kernel a call runs
struct DecodeVariant {
    bool chunked;      // tdt_greedy_decode_chunk
    bool frame_loop;   // TDT_ALG_FRAME_LOOPING
    bool on_the_fly;   // TDT_PROJ_ON_THE_FLY
    bool wide_joint;   // the joint pass streams the output matrix (TDT_JOINT_STREAMING)
};
hipError_t launch_decode(const DecodeParams &p, const tdt_weights_t *w, DecodeVariant v, int grid,
                         hipStream_t stream);
// the same for label_loop.hip's kernel (label_kernel_takes)
hipError_t launch_label(const DecodeParams &p, const tdt_weights_t *w, bool chunked, bool wide, int grid, hipStream_t stream);
// largest grid the decode kernel can run with all workgroups resident, 0 on error
int decode_max_grid(const tdt_weights_t *w, DecodeVariant v);
#if TDT_TRACE
hipError_t copy_trace_general(long long *out, int n);
hipError_t copy_trace_label(long long *out, int n);
#endif
// ticks per millisecond of the device wall clock the kernels read (100000 if the query fails)
int wall_clock_khz();

}  // namespace tdt
