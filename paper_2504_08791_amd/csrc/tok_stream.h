// Launchers of the projections of a window of several tokens (tok_stream.hip).
#pragma once
#include "common.h"

namespace prima {

// where a matrix's sums lie: share p of token t, row r of the matrix at part[(p * T + t) * rows + row0 + r]
struct TokPart {
    const float *part;
    int n_parts;
    int64_t rows, row0;
};
struct TokNorm {
    const float *ss; // sums of squares [nb][token slots] that tok_prepare_kernel left (null: none)
    int nb;
    float eps;
};
struct TokMat {
    const uint8_t *W;
    int64_t n_rows; // a multiple of 16
};

enum { TOK_PLAIN = 0, TOK_RESIDUAL = 1, TOK_SWIGLU = 2, TOK_ATTENTION = 3 };
struct TokPrepare {
    int mode, T, nb;  // v: [T][256 nb]
    const float *x;   // TOK_PLAIN: v; TOK_RESIDUAL: added to the shares of p[0]
    TokPart p[2];     // TOK_SWIGLU: silu(gate / rms) * up / rms of p[0] (gate), p[1] (up)
    TokNorm norm;     // TOK_SWIGLU
    AttnRecords att;  // TOK_ATTENTION: v from the key ranges' records of heads of D columns
    int D;
    float *out;       // v stored (null: not); may be x
    const float *gain; // null: none; else ss gets the sums of squares of v, and v * gain is laid out
    float *ss;
    uint8_t *rec[2]; // activations laid out for Q4_K and for the other formats (null: not)
};
struct TokSum {
    int n, T, nt; // nt: token slots of norm.ss
    TokPart p[3];
    int64_t rows[3]; // multiples of 16
    float *y[3];     // [T][rows]
    TokNorm norm;
    const float *resid; // [T][rows[0]], with n == 1 (null: none)
};

int tok_max_parts(int nb, int nt, int64_t n_rows); // shares of K of a launch of n_rows rows in all, at most (fewer rows: not fewer)
int tok_slots(int T);
size_t tok_rec_bytes(int64_t n_cols, int T);
size_t tok_part_floats(int64_t n_rows, int64_t n_cols, int T); // for one matrix; matrices launched together take no more than the sum of theirs
size_t tok_ss_bytes(int64_t n_cols, int T);
// sums of up to three matrices of one format (all but FP32) and equal columns with the activations rec; out[i]: where they lie
prima_status launch_tok_stream(int fmt, const TokMat *mats, int n_mats, int64_t n_cols, const uint8_t *rec, int T, float *part, size_t part_floats,
                               TokPart *out, hipStream_t st);
// host only: whether matrices of n_rows rows in all find a plan whose shares fit
prima_status tok_stream_plan_status(int fmt, int64_t n_rows, int64_t n_cols, int T, size_t part_floats);
// init: a window's first launch does what a step needs in front of it too (tab null: not)
prima_status launch_tok_prepare(const TokPrepare &a, const StepInit &init, hipStream_t st);
prima_status launch_tok_sum(const TokSum &a, hipStream_t st);

} // namespace prima
