// Host interface of the matrix-core kernel for CSR filters (matrix.hip);
// internal header.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstddef>
#include <cstdint>

#include "spconv.h"

// Tiling of one launch (see MatArgs).
struct MatrixPlan {
    int RB = 0, NBX = 0, wm = 0, wp = 0, ksr = 0, M = 0, O = 0, nchunks = 0, nunits = 0, TH = 0, TW = 0, nty = 0,
        ntx = 0, rows = 0, vp = 0, PX = 0, stepy = 0, stepx = 0, lsy = 0, lsx = 0, hw = 0, pitch = 0, bufs = 0, a_bytes = 0,
        b_bytes = 0, nkt = 0, total_wgs = 0;
    size_t lds_bytes = 0;
    double time = 0.0;  // modelled cycles
};

// The call a plan is launched for: shapes, epilogue and input layout.
struct MatrixCall {
    int N, C, H, W, K, R, S, stride, pad, Ho, Wo;
    bool pool, unpadded;
    int relu;
    int out_pad, opitch, res_pad, rpitch;
    size_t oplane, rplane;
};

// Least modelled time over the tilings; false when none fits.
bool matrix_plan(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, bool pool, long long nnz,
                 MatrixPlan *out);

// What was decided for recent calls of these shapes (thread safe, bounded):
// recall fills *plan and *use (whether they run on this kernel) and returns true
// when it remembers one.
bool matrix_recall(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, bool pool, long long nnz,
                   MatrixPlan *plan, bool *use);
void matrix_remember(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, bool pool, long long nnz,
                     const MatrixPlan &plan, bool use);

// (16-pixel blocks per wave, 0, channels per wave, pool) of the compiled instances.
void matrix_variants(int32_t *variants, int32_t capacity, int32_t *count);

int matrix_launch(const MatrixPlan &pl, const MatrixCall &c, const float *in, const int32_t *rowptr,
                  const int32_t *offset, const float *vals, const float *bias, const float *res, float *out,
                  hipStream_t stream);
