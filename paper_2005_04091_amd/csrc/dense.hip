// Dense path of the fused convolution on the matrix cores (gfx950 MFMA), for
// filters dense enough that skipping zeros no longer pays, and the host model
// that chooses between it and the sparse path (spconv_select_path).
//
// The convolution is the implicit GEMM  out[k, p] = sum over (c, r, s) of
// W[k, c, r, s] * Xp[c, p + r*Wp + s]  (stride 1, p = y*Wp + x, the paper's
// offset trick with the padded row pitch as pixel pitch; columns x >= Wo are
// computed and dropped). Products are formed exactly enough for fp32: every
// value is the sum of three bf16 parts, x = h + m + l (each the bf16 rounding
// of what the parts before it leave, so the sum is exact), and a product takes
// the six part products of weight 2^-16 or more, hh + hm + mh + mm + hl + lh,
// on v_mfma_f32_32x32x16_bf16 with fp32 sums (what is dropped is at most
// 2^-23 of the product and 2^-26 on average). Six of them take 192 cycles for 16 channels, where the fp32
// MFMA (32x32x2) takes 512.
//  * a workgroup owns (image, tile of TH output rows, 32*nw output channels);
//    the tile's NB blocks of 32 consecutive virtual pixels are dealt to ksp
//    waves per channel tile (NBW blocks each, one 32x32 accumulator tile per
//    block) and the reduction's groups of 16 channels to ksr waves; the ksr
//    partial sums of a tile are added through LDS in a fixed order at the end;
//  * the tile's input rows are loaded one chunk of channel groups ahead into
//    registers, split there and stored to LDS as [part][8-channel half][pixel]
//    [8 bf16], so a B fragment (8 channels of a pixel shifted by the tap) is
//    one 16-byte LDS read per part, consecutive over the lanes;
//  * the A fragment of (group, tap) is four 8-byte loads from the filter
//    packed by spconv_pack_dense, three steps ahead, split in registers;
//  * the epilogue adds bias (and a residual), applies ReLU, pools 2x2 windows
//    through LDS when asked, and stores once. Sums that are not finite are taken
//    again on the fp32 MFMA: infinities (and values that round to one in bf16)
//    have no finite parts, and near the top of the range h rounds up past the
//    value, so that hh can overflow where the product does not.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "common.h"
#include "dense_layout.h"
#include "split.h"
#include "spconv.h"

__attribute__((visibility("hidden"))) int dense_kernel_variants(int32_t *variants, int32_t capacity, int32_t *count);
// Modelled time of the sparse path (spconv.hip).
__attribute__((visibility("hidden"))) bool sparse_layer_us(int N, int C, int H, int W, int K, int R, int S, int pad,
                                                           int Ho, int Wo, bool pool, bool unpadded, long long nnz,
                                                           double *us, bool *walk);

namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kDnsTile = dense_layout::kTile;  // MFMA tile: 32 channels x 32 pixels
constexpr int kDnsMaxThreads = 512;       // nw * ksr * ksp waves per workgroup, at most 8
constexpr int kDnsMaxBlocks = 8;          // pixel blocks per tile
constexpr int kDnsWaveBlocks = 4;         // pixel blocks per wave (16 accumulator VGPRs each)
constexpr int kDnsGroup = 16;             // channels per MFMA (one reduction group)
constexpr int kDnsPxBytes = 6 * kDnsGroup;  // LDS bytes of a group's pixel: three bf16 parts of 16 channels
constexpr int kDnsLdsBytes = 64 * 1024;   // per workgroup: two fit a CU, where their registers do (at most four waves each)
constexpr int kDnsCuLds = 160 * 1024;     // LDS of a CU
constexpr int kDnsLdsMax = 80 * 1024;     // one group of the widest rows (256 padded columns, 3 rows)
constexpr int kDnsPoolCh = 8;             // channels of one pooled staging round (4 accumulator rows x 2 halves)
constexpr int kDnsRounds = 3;             // staging tasks per thread whose loads run a chunk ahead

struct DenseArgs {
    int N, C, K, Kp, Hp, Wp, Ho, Wo, Hq, Wq;
    int relu;
    int TH;          // output rows per tile
    int ntiles_y;    // tiles per image
    int nw;          // channel tiles of 32 per workgroup
    int ksr;         // waves splitting the reduction over channel groups
    int ksp;         // waves splitting the tile's pixel blocks
    int nkt;         // channel tiles of 32*nw
    int Cg;          // channel groups per LDS chunk (a multiple of ksr)
    int nchunks;
    int nbuf;        // LDS chunk buffers, 1 or 2
    int PX;          // staged pixels per channel
    int tasks;       // staging tasks of a chunk: (octet of channels, pixel), 2*Cg*PX
    int buf_bytes;   // Cg * PX * kDnsPxBytes
    int total_wgs;
    int out_pad, opitch;
    size_t oplane;
    int res_pad, rpitch;
    size_t rplane;
    int wpk_bytes;   // bytes of the packed filter (below 2^31)
    // x / PX (staging), x / Wp, and the pooled epilogue's x / ((TH/2) * Wq)
    // and x / Wq as multiply-shift
    uint32_t px_magic, wp_magic, pch_magic, wq_magic;
    int px_shift, wp_shift, pch_shift, wq_shift;
    // input planes: IH x IW with the tile's padded row i, column x at plane
    // row i - ipad, column x - ipad (the padded tensor itself: ipad = 0)
    int IH, IW, ipad;
};

// One staging task: eight channels of one staged pixel of a chunk.
struct StageTask {
    uint32_t voff;  // byte offset of the first channel's pixel from the chunk's first channel, or past its end
    int lds;        // byte offset of the h part in the chunk buffer, or -1 (no task)
};

__device__ __forceinline__ StageTask dense_task(const DenseArgs &a, int id, int y0) {
    StageTask t;
    t.lds = -1;
    t.voff = 0xfffffff0u;
    if (id < a.tasks) {
        const int oct = (int)fast_div((uint32_t)id, a.px_magic, a.px_shift);
        const int px = id - oct * a.PX;
        const int i = (int)fast_div((uint32_t)px, a.wp_magic, a.wp_shift);
        const int y = y0 + i - a.ipad, x = px - i * a.Wp - a.ipad;
        t.lds = (oct >> 1) * a.PX * kDnsPxBytes + ((oct & 1) * a.PX + px) * 16;
        if (oct * 8 < a.C && y >= 0 && y < a.IH && x >= 0 && x < a.IW)
            t.voff = (uint32_t)((oct * 8 * a.IH + y) * a.IW + x) * (uint32_t)sizeof(float);
    }
    return t;
}

// The chunk's input through a descriptor over its channels of image n: border
// pixels and channels past C read as zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dense_chunk_rsrc(const DenseArgs &a, const float *__restrict__ xp,
                                                                   int ch, int n) {
    const int c0 = ch * a.Cg * kDnsGroup;
    const int cn = min(a.Cg * kDnsGroup, a.C - c0);
    const size_t plane = (size_t)a.IH * a.IW;
    return uniform_rsrc(xp + ((size_t)n * a.C + c0) * plane, (uint32_t)(cn * plane * sizeof(float)));
}

__device__ __forceinline__ void dense_load(const DenseArgs &a, const __amdgpu_buffer_rsrc_t &rsrc, const StageTask &t,
                                           float (&v)[8]) {
    const uint32_t pb = (uint32_t)(a.IH * a.IW) * (uint32_t)sizeof(float);
    // Saturating steps: offsets past the range (border pixels, channels past C)
    // stay there and do not wrap.
    uint32_t off = t.voff;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0));
        off = __builtin_elementwise_add_sat(off, pb);
    }
}

__device__ __forceinline__ void dense_put(const DenseArgs &a, char *buf, const StageTask &t, const float (&v)[8]) {
    if (t.lds < 0) return;
    Parts p;
#pragma unroll
    for (int i = 0; i < 4; ++i) split2(p, i, v[2 * i], v[2 * i + 1]);
    char *d = buf + t.lds;
    *reinterpret_cast<u32x4_t *>(d) = p.h;
    *reinterpret_cast<u32x4_t *>(d + a.PX * 32) = p.m;
    *reinterpret_cast<u32x4_t *>(d + a.PX * 64) = p.l;
}

// What bounds it: at 14x14 (256 channels, batch 32, one workgroup per CU) the
// MFMAs alone take about 33 us (the chip holds 1.65 PFLOP/s on this MFMA form)
// and everything else (the A loads and their split, LDS reads, staging) about
// 35 us without them; together 56 us, where the fp32 MFMA kernel before it
// took 88 us. Other layers, batch 32, fp32 MFMA kernel and this one: 56x56, 64
// channels 98 and 63 us; 28x28, 128 channels, pooled 82 and 52 us; 7x7, 512
// channels 171 and 112 us; 112x112, 64 channels (batch 8) 97 and 76 us. Against
// float64 the sums are two to three times closer than that kernel's (14x14: 1.5e-7
// against 4.1e-7 relative), because the hh products round into the main sum once
// per 16 channels and tap. Chunks of 32 to 96 channels take the same time.
//
// Registers: 191 to 256 (tap pairs 138 to 256), so two waves a SIMD. With four
// blocks a wave they do not suffice: 42 to 52 are spilled (3x3; 19 with three
// blocks, 8 for 1x1, 13 for tap pairs), mostly the next chunk's loads: some 30
// scratch stores before a chunk's MFMAs and as many loads after them, 6 loads to a
// group's 216 MFMAs, none between these. Tiles of at most three blocks a wave took
// 68 us for the 56x56 layer's 63, and 65 for the 112x112 one's 76; the planner does
// not tell them apart yet.
//
// PAIR (filters of several taps, at most 8 channels): the second half of an
// MFMA's 16 channels would be padding, so it takes the next tap instead, 5 MFMA
// steps for 3x3 where there were 9, and only one octet is staged.
// 3x3 on 3 channels, 64 outputs, 224x224 batch 32: 297 us (396 without pairs, fp32
// MFMA kernel 374); 56x56 batch 8 10.3 us (14.4); 8 channels at 112x112, batch 4,
// 15.1 us (32.8). The output's stores are most of what is left.
template <int R, int S, int NBW, bool POOL, bool PAIR>
__global__ __launch_bounds__(kDnsMaxThreads) void spconv_dense_kernel(DenseArgs a, const float *__restrict__ xp,
                                                                            const float *__restrict__ wpk,
                                                                            const float *__restrict__ bias,
                                                                            const float *__restrict__ res,
                                                                            float *__restrict__ out) {
    extern __shared__ float lds[];
    constexpr int RS = R * S;
    constexpr int T = PAIR ? (RS + 1) / 2 : RS;  // MFMA steps of a channel group
    char *ldsb = reinterpret_cast<char *>(lds);
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int work = xcd_linear_id((int)blockIdx.x, a.total_wgs);
    const int kt = __builtin_amdgcn_readfirstlane(work % a.nkt);
    const int rest = work / a.nkt;
    const int ty = __builtin_amdgcn_readfirstlane(rest % a.ntiles_y);
    const int n = __builtin_amdgcn_readfirstlane(rest / a.ntiles_y);
    const int y0 = ty * a.TH;
    // channel tile, reduction share, pixel share
    const int wn = __builtin_amdgcn_readfirstlane(wave % a.nw);
    const int wr = __builtin_amdgcn_readfirstlane((wave / a.nw) % a.ksr);
    const int wp = __builtin_amdgcn_readfirstlane(wave / (a.nw * a.ksr));
    const int k0 = (kt * a.nw + wn) * kDnsTile;
    const int q0 = wp * NBW * kDnsTile;  // first virtual pixel of the wave
    const int half = lane >> 5, col = lane & 31;
    const int nthreads = (int)blockDim.x;
    // A wave whose blocks hold no stored pixel computes nothing.
    const bool active = q0 < (min(a.TH, a.Ho - y0) - 1) * a.Wp + a.Wo;

    // Sums of the hh products, and of the five smaller ones: added once at the
    // end, so that the main sum rounds once per 16 channels and tap.
    f32x16_t acc[NBW], low[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = low[b][r] = 0.0f;

    // A fragment of (group g, tap t), channel pair j of the lane's half:
    // wpk[(((8g + 4*half + j)*RS + t)*Kp + k0 + col)*2 ..]. The descriptor
    // starts at the group and the lane's offset counts its pair, so pairs past
    // the filter (C not a multiple of 16, or a group past the last) read zeros
    // whatever the scalar tap offset.
    const int npairs = (a.C + 1) / 2;
    const uint32_t wtap = (uint32_t)a.Kp * 8u, wpair = wtap * RS;
    uint32_t wlane[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        wlane[j] = (uint32_t)(k0 + col) * 8u + (uint32_t)(PAIR ? j : 4 * half + j) * wpair + (PAIR ? half * wtap : 0u);
    // (a group past the last, whose values are not used, reads the first)
    auto a_rsrc = [&](int g) {
        const int g0 = 8 * g < npairs ? 8 * g : 0;
        return uniform_rsrc(wpk + (size_t)g0 * (wpair / 4), (uint32_t)min(npairs - g0, 8) * wpair);
    };
    // A fragment of step t; with PAIR taps 2t and 2t + 1, zeros past the last
    // tap (an offset past any range: the packed filter is below 2^31 bytes).
    auto load_a = [&](f32x2_t(&av)[4], const __amdgpu_buffer_rsrc_t &rs, int t) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = PAIR && 2 * t + 1 >= RS && half ? 0x7ffffff0u : wlane[j];
            av[j] = __builtin_bit_cast(f32x2_t,
                                       __builtin_amdgcn_raw_buffer_load_b64(rs, v, (PAIR ? 2 * t : t) * wtap, 0));
        }
    };

    StageTask task[kDnsRounds];
    float xin[kDnsRounds][8];
#pragma unroll
    for (int i = 0; i < kDnsRounds; ++i) task[i] = dense_task(a, (int)threadIdx.x + i * nthreads, y0);
    auto stage_load = [&](int ch) {
        const __amdgpu_buffer_rsrc_t rsrc = dense_chunk_rsrc(a, xp, ch, n);
#pragma unroll
        for (int i = 0; i < kDnsRounds; ++i)
            if (i * nthreads < a.tasks) dense_load(a, rsrc, task[i], xin[i]);
    };
    // Split and store the loaded chunk, and the tasks past the rounds kept in registers.
    auto stage_put = [&](int ch, char *buf) {
#pragma unroll
        for (int i = 0; i < kDnsRounds; ++i)
            if (i * nthreads < a.tasks) dense_put(a, buf, task[i], xin[i]);
        if (kDnsRounds * nthreads < a.tasks) {
            const __amdgpu_buffer_rsrc_t rsrc = dense_chunk_rsrc(a, xp, ch, n);
            for (int id = (int)threadIdx.x + kDnsRounds * nthreads; id < a.tasks; id += kDnsRounds * nthreads) {
                StageTask t[kDnsRounds];
                float v[kDnsRounds][8];
#pragma unroll
                for (int i = 0; i < kDnsRounds; ++i) {
                    t[i] = dense_task(a, id + i * nthreads, y0);
                    dense_load(a, rsrc, t[i], v[i]);
                }
#pragma unroll
                for (int i = 0; i < kDnsRounds; ++i) dense_put(a, buf, t[i], v[i]);
            }
        }
    };

    stage_load(0);
    const int ngroups = (a.C + kDnsGroup - 1) / kDnsGroup;
    const int lane_b = ((PAIR ? 0 : half * a.PX) + q0 + col) * 16;
    // Steps of this wave: (group, tap), groups wr, wr + ksr, ... over all
    // chunks. A wave runs them as one pipeline: the A loads three steps ahead,
    // the split of the next step's A and the B reads of the next unit (one
    // block of a step) between the six MFMAs of the current unit.
    f32x2_t araw[3][4];
    Parts A;
    if (active) {
        load_a(araw[0], a_rsrc(wr), 0);
        load_a(araw[1], a_rsrc(wr + 1 / T * a.ksr), 1 % T);
        load_a(araw[2], a_rsrc(wr + 2 / T * a.ksr), 2 % T);
    }
    stage_put(0, ldsb);
    if (active)
#pragma unroll
        for (int j = 0; j < 4; ++j) split2(A, j, araw[0][j].x, araw[0][j].y);
    __syncthreads();

    // The wave's last block may lie past the stored pixels: it then reads the
    // first block's pixels again (its sums are dropped).
    const int valid_px = (a.TH - 1) * a.Wp + a.Wo;
    const int last_off = q0 + (NBW - 1) * kDnsTile < valid_px ? (NBW - 1) * kDnsTile * 16 : 0;
    auto read_b = [&](Parts &u, const char *bp, int b) {
        const char *bb = bp + (NBW > 1 && b == NBW - 1 ? last_off : b * kDnsTile * 16);
        u.h = *reinterpret_cast<const u32x4_t *>(bb);
        u.m = *reinterpret_cast<const u32x4_t *>(bb + a.PX * 32);
        u.l = *reinterpret_cast<const u32x4_t *>(bb + a.PX * 64);
    };
    auto mma = [&](f32x16_t &c, const u32x4_t &x, const u32x4_t &y) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, y), c,
                                                    0, 0, 0);
    };

    // B bytes from the lane's pixel to the pixel under step t's tap.
    auto tap_at = [&](int t) {
        if constexpr (!PAIR) return ((t / S) * a.Wp + t % S) * 16;
        const int t0 = 2 * t, t1 = min(2 * t + 1, RS - 1);  // (past the last tap: the last, times zeros)
        return (half ? (t1 / S) * a.Wp + t1 % S : (t0 / S) * a.Wp + t0 % S) * 16;
    };
    for (int ch = 0; ch < a.nchunks; ++ch) {
        const bool more = !PAIR && ch + 1 < a.nchunks;  // (one group is one chunk)
        if (more) stage_load(ch + 1);
        const char *buf = ldsb + (a.nbuf == 2 ? (ch & 1) * a.buf_bytes : 0) + lane_b;
        const int gn = min(a.Cg, ngroups - ch * a.Cg);
        const int gstride = a.PX * kDnsPxBytes;
        if (active && wr < gn) {
            Parts B[2];
            read_b(B[0], buf + wr * gstride + tap_at(0), 0);
            for (int g = wr; g < gn; g += a.ksr) {
                const char *gb = buf + g * gstride;
                const char *gnext = g + a.ksr < gn ? gb + a.ksr * gstride : gb;  // (the last group's reads repeat)
                const int gg = ch * a.Cg + g;
                const __amdgpu_buffer_rsrc_t rs0 = a_rsrc(gg), rs1 = a_rsrc(gg + (T == 1 ? 3 : 1) * a.ksr);
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    // araw[t % 3] is split already: its registers take step t + 3.
                    if (!PAIR || t + 3 < T) load_a(araw[t % 3], t + 3 < T ? rs0 : rs1, (t + 3) % T);
                    Parts An;
#pragma unroll
                    for (int b = 0; b < NBW; ++b) {
                        const int un = t * NBW + b, tn = (un + 1) / NBW, bn = (un + 1) % NBW;
                        read_b(B[(un + 1) & 1], tn < T ? gb + tap_at(tn) : gnext, bn);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (j * NBW / 4 == b) {  // the split's four pairs, dealt to the units
                                split2(An, j, araw[(t + 1) % 3][j].x, araw[(t + 1) % 3][j].y);
                                // (kept in this unit: the compiler would sink it to the next step's first use)
                                asm volatile("" : "+v"(An.h[j]), "+v"(An.m[j]), "+v"(An.l[j]));
                            }
                        const Parts &Bu = B[un & 1];
                        mma(low[b], A.l, Bu.h);
                        mma(low[b], A.h, Bu.l);
                        mma(low[b], A.m, Bu.m);
                        mma(low[b], A.m, Bu.h);
                        mma(low[b], A.h, Bu.m);
                        mma(acc[b], A.h, Bu.h);
                        if constexpr (RS > 1) {
                            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);              // LDS reads
                            if (b == 0 && (!PAIR || t + 3 < T))
                                __builtin_amdgcn_sched_group_barrier(0x020, 4, 0);  // A loads
#pragma unroll
                            for (int k = 0; k < 6; ++k) {
                                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                                __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);  // VALU
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    A = An;
                }
                if constexpr ((T * NBW) % 2 == 1) B[0] = B[1];
                if constexpr (T % 3 != 0 && !PAIR) {  // one tap: the ring turns by copies
                    static_assert(RS == 1, "filters of the dense kernel");
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x2_t v = araw[0][j];
                        araw[0][j] = araw[1][j];
                        araw[1][j] = araw[2][j];
                        araw[2][j] = v;
                    }
                }
            }
        }
        if (more) {
            if (a.nbuf == 1) __syncthreads();
            stage_put(ch + 1, ldsb + (a.nbuf == 2 ? ((ch + 1) & 1) * a.buf_bytes : 0));
            __syncthreads();
        }
    }
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] += low[b][r];

    // (The lane counted again: the values above would stay in registers through the loop.)
    const int elane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int ehalf = elane >> 5, ecol = elane & 31;
    // Row and column of the lane's pixel in each block, virtual pixel q0 + 32*b of
    // the tile and on (row -1: not stored).
    int ys[NBW], xs[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
        const int q = q0 + kDnsTile * b + ecol;
        const int yl = (int)fast_div((uint32_t)q, a.wp_magic, a.wp_shift), x = q - yl * a.Wp;
        const bool in = yl < a.TH && x < a.Wo && y0 + yl < a.Ho;
        ys[b] = in ? y0 + yl : -1;
        xs[b] = x;
    }
    // A wave with a sum that is not finite takes its share of the sums again on the
    // fp32 MFMA (see the file comment), a filter row of a channel pair at a time
    // from global memory, and keeps the new value where the old one is not finite.
    // With NaN in every pixel 14x14, 256 channels, batch 32 takes 211 us (59 without;
    // 1623 where each lane summed its outputs one after another).
    bool bad = false;
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) bad |= ys[b] >= 0 && !(fabsf(acc[b][r]) < INFINITY);
    if (__builtin_amdgcn_ballot_w64(bad)) {
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) low[b][r] = 0.0f;
        for (int g = wr; g < ngroups; g += a.ksr)
            for (int cp = 8 * g; cp < min(8 * g + 8, npairs); ++cp) {
                const int c = 2 * cp + ehalf;  // (past the last channel of an odd count: zeros)
                const float *plane = xp + ((size_t)n * a.C + min(c, a.C - 1)) * a.IH * a.IW;
#pragma unroll 1
                for (int r = 0; r < R; ++r) {
                    float w[S], v[S][NBW];
                    int at[S][NBW];
#pragma unroll
                    for (int t = 0; t < S; ++t) {
                        w[t] = wpk[((size_t)(cp * RS + r * S + t) * a.Kp + k0 + ecol) * 2 + ehalf];
#pragma unroll
                        for (int b = 0; b < NBW; ++b) {
                            const int y = ys[b] + r - a.ipad, x = xs[b] + t - a.ipad;
                            const bool in = ys[b] >= 0 && c < a.C && y >= 0 && y < a.IH && x >= 0 && x < a.IW;
                            at[t][b] = in ? y * a.IW + x : -1;
                            v[t][b] = plane[max(at[t][b], 0)];  // (no branch around the load)
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);  // (the compiler would wait for each load in turn)
#pragma unroll
                    for (int t = 0; t < S; ++t)
#pragma unroll
                        for (int b = 0; b < NBW; ++b)
                            low[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[t], at[t][b] >= 0 ? v[t][b] : 0.0f, low[b], 0, 0, 0);
                }
            }
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[b][r] = fabsf(acc[b][r]) < INFINITY ? acc[b][r] : low[b][r];
    }

    // Sum the ksr partial tiles, in order 0, 1, ..., through LDS; wave wr keeps
    // accumulator registers wr*J .. wr*J + J - 1 (fin[b][jj], J = 16 / ksr), so
    // every wave has a share of the epilogue.
    const int J = 16 / a.ksr, j0 = wr * J;
    if (a.ksr > 1) {
        __syncthreads();  // the chunk buffers are free
        float *red = lds + (size_t)(wp * a.nw + wn) * a.ksr * NBW * 16 * kWave + elane;
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int j = 0; j < 16; ++j) red[((wr * NBW + b) * 16 + j) * kWave] = acc[b][j];
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            if (jj >= J) break;
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                float s = red[(b * 16 + j0 + jj) * kWave];
                for (int k = 1; k < a.ksr; ++k) s += red[((k * NBW + b) * 16 + j0 + jj) * kWave];
                acc[b][jj] = s;
            }
        }
    }

    // acc[b][jj] is channel chan(jj) of pixel (ys[b], xs[b]).
    auto chan = [&](int jj) {
        const int j = j0 + jj;
        return k0 + 8 * (j >> 2) + 4 * ehalf + (j & 3);
    };

    // Bias, residual and ReLU of registers 4*gq .. 4*gq + 3 (the residuals of
    // all blocks are loaded before the first is used).
    auto finish4 = [&](int gq) {
        float rv[4][NBW], bk[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = chan(4 * gq + u);
            bk[u] = (bias && k < a.K) ? bias[k] : 0.0f;
            if (res) {
                const float *rplane = res + ((size_t)n * a.K + k) * a.rplane + a.res_pad * (a.rpitch + 1);
#pragma unroll
                for (int b = 0; b < NBW; ++b)
                    rv[u][b] = (ys[b] >= 0 && k < a.K) ? rplane[(size_t)ys[b] * a.rpitch + xs[b]] : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                float v = acc[b][4 * gq + u] + bk[u];
                if (res) v += rv[u][b];
                if (a.relu) v = v > 0.0f ? v : 0.0f;
                acc[b][4 * gq + u] = v;
            }
    };
    const bool stream = a.out_pad == 0;
    const int share = wr * a.ksp + wp, shares = a.ksr * a.ksp;  // this wave among its channel tile's
    if constexpr (!POOL) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            if (4 * gq >= J) break;
            finish4(gq);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = chan(4 * gq + u);
                if (k >= a.K) continue;
                float *plane = out + ((size_t)n * a.K + k) * a.oplane + a.out_pad * (a.opitch + 1);
#pragma unroll
                for (int b = 0; b < NBW; ++b)
                    if (ys[b] >= 0) store_out(plane + (size_t)ys[b] * a.opitch + xs[b], acc[b][4 * gq + u], stream);
            }
        }
        if (a.out_pad) {
            const int r1 = min(y0 + a.TH, a.Ho);
            for (int kk = k0 + share; kk < min(k0 + kDnsTile, a.K); kk += shares)
                zero_border(out + ((size_t)n * a.K + kk) * a.oplane, y0, r1, a.Ho, a.Wo, a.out_pad, a.opitch, ty == 0,
                            ty == a.ntiles_y - 1, elane, kWave);
        }
    } else {
        // Pool through LDS, 8 channels of each (channel tile, reduction share)
        // at a time: its ksp waves stage the activated values of their blocks,
        // then take the max of each 2x2 window between them.
        const int px = a.ksp * NBW * kDnsTile;
        float *st = lds + (size_t)(wn * a.ksr + wr) * kDnsPoolCh * px;
        const int prow0 = y0 / 2;
        const int prows = a.TH / 2;
        const int per_ch = prows * a.Wq;
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            if (4 * gq >= J) break;
            finish4(gq);
            __syncthreads();  // the chunk buffers, or the previous round's values, are read
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int b = 0; b < NBW; ++b)
                    st[(4 * ehalf + u) * px + q0 + kDnsTile * b + ecol] = acc[b][4 * gq + u];
            __syncthreads();
            for (int t = wp * kWave + elane; t < kDnsPoolCh * per_ch; t += a.ksp * kWave) {
                const int cc = (int)fast_div((uint32_t)t, a.pch_magic, a.pch_shift);
                const int rem = t - cc * per_ch;
                const int r = (int)fast_div((uint32_t)rem, a.wq_magic, a.wq_shift), jq = rem - r * a.Wq;
                const int k = k0 + 8 * ((j0 >> 2) + gq) + cc;
                const int pr = prow0 + r;
                if (k < a.K && pr < a.Hq) {
                    const float *s0 = st + cc * px + 2 * r * a.Wp + 2 * jq;
                    const float m = fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[a.Wp], s0[a.Wp + 1]));
                    store_out(out + ((size_t)n * a.K + k) * a.oplane + (size_t)(pr + a.out_pad) * a.opitch + jq +
                                  a.out_pad,
                              m, stream);
                }
            }
        }
        if (a.out_pad) {
            const int r1 = min(prow0 + prows, a.Hq);
            for (int kk = k0 + share; kk < min(k0 + kDnsTile, a.K); kk += shares)
                zero_border(out + ((size_t)n * a.K + kk) * a.oplane, prow0, r1, a.Hq, a.Wq, a.out_pad, a.opitch,
                            ty == 0, ty == a.ntiles_y - 1, elane, kWave);
        }
    }
}

using DenseKernel = void (*)(DenseArgs, const float *, const float *, const float *, const float *, float *);

template <int R, int S, int NBW, bool PAIR>
DenseKernel pick_dense_pool(bool pool) {
    return pool ? spconv_dense_kernel<R, S, NBW, true, PAIR> : spconv_dense_kernel<R, S, NBW, false, PAIR>;
}

template <int R, int S, bool PAIR>
DenseKernel pick_dense_nbw(int NBW, bool pool) {
    switch (NBW) {
        case 1: return pick_dense_pool<R, S, 1, PAIR>(pool);
        case 2: return pick_dense_pool<R, S, 2, PAIR>(pool);
        case 3: return pick_dense_pool<R, S, 3, PAIR>(pool);
        case 4: return pick_dense_pool<R, S, kDnsWaveBlocks, PAIR>(pool);
        default: return nullptr;
    }
}

// Two taps per MFMA step: one octet of channels, several taps.
bool dense_pairs(int C, int R, int S) { return C <= 8 && R * S > 1; }

// Filter shapes the dense kernel is built for.
DenseKernel pick_dense(int C, int R, int S, int NBW, bool pool) {
    if (R == 3 && S == 3)
        return dense_pairs(C, R, S) ? pick_dense_nbw<3, 3, true>(NBW, pool) : pick_dense_nbw<3, 3, false>(NBW, pool);
    if (R == 1 && S == 1) return pick_dense_nbw<1, 1, false>(NBW, pool);
    return nullptr;
}

}  // namespace

// (R, S, blocks per tile, pool) of every tile shape of the dense kernel (a
// library-internal helper of spconv_kernel_variants, not exported). Tiles of
// more than one block share them between waves, so several tile shapes run one
// compiled instance.
__attribute__((visibility("hidden"))) int dense_kernel_variants(int32_t *variants, int32_t capacity, int32_t *count) {
    int n = 0;
    for (int rs : {3, 1})
        for (int nb = 1; nb <= kDnsMaxBlocks; ++nb)
            for (int pool = 0; pool < 2; ++pool) {
                    if (n < capacity) {
                        variants[4 * n] = rs;
                        variants[4 * n + 1] = rs;
                        variants[4 * n + 2] = nb;
                        variants[4 * n + 3] = pool;
                    }
                    ++n;
                }
    *count = n;
    return SPCONV_OK;
}

namespace {

struct DensePlan {
    int TH = 0, ntiles_y = 0, NB = 0, NBW = 0, nw = 0, ksr = 1, ksp = 1, nkt = 0, Cg = 0, nchunks = 0, nbuf = 1;
    int PX = 0, total_wgs = 0;
    size_t lds_bytes = 0;
};

using dense_layout::round_up;

int dense_waves(int K) { return dense_layout::waves(K); }

// Kp of the packed filter: K rounded up to whole workgroup channel tiles.
int dense_kp(int K) { return dense_layout::kp(K); }

// Waves per channel tile (1, 2 or 4): two where the workgroup has room, four
// only when even two would leave the grid under 1024 waves.
int dense_split(long long base_waves, int nw) {
    int ws = nw * 2 * kWave <= kDnsMaxThreads ? 2 : 1;
    if (ws == 2 && base_waves * 2 < 1024 && nw * 4 * kWave <= kDnsMaxThreads) ws = 4;
    return ws;
}

// Splits a tile's waves and LDS. The ws waves of a channel tile share its pixel
// blocks until each has at most four (accumulators; with three or four an A
// fragment's split and loads are small next to its MFMAs), and the reduction
// from there on; where the partial tiles or a chunk of that many groups do not
// fit the LDS they share pixels only. A chunk holds as many channel groups as
// threads can load ahead (kDnsRounds tasks each), in two buffers where they fit.
// A chunk's channels lie within 32-bit byte offsets (`plane_bytes` each).
bool dense_layout_tile(int C, long long plane_bytes, int Wp, int Wo, int R, int S, bool pool, int ws, DensePlan *q) {
    const long long range = 0xfffffff0LL / plane_bytes;  // channels in reach
    const int valid = (q->TH - 1) * Wp + Wo;  // virtual pixels up to the last stored one
    const int nbv = (valid + kDnsTile - 1) / kDnsTile;
    const int ngroups = (C + kDnsGroup - 1) / kDnsGroup;
    q->PX = valid + (R - 1) * Wp + S - 1;
    const long long unit = (long long)q->PX * kDnsPxBytes;
    for (int ksr = ws; ksr >= 1; ksr /= 2) {
        const int ksp = ws / ksr;
        const int nbw = (nbv + ksp - 1) / ksp;
        if (nbw > kDnsWaveBlocks || ksr > ngroups) continue;
        // Lanes of the last block past the stored pixels read on past PX.
        const int slack = std::max(0, nbv * kDnsTile + (R - 1) * Wp + S - 1 - q->PX) * 16;
        size_t epi = pool ? (size_t)q->nw * ksr * kDnsPoolCh * ksp * nbw * kDnsTile * sizeof(float) : 0;
        if (ksr > 1) epi = std::max(epi, (size_t)q->nw * ws * nbw * 16 * kWave * sizeof(float));
        if (epi > (size_t)kDnsLdsBytes) continue;
        const int threads = q->nw * ws * kWave;
        int gmax = (int)std::min<long long>((kDnsLdsBytes - slack) / unit, 1 << 20);
        if (gmax < 1 && unit + slack <= kDnsLdsMax) gmax = 1;
        if (std::min(C, kDnsGroup) > range) return false;
        if (C > range) gmax = std::min(gmax, (int)(range / kDnsGroup));
        if (gmax < ksr) continue;
        const int ahead = std::max(1, kDnsRounds * threads / (2 * q->PX));  // groups loaded ahead
        int Cg = std::min({ahead, gmax, ngroups});
        if (Cg < ngroups && gmax / 2 >= ksr) Cg = std::min(Cg, gmax / 2);
        Cg = std::max(ksr, Cg / ksr * ksr);
        q->ksr = ksr;
        q->ksp = ksp;
        q->NBW = nbw;
        q->Cg = Cg;
        q->nchunks = (ngroups + Cg - 1) / Cg;
        q->nbuf = (q->nchunks > 1 && 2 * Cg <= gmax) ? 2 : 1;
        q->lds_bytes = std::max((size_t)(q->nbuf * Cg * unit + slack), epi);
        return true;
    }
    return false;
}

// Tile rows: among the heights whose tile fits 8 pixel blocks (even heights
// when pooling), the least modelled work, tiles x (blocks + 1): a wave's MFMAs
// per channel group (one set per block and tap) plus about one block's worth
// for the group's A fragments, which each block reuses; provided the grid keeps
// at least 1536 waves (six per SIMD over the run) when any height can, ties
// going to the grid with more waves. Measured on 14x14 (256 channels), 28x28
// pooled and 56x56 layers: the picks are each layer's fastest tiling of the sweep.
bool plan_dense(int N, int C, int K, int H, int W, int pad, int Wp, int Ho, int Wo, int R, int S, bool pool,
                DensePlan *pl) {
    DensePlan p;
    p.nw = dense_waves(K);
    p.nkt = (K + kDnsTile * p.nw - 1) / (kDnsTile * p.nw);
    const long long kMinWaves = 1536;
    DensePlan best;
    long long best_cost = 0, best_waves = 0;
    for (int th = pool ? 2 : 1; th <= (pool ? round_up(Ho, 2) : Ho); th += pool ? 2 : 1) {
        DensePlan q = p;
        q.TH = th;
        q.NB = (th * Wp + kDnsTile - 1) / kDnsTile;
        if (q.NB > kDnsMaxBlocks) break;
        q.ntiles_y = (Ho + th - 1) / th;
        const long long base_waves = (long long)N * q.ntiles_y * q.nkt * q.nw;
        if (!dense_layout_tile(C, (H + 2LL * pad) * Wp * (long long)sizeof(float), Wp, Wo, R, S, pool,
                               dense_split(base_waves, q.nw), &q))
            continue;
        const long long waves = base_waves * q.ksr * q.ksp;
        const long long cost = (long long)q.ntiles_y * (q.NB + 1);
        bool better;
        if (best.TH == 0) {
            better = true;
        } else {
            const bool ok = waves >= kMinWaves, best_ok = best_waves >= kMinWaves;
            if (ok != best_ok)
                better = ok;
            else if (!ok)
                better = waves > best_waves;
            else
                better = cost < best_cost || (cost == best_cost && waves > best_waves);
        }
        if (better) {
            best = q;
            best_cost = cost;
            best_waves = waves;
        }
    }
    if (best.TH == 0) return false;
    p = best;
    const long long wgs = (long long)N * p.ntiles_y * p.nkt;
    if (wgs > 0x7fffffffLL) return false;
    p.total_wgs = (int)wgs;
    *pl = p;
    return true;
}

bool out_extent(int in, int k, int pad, int *o) {
    const long long v = (long long)in + 2LL * pad - k + 1;
    if (v < 1 || v > 0x7fffffffLL) return false;
    *o = (int)v;
    return true;
}

// Checks and plan of a dense forward call (everything but the buffers).
int prepare_dense(int N, int C, int H, int W, int K, int R, int S, int pad, uint32_t flags,
                  const spconv_options *opt, DensePlan *plp, DenseArgs *ap) {
    if (N < 1 || C < 1 || H < 1 || W < 1 || K < 1 || R < 1 || S < 1 || pad < 0) return SPCONV_EINVAL;
    if (flags & ~(SPCONV_RELU | SPCONV_MAXPOOL2X2 | SPCONV_UNPADDED_INPUT)) return SPCONV_EINVAL;
    const long long Hp = (long long)H + 2LL * pad, Wp = (long long)W + 2LL * pad;
    if ((long long)C * Hp * Wp >= (1LL << 31)) return SPCONV_EINVAL;
    const bool pool = (flags & SPCONV_MAXPOOL2X2) != 0;
    int Ho, Wo;
    if (!out_extent(H, R, pad, &Ho) || !out_extent(W, S, pad, &Wo)) return SPCONV_EINVAL;
    if (pool && (Ho < 2 || Wo < 2)) return SPCONV_EINVAL;
    DensePlan pl;
    if (!plan_dense(N, C, K, H, W, pad, (int)Wp, Ho, Wo, R, S, pool, &pl)) return SPCONV_EINVAL;
    if (!pick_dense(C, R, S, pl.NBW, pool)) return SPCONV_EINVAL;
    DenseArgs a;
    a.N = N;
    a.C = C;
    a.K = K;
    a.Kp = dense_kp(K);
    const long long wbytes = (long long)((C + 1) / 2) * R * S * a.Kp * 2 * (long long)sizeof(float);
    if (wbytes >= (1LL << 31)) return SPCONV_EINVAL;
    a.wpk_bytes = (int)wbytes;
    a.Hp = (int)Hp;
    a.Wp = (int)Wp;
    a.Ho = Ho;
    a.Wo = Wo;
    a.Hq = pool ? Ho / 2 : Ho;
    a.Wq = pool ? Wo / 2 : Wo;
    a.pch_magic = a.wq_magic = 1;
    a.pch_shift = a.wq_shift = 0;
    if (!div_magic((uint32_t)a.Wp, &a.wp_magic, &a.wp_shift) ||
        (pool && (!div_magic((uint32_t)((pl.TH / 2) * a.Wq), &a.pch_magic, &a.pch_shift) ||
                  !div_magic((uint32_t)a.Wq, &a.wq_magic, &a.wq_shift))))
        return SPCONV_EINVAL;
    a.relu = (flags & SPCONV_RELU) ? 1 : 0;
    const bool unpadded = (flags & SPCONV_UNPADDED_INPUT) != 0;
    a.IH = unpadded ? H : (int)Hp;
    a.IW = unpadded ? W : (int)Wp;
    a.ipad = unpadded ? pad : 0;
    a.TH = pl.TH;
    a.ntiles_y = pl.ntiles_y;
    a.nw = pl.nw;
    a.ksr = pl.ksr;
    a.ksp = pl.ksp;
    a.nkt = pl.nkt;
    a.Cg = pl.Cg;
    a.nchunks = pl.nchunks;
    a.nbuf = pl.nbuf;
    a.PX = pl.PX;
    a.tasks = (dense_pairs(C, R, S) ? 1 : 2 * pl.Cg) * pl.PX;
    a.buf_bytes = pl.Cg * pl.PX * kDnsPxBytes;
    if (!div_magic((uint32_t)pl.PX, &a.px_magic, &a.px_shift)) return SPCONV_EINVAL;
    a.total_wgs = pl.total_wgs;
    const long long op = opt ? opt->out_pad : 0;
    const long long rp = (opt && opt->residual) ? opt->residual_pad : 0;
    if (op < 0 || rp < 0) return SPCONV_EINVAL;
    const long long oh = a.Hq + 2 * op, ow = a.Wq + 2 * op;
    const long long rh = a.Ho + 2 * rp, rw = a.Wo + 2 * rp;
    if (oh * ow >= (1LL << 31) || rh * rw >= (1LL << 31)) return SPCONV_EINVAL;
    a.out_pad = (int)op;
    a.opitch = (int)ow;
    a.oplane = (size_t)(oh * ow);
    a.res_pad = (int)rp;
    a.rpitch = (int)rw;
    a.rplane = (size_t)(rh * rw);
    *plp = pl;
    *ap = a;
    return SPCONV_OK;
}

}  // namespace

extern "C" int spconv_forward_dense(const float *in_padded, int N, int C, int H, int W, const float *packed, int K,
                                    int R, int S, int pad, const float *bias, uint32_t flags,
                                    const spconv_options *opt, float *out, hipStream_t stream) {
    if (!in_padded || !packed || !out) return SPCONV_EINVAL;
    DensePlan pl;
    DenseArgs a;
    const int rc = prepare_dense(N, C, H, W, K, R, S, pad, flags, opt, &pl, &a);
    if (rc != SPCONV_OK) return rc;
    DenseKernel kern = pick_dense(C, R, S, pl.NBW, (flags & SPCONV_MAXPOOL2X2) != 0);
    const float *residual = opt ? opt->residual : nullptr;
    // Raised once per instance to the family's budget (see raise_lds_limit).
    if (!raise_lds_limit((const void *)kern, kDnsLdsMax)) return SPCONV_EHIP;
    // A launch counts its threads in 32 bits: tens of millions of images take
    // several, each of as many whole images as fit.
    const int threads = pl.nw * pl.ksr * pl.ksp * kWave, per_image = pl.total_wgs / N;
    const int most = (int)std::min<long long>(N, std::max(1LL, 0xffffffffLL / threads / per_image));
    for (int n0 = 0; n0 < N; n0 += most) {
        a.N = std::min(most, N - n0);
        a.total_wgs = a.N * per_image;
        hipLaunchKernelGGL(kern, dim3((unsigned)a.total_wgs), dim3((unsigned)threads), pl.lds_bytes, stream, a,
                           in_padded + (size_t)n0 * C * a.IH * a.IW, packed, bias,
                           residual ? residual + (size_t)n0 * K * a.rplane : nullptr, out + (size_t)n0 * K * a.oplane);
        if (hipGetLastError() != hipSuccess) return SPCONV_EHIP;
        if (N - n0 <= most) break;  // (n0 + most may pass int)
    }
    return SPCONV_OK;
}

extern "C" int spconv_dense_plan(int N, int C, int H, int W, int K, int R, int S, int pad, uint32_t flags,
                                 spconv_plan_info *info) {
    if (!info) return SPCONV_EINVAL;
    DensePlan pl;
    DenseArgs a;
    const int rc = prepare_dense(N, C, H, W, K, R, S, pad, flags, nullptr, &pl, &a);
    if (rc != SPCONV_OK) return rc;
    info->kernel = SPCONV_KERNEL_DENSE;
    info->pixels_per_lane = pl.NB;
    info->images_per_group = 1;
    info->channels_per_wave = kDnsTile;
    info->tile_rows = pl.TH;
    info->tiles_per_image = pl.ntiles_y;
    info->channels_per_chunk = std::min(pl.Cg * kDnsGroup, C);
    info->chunks = pl.nchunks;
    info->workgroups = pl.total_wgs;
    info->threads_per_workgroup = pl.nw * pl.ksr * pl.ksp * kWave;
    info->lds_bytes = (int64_t)pl.lds_bytes;
    info->lds_channel_floats = info->lds_row_pitch = info->lds_col_shift = 0;
    info->launch_workgroups = pl.total_wgs;
    info->tile_pixels = 0;
    return SPCONV_OK;
}

namespace {

// Microseconds of the dense kernel on a plan: per round of workgroups (one or two a
// CU) 7.2, the MFMAs of a SIMD's waves at 59 % of their rate, and 0.55 for each
// round of staging loads past those that run a chunk ahead; the bytes of the planes
// and of the filter; and the input's that the 256 MB of Infinity Cache do not
// hold, which neighbouring tiles fetch again. Against 422 layers (those of
// sparse_layer_us) half are within 7 % and nine in ten within 20 %.
double dense_us(const DensePlan &pl, const DenseArgs &a, int R, int S) {
    const int waves = pl.nw * pl.ksr * pl.ksp;
    const int ngroups = (a.C + kDnsGroup - 1) / kDnsGroup;
    const bool pairs = dense_pairs(a.C, R, S);
    const int resident = std::max(1, std::min(8 / waves, kDnsCuLds / (int)pl.lds_bytes));
    const double rounds = std::ceil(pl.total_wgs / (256.0 * resident));
    const double per_simd = std::max(1.0, std::min((double)resident, std::ceil(pl.total_wgs / 256.0)) * waves / 4.0);
    const int steps = (ngroups + pl.ksr - 1) / pl.ksr * (pairs ? (R * S + 1) / 2 : R * S);
    const double mfma = 6.0 * 32.0 * steps * pl.NBW * per_simd;
    const int tasks = (pairs ? 1 : 2 * std::min(pl.Cg, ngroups)) * pl.PX;
    const int threads = waves * kWave;
    const double late = std::max(0, (tasks + threads - 1) / threads - kDnsRounds) * (double)pl.nchunks;
    const double in = 4e-6 * a.N * ((double)a.C * a.Hp * a.Wp), out = 4e-6 * a.N * ((double)a.K * a.Hq * a.Wq);
    const double filter = 4e-6 * round_up(a.K, kDnsTile) * (double)a.C * R * S;
    return rounds * (7.2 + 0.704e-3 * mfma + 0.55 * late) + 0.33 * (in + out) + 1.9 * std::max(0.0, in - 256.0) +
           0.94 * filter;
}

// Filter density from which a layer stays dense where the other choice is the
// stride-1 walk, also if that is modelled faster: the dense sums are closer, 1.05 to
// 2.4 times and half of them 1.5 times, than the walk's chains of fp32 products
// (against float64 on 42 layers of densities 0.26 to 0.7), and layers this dense
// have always had them. (The line is where the fp32 MFMA kernel before this one
// broke even: 14x14, 28x28, 56x56 and 224x224 in batches of 32, log-linear in
// output pixels between.) What it costs: 3 to 16 channels, above all, 3 channels at
// 224x224 in a batch of 32 298 against 159 us.
double kept_dense_density(int Ho, int Wo) {
    struct Anchor {
        double px, d;
    };
    static constexpr Anchor kAnchors[] = {{196.0, 0.245}, {784.0, 0.44}, {3136.0, 0.43}, {50176.0, 0.67}};
    constexpr int n = (int)(sizeof(kAnchors) / sizeof(kAnchors[0]));
    const double px = std::max(1.0, (double)Ho * Wo);
    if (px <= kAnchors[0].px) return kAnchors[0].d;
    for (int i = 1; i < n; ++i)
        if (px <= kAnchors[i].px) {
            const double t = std::log2(px / kAnchors[i - 1].px) / std::log2(kAnchors[i].px / kAnchors[i - 1].px);
            return kAnchors[i - 1].d + t * (kAnchors[i].d - kAnchors[i - 1].d);
        }
    return kAnchors[n - 1].d;
}

}  // namespace

extern "C" int spconv_select_path(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int64_t nnz,
                                  uint32_t flags, int *path) {
    if (!path || N < 1 || C < 1 || H < 1 || W < 1 || K < 1 || R < 1 || S < 1 || stride < 1 || pad < 0 || nnz < 0 ||
        nnz > (int64_t)K * C * R * S || (flags & ~(SPCONV_RELU | SPCONV_MAXPOOL2X2 | SPCONV_UNPADDED_INPUT)))
        return SPCONV_EINVAL;
    *path = SPCONV_PATH_SPARSE;
    if (stride != 1) return SPCONV_OK;
    DensePlan pl;
    DenseArgs a;
    if (prepare_dense(N, C, H, W, K, R, S, pad, flags & ~SPCONV_UNPADDED_INPUT, nullptr, &pl, &a) != SPCONV_OK)
        return SPCONV_OK;
    double sparse;
    bool walk;
    if (!sparse_layer_us(N, C, H, W, K, R, S, pad, a.Ho, a.Wo, (flags & SPCONV_MAXPOOL2X2) != 0,
                         (flags & SPCONV_UNPADDED_INPUT) != 0, nnz, &sparse, &walk) ||
        dense_us(pl, a, R, S) < sparse ||
        (walk && (double)nnz > kept_dense_density(a.Ho, a.Wo) * (double)K * C * R * S))
        *path = SPCONV_PATH_DENSE;
    return SPCONV_OK;
}
