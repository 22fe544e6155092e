// Sparse convolution on the matrix cores (gfx950 MFMA) from the CSR filter, any
// filter shape and stride: for strided layers, whose entries the vector units
// would gather at a step, and wherever multiplying the zeros of a small tile
// costs less than walking its entries.
//
// A workgroup owns (image, tile of TH x TW output pixels, M output channels) and
// takes the input channels in chunks of O octets. For each chunk it holds in LDS
//  * the tile's input window, every value split into three bf16 parts (split.h),
//    as [octet][pixel][part][8 channels] (48 bytes per octet and pixel: 16 pixels
//    side by side start in the 16 different 16-byte bank groups);
//  * the chunk's part of the filter as dense fragments: zeros, and the CSR
//    entries scattered over them, split the same way.
// The product then runs over octet-taps (8 channels under one filter tap), four
// to an MFMA (v_mfma_f32_16x16x32_bf16, one per quarter of the lanes): a lane
// reads 8 channels of its pixel under its quarter's tap, at the pixel's base plus
// an offset per (unit of four octet-taps, quarter) from a table, so tiles need
// no padded columns, and strides only change the bases. Six part products per
// unit give fp32 products (split.h); the hh products and the smaller ones have
// separate fp32 sums, so the main sum rounds once per unit.
// An output that came out infinite or NaN is summed again from its CSR entries in
// fp32: infinities have no finite parts, zeros of the tile do not count, and near
// the top of the range h rounds up past the value, so that hh can overflow where
// the product does not.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>

#include "common.h"
#include "matrix.h"
#include "split.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMatThreads = 512;
constexpr int kMatWaves = kMatThreads / kWave;
constexpr int kMatPx = 48;               // LDS bytes of one octet of one staged pixel
constexpr int kMatFrag = 3 * 1024;       // LDS bytes of one filter fragment: 16 channels x 32 values x three parts
constexpr int kMatRounds = 2;            // input tasks per thread loaded a chunk ahead
constexpr int kMatQueue = 6;             // filter entries per thread loaded a chunk ahead
constexpr int kMatLdsBytes = 160 * 1024;

struct MatArgs {
    int N, C, K, R, S, stride;
    int IH, IW, ipad;     // input planes: padded row y, column x at plane row y - ipad, column x - ipad
    int Ho, Wo, Hq, Wq;   // output grid, stored grid
    int relu;
    int TH, TW, nty, ntx; // output tile and tiles per image
    int pitch;            // pixels from one tile row to the next in the lanes' order: TW, or up to 7 more
    int nkt, M;           // channel tiles and channels per tile
    int wm, wp, ksr;      // waves over channels, pixels, and units of the reduction
    int O, oshift, nchunks; // octets per chunk (a power of two)
    int nunits;           // MFMA units per chunk: ceil(O*R*S / 4)
    int rows, vp, PX;     // staged window: rows, columns, pixels
    int stepy, stepx;     // input rows/columns per staged row/column
    int lsy, lsx;         // staged rows/columns per output row/column
    int hw;               // LDS pixels of a staged row's columns x, x + lsx, x + 2*lsx, ... (vp = lsx * hw)
    int tasks;            // O * PX input tasks (8 channels of a pixel)
    int a_bytes, b_bytes; // LDS of one filter / input buffer
    int bufs;             // buffers of both, 1 or 2
    int Wp, plane;        // padded row pitch and plane of the CSR offsets
    int total_wgs;
    int out_pad, opitch;
    size_t oplane;
    int res_pad, rpitch;
    size_t rplane;
    // x / PX, x / vp, x / pitch, x / plane, x / Wp and the pooled x / ((TH/2)*(TW/2)), x / (TW/2)
    uint32_t px_magic, vp_magic, pt_magic, plane_magic, wp_magic, pw_magic, pq_magic;
    int px_shift, vp_shift, pt_shift, plane_shift, wp_shift, pw_shift, pq_shift;
};

// A fragment (16 rows x 4 octet-taps x 8 channels, three parts) is stored as
// slots of 16 rows x 16 bytes per (unit, part, quarter), slot s = unit * 12 +
// part * 4 + quarter at s * 256 bytes; row i sits at position (i + s) & 15 of
// its slots, so that one row's slots, cleared together, lie in different banks.

// x / d for 0 <= x < 2^31 and d >= 2 (whose reciprocal's shift is 32 or more).
__device__ __forceinline__ int fast_div_hi(int x, uint32_t magic, int shift) {
    return (int)(__umulhi((uint32_t)x, magic) >> (shift - 32));
}

struct MatTask {
    uint32_t voff;  // byte offset of the octet's first channel from the chunk's, or past its end
    int lds;        // byte offset in the input buffer, or -1 (no task)
};

constexpr uint32_t kMatNone = 0xfffffff0u;

// LDS position of staged column x: the columns one output row reads under a tap
// (every lsx-th) lie side by side, as with stride 1.
__device__ __forceinline__ int column(const MatArgs &a, int x) {
    return a.lsx == 1 ? x : x % a.lsx * a.hw + x / a.lsx;
}

__device__ __forceinline__ MatTask mat_task(const MatArgs &a, int id, int y0, int x0) {
    MatTask t;
    t.lds = -1;
    t.voff = kMatNone;
    if (id < a.tasks) {
        const int oct = (int)fast_div((uint32_t)id, a.px_magic, a.px_shift);
        const int px = id - oct * a.PX;
        const int i = (int)fast_div((uint32_t)px, a.vp_magic, a.vp_shift);
        const int xi = px - i * a.vp;
        const int y = y0 * a.stride + i * a.stepy - a.ipad, x = x0 * a.stride + xi * a.stepx - a.ipad;
        t.lds = (oct * a.PX + i * a.vp + column(a, xi)) * kMatPx;
        if (y >= 0 && y < a.IH && x >= 0 && x < a.IW)
            t.voff = (uint32_t)((oct * 8 * a.IH + y) * a.IW + x) * (uint32_t)sizeof(float);
    }
    return t;
}

__device__ __forceinline__ void mat_load(const MatArgs &a, const __amdgpu_buffer_rsrc_t &rsrc, const MatTask &t,
                                         float (&v)[8]) {
    const uint32_t step = t.voff == kMatNone ? 0u : (uint32_t)(a.IH * a.IW) * (uint32_t)sizeof(float);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, t.voff + j * step, 0, 0));
}

__device__ __forceinline__ void mat_put(char *buf, const MatTask &t, const float (&v)[8]) {
    if (t.lds < 0) return;
    Parts p;
#pragma unroll
    for (int i = 0; i < 4; ++i) split2(p, i, v[2 * i], v[2 * i + 1]);
    char *d = buf + t.lds;
    *reinterpret_cast<u32x4_t *>(d) = p.h;
    *reinterpret_cast<u32x4_t *>(d + 16) = p.m;
    *reinterpret_cast<u32x4_t *>(d + 32) = p.l;
}

// Plain fp32 sums, in CSR order, of four output channels (row entries j[i] .. e[i] -
// 1, the same for the whole wave) at the lanes' pixels (padded input rows y,
// columns x; y < 0: none), for results that are not finite. A wave decodes 64
// entries of each row at once, one to a lane, and takes them in turn from those
// lanes; four rows side by side meet the same input channels while these are in
// the L1. With NaN in every pixel 56x56 of stride 2, 64 to 128 channels, batch 32,
// density 0.2 takes 391 us (61 without; 1124 where each lane summed its outputs
// one after another), 28x28, 128 channels, density 0.35 1048 us (62; 3328).
template <int P>
__device__ __forceinline__ void mat_sums_fp32(const MatArgs &a, const float *__restrict__ img,
                                              const int32_t *__restrict__ offset, const float *__restrict__ vals,
                                              const int (&j)[4], const int (&e)[4], int lane, const int (&y)[P],
                                              const int (&x)[P], float (&s)[4][P]) {
    constexpr int U = 4;
    int most = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        most = max(most, e[i] - j[i]);
#pragma unroll
        for (int p = 0; p < P; ++p) s[i][p] = 0.0f;
    }
    int pix[P];
#pragma unroll
    for (int p = 0; p < P; ++p) pix[p] = y[p] * a.IW + x[p];
#pragma unroll 1
    for (int t0 = 0; t0 < most; t0 += kWave) {
        int wt[4], dy[4], dx[4], base[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = max(min(j[i] + t0 + lane, e[i] - 1), 0);  // (past the row: another entry, not added)
            const int o = offset[at];
            wt[i] = (int)__float_as_uint(vals[at]);
            const int c = (int)fast_div((uint32_t)o, a.plane_magic, a.plane_shift);
            const int rem = o - c * a.plane;
            const int r = (int)fast_div((uint32_t)rem, a.wp_magic, a.wp_shift);
            dy[i] = r - a.ipad;
            dx[i] = rem - r * a.Wp - a.ipad;
            base[i] = (c * a.IH + dy[i]) * a.IW + dx[i];
        }
#pragma unroll 1
        for (int t = t0; t < min(most, t0 + kWave); t += U) {
            float in[U][4][P];
            int at[U][4][P];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int by = __builtin_amdgcn_readlane(dy[i], t - t0 + u);
                    const int bx = __builtin_amdgcn_readlane(dx[i], t - t0 + u);
                    const int bb = __builtin_amdgcn_readlane(base[i], t - t0 + u);
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const bool inside = y[p] >= 0 && (uint32_t)(y[p] + by) < (uint32_t)a.IH &&
                                            (uint32_t)(x[p] + bx) < (uint32_t)a.IW;
                        at[u][i][p] = inside ? bb + pix[p] : -1;
                        in[u][i][p] = img[max(at[u][i][p], 0)];  // (no branch around the load)
                    }
                }
            __builtin_amdgcn_sched_barrier(0);  // (the compiler would wait for each load in turn)
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = __uint_as_float((uint32_t)__builtin_amdgcn_readlane(wt[i], t - t0 + u));
#pragma unroll
                    for (int p = 0; p < P; ++p)
                        s[i][p] = j[i] + t + u < e[i] ? fmaf(v, at[u][i][p] >= 0 ? in[u][i][p] : 0.0f, s[i][p]) : s[i][p];
                }
        }
    }
}

// What bounds it: on a 56x56 layer of stride 2 (64 to 128 channels, batch 32,
// density 0.2) 43 us back to back (48 in a kernel trace), of which the MFMAs take
// 12; per chunk the staging (the scatter and the input's split, both vector
// instructions) and two barriers cost as much again as the MFMAs, and a launch
// about 12 us beside its chunks. 46 % of its LDS cycles are bank conflicts; which of
// the scatter, the input's stores and the reads make them has not been told apart. The
// any-stride kernel walks the entries of that layer in 261 us (154 us at density
// 0.05, 473 us at 0.5; here 40 and 50 us). Reads a block ahead and the 48-byte
// pixel rows took 3 to 5 % each; loads further ahead than one chunk, three tilings
// of 32 x 112 per wave and entry windows per wave instead of per lane were
// slower or no faster.
template <int RB, int NBX, bool POOL>
__global__ __launch_bounds__(kMatThreads) void spconv_matrix_kernel(MatArgs a, const float *__restrict__ xp,
                                                                    const int32_t *__restrict__ rowptr,
                                                                    const int32_t *__restrict__ offset,
                                                                    const float *__restrict__ vals,
                                                                    const float *__restrict__ bias,
                                                                    const float *__restrict__ res,
                                                                    float *__restrict__ out) {
    extern __shared__ float lds[];
    char *abuf = reinterpret_cast<char *>(lds);
    char *bbuf = abuf + a.bufs * a.a_bytes;
    int *table = reinterpret_cast<int *>(bbuf + a.bufs * a.b_bytes);
    const int tid = (int)threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int quarter = lane >> 4, col = lane & 15;
    const int work = xcd_linear_id((int)blockIdx.x, a.total_wgs);
    const int kt = __builtin_amdgcn_readfirstlane(work % a.nkt);
    const int tile = work / a.nkt;
    const int tx = __builtin_amdgcn_readfirstlane(tile % a.ntx);
    const int ty = __builtin_amdgcn_readfirstlane((tile / a.ntx) % a.nty);
    const int n = __builtin_amdgcn_readfirstlane(tile / (a.ntx * a.nty));
    const int y0 = ty * a.TH, x0 = tx * a.TW;
    const int wm = __builtin_amdgcn_readfirstlane(wave % a.wm);
    const int wr = __builtin_amdgcn_readfirstlane((wave / a.wm) % a.ksr);
    const int wp = __builtin_amdgcn_readfirstlane(wave / (a.wm * a.ksr));
    const int k0 = kt * a.M;
    const int taps = a.R * a.S;

    // Octet-tap offsets: unit u, quarter q takes octet-tap 4u + q = tap * O + octet.
    for (int i = tid; i < 4 * a.nunits; i += kMatThreads) {
        const int t = i / a.O, o = i - t * a.O;
        table[i] = t < taps ? (o * a.PX + t / a.S * a.vp + column(a, t % a.S)) * kMatPx : 0;
    }
    // This lane's pixels: LDS base, and output row (-1: not stored) and column.
    int pbase[NBX], ys[NBX], xs[NBX];
    const int th = min(a.TH, a.Ho - y0), tw = min(a.TW, a.Wo - x0);
    const int reach = (a.R - 1) * a.vp + (a.lsx - 1) * a.hw + (a.S - 1) / a.lsx;  // a tap's largest offset, or more
#pragma unroll
    for (int b = 0; b < NBX; ++b) {
        const int q = (wp * NBX + b) * 16 + col;
        const int yl = (int)fast_div((uint32_t)q, a.pt_magic, a.pt_shift), xl = q - yl * a.pitch;
        const bool in = yl < th && xl < tw;
        // (a dropped pixel reads on where it can: its lane's banks are then its own)
        const int px = yl * a.lsy * a.vp + xl;
        pbase[b] = in || px + reach < a.PX ? px * kMatPx : 0;
        ys[b] = in ? y0 + yl : -1;
        xs[b] = x0 + xl;
    }
    const bool active = wp * NBX * 16 < (th - 1) * a.pitch + tw;

    // Filter rows of the tile: `lpr` consecutive lanes share row `frow` (lanes
    // of one wave); lane `sub` of them takes the row's entries sub, sub + lpr,
    // ... in turn, `next` being its first one of the chunks to come.
    const int lpr = kMatThreads / a.M;
    const int frow = tid / lpr, sub = tid - frow * lpr;
    const int fbase = (frow >> 4) * a.nunits * kMatFrag;
    int next = 0, end = 0;
    if (k0 + frow < a.K) {
        next = rowptr[k0 + frow] + sub;
        end = rowptr[k0 + frow + 1];
    }
    int eo[kMatQueue];
    float ev[kMatQueue];
    auto load_a = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kMatQueue; ++i) {
            const int j = next + i * lpr;
            eo[i] = j < end ? offset[j] : 0x7fffffff;
            ev[i] = j < end ? vals[j] : 0.0f;
        }
    };
    // Stores entry (o, v) of the thread's row to its place in the fragments of
    // the chunk starting at channel c0.
    auto scatter = [&](char *buf, int c0, int o, float v) __attribute__((always_inline)) {
        const int c = fast_div_hi(o, a.plane_magic, a.plane_shift);
        const int rem = o - (int)__umul24(c, a.plane);
        const int r = fast_div_hi(rem, a.wp_magic, a.wp_shift), s = rem - (int)__umul24(r, a.Wp);
        const int cl = c - c0;
        if (r < a.R && s < a.S && cl >= 0) {
            const int u = ((int)__umul24(r, a.S) + s << a.oshift) + (cl >> 3);
            Parts p;
            split2(p, 0, v, 0.0f);
            const int row = (frow & 15) + (int)__umul24(u >> 2, 12) + (u & 3);
            char *d = buf + fbase + (int)__umul24(u >> 2, kMatFrag) + (u & 3) * 256 + (cl & 7) * 2;
            *reinterpret_cast<uint16_t *>(d + (row & 15) * 16) = (uint16_t)p.h[0];
            *reinterpret_cast<uint16_t *>(d + 1024 + ((row + 4) & 15) * 16) = (uint16_t)p.m[0];
            *reinterpret_cast<uint16_t *>(d + 2048 + ((row + 8) & 15) * 16) = (uint16_t)p.l[0];
        }
    };
    // Filter fragments of chunk ch: a row's lanes clear its slots and store its
    // entries there (no other wave touches them, and a wave's LDS operations
    // run in order), from the queue loaded before, then the queue moves on. A
    // lane's entries fall in slots that another lane cleared, which neither its
    // own addresses nor the types tell the compiler: the wavefront fence, no
    // instruction, keeps the clears first.
    auto put_a = [&](char *buf, int ch) __attribute__((always_inline)) {
        const int c0 = ch * a.O * 8;
        const int bound = min(c0 + a.O * 8, a.C) * a.plane;
        for (int s = sub; s < a.nunits * 12; s += lpr)  // slot s: (unit, part, quarter)
            *reinterpret_cast<u32x4_t *>(buf + fbase + s * 256 + ((frow + s) & 15) * 16) =
                (u32x4_t){0u, 0u, 0u, 0u};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        int got = 0;
#pragma unroll
        for (int i = 0; i < kMatQueue; ++i)
            if (eo[i] < bound) {
                scatter(buf, c0, eo[i], ev[i]);
                got = i + 1;
            }
        next += got * lpr;
        if (got == kMatQueue)  // the row has more entries in the chunk
            for (; next < end; next += lpr) {
                const int o = offset[next];
                if (o >= bound) break;
                scatter(buf, c0, o, vals[next]);
            }
    };

    MatTask task[kMatRounds];
    float xin[kMatRounds][8];
#pragma unroll
    for (int i = 0; i < kMatRounds; ++i) task[i] = mat_task(a, tid + i * kMatThreads, y0, x0);
    const size_t iplane = (size_t)a.IH * a.IW;
    auto chunk_rsrc = [&](int ch) __attribute__((always_inline)) {
        const int c0 = ch * a.O * 8, cn = min(a.O * 8, a.C - c0);
        return uniform_rsrc(xp + ((size_t)n * a.C + c0) * iplane, (uint32_t)(cn * iplane * sizeof(float)));
    };
    auto load_b = [&](int ch) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rsrc = chunk_rsrc(ch);
#pragma unroll
        for (int i = 0; i < kMatRounds; ++i)
            if (i * kMatThreads < a.tasks) mat_load(a, rsrc, task[i], xin[i]);
    };
    auto put_b = [&](char *buf, int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kMatRounds; ++i)
            if (i * kMatThreads < a.tasks) mat_put(buf, task[i], xin[i]);
        if (kMatRounds * kMatThreads < a.tasks) {
            const __amdgpu_buffer_rsrc_t rsrc = chunk_rsrc(ch);
            for (int id = tid + kMatRounds * kMatThreads; id < a.tasks; id += kMatRounds * kMatThreads) {
                MatTask t[kMatRounds];
                float v[kMatRounds][8];
#pragma unroll
                for (int i = 0; i < kMatRounds; ++i) {
                    t[i] = mat_task(a, id + i * kMatThreads, y0, x0);
                    mat_load(a, rsrc, t[i], v[i]);
                }
#pragma unroll
                for (int i = 0; i < kMatRounds; ++i) mat_put(buf, t[i], v[i]);
            }
        }
    };

    auto read_a = [&](Parts(&f)[RB], const char *A, int u) __attribute__((always_inline)) {
        const int turn = col + u * 12 + quarter;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const char *p = A + (rb * a.nunits + u) * kMatFrag;
            f[rb].h = *reinterpret_cast<const u32x4_t *>(p + (turn & 15) * 16);
            f[rb].m = *reinterpret_cast<const u32x4_t *>(p + 1024 + ((turn + 4) & 15) * 16);
            f[rb].l = *reinterpret_cast<const u32x4_t *>(p + 2048 + ((turn + 8) & 15) * 16);
        }
    };
    auto read_b = [&](Parts &f, const char *p) __attribute__((always_inline)) {
        f.h = *reinterpret_cast<const u32x4_t *>(p);
        f.m = *reinterpret_cast<const u32x4_t *>(p + 16);
        f.l = *reinterpret_cast<const u32x4_t *>(p + 32);
    };
    f32x4 acc[RB][NBX], low[RB][NBX];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int b = 0; b < NBX; ++b) acc[rb][b] = low[rb][b] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    auto mma = [&](f32x4 &c, const u32x4_t &x, const u32x4_t &y) __attribute__((always_inline)) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, y), c, 0,
                                                    0, 0);
    };

    // The buffers of chunk ch + 1 are filled, from registers loaded a chunk
    // before, while chunk ch is multiplied, where they are its own: by the older
    // wave of each SIMD before its MFMAs (phase 0), by the younger after them
    // (phase 1), so that the two overlap. A buffer shared with chunk ch is
    // filled once every wave is done with it (phase 2). Chunk -1 fills the first
    // buffers. (One loop over the phases, so that the code of each part exists
    // once: three copies of it did not fit the instruction cache.)
    const int mine = wave < kMatWaves / 2 ? 0 : 1;
    int turned = 0;  // units before this chunk, modulo ksr
    load_b(0);
    load_a();
#pragma unroll 1
    for (int ch = -1; ch < a.nchunks; ++ch) {
        const bool more = ch + 1 < a.nchunks;
#pragma unroll 1
        for (int phase = 0; phase < 3; ++phase) {
            if (phase == 2) {
                if (!more || a.bufs == 2) break;
                __syncthreads();
            }
            if (phase == 1 && ch >= 0) {
                const char *A = abuf + (a.bufs == 2 ? (ch & 1) * a.a_bytes : 0) + wm * RB * a.nunits * kMatFrag + quarter * 256;
                const char *B = bbuf + (a.bufs == 2 ? (ch & 1) * a.b_bytes : 0);
                int u = wr - turned;
                if (u < 0) u += a.ksr;
                if (active && u < a.nunits) {
                    // One pipeline over (unit, pixel block): the reads of the next
                    // block (or of the next unit's first, and of its filter
                    // fragments) are in flight under the MFMAs of the current one.
                    Parts fa[RB], fb[2];
                    const char *bu = B + table[4 * u + quarter];
                    read_a(fa, A, u);
                    read_b(fb[0], bu + pbase[0]);
                    for (; u < a.nunits; u += a.ksr) {
                        const int un = u + a.ksr < a.nunits ? u + a.ksr : u;  // (the last unit's reads repeat)
                        const int tn = table[4 * un + quarter];
                        const char *bn = bu;
                        Parts fn[RB];
#pragma unroll
                        for (int b = 0; b < NBX; ++b) {
                            if (b + 1 == NBX) bn = B + tn;
                            read_b(fb[(b + 1) & 1], (b + 1 < NBX ? bu : bn) + pbase[(b + 1) % NBX]);
                            if (b == NBX - 1) read_a(fn, A, un);
                            const Parts &f = fb[b & 1];
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma(low[rb][b], fa[rb].l, f.h);
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma(low[rb][b], fa[rb].h, f.l);
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma(low[rb][b], fa[rb].m, f.m);
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma(low[rb][b], fa[rb].m, f.h);
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma(low[rb][b], fa[rb].h, f.m);
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) mma(acc[rb][b], fa[rb].h, f.h);
                            // (the compiler would issue the reads last)
                            if (b == 0)
                                __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
                            else if (b == NBX - 1)
                                __builtin_amdgcn_sched_group_barrier(0x100, 3 + 3 * RB, 0);
                            else
                                __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                            __builtin_amdgcn_sched_group_barrier(0x008, 6 * RB, 0);
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) fa[rb] = fn[rb];
                        bu = bn;
                        if (NBX & 1) fb[0] = fb[1];
                    }
                }
                turned = (turned + a.nunits) % a.ksr;
            }
            if (more && phase == (a.bufs == 2 || ch < 0 ? mine : 2)) {
                // (Both puts before the loads: a put waits for every load before it.)
                const int buf = a.bufs == 2 ? (ch + 1) & 1 : 0;
                put_a(abuf + buf * a.a_bytes, ch + 1);
                put_b(bbuf + buf * a.b_bytes, ch + 1);
                load_a();
                if (ch + 2 < a.nchunks) load_b(ch + 2);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int b = 0; b < NBX; ++b) acc[rb][b] += low[rb][b];

    // Sum the ksr partial tiles in order through LDS; wave wr keeps accumulator
    // registers wr*J .. wr*J + J - 1.
    const int J = 4 / a.ksr, j0 = wr * J;
    if (a.ksr > 1) {
        __syncthreads();
        float *red = lds + (size_t)(wp * a.wm + wm) * a.ksr * RB * NBX * 4 * kWave + lane;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int b = 0; b < NBX; ++b)
#pragma unroll
                for (int j = 0; j < 4; ++j) red[(((wr * RB + rb) * NBX + b) * 4 + j) * kWave] = acc[rb][b][j];
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int b = 0; b < NBX; ++b)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    if (jj >= J) break;
                    float s = red[((rb * NBX + b) * 4 + j0 + jj) * kWave];
                    for (int k = 1; k < a.ksr; ++k) s += red[(((k * RB + rb) * NBX + b) * 4 + j0 + jj) * kWave];
                    acc[rb][b][jj] = s;
                }
    }

    // acc[rb][b][jj] is channel chan(rb, jj) of pixel (ys[b], xs[b]).
    auto chan = [&](int rb, int jj) { return k0 + (wm * RB + rb) * 16 + 4 * quarter + j0 + jj; };
    // Sums that are not finite are taken again in fp32 (see the file comment), four
    // channels at a time, the lanes then being the wave's pixels.
    uint32_t redo[RB * 4];
    bool any = false;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            uint32_t m = 0;
#pragma unroll
            for (int b = 0; b < NBX; ++b)
                if (!(fabsf(acc[rb][b][jj]) < INFINITY) && ys[b] >= 0) m |= 1u << b;
            redo[rb * 4 + jj] = jj < J && chan(rb, jj) < a.K ? m : 0u;
            any |= redo[rb * 4 + jj] != 0;
        }
    if (__builtin_amdgcn_ballot_w64(any)) {
        const float *img = xp + (size_t)n * a.C * iplane;
        constexpr int P = (NBX * 16 + kWave - 1) / kWave;
        int yi[P], xi[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int pw = i * kWave + lane, q = wp * NBX * 16 + pw;
            const int yl = (int)fast_div((uint32_t)q, a.pt_magic, a.pt_shift), xl = q - yl * a.pitch;
            yi[i] = pw < NBX * 16 && yl < th && xl < tw ? (y0 + yl) * a.stride : -1;
            xi[i] = (x0 + xl) * a.stride;
        }
#pragma unroll 1
        for (int g = 0; g < RB * 4; ++g) {  // channels of row block g >> 2 in quarter g & 3
            uint32_t m[4];
            int j[4], e[4];
            bool some = false;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                m[jj] = 0;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    if (rb == g >> 2 && quarter == (g & 3)) m[jj] = redo[rb * 4 + jj];
                const bool take = __builtin_amdgcn_ballot_w64(m[jj] != 0) != 0;
                const int k = k0 + (wm * RB * 4 + g) * 4 + j0 + jj;
                j[jj] = take ? __builtin_amdgcn_readfirstlane(rowptr[k]) : 0;
                e[jj] = take ? __builtin_amdgcn_readfirstlane(rowptr[k + 1]) : 0;
                some |= take;
            }
            if (!some) continue;
            float s[4][P];
            mat_sums_fp32<P>(a, img, offset, vals, j, e, lane, yi, xi, s);
#pragma unroll
            for (int b = 0; b < NBX; ++b)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const float t = __shfl(s[jj][b * 16 / kWave], b * 16 % kWave + col);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        if (rb == g >> 2 && m[jj] >> b & 1) acc[rb][b][jj] = t;
                }
        }
    }

    // Bias, residual, ReLU; then the stores, or the values to LDS for the pool.
    const bool stream = a.out_pad == 0;
    float *st = lds;
    const int PP = a.wp * NBX * 16;
    if (POOL) __syncthreads();  // the buffers (or the partial tiles) are read
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        float rv[4][NBX];
        if (res) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int b = 0; b < NBX; ++b) {
                    const int k = chan(rb, jj);
                    rv[jj][b] = (jj < J && ys[b] >= 0 && k < a.K)
                                    ? res[((size_t)n * a.K + k) * a.rplane + (size_t)(ys[b] + a.res_pad) * a.rpitch +
                                          xs[b] + a.res_pad]
                                    : 0.0f;
                }
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            if (jj >= J) break;
            const int k = chan(rb, jj);
            const float bk = (bias && k < a.K) ? bias[k] : 0.0f;
#pragma unroll
            for (int b = 0; b < NBX; ++b) {
                float v = acc[rb][b][jj] + bk;
                if (res) v += rv[jj][b];
                if (a.relu) v = v > 0.0f ? v : 0.0f;
                if constexpr (POOL) {
                    st[(k - k0) * PP + (wp * NBX + b) * 16 + col] = v;
                } else {
                    if (ys[b] >= 0 && k < a.K)
                        store_out(out + ((size_t)n * a.K + k) * a.oplane + (size_t)(ys[b] + a.out_pad) * a.opitch +
                                      xs[b] + a.out_pad,
                                  v, stream);
                }
            }
        }
    }
    // Stored rows and columns of the tile.
    const int sy0 = POOL ? y0 / 2 : y0, sx0 = POOL ? x0 / 2 : x0;
    const int sy1 = min(sy0 + (POOL ? a.TH / 2 : a.TH), a.Hq), sx1 = min(sx0 + (POOL ? a.TW / 2 : a.TW), a.Wq);
    if constexpr (POOL) {
        __syncthreads();
        const int pw = a.TW / 2, pq = (a.TH / 2) * pw;
        for (int t = tid; t < a.M * pq; t += kMatThreads) {
            const int kl = (int)fast_div((uint32_t)t, a.pq_magic, a.pq_shift);
            const int rem = t - kl * pq;
            const int r = (int)fast_div((uint32_t)rem, a.pw_magic, a.pw_shift), c = rem - r * pw;
            if (k0 + kl < a.K && sy0 + r < a.Hq && sx0 + c < a.Wq) {
                const float *s0 = st + kl * PP + 2 * r * a.pitch + 2 * c;
                const float m = fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[a.pitch], s0[a.pitch + 1]));
                store_out(out + ((size_t)n * a.K + k0 + kl) * a.oplane + (size_t)(sy0 + r + a.out_pad) * a.opitch + sx0 +
                              c + a.out_pad,
                          m, stream);
            }
        }
    }
    if (a.out_pad) {
        // The tile's rows and columns, reaching over the border at the plane's
        // edges: every element outside the plane is zeroed, by one tile.
        const int ey0 = ty == 0 ? -a.out_pad : sy0, ey1 = ty == a.nty - 1 ? a.Hq + a.out_pad : sy1;
        const int ex0 = tx == 0 ? -a.out_pad : sx0, ex1 = tx == a.ntx - 1 ? a.Wq + a.out_pad : sx1;
        for (int k = k0 + wave; k < min(k0 + a.M, a.K); k += kMatWaves) {
            float *plane = out + ((size_t)n * a.K + k) * a.oplane + a.out_pad * (a.opitch + 1);
            for (int y = ey0; y < ey1; ++y) {
                const bool inside = y >= 0 && y < a.Hq;
                if (inside && ex0 >= 0 && ex1 <= a.Wq) continue;
                for (int x = ex0 + lane; x < ex1; x += kWave)
                    if (!inside || x < 0 || x >= a.Wq) plane[(ptrdiff_t)y * a.opitch + x] = 0.0f;
            }
        }
    }
}

using MatKernel = void (*)(MatArgs, const float *, const int32_t *, const int32_t *, const float *, const float *,
                           const float *, float *);

template <int RB, int NBX>
MatKernel pick_mat_pool(bool pool) {
    return pool ? spconv_matrix_kernel<RB, NBX, true> : spconv_matrix_kernel<RB, NBX, false>;
}

// Wave tiles: row blocks of 16 channels x blocks of 16 pixels.
constexpr int kMatTiles[][2] = {{2, 4}, {1, 7}, {1, 4}, {1, 2}};

MatKernel pick_mat(int RB, int NBX, bool pool) {
    if (RB == 2 && NBX == 4) return pick_mat_pool<2, 4>(pool);
    if (RB == 1 && NBX == 7) return pick_mat_pool<1, 7>(pool);
    if (RB == 1 && NBX == 4) return pick_mat_pool<1, 4>(pool);
    if (RB == 1 && NBX == 2) return pick_mat_pool<1, 2>(pool);
    return nullptr;
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// The tiling of least modelled time. A workgroup's cycles are the longer of its
// MFMAs (20 cycles each for the two waves of a SIMD: the chip holds 2.05 of the
// nominal 2.5 PFLOP/s on them) and its LDS reads, plus the staging between them
// (80 instructions per 64 input tasks, 45 per 64 filter entries, the clearing),
// 1500 cycles per chunk and 12000 per workgroup (its first loads and its
// epilogue); one workgroup per CU (its registers allow no second). Over
// 20 tilings of five layers (14x14, 28x28 pooled, 56x56, 56x56 of stride 2,
// 224x224) a million modelled cycles take 520 to 560 us, and the pick is each
// layer's fastest.
bool search_plan(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, bool pool, long long nnz,
                 MatrixPlan *out) {
    const long long plane = (H + 2LL * pad) * (W + 2LL * pad);
    // 24-bit products and reciprocals of two or more in the entries' decoding.
    if (plane >= (1 << 24) || C >= (1 << 24) || W + 2LL * pad < 2) return false;
    const int Hp = H + 2 * pad, Wp = W + 2 * pad;
    const int Ho = (Hp - R) / stride + 1, Wo = (Wp - S) / stride + 1;
    // One output row (column) reads the window of one position, however far the
    // next would be: a stride past the plane would be a window pitch past any LDS.
    const int sy = Ho > 1 ? stride : 1, sx = Wo > 1 ? stride : 1;
    const int taps = R * S;
    const int noct = ceil_div(C, 8);
    const double per_row_chan = (double)nnz / K / C;  // entries per (row, channel)
    MatrixPlan best;
    double best_time = -1.0;
    for (const auto &wt : kMatTiles)
        for (int wm : {1, 2, 4, 8})
            for (int ksr : {1, 2, 4}) {
                const int RB = wt[0], NBX = wt[1];
                if (wm * ksr > kMatWaves) continue;
                const int wp = kMatWaves / (wm * ksr);
                const int M = 16 * RB * wm, P = 16 * NBX * wp;
                if (M > 16 && M / 2 >= K) continue;  // half the channels would do
                const size_t epi = std::max(pool ? (size_t)M * P * 4 : 0,
                                            ksr > 1 ? (size_t)kMatWaves * RB * NBX * 4 * kWave * 4 : 0);
                if (epi > (size_t)kMatLdsBytes) continue;
                // Tile widths: even shares of the row, from the widest that fits.
                const int nx0 = ceil_div(Wo, P);
                for (int ntx = nx0; ntx < nx0 + 16; ++ntx) {
                    int TW = ceil_div(Wo, ntx);
                    if (pool && (TW & 1)) ++TW;
                    if (ntx > nx0 && TW < 4) break;
                    // Lane rows of whole 8-pixel groups where the tile is wide enough
                    // for that to cost little: 8 lanes' LDS reads then never cross a row.
                    const int pitch = TW > 8 ? ceil_div(TW, 8) * 8 : TW;
                    if (pitch > P) continue;
                    int th_max = std::min(P / pitch, pool ? (Ho + 1) / 2 * 2 : Ho);
                    if (pool) th_max &= ~1;
                    if (th_max < 1) continue;
                    const int nty = ceil_div(Ho, th_max);
                    int TH = ceil_div(Ho, nty);
                    if (pool && (TH & 1)) ++TH;
                    const int nx = ceil_div(Wo, TW), ny = ceil_div(Ho, TH);
                    const int stepy = R == 1 ? sy : 1, stepx = S == 1 ? sx : 1;
                    const int lsy = R == 1 ? 1 : sy, lsx = S == 1 ? 1 : sx;
                    const int rows = (TH - 1) * lsy + R, hw = ceil_div((TW - 1) * lsx + S, lsx), vp = lsx * hw;
                    const int PX = rows * vp;
                    for (int O : {16, 8, 4, 2, 1}) {
                        if (O > 1 && O / 2 >= noct) continue;
                        const int nunits = ceil_div(O * taps, 4);
                        const long long a_bytes = (long long)(M / 16) * nunits * kMatFrag;
                        const long long b_bytes = ((long long)O * PX * kMatPx + 15) / 16 * 16;
                        const long long tab = 16LL * nunits;
                        const int nchunks = ceil_div(noct, O);
                        if (a_bytes + b_bytes + tab > kMatLdsBytes) continue;
                        const int bufs = nchunks > 1 && 2 * (a_bytes + b_bytes) + tab <= kMatLdsBytes ? 2 : 1;
                        if ((long long)O * 8 * Hp * Wp * 4 >= (1LL << 31)) continue;
                        const long long wgs = (long long)N * nx * ny * ceil_div(K, M);
                        // A launch counts its threads in 32 bits (the other kernels hold
                        // several small images in a workgroup, and so reach further).
                        if (wgs * kMatThreads >= (1LL << 32)) continue;
                        const size_t lds = std::max((size_t)(bufs * (a_bytes + b_bytes) + tab), epi);
                        const double units = (double)nchunks * nunits / ksr;
                        const double mfma = 2.0 * units * RB * NBX * 6 * 20;
                        const double ldsr = kMatWaves * units * (RB + NBX) * 3072.0 / 200.0;
                        const double stage = nchunks * ((double)O * PX / 64.0 * 80 +
                                                        (double)M * (1.0 + std::max(1.0, per_row_chan * O * 8 / 64)) * 45 +
                                                        (double)M * nunits * 12 / 64 * 12);
                        const double bar = nchunks * 1500.0;
                        const double wg = std::max(mfma, ldsr) + (bufs == 2 ? 0.6 : 1.0) * stage + bar + 12000.0;
                        const double time = (double)((wgs + 255) / 256) * wg;
                        if (best_time < 0 || time < best_time) {
                            best_time = time;
                            best = MatrixPlan{};
                            best.RB = RB; best.NBX = NBX; best.wm = wm; best.wp = wp; best.ksr = ksr; best.M = M;
                            best.O = O; best.nchunks = nchunks; best.nunits = nunits; best.TH = TH; best.TW = TW;
                            best.nty = ny; best.ntx = nx; best.rows = rows; best.vp = vp; best.PX = PX;
                            best.stepy = stepy; best.stepx = stepx; best.lsy = lsy; best.lsx = lsx; best.hw = hw; best.pitch = pitch;
                            best.bufs = bufs; best.a_bytes = (int)a_bytes; best.b_bytes = (int)b_bytes;
                            best.nkt = ceil_div(K, M); best.total_wgs = (int)wgs; best.lds_bytes = lds;
                            best.time = time;
                        }
                    }
                }
            }
    if (best_time < 0) return false;
    *out = best;
    return true;
}

// Choices of recent calls: whether a call runs here, and on which plan. They are
// functions of its shapes and entry count alone, and finding one takes the host
// some thousand tilings (11 to 34 us, as much as a launch), while a program calls
// the same layers again and again. 128 sets of eight, the least recently used one
// of a set replaced: a network's layers at a few batch sizes stay (a table of 64
// single slots lost half of ten layers to each other).
struct ChoiceKey {
    int v[10];
    long long nnz;
    bool operator==(const ChoiceKey &o) const { return std::equal(v, v + 10, o.v) && nnz == o.nnz; }
};

struct Choice {
    ChoiceKey key{};
    MatrixPlan plan;
    bool use = false;
    uint64_t used = 0;  // turn of the last use, 0: empty
};

constexpr int kChoiceSets = 128, kChoiceWays = 8;
std::mutex choice_mutex;
Choice choices[kChoiceSets][kChoiceWays];
uint64_t choice_turn = 0;

ChoiceKey choice_key(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, bool pool, long long nnz) {
    return {{N, C, H, W, K, R, S, stride, pad, pool ? 1 : 0}, nnz};
}

Choice *choice_set(const ChoiceKey &key) {
    uint64_t h = (uint64_t)key.nnz;
    for (int v : key.v) h = (h ^ (uint64_t)(uint32_t)v) * 0x9e3779b97f4a7c15ull;
    return choices[(h >> 40) % kChoiceSets];
}

}  // namespace

__attribute__((visibility("hidden"))) bool matrix_plan(int N, int C, int H, int W, int K, int R, int S, int stride,
                                                       int pad, bool pool, long long nnz, MatrixPlan *out) {
    return search_plan(N, C, H, W, K, R, S, stride, pad, pool, nnz, out);
}

__attribute__((visibility("hidden"))) bool matrix_recall(int N, int C, int H, int W, int K, int R, int S, int stride,
                                                         int pad, bool pool, long long nnz, MatrixPlan *plan, bool *use) {
    const ChoiceKey key = choice_key(N, C, H, W, K, R, S, stride, pad, pool, nnz);
    Choice *set = choice_set(key);
    std::lock_guard<std::mutex> lock(choice_mutex);
    for (int i = 0; i < kChoiceWays; ++i)
        if (set[i].used && set[i].key == key) {
            set[i].used = ++choice_turn;
            *plan = set[i].plan;
            *use = set[i].use;
            return true;
        }
    return false;
}

__attribute__((visibility("hidden"))) void matrix_remember(int N, int C, int H, int W, int K, int R, int S, int stride,
                                                           int pad, bool pool, long long nnz, const MatrixPlan &plan,
                                                           bool use) {
    const ChoiceKey key = choice_key(N, C, H, W, K, R, S, stride, pad, pool, nnz);
    Choice *set = choice_set(key);
    std::lock_guard<std::mutex> lock(choice_mutex);
    Choice *slot = set;
    for (int i = 0; i < kChoiceWays; ++i) {
        if (set[i].used && set[i].key == key) {  // (another thread was first)
            slot = set + i;
            break;
        }
        if (set[i].used < slot->used) slot = set + i;
    }
    slot->key = key;
    slot->plan = plan;
    slot->use = use;
    slot->used = ++choice_turn;
}

__attribute__((visibility("hidden"))) void matrix_variants(int32_t *variants, int32_t capacity, int32_t *count) {
    int n = 0;
    for (const auto &t : kMatTiles)
        for (int pool = 0; pool < 2; ++pool, ++n)
            if (n < capacity) {
                variants[4 * n] = t[1];
                variants[4 * n + 1] = 0;
                variants[4 * n + 2] = 16 * t[0];
                variants[4 * n + 3] = pool;
            }
    *count = n;
}

__attribute__((visibility("hidden"))) int matrix_launch(const MatrixPlan &pl, const MatrixCall &c, const float *in,
                                                        const int32_t *rowptr, const int32_t *offset,
                                                        const float *vals, const float *bias, const float *res,
                                                        float *out, hipStream_t stream) {
    MatArgs a;
    a.N = c.N; a.C = c.C; a.K = c.K; a.R = c.R; a.S = c.S; a.stride = c.stride;
    a.Wp = c.W + 2 * c.pad;
    a.plane = (c.H + 2 * c.pad) * a.Wp;
    a.IH = c.unpadded ? c.H : c.H + 2 * c.pad;
    a.IW = c.unpadded ? c.W : a.Wp;
    a.ipad = c.unpadded ? c.pad : 0;
    a.Ho = c.Ho; a.Wo = c.Wo;
    a.Hq = c.pool ? c.Ho / 2 : c.Ho;
    a.Wq = c.pool ? c.Wo / 2 : c.Wo;
    a.relu = c.relu;
    a.TH = pl.TH; a.TW = pl.TW; a.nty = pl.nty; a.ntx = pl.ntx;
    a.nkt = pl.nkt; a.M = pl.M; a.wm = pl.wm; a.wp = pl.wp; a.ksr = pl.ksr;
    a.O = pl.O; a.oshift = __builtin_ctz(pl.O); a.nchunks = pl.nchunks; a.nunits = pl.nunits;
    a.rows = pl.rows; a.vp = pl.vp; a.PX = pl.PX;
    a.stepy = pl.stepy; a.stepx = pl.stepx; a.lsy = pl.lsy; a.lsx = pl.lsx; a.hw = pl.hw; a.pitch = pl.pitch;
    a.tasks = pl.O * pl.PX;
    a.a_bytes = pl.a_bytes; a.b_bytes = pl.b_bytes; a.bufs = pl.bufs;
    a.total_wgs = pl.total_wgs;
    a.out_pad = c.out_pad; a.opitch = c.opitch; a.oplane = c.oplane;
    a.res_pad = c.res_pad; a.rpitch = c.rpitch; a.rplane = c.rplane;
    a.pw_magic = a.pq_magic = 1;
    a.pw_shift = a.pq_shift = 0;
    if (!div_magic((uint32_t)a.PX, &a.px_magic, &a.px_shift) || !div_magic((uint32_t)a.vp, &a.vp_magic, &a.vp_shift) ||
        !div_magic((uint32_t)a.pitch, &a.pt_magic, &a.pt_shift) ||
        !div_magic((uint32_t)a.plane, &a.plane_magic, &a.plane_shift) ||
        !div_magic((uint32_t)a.Wp, &a.wp_magic, &a.wp_shift) ||
        (c.pool && (!div_magic((uint32_t)(a.TW / 2), &a.pw_magic, &a.pw_shift) ||
                    !div_magic((uint32_t)((a.TH / 2) * (a.TW / 2)), &a.pq_magic, &a.pq_shift))))
        return SPCONV_EINVAL;
    const MatKernel kern = pick_mat(pl.RB, pl.NBX, c.pool);
    if (!kern) return SPCONV_EINVAL;
    if (!raise_lds_limit((const void *)kern, kMatLdsBytes)) return SPCONV_EHIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)pl.total_wgs), dim3(kMatThreads), pl.lds_bytes, stream, a, in, rowptr, offset,
                       vals, bias, res, out);
    return hipGetLastError() == hipSuccess ? SPCONV_OK : SPCONV_EHIP;
}
