// Activation predictor (PowerInfer Sec. 5.1: input layer, one hidden layer, output layer)
// and active-index compaction.
//   hidden : t[b][m]     = ReLU(p1[m] . x[b])                          r rows of d fp16
//   output : logit[b][i] = p2[i] . t[b] + p_bias[i]                     ffn rows of r fp16
//            bit i of the mask = any_b(logit[b][i] > logit(threshold))  (wave ballot)
//   compact: idx[] = ascending positions of the set bits, count = popcount
// Both GEMVs are HBM-bound streams of fp16 rows, 16-byte loads per lane, fp32 accumulation.  Two forms:
// batch 1 .. 3 holds the activations by column in registers (hidden_cols_body, pred_out_cols_body); rows longer
// than that covers, and batches of 4 to 8 below the matrix cores' line, take one wave per row with the
// activations staged once per workgroup in LDS and a DPP reduction (pred_hidden_body, pred_out_body).
// No kernel here uses device-scope fences: data crosses workgroups only at kernel ends.
#pragma once
#include "dev_util.h"

namespace pf {

constexpr int kPredThreads = 256;  // 4 waves per workgroup
constexpr int kGlueMaxParts = 4;   // FC2 may hand its output over as up to 4 partial sums
constexpr int kPredWaves = kPredThreads / kWave;

// ---------------------------------------------------------------------------------------
// One pass of the stack glue inside a consumer kernel: S strides of NT * 4 elements of
// v = sign * (x_prev + sum of FC2's partial sums), for B tokens.  glue_issue puts the loads in
// flight (x and up to kGlueMaxParts partial sums per element, partials added in the fixed
// order 0 .. ny-1), glue_commit adds them up, accumulates ||v||^2 per token into ss and
// stores v in the staged-activation layout of dev_util.h (scrap slot for strides past the
// vector).  The caller reduces ss over the block and applies sqrt(d / ss) to its dot products.
template <int B, int S>
struct GluePass {
    float4 va[S][B], vc[S][B], vp[S][B][kGlueMaxParts - 1];
};

template <int B, int S, int NT>
__device__ __forceinline__ void glue_issue(GluePass<B, S> &gp, rsrc_t xr, rsrc_t yr, uint32_t pbytes,
                                           int ny, int d, int e0)
{
    constexpr int step = NT * 4;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int e = e0 + s * step;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const uint32_t off = e < d ? (uint32_t)(b * d + e) * 4u : kOobOffset;
            gp.va[s][b] = ld16_f32(xr, off);
            gp.vc[s][b] = ld16_f32(yr, off);
#pragma unroll
            for (int p = 1; p < kGlueMaxParts; ++p)  // partial sums of FC2, in order
                gp.vp[s][b][p - 1] = ld16_f32(yr, (e < d && p < ny) ? off + (uint32_t)p * pbytes : kOobOffset);
        }
    }
}

template <int B, int S, int NT>
__device__ __forceinline__ void glue_commit(const GluePass<B, S> &gp, float *__restrict__ xs, int kpad,
                                            int b0, int e0, float (&ss)[B])
{
    constexpr int step = NT * 4;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int e = e0 + s * step;
#pragma unroll
        for (int b = 0; b < B; ++b) {  // strides past the vector hold zeros: scrap slot
            const float4 a = gp.va[s][b];
            float4 c = gp.vc[s][b];
#pragma unroll
            for (int p = 1; p < kGlueMaxParts; ++p) {
                const float4 q = gp.vp[s][b][p - 1];
                c = make_float4(c.x + q.x, c.y + q.y, c.z + q.z, c.w + q.w);
            }
            const float4 v = glue_signed(make_float4(a.x + c.x, a.y + c.y, a.z + c.z, a.w + c.w),
                                         (uint32_t)b0 + (uint32_t)b, (uint32_t)e);
            ss[b] = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, ss[b]))));
            *reinterpret_cast<float4 *>(xs + (e < kpad ? b * kpad + lds_slot(e) : B * kpad)) = v;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Hidden layer.  grid = ceil(r / 4); wave w of block g owns row 4g + w.
// With GLUE the input of the layer is formed on the fly from the previous layer's input and
// FFN output, x = (xp + yp) * sqrt(d) / ||xp + yp||_2 per token (the stack's residual +
// scale-only RMS norm): every block stages v = xp + yp, reduces ||v||^2 itself and applies
// the scale to its dot products; block 0 also writes x for the kernels that follow.
// yp may arrive as ny <= 4 partial sums, ypstride floats apart (row-split FC2): they are
// added in the fixed order 0 .. ny-1.  b0 = batch row of the first token this launch handles
// (the glue's sign pattern depends on the row).
// GS = strides of 1024 elements whose glue loads (x and up to 4 partial sums each) a thread
// issues together: 4 covers d <= 4096 in a single round trip, at 80 registers.
// The body takes the block's number explicitly (bid) so that a launch can run it in a range of
// its blocks beside another role; write_x: this block also writes x for the kernels that follow.
// NT = threads of the launch (a block owns NT / 64 rows).
template <int B, bool GLUE, int GS, int NT = kPredThreads>
__device__ __forceinline__ void pred_hidden_body(float *xs, float (*ss_w)[B], const int bid, const bool write_x,
                                                 const __half *__restrict__ p1,
                                                 const float *__restrict__ x,
                                                 const float *__restrict__ yp, int ny,
                                                 int ypstride, float *__restrict__ x_new,
                                                 float *__restrict__ t, int d, int r, int b0)
{
    constexpr int U = 8;
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    const int nch = (d + kChunk - 1) / kChunk, kpad = nch * kChunk;
    const int m = bid * (NT / kWave) + wave;
    const bool live = m < r;
    const rsrc_t row = row_rsrc(p1, live ? m : 0, d, live);

    PF_TSTAMP(0, 0);
    if (!GLUE) stage_dma<B>(xs, x, d, kpad);
    WGroup<U> g;
    float scale[B];
    if (GLUE) {
        float ss[B];
#pragma unroll
        for (int b = 0; b < B; ++b) ss[b] = 0.f;
        constexpr int S = GS;  // strides whose loads are issued together
        constexpr int step = NT * 4;
        bool issued = false;
        const rsrc_t xr = make_rsrc(x, (uint32_t)B * (uint32_t)d * 4u);
        const uint32_t pbytes = (uint32_t)ypstride * 4u;  // distance between partials
        const rsrc_t yr = make_rsrc(yp, (uint32_t)(ny - 1) * pbytes + (uint32_t)B * (uint32_t)d * 4u);
        for (int e0 = threadIdx.x * 4; e0 < kpad; e0 += step * S) {
            GluePass<B, S> gp;
            glue_issue<B, S, NT>(gp, xr, yr, pbytes, ny, d, e0);
            // the row's own loads queue up behind the first pass of activations
            if (!issued) {
                load_group<U>(g, row, 0, lane);
                issued = true;
            }
            glue_commit<B, S, NT>(gp, xs, kpad, b0, e0, ss);
        }
        if (!issued) load_group<U>(g, row, 0, lane);  // threads past a short vector
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float s = wave_sum(ss[b]);
            if (lane == 0) ss_w[wave][b] = s;
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B; ++b) {
            float tot = 0.f;
#pragma unroll
            for (int k = 0; k < NT / kWave; ++k) tot += ss_w[k][b];
            scale[b] = tot > 0.f ? sqrtf((float)d / tot) : 0.f;
        }
        if (write_x) {
            for (int e = threadIdx.x * 4; e < d; e += NT * 4) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const float4 v = *reinterpret_cast<const float4 *>(xs + b * kpad + lds_slot(e));
                    *reinterpret_cast<float4 *>(x_new + (size_t)b * d + e) =
                        make_float4(v.x * scale[b], v.y * scale[b], v.z * scale[b], v.w * scale[b]);
                }
            }
        }
    } else {
        load_group<U>(g, row, 0, lane);
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B; ++b) scale[b] = 1.f;
    }

    PF_TSTAMP(0, 1);
    float acc[B];
#pragma unroll
    for (int b = 0; b < B; ++b) acc[b] = 0.f;
    fma_group<B, U>(g, xs, kpad, 0, nch, lane, acc);
    for (int it0 = U; it0 < nch; it0 += U) {
        load_group<U>(g, row, it0, lane);
        fma_group<B, U>(g, xs, kpad, it0, nch, lane, acc);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const float s = wave_sum(acc[b]) * scale[b];
        if (live && lane == 0) t[(size_t)b * r + m] = fmaxf(s, 0.f);
    }
    PF_TSTAMP(0, 2);
}

template <int B, bool GLUE, int GS = (B >= 2 ? 1 : 2)>
__global__ __launch_bounds__(kPredThreads) void k_pred_hidden(const __half *__restrict__ p1,
                                                              const float *__restrict__ x,
                                                              const float *__restrict__ yp, int ny,
                                                              int ypstride,
                                                              float *__restrict__ x_new,
                                                              float *__restrict__ t, int d, int r,
                                                              int b0, const int32_t *__restrict__ skip)
{
    extern __shared__ float xs[];
    __shared__ float ss_w[kPredWaves][B];
    // adaptive layer step: a set flag means this step runs dense and needs no prediction
    if (skip != nullptr && *skip != 0) return;
    pred_hidden_body<B, GLUE, GS>(xs, ss_w, (int)blockIdx.x, blockIdx.x == 0, p1, x, yp, ny, ypstride,
                                  x_new, t, d, r, b0);
}

// ---------------------------------------------------------------------------------------
// Activations held by column: the waves of a workgroup split a row's columns between them -- wave w takes
// the chunks w, w + W, ... of 512 -- and a lane multiplies the same 8 columns of every row, so that it keeps
// its activations in registers and all rows of the workgroup are in flight at once, whatever their
// length.  (One wave per row wants the whole vector in LDS: a barrier in front of the first sum, twice
// the weights' bytes per token through LDS, and loads past the row's end where its length is no
// multiple of the wave's share.)  The waves' sums of a row meet in LDS once at the end.
constexpr int kColsMaxWaves = 8;

// Waves of a workgroup for rows of K elements, and chunks per wave that cover the row in one pass.
inline int cols_waves(int K)
{
    const int nch = (K + kChunk - 1) / kChunk, cpw = (nch + kColsMaxWaves - 1) / kColsMaxWaves;
    return (nch + cpw - 1) / cpw;
}
inline int cols_per_wave(int K)
{
    const int nch = (K + kChunk - 1) / kChunk;
    return (nch + kColsMaxWaves - 1) / kColsMaxWaves;
}

template <int B>
struct ColX {
    float4 lo[B], hi[B];  // 8 columns of every token
};

// fp32 vectors are read 16 bytes a lane in one run -- lane l the elements 4 l .. 4 l + 3 of each half of a
// chunk (a lane's own 32 bytes would cost twice the line look-ups) -- and handed to the lanes whose
// columns they are through 2 KB of LDS per wave, without a barrier.
constexpr int kColsXFloats = kChunk;

__device__ __forceinline__ void cols_exchange(float *xw, float4 &lo, float4 &hi, int lane)
{
    float4 *to = reinterpret_cast<float4 *>(xw);
    to[lane] = lo;
    to[64 + lane] = hi;
    __builtin_amdgcn_wave_barrier();
    lo = to[2 * lane];
    hi = to[2 * lane + 1];
    __builtin_amdgcn_wave_barrier();
}

// Elements e .. e + 3 and e + 256 .. e + 259 of x[B][d] (zeros from d on), e = 512 chunk + 4 lane.
template <int B>
__device__ __forceinline__ void colx_load(ColX<B> &v, rsrc_t xr, int e, int d)
{
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const uint32_t off = (uint32_t)(b * d + e) * 4u;
        v.lo[b] = ld16_f32(xr, e < d ? off : kOobOffset);
        v.hi[b] = ld16_f32(xr, e + 256 < d ? off + 1024u : kOobOffset);
    }
}

// The same of the stack glue's sum x + (y_0 + y_1 + ..) with its signs, not yet normalised: NY partial
// sums, pbytes apart.  issue puts the loads in flight, commit adds up and leaves ||v||^2 in ss.
template <int B, int NY>
struct ColGlue {
    float4 lo[B][NY + 1], hi[B][NY + 1];
    uint32_t slo[B], shi[B];
};

// Tokens T0 .. T0 + N - 1.
template <int N, int NY, int T0 = 0>
__device__ __forceinline__ void colglue_issue(ColGlue<N, NY> &g, rsrc_t xr, rsrc_t yr, rsrc_t sr, uint32_t sstride,
                                              uint32_t pbytes, int e, int d)
{
    const bool ok = e < d, ok2 = e + 256 < d;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int b = T0 + i;
        const uint32_t off = (uint32_t)(b * d + e) * 4u, soff = (uint32_t)b * sstride + ((uint32_t)e >> 3);
        g.lo[i][NY] = ld16_f32(xr, ok ? off : kOobOffset);
        g.hi[i][NY] = ld16_f32(xr, ok2 ? off + 1024u : kOobOffset);
#pragma unroll
        for (int p = 0; p < NY; ++p) {
            g.lo[i][p] = ld16_f32(yr, ok ? off + (uint32_t)p * pbytes : kOobOffset);
            g.hi[i][p] = ld16_f32(yr, ok2 ? off + (uint32_t)p * pbytes + 1024u : kOobOffset);
        }
        if (b > 0) {  // row 0 keeps its signs
            g.slo[i] = __builtin_amdgcn_raw_buffer_load_b8(sr, (int)(ok ? soff : kOobOffset), 0, 0);
            g.shi[i] = __builtin_amdgcn_raw_buffer_load_b8(sr, (int)(ok2 ? soff + 32u : kOobOffset), 0, 0);
        }
    }
}

__device__ __forceinline__ float4 with_signs(const float4 &v, uint32_t bits)
{
    auto one = [&](float a, int e) {
        return __uint_as_float(__float_as_uint(a) ^ ((bits << (31 - e)) & 0x80000000u));
    };
    return make_float4(one(v.x, 0), one(v.y, 1), one(v.z, 2), one(v.w, 3));
}

template <int B, int N, int NY, int T0 = 0>
__device__ __forceinline__ void colglue_commit(const ColGlue<N, NY> &g, ColX<B> &v, float *ss, int lane)
{
    auto sum4 = [&](const float4 (&q)[NY + 1]) {
        float4 c = q[0];
#pragma unroll
        for (int p = 1; p < NY; ++p) c = make_float4(c.x + q[p].x, c.y + q[p].y, c.z + q[p].z, c.w + q[p].w);
        return make_float4(q[NY].x + c.x, q[NY].y + c.y, q[NY].z + c.z, q[NY].w + c.w);
    };
    const int sh = (lane & 1) * 4;  // e & 4
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int b = T0 + i;
        float4 a = sum4(g.lo[i]), c = sum4(g.hi[i]);
        if (b > 0) {
            a = with_signs(a, g.slo[i] >> sh);
            c = with_signs(c, g.shi[i] >> sh);
        }
        ss[b] = fmaf(a.x, a.x, fmaf(a.y, a.y, fmaf(a.z, a.z, fmaf(a.w, a.w, ss[b]))));
        ss[b] = fmaf(c.x, c.x, fmaf(c.y, c.y, fmaf(c.z, c.z, fmaf(c.w, c.w, ss[b]))));
        v.lo[b] = a;
        v.hi[b] = c;
    }
}

// One chunk's glue for all tokens, N of them at a time (the rest of B last).
template <int B, int NY, int N, int T0 = 0>
__device__ __forceinline__ void colglue_chunk(ColX<B> &v, float *ss, rsrc_t xr, rsrc_t yr, rsrc_t sr, uint32_t sstride,
                                              uint32_t pbytes, int e, int d, int lane)
{
    if constexpr (T0 < B) {
        constexpr int M = B - T0 < N ? B - T0 : N;
        ColGlue<M, NY> g;
        colglue_issue<M, NY, T0>(g, xr, yr, sr, sstride, pbytes, e, d);
        colglue_commit<B, M, NY, T0>(g, v, ss, lane);
        __builtin_amdgcn_sched_barrier(0);
        colglue_chunk<B, NY, N, T0 + M>(v, ss, xr, yr, sr, sstride, pbytes, e, d, lane);
    }
}

// The glue's inputs of a launch.
struct GlueIn {
    const float *x, *yp;
    const uint8_t *sign;  // [kSignRows][sstride]
    int ny, ypstride, sstride;
};

// ---------------------------------------------------------------------------------------
// Hidden layer.  grid = ceil(r / R), block = 64 * cols_waves(d).  Block g owns the rows R g .. R g + R - 1.
// With GLUE the input of the layer is formed on the fly from the previous layer's input and
// FFN output, x = (xp + yp) * sqrt(d) / ||xp + yp||_2 per token (the stack's residual +
// scale-only RMS norm): a lane forms v = xp + yp for its columns, ||v||^2 is summed with the rows' sums
// and the norm applied to them; the block with write_x set also writes x for the kernels that follow.
// yp may arrive as ny <= 4 partial sums, ypstride floats apart (row-split FC2): they are
// added in the fixed order 0 .. ny-1.
// The body takes the block's number explicitly (bid) so that a launch can run it in a range of
// its blocks beside another role.  red = [waves][cols_red_floats(R * B + B)] floats of LDS, xw = this wave's
// kColsXFloats.
// Bound by the glue's bytes through each workgroup's memory path and one trip to memory.  One wave per row
// with x staged in LDS -> this, us (glue included): d 5120, r 1024 batch 1 6.7 -> 5.3; d 7168, r 1536 9.0 ->
// 7.5; d 12288, r 2048 15.0 -> 12.5; d 768, r 128 batch 2 3.8 -> 3.5; d 4096, r 1024
// batch 3 8.5 -> 7.6, batch 1 4.2 -> 4.4 (the one shape behind; the stack is 2 % faster all the same).  With a loop
// around the one pass these two were 4.4 and 4.6.
__host__ __device__ constexpr int cols_red_floats(int n) { return (n + 3) / 4 * 4; }

// Sum of one value of the W <= MAX waves, `pitch` floats apart: all reads in flight at once.
template <int MAX = kColsMaxWaves>
__device__ __forceinline__ float cols_total(const float *p, int pitch, int W)
{
    float s[MAX];
#pragma unroll
    for (int k = 0; k < MAX; ++k) s[k] = p[min(k, W - 1) * pitch];
    float a = s[0];
#pragma unroll
    for (int k = 1; k < MAX; ++k) a += k < W ? s[k] : 0.f;
    return a;
}

// SEQ: the glue chunk by chunk and GT tokens at a time, for fewer registers.  ONE: d <= 512 CPW waves, one pass.
template <int B, bool GLUE, int CPW, int R, bool SEQ = (CPW * B > 3), int GT = B, bool ONE = false>
__device__ __forceinline__ void hidden_cols_body(float *red, float *xw, const int bid, const bool write_x,
                                                 const __half *__restrict__ p1, const float *__restrict__ x,
                                                 const GlueIn gi, float *__restrict__ x_new,
                                                 float *__restrict__ t, int d, int r)
{
    constexpr int N = R * B + (GLUE ? B : 0), NP = cols_red_floats(N);
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6), W = (int)(blockDim.x >> 6);
    const int nch = (d + kChunk - 1) / kChunk;
    const int m0 = bid * R, nrows = min(R, r - m0);
    const rsrc_t rows = make_rsrc(p1 + (size_t)m0 * d, (uint32_t)nrows * (uint32_t)d * 2u);
    const uint32_t pbytes = GLUE ? (uint32_t)gi.ypstride * 4u : 0u;
    const rsrc_t xr = make_rsrc(GLUE ? gi.x : x, (uint32_t)B * (uint32_t)d * 4u);
    const rsrc_t yr = make_rsrc(gi.yp, GLUE ? (uint32_t)(gi.ny - 1) * pbytes + (uint32_t)B * (uint32_t)d * 4u : 0u);
    const rsrc_t sr = make_rsrc(gi.sign, GLUE ? (uint32_t)kSignRows * (uint32_t)gi.sstride : 0u);

    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
    ColX<B> v[CPW];
    const int step = W * CPW;  // chunks of a pass; one pass up to d = 4096 CPW
    for (int c0 = 0; c0 < nch; c0 += step) {
        int col[CPW], e0[CPW];
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            col[c] = (c0 + c * W + wave) * kChunk + lane * 8;
            e0[c] = (c0 + c * W + wave) * kChunk + lane * 4;
        }
        uint4 w[CPW][R];
        auto load_rows = [&]() {
#pragma unroll
            for (int c = 0; c < CPW; ++c)
#pragma unroll
                for (int q = 0; q < R; ++q)
                    w[c][q] = ld16_stream(rows, col[c] < d ? (uint32_t)(q * d + col[c]) * 2u : kOobOffset);
        };
        if constexpr (GLUE) {
            // a copy of this piece per number of partial sums: a load whose lanes are all past the end costs
            // the address unit as much as any
            auto piece = [&](auto nyc) {
                constexpr int NY = decltype(nyc)::value;
                if constexpr (!SEQ) {
                    ColGlue<B, NY> g[CPW];
#pragma unroll
                    for (int c = 0; c < CPW; ++c)
                        colglue_issue<B, NY>(g[c], xr, yr, sr, (uint32_t)gi.sstride, pbytes, e0[c], d);
                    load_rows();  // queue up behind the activations
#pragma unroll
                    for (int c = 0; c < CPW; ++c) colglue_commit(g[c], v[c], acc + R * B, lane);
                } else {  // not enough registers for all of them at once
                    load_rows();
#pragma unroll
                    for (int c = 0; c < CPW; ++c)
                        colglue_chunk<B, NY, GT>(v[c], acc + R * B, xr, yr, sr, (uint32_t)gi.sstride, pbytes, e0[c], d, lane);
                }
            };
            if (gi.ny == 4) piece(IntC<4>());
            else if (gi.ny == 3) piece(IntC<3>());
            else if (gi.ny == 2) piece(IntC<2>());
            else piece(IntC<1>());
#pragma unroll
            for (int c = 0; c < CPW; ++c)
#pragma unroll
                for (int b = 0; b < B; ++b) cols_exchange(xw, v[c].lo[b], v[c].hi[b], lane);
            if (!ONE && write_x && nch > step) {  // scaled in place below
#pragma unroll
                for (int c = 0; c < CPW; ++c)
                    if (col[c] < d)
#pragma unroll
                        for (int b = 0; b < B; ++b) {
                            *reinterpret_cast<float4 *>(x_new + (size_t)b * d + col[c]) = v[c].lo[b];
                            *reinterpret_cast<float4 *>(x_new + (size_t)b * d + col[c] + 4) = v[c].hi[b];
                        }
            }
        } else {
#pragma unroll
            for (int c = 0; c < CPW; ++c) colx_load<B>(v[c], xr, e0[c], d);
            load_rows();
#pragma unroll
            for (int c = 0; c < CPW; ++c)
#pragma unroll
                for (int b = 0; b < B; ++b) cols_exchange(xw, v[c].lo[b], v[c].hi[b], lane);
        }
#pragma unroll
        for (int c = 0; c < CPW; ++c)
#pragma unroll
            for (int q = 0; q < R; ++q)
#pragma unroll
                for (int b = 0; b < B; ++b)
                    acc[q * B + b] = dot8(w[c][q], v[c].lo[b], v[c].hi[b], acc[q * B + b]);
        if (ONE) break;
    }
    float s[NP / 4];
    wave_sums<N>(acc, s);
    if ((lane & 15) == 0) {
#pragma unroll
        for (int i = 0; i < NP / 4; ++i) red[wave * NP + 4 * i + wave_sums_value(lane >> 4)] = s[i];
    }
    __syncthreads();
    auto scale_of = [&](int b) {
        const float ss = cols_total(red + R * B + b, NP, W);
        return ss > 0.f ? sqrtf((float)d / ss) : 0.f;
    };
    if ((int)threadIdx.x < R * B) {
        const int q = (int)threadIdx.x % R, b = (int)threadIdx.x / R;
        float a = cols_total(red + q * B + b, NP, W);
        if (GLUE) a *= scale_of(b);
        if (q < nrows) t[(size_t)b * r + m0 + q] = fmaxf(a, 0.f);
    }
    if (GLUE && write_x) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float sc = scale_of(b);
            for (int c0 = 0; c0 < (ONE ? 1 : nch); c0 += step)
#pragma unroll
                for (int c = 0; c < CPW; ++c) {
                    const int col = ((c0 + c * W + wave) * 64 + lane) * 8;
                    if (col >= d) continue;
                    float4 *to = reinterpret_cast<float4 *>(x_new + (size_t)b * d + col);
                    const bool again = !ONE && nch > step;
                    const float4 a = again ? to[0] : v[c].lo[b], e = again ? to[1] : v[c].hi[b];
                    to[0] = make_float4(a.x * sc, a.y * sc, a.z * sc, a.w * sc);
                    to[1] = make_float4(e.x * sc, e.y * sc, e.z * sc, e.w * sc);
                }
        }
    }
}

template <int B, bool GLUE, int CPW, int R>
__global__ __launch_bounds__(64 * kColsMaxWaves) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_hidden_cols(
    const __half *__restrict__ p1, const float *__restrict__ x, GlueIn gi, float *__restrict__ x_new,
    float *__restrict__ t, int d, int r, const int32_t *__restrict__ skip)
{
    __shared__ float red[kColsMaxWaves * cols_red_floats(R * B + B)];
    __shared__ __align__(16) float xch[kColsMaxWaves * kColsXFloats];
    // adaptive layer step: a set flag means this step runs dense and needs no prediction
    if (skip != nullptr && *skip != 0) return;
    // (two tokens of rows longer than 8192 take two passes)
    hidden_cols_body<B, GLUE, CPW, R, (CPW * B > 3), B, !(B == 2 && CPW == 2)>(red, xch + (threadIdx.x >> 6) * kColsXFloats, (int)blockIdx.x, blockIdx.x == 0, p1, x, gi, x_new, t, d, r);
}

// ---------------------------------------------------------------------------------------
// Output layer + threshold + ballot.  grid = (ffn - 64 first_word) / NB; block g owns the NB
// neurons from 64 first_word + NB*g on (NB = 16, 32 or 64: a quarter, half or whole mask word), wave w of it rows
// 4w .. 4w+3, all in flight at once; wave 0 turns the NB decisions into its piece of the
// mask word with a ballot.
constexpr int kPredOutNeurons = 64;
constexpr int kPredOutThreads = kPredOutNeurons * 16;
static_assert(kPredOutNeurons == 16 || kPredOutNeurons == 32 || kPredOutNeurons == 64, "mask piece");
template <int NB> struct MaskPiece { typedef uint64_t type; };
template <> struct MaskPiece<32> { typedef uint32_t type; };
template <> struct MaskPiece<16> { typedef uint16_t type; };

// Writes "always on" for the first `words` mask words (and score 1 for their neurons): the
// neurons of an always-on prefix are not evaluated by the predictor's output layer at all.
// Called by one workgroup of the output-layer kernels.
template <int B>
__device__ __forceinline__ void mark_always_on(int words, int ffn, float *__restrict__ scores,
                                               uint64_t *__restrict__ mask_words)
{
    for (int w = threadIdx.x; w < words; w += blockDim.x) mask_words[w] = ~0ull;
    if (scores != nullptr)
        for (int e = threadIdx.x; e < B * words * 64; e += blockDim.x)
            scores[(size_t)(e / (words * 64)) * ffn + e % (words * 64)] = 1.f;
}

// Body for a block of NB neurons (NB * 16 threads: 4 rows per wave); bid = which NB neurons.
// The launch covers the neurons from 64 * first_word on; its first block marks the words below.
template <int B, int NB>
__device__ __forceinline__ void pred_out_body(float *ts, float (*logit_s)[NB], const int bid0,
                                              const __half *__restrict__ p2,
                                              const float *__restrict__ p_bias,
                                              const float *__restrict__ t, int r, int ffn,
                                              float thr_logit, float *__restrict__ scores,
                                              uint64_t *__restrict__ mask_words, const int first_word)
{
    constexpr int NT = NB * 16;
    const int bid = bid0 + first_word * (64 / NB);
    if (bid0 == 0 && first_word > 0) mark_always_on<B>(first_word, ffn, scores, mask_words);
    // 16 waves per block leave 128 VGPRs per lane: fewer loads in flight at larger batch
    constexpr int U = (B <= 2) ? 4 : 2, R = NB / (NT / kWave);
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    const int nch = (r + kChunk - 1) / kChunk, kpad = nch * kChunk;
    const int n0 = bid * NB + wave * R;
    rsrc_t rows[R];
#pragma unroll
    for (int q = 0; q < R; ++q) rows[q] = row_rsrc(p2, n0 + q, r, true);

    PF_TSTAMP(1, 0);
    stage_dma<B>(ts, t, r, kpad);
    constexpr int PRE = 2;  // rows whose loads are issued before the block barrier
    WGroup<U> g[R];
#pragma unroll
    for (int q = 0; q < PRE; ++q) load_group<U>(g[q], rows[q], 0, lane);
    // lane q: the bias of the wave's row q
    const float pbl = ld4_f32(bias_rsrc(p_bias, ffn), lane < R ? (uint32_t)(n0 + lane) * 4u : kOobOffset);
    __syncthreads();
#pragma unroll
    for (int q = PRE; q < R; ++q) load_group<U>(g[q], rows[q], 0, lane);
    PF_TSTAMP(1, 1);

    float acc[R][B];
#pragma unroll
    for (int q = 0; q < R; ++q) {
#pragma unroll
        for (int b = 0; b < B; ++b) acc[q][b] = 0.f;
        fma_group<B, U>(g[q], ts, kpad, 0, nch, lane, acc[q]);
    }
    for (int it0 = U; it0 < nch; it0 += U) {
#pragma unroll
        for (int q = 0; q < R; ++q) load_group<U>(g[q], rows[q], it0, lane);
#pragma unroll
        for (int q = 0; q < R; ++q) fma_group<B, U>(g[q], ts, kpad, it0, nch, lane, acc[q]);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const float pb = lane_value(pbl, q);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float s = wave_sum(acc[q][b]) + pb;
            if (lane == 0) logit_s[b][wave * R + q] = s;
        }
    }
    __syncthreads();

    if (scores != nullptr) {
        for (int e = threadIdx.x; e < B * NB; e += NT) {
            const int b = e / NB, q = e % NB;
            scores[(size_t)b * ffn + bid * NB + q] = 1.f / (1.f + __expf(-logit_s[b][q]));
        }
    }
    if (wave == 0) {
        bool on = false;
#pragma unroll
        for (int b = 0; b < B; ++b) on = on || (lane < NB && logit_s[b][lane % NB] > thr_logit);
        const uint64_t word = __ballot(on);
        typedef typename MaskPiece<NB>::type piece_t;  // little endian: piece g of the words
        if (lane == 0) reinterpret_cast<piece_t *>(mask_words)[bid] = (piece_t)word;
    }
    PF_TSTAMP(1, 2);
}

// The same with the hidden vector held by column, batch 1 .. 3 and r <= 2048: the waves form C column
// chunks x row groups, a wave has all of its rows (4 at C = 1, 8 at C = 2, else 16) of one chunk in flight
// behind its piece of t, and nothing waits for the block before the first sum.  logits_cols leaves the
// partial sums in red [B][C][NB]; logit_cols adds them up for one neuron behind a barrier.
// One wave per 4 rows with t in LDS, four loads a row whatever r (half of them past its end at r = 1024)
// -> this, a step of the stack, us: 175B-class int4 (r 2048) 762 -> 729, 30B-class batch 1 (r 1536, 8
// layers) 327 -> 310, 13B-class gated batch 1 (r 1024) 612 -> 596.
template <int B, int NB, int C>
struct PredOutCols {
    static constexpr int WAVES = C == 3 ? NB * 3 / 16 : NB / 4;  // that have work
    static constexpr int GROUPS = WAVES / C, ROWS = NB / GROUPS;
    static constexpr int RED = C * NB * B;  // floats
};

// row_of(q): number of the block's row q in p2; valid(q): whether it is read.
template <int B, int NB, int C, typename RowOf, typename Valid>
__device__ __forceinline__ void logits_cols(float *red, float *xw, const __half *__restrict__ p2,
                                            const float *__restrict__ t, int r, RowOf row_of, Valid valid)
{
    typedef PredOutCols<B, NB, C> S;
    constexpr int RF = (B == 3 && S::ROWS == 16) ? 8 : S::ROWS;  // in flight: what 128 registers hold
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    if (wave >= S::WAVES) return;
    const int c = wave % C, q0 = wave / C * S::ROWS, col = c * kChunk + lane * 8;
    ColX<B> v;
    colx_load<B>(v, make_rsrc(t, (uint32_t)B * (uint32_t)r * 4u), c * kChunk + lane * 4, r);
#pragma unroll
    for (int h = 0; h < S::ROWS; h += RF) {
        uint4 w[RF];
#pragma unroll
        for (int q = 0; q < RF; ++q) {
            const int qq = q0 + h + q;
            w[q] = ld16_stream(row_rsrc(p2, row_of(qq), r, valid(qq)), (uint32_t)col * 2u);
        }
        if (h == 0) {
#pragma unroll
            for (int b = 0; b < B; ++b) cols_exchange(xw, v.lo[b], v.hi[b], lane);
        }
#pragma unroll
        for (int q = 0; q < RF; q += 4) {
            float acc[4 * B], s[B];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int b = 0; b < B; ++b) acc[b * 4 + i] = dot8(w[q + i], v.lo[b], v.hi[b], 0.f);
            wave_sums<4 * B>(acc, s);
            if ((lane & 15) == 0) {
#pragma unroll
                for (int b = 0; b < B; ++b)
                    red[(b * C + c) * NB + q0 + h + q + wave_sums_value(lane >> 4)] = s[b];
            }
        }
    }
}
template <int NB, int C>
__device__ __forceinline__ float logit_cols(const float *red, int b, int q, float bias)
{
    float a = red[b * C * NB + q];
#pragma unroll
    for (int c = 1; c < C; ++c) a += red[(b * C + c) * NB + q];
    return a + bias;
}

// Body for a block of NB neurons, as pred_out_body; xch = kColsXFloats floats of LDS per wave.
template <int B, int NB, int C>
__device__ __forceinline__ void pred_out_cols_body(float *red, float *xch, const int bid0,
                                                   const __half *__restrict__ p2, const float *__restrict__ p_bias,
                                                   const float *__restrict__ t, int r, int ffn, float thr_logit,
                                                   float *__restrict__ scores, uint64_t *__restrict__ mask_words,
                                                   const int first_word)
{
    const int bid = bid0 + first_word * (64 / NB);
    if (bid0 == 0 && first_word > 0) mark_always_on<B>(first_word, ffn, scores, mask_words);
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    PF_TSTAMP(1, 0);
    logits_cols<B, NB, C>(red, xch + wave * kColsXFloats, p2, t, r, [&](int q) { return bid * NB + q; },
                          [&](int) { return true; });
    const float bias = ld4_f32(bias_rsrc(p_bias, ffn), lane < NB ? (uint32_t)(bid * NB + lane) * 4u : kOobOffset);
    __syncthreads();
    PF_TSTAMP(1, 1);
    if (wave == 0) {
        bool on = false;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float lg = logit_cols<NB, C>(red, b, lane % NB, bias);
            on = on || (lane < NB && lg > thr_logit);
            if (scores != nullptr && lane < NB) scores[(size_t)b * ffn + bid * NB + lane] = 1.f / (1.f + __expf(-lg));
        }
        const uint64_t word = __ballot(on);
        typedef typename MaskPiece<NB>::type piece_t;  // little endian: piece g of the words
        if (lane == 0) reinterpret_cast<piece_t *>(mask_words)[bid] = (piece_t)word;
    }
    PF_TSTAMP(1, 2);
}

template <int B, int C>
__global__ __launch_bounds__((64 * PredOutCols<B, kPredOutNeurons, C>::WAVES)) void k_pred_out_cols(
    const __half *__restrict__ p2, const float *__restrict__ p_bias, const float *__restrict__ t, int r, int ffn,
    float thr_logit, float *__restrict__ scores, uint64_t *__restrict__ mask_words, int first_word,
    const int32_t *__restrict__ skip)
{
    typedef PredOutCols<B, kPredOutNeurons, C> S;
    __shared__ __align__(16) float xch[S::WAVES * kColsXFloats];
    __shared__ float red[S::RED];
    // adaptive layer step: a set flag means this step runs dense -- every neuron is marked
    if (skip != nullptr && *skip != 0) {
        if (threadIdx.x == 0) mask_words[first_word + (int)blockIdx.x] = ~0ull;
        if (blockIdx.x == 0 && first_word > 0) mark_always_on<B>(first_word, ffn, nullptr, mask_words);
        return;
    }
    pred_out_cols_body<B, kPredOutNeurons, C>(red, xch, (int)blockIdx.x, p2, p_bias, t, r, ffn, thr_logit, scores,
                                              mask_words, first_word);
}

template <int B>
__global__ __launch_bounds__(kPredOutThreads) void k_pred_out(
    const __half *__restrict__ p2, const float *__restrict__ p_bias, const float *__restrict__ t,
    int r, int ffn, float thr_logit, float *__restrict__ scores, uint64_t *__restrict__ mask_words,
    int first_word, const int32_t *__restrict__ skip)
{
    extern __shared__ float ts[];  // [B][kpad] staged hidden vector
    __shared__ float logit_s[B][kPredOutNeurons];
    // adaptive layer step: a set flag means this step runs dense -- every neuron is marked
    if (skip != nullptr && *skip != 0) {
        if (threadIdx.x == 0) mask_words[first_word + (int)blockIdx.x] = ~0ull;
        if (blockIdx.x == 0 && first_word > 0) mark_always_on<B>(first_word, ffn, nullptr, mask_words);
        return;
    }
    pred_out_body<B, kPredOutNeurons>(ts, logit_s, (int)blockIdx.x, p2, p_bias, t, r, ffn, thr_logit,
                                      scores, mask_words, first_word);
}

// ---------------------------------------------------------------------------------------
// Block-wide exclusive prefix of the popcounts of mask words: pre[w] = set bits in words
// [0, w) for w in [0, nwords]; the words are kept in LDS beside it.  Returns pre[nwords].
// Thread t scans the contiguous words [t*per, (t+1)*per); wave scan + LDS across waves.
template <int NT>
__device__ __forceinline__ uint32_t mask_prefix(const uint64_t *__restrict__ mask_words, int nwords,
                                                uint64_t *words_lds, uint32_t *pre_lds,
                                                uint32_t *wave_tot /* [NT / 64] */)
{
    constexpr int NW = NT / kWave;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (nwords + NT - 1) / NT;
    const int w0 = tid * per, w1 = min(nwords, w0 + per);
    uint32_t mine = 0;
    for (int w = w0; w < w1; ++w) {
        const uint64_t word = mask_words[w];
        words_lds[w] = word;
        mine += (uint32_t)__popcll(word);
    }
    uint32_t inc = mine;  // inclusive scan inside the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)inc, o, 64);
        if (lane >= o) inc += up;
    }
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t v = wave_tot[k];
        if (k < wave) before += v;
        total += v;
    }
    uint32_t run = before + inc - mine;
    for (int w = w0; w < w1; ++w) {
        pre_lds[w] = run;
        run += (uint32_t)__popcll(words_lds[w]);
    }
    if (tid == NT - 1) pre_lds[nwords] = total;
    __syncthreads();
    return total;
}

// Position of the j-th set bit (j < total) given the prefix above; all 64 lanes of a wave
// call it with the same j and get the same answer.  Two ballots find the word (coarse
// stride, then within the stride; nwords <= 4096), a third the bit inside the word.
__device__ __forceinline__ int select_set_bit(const uint64_t *words_lds, const uint32_t *pre_lds,
                                              int nwords, uint32_t j, int lane)
{
    const int step = (nwords + 63) >> 6;
    const int wc = min(lane * step, nwords);
    const int coarse = __popcll(__ballot(lane * step < nwords && pre_lds[wc] <= j)) - 1;
    const int wf = coarse * step + lane;
    const bool ok = lane < step && wf < nwords && pre_lds[min(wf, nwords)] <= j;
    const int w = coarse * step + __popcll(__ballot(ok)) - 1;
    const uint64_t word = words_lds[w];
    const uint32_t rank = j - pre_lds[w];
    const uint64_t below = word & ((1ull << lane) - 1ull);
    const uint64_t hit = __ballot(((word >> lane) & 1ull) && (uint32_t)__popcll(below) == rank);
    return w * 64 + (int)__builtin_ctzll(hit);
}

// ---------------------------------------------------------------------------------------
// The same compaction by every wave for itself, with one barrier: the mask words go to LDS straight from
// memory (list_words_issue; the caller synchronises the block), then each wave scans them -- lane l owns
// the words [l per, (l + 1) per) -- and looks up the slots it wants, one per lane, with three dependent
// LDS reads: 16 coarse prefixes, 4 fine ones, the words of the lane found.
constexpr int kListPriv = 80;  // floats of LDS of a wave: prefix per lane, and every fourth of them
__host__ __device__ constexpr int list_words_alloc(int nwords) { return (nwords + 127) / 128 * 128; }

__device__ __forceinline__ void list_words_issue(uint64_t *words, const uint64_t *__restrict__ mask_words, int nwords)
{
    const rsrc_t r = make_rsrc(mask_words, (uint32_t)nwords * 8u);
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6), W = (int)(blockDim.x >> 6);
    for (int c = wave; c < list_words_alloc(nwords) / 128; c += W)  // words past the mask read as zeros
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(words + c * 128), 16, c * 1024 + lane * 16, 0, 0, 0);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_rows_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v)
{
    v += dpp_rows_u32<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
    v += dpp_rows_u32<0x112, 0xf>(v);
    v += dpp_rows_u32<0x114, 0xf>(v);
    v += dpp_rows_u32<0x118, 0xf>(v);
    v += dpp_rows_u32<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
    v += dpp_rows_u32<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
    return v;
}

// Scans the words; returns the number of set bits.  priv: kListPriv words of LDS of this wave.
__device__ __forceinline__ int list_scan(const uint64_t *words, int nwords, uint32_t *priv, int lane)
{
    const int per = (nwords + 63) >> 6;
    uint32_t cnt = 0;
    for (int q = 0; q < per; ++q) cnt += (uint32_t)__popcll(words[lane * per + q]);
    const uint32_t inc = wave_prefix(cnt);
    priv[lane] = inc - cnt;
    if ((lane & 3) == 0) priv[64 + (lane >> 2)] = inc - cnt;
    __builtin_amdgcn_wave_barrier();
    return __builtin_amdgcn_readlane((int)inc, 63);
}

// Neuron of list slot j (of `total`), -1 past the end.
__device__ __forceinline__ int list_select(const uint64_t *words, int nwords, const uint32_t *priv, int j, int total)
{
    const int per = (nwords + 63) >> 6;
    const uint32_t ju = (uint32_t)max(j, 0);
    const uint4 *coarse = reinterpret_cast<const uint4 *>(priv + 64);
    int c = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 p = coarse[i];
        c += (p.x <= ju) + (p.y <= ju) + (p.z <= ju) + (p.w <= ju);
    }
    c = max(c - 1, 0);
    const uint4 f = reinterpret_cast<const uint4 *>(priv)[c];
    const int fi = max((f.x <= ju) + (f.y <= ju) + (f.z <= ju) + (f.w <= ju) - 1, 0);
    uint32_t rank = ju - (fi == 0 ? f.x : fi == 1 ? f.y : fi == 2 ? f.z : f.w);
    int at = (4 * c + fi) * per;
    uint64_t w = words[at];
    bool found = false;
    int wi = at;
    for (int q = 0; q < per; ++q) {  // the first word with more than `rank` bits left
        const uint64_t wq = words[at + q];
        const uint32_t n = (uint32_t)__popcll(wq);
        if (!found) {
            w = wq;
            wi = at + q;
            found = rank < n;
            if (!found) rank -= n;
        }
    }
    int pos = 0;
#pragma unroll
    for (int width = 32; width >= 1; width >>= 1) {
        const uint32_t n = (uint32_t)__popcll(w & ((1ull << width) - 1ull));
        if (rank >= n) {  // the bit lies in the upper half
            rank -= n;
            w >>= width;
            pos += width;
        }
    }
    return j < total ? wi * 64 + pos : -1;
}

// ---------------------------------------------------------------------------------------
// Stand-alone compaction of mask words into an ascending index list, by one workgroup.
// Per pass of NT words: popcount prefix as above, then one wave per word; lane l owns
// bit l and its rank inside the word is the popcount of the lower bits (what a ballot +
// mbcnt pair gives for a live predicate).
constexpr int kCompactThreads = 1024;

__global__ __launch_bounds__(kCompactThreads) void k_compact(const uint64_t *__restrict__ mask_words,
                                                             int nwords, int32_t *__restrict__ idx,
                                                             int32_t *__restrict__ count)
{
    constexpr int NT = kCompactThreads, NW = NT / kWave;
    __shared__ uint64_t words_lds[NT];
    __shared__ uint32_t pre_lds[NT + 1];
    __shared__ uint32_t wave_tot[NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int w0 = 0; w0 < nwords; w0 += NT) {
        const int nhere = min(NT, nwords - w0);
        const uint32_t total = mask_prefix<NT>(mask_words + w0, nhere, words_lds, pre_lds, wave_tot);
        for (int q = wave; q < nhere; q += NW) {
            const uint64_t wq = words_lds[q];
            const uint64_t below = wq & ((1ull << lane) - 1ull);
            if ((wq >> lane) & 1ull)
                idx[carry + pre_lds[q] + (uint32_t)__popcll(below)] = (w0 + q) * 64 + lane;
        }
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *count = (int32_t)carry;
}

}  // namespace pf
