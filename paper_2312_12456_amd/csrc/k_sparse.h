// Neuron-aware sparse FFN over the active neurons (PowerInfer Sec. 5.4; the FFN block
// itself is Sec. 2.1, Fig. "bg-mlp"): only the FC1 / gate rows and FC2 columns of the listed
// neurons are read.  All three matrices are neuron-major [ffn][d] fp16, so one neuron is one
// contiguous run of 2d bytes (a multiple of 128 B at every model width used).
//   k_up   : h[b][j] = act(row idx[j] . x[b] + bias)           one wave per listed neuron
//   k_down2: y[b][:] = b_down + sum_j h[b][j] * FC2^T[idx[j]]  64 columns x every P-th slot per workgroup
// The number of listed neurons is read from device memory; grids are fixed.  No kernel
// uses device-scope fences or atomics: every sum has one owner and a fixed order.
#pragma once
#include "dev_util.h"
#include "k_predict.h"

namespace pf {

constexpr int kUpThreads = 256;
constexpr int kUpWaves = kUpThreads / kWave;

// LDS bytes the up kernel needs beyond the staged activations when it compacts itself.
inline size_t up_mask_lds_bytes(int ffn)
{
    const size_t nwords = (size_t)ffn / 64;
    return nwords * sizeof(uint64_t) + (nwords + 1) * sizeof(uint32_t) + 64;
}

// ---------------------------------------------------------------------------------------
// grid = any; waves stride over the list.  x is staged once per workgroup in LDS while the
// first row of every wave is already in flight.
// FROM_MASK: the list is not given; every workgroup derives it from the predictor's mask
// words (popcount prefix in LDS, then each wave selects its j-th set bit), writes the
// entries it owns to idx_out and block 0 writes the count -- the compaction fused into its
// consumer, so the layer step needs no separate compaction launch.
// Gated forms (ACT == 1): h = ReLU(gate . x + bias) * max(up . x, up_floor); up_floor is
// -infinity for the plain ReLU-gated block and 0 for dReLU (ReLU on both branches).
// GLUE (only with FROM_MASK, inside a stack): the layer input is formed in the kernel from the
// previous layer's input and FC2 partial sums, like the predictor's hidden kernel does, and
// applied as a scale on the dot products; the block with write_x set stores it for later kernels.
// The body takes its block number and the number of blocks of its role explicitly, so that a
// launch can run it in a range of its blocks beside another role.
template <int B, int ACT, bool FROM_MASK, bool GLUE>
__device__ __forceinline__ void up_body(
    float *xs, uint32_t *wave_tot, float (*ss_w)[B], const int bid, const int nblocks, const bool write_x,
    const __half *__restrict__ w_up, const __half *__restrict__ w_gate,
    const float *__restrict__ b_up, const float *__restrict__ x,
    const int32_t *__restrict__ idx_in, const int32_t *__restrict__ count_in,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d, int ffn, float up_floor,
    const float *__restrict__ yp, int ny, int ypstride, float *__restrict__ x_new)
{
    constexpr int U = 8;
    constexpr bool GATED = (ACT == 1);
    const int lane = threadIdx.x & 63;
    const int wave = wave_uniform(threadIdx.x >> 6);
    const int nch = (d + kChunk - 1) / kChunk, kpad = nch * kChunk;
    const int stride = nblocks * kUpWaves;
    const int nwords = ffn / 64;
    uint64_t *words_lds = reinterpret_cast<uint64_t *>(xs + (size_t)B * kpad + kStageScrap);
    uint32_t *pre_lds = reinterpret_cast<uint32_t *>(words_lds + nwords);

    PF_TSTAMP(2, 0);
    // Through registers rather than straight to LDS: a global -> LDS copy has to be waited
    // for at the first barrier of the mask scan, the register copy only at the commit
    // (measured: 3 % of the stack's time at batch 1, more at larger batches).
    constexpr int SS = (B >= 4) ? 1 : 4 / B;
    Staged<B, SS> st;
    // glue: strides of 1024 elements whose loads are in flight together (all of d <= 4096 at
    // batch 1, as in the hidden kernel)
    constexpr int GS = GLUE ? (B >= 2 ? 1 : 4) : 1;
    GluePass<B, GS> gp;
    const rsrc_t xr = make_rsrc(x, (uint32_t)B * (uint32_t)d * 4u);
    const uint32_t pbytes = (uint32_t)ypstride * 4u;
    const rsrc_t yr = make_rsrc(yp, GLUE ? (uint32_t)(ny - 1) * pbytes + (uint32_t)B * (uint32_t)d * 4u : 0u);
    if (GLUE)
        glue_issue<B, GS, kUpThreads>(gp, xr, yr, pbytes, ny, d, threadIdx.x * 4);
    else
        stage_issue<B, SS>(st, x, d);  // in flight during the mask scan; lands before any weight
    int n;
    if (FROM_MASK) {
        n = (int)mask_prefix<kUpThreads>(mask_words, nwords, words_lds, pre_lds, wave_tot);
        if (bid == 0 && threadIdx.x == 0) *count_out = n;
    } else {
        n = min(max(*count_in, 0), ffn);
    }
    if (bid * kUpWaves >= n && !(GLUE && write_x)) return;  // uniform over the block
    PF_TSTAMP(2, 1);

    auto neuron_of = [&](int j) -> int {
        if (FROM_MASK) {
            const int i = select_set_bit(words_lds, pre_lds, nwords, (uint32_t)j, lane);
            if (lane == 0) idx_out[j] = i;
            return i;
        }
        return idx_in[j];
    };

    int j = bid * kUpWaves + wave;
    int i = 0;
    bool valid = false;
    if (j < n) {
        i = wave_uniform(neuron_of(j));
        valid = (unsigned)i < (unsigned)ffn;
        if (!valid) i = 0;
    }
    PF_TSTAMP(2, 5);
    WGroup<U> gu, gg;
    rsrc_t ru = row_rsrc(w_up, i, d, valid), rg = row_rsrc(GATED ? w_gate : w_up, i, d, valid);
    // The first row's bias is requested in front of its weights and kept as a scalar: behind the sums it was a trip to
    // HBM of its own.  Those of later rows are scalar loads behind their sums, which other waves' work hides; as
    // vector loads beside the next row's weights they cost lists of many rows a wave 4 - 6 % (pf_dense_ffn of 7176 x
    // 22912 at batch 8, FC1 alone 122 / 130 us).
    const float bias_first = ld4_f32(bias_rsrc(b_up, ffn), valid ? (uint32_t)i * 4u : kOobOffset);
    load_group<U>(gu, ru, 0, lane);
    if (GATED) load_group<U>(gg, rg, 0, lane);

    PF_TSTAMP(2, 2);
    float scale[B];
    if (GLUE) {
        float ss[B];
#pragma unroll
        for (int b = 0; b < B; ++b) ss[b] = 0.f;
        glue_commit<B, GS, kUpThreads>(gp, xs, kpad, 0, threadIdx.x * 4, ss);
        for (int e0 = threadIdx.x * 4 + kUpThreads * 4 * GS; e0 < kpad; e0 += kUpThreads * 4 * GS) {
            glue_issue<B, GS, kUpThreads>(gp, xr, yr, pbytes, ny, d, e0);
            glue_commit<B, GS, kUpThreads>(gp, xs, kpad, 0, e0, ss);
        }
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
            for (int k = 0; k < kUpWaves; ++k) tot += ss_w[k][b];
            scale[b] = tot > 0.f ? sqrtf((float)d / tot) : 0.f;
        }
        if (write_x) {
            for (int e = threadIdx.x * 4; e < d; e += kUpThreads * 4) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const float4 v = *reinterpret_cast<const float4 *>(xs + b * kpad + lds_slot(e));
                    *reinterpret_cast<float4 *>(x_new + (size_t)b * d + e) =
                        make_float4(v.x * scale[b], v.y * scale[b], v.z * scale[b], v.w * scale[b]);
                }
            }
        }
    } else {
        stage_commit<B, SS>(st, xs, x, d, kpad);
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B; ++b) scale[b] = 1.f;
    }
    PF_TSTAMP(2, 3);
    const float bias0 = lane_value(bias_first, 0);
    bool first = true;

    while (j < n) {  // wave-uniform; no block-level synchronisation inside
        float au[B], ag[B];
#pragma unroll
        for (int b = 0; b < B; ++b) au[b] = ag[b] = 0.f;
        fma_group<B, U>(gu, xs, kpad, 0, nch, lane, au);
        if (GATED) fma_group<B, U>(gg, xs, kpad, 0, nch, lane, ag);
        for (int it0 = U; it0 < nch; it0 += U) {
            load_group<U>(gu, ru, it0, lane);
            if (GATED) load_group<U>(gg, rg, it0, lane);
            fma_group<B, U>(gu, xs, kpad, it0, nch, lane, au);
            if (GATED) fma_group<B, U>(gg, xs, kpad, it0, nch, lane, ag);
        }
        const int jcur = j, icur = i;
        const bool vcur = valid;
        j += stride;
        if (j < n) {  // next row in flight before this row's reductions
            i = wave_uniform(neuron_of(j));
            valid = (unsigned)i < (unsigned)ffn;
            if (!valid) i = 0;
            ru = row_rsrc(w_up, i, d, valid);
            rg = row_rsrc(GATED ? w_gate : w_up, i, d, valid);
            load_group<U>(gu, ru, 0, lane);
            if (GATED) load_group<U>(gg, rg, 0, lane);
        }
        const float bcur = first ? bias0 : (b_up != nullptr && vcur) ? b_up[icur] : 0.f;
        first = false;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            float v;
            if (GATED) {
                const float gsum = (GLUE ? wave_sum(ag[b]) * scale[b] : wave_sum(ag[b])) + bcur;
                const float usum = GLUE ? wave_sum(au[b]) * scale[b] : wave_sum(au[b]);
                v = fmaxf(gsum, 0.f) * fmaxf(usum, up_floor);
            } else {
                v = fmaxf((GLUE ? wave_sum(au[b]) * scale[b] : wave_sum(au[b])) + bcur, 0.f);
            }
            if (lane == 0) h[(size_t)jcur * hs + b] = vcur ? v : 0.f;
        }
    }
    PF_TSTAMP(2, 4);
}

template <int B, int ACT, bool FROM_MASK>
__global__ __launch_bounds__(kUpThreads) void k_up(
    const __half *__restrict__ w_up, const __half *__restrict__ w_gate,
    const float *__restrict__ b_up, const float *__restrict__ x,
    const int32_t *__restrict__ idx_in, const int32_t *__restrict__ count_in,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d, int ffn, float up_floor)
{
    extern __shared__ float xs[];
    __shared__ uint32_t wave_tot[kUpWaves];
    up_body<B, ACT, FROM_MASK, false>(xs, wave_tot, nullptr, (int)blockIdx.x, (int)gridDim.x, false, w_up,
                                      w_gate, b_up, x, idx_in, count_in, mask_words, idx_out, count_out,
                                      h, hs, d, ffn, up_floor, nullptr, 1, 0, nullptr);
}

// ---------------------------------------------------------------------------------------
// FC1 over the listed neurons with the activations held by column (k_predict.h), batch 1 .. 3: block b of
// G owns the list slots [n b / G, n (b + 1) / G), all of its waves work on the same rows, R of them in
// flight while the R before are multiplied.  The rows' sums meet in LDS every kUpColsRows rows.
// Arguments as in up_body.  lds: up_cols_lds_bytes.  d <= 512 CPW waves.
// One workgroup per CU: with whole rows dealt to waves some CUs got half as many rows again as others.
// One wave per row with x in LDS -> this, us: d 5120 gated, 2073 rows (42 MB) batch 1 12.4 -> 10.4, batch 2 18 ->
// 14; d 4096 gated batch 3 14.7 -> 12.0; d 7168, 1700 rows 8.7 -> 8.3; d 4096, 1307 rows 5.9 -> 6.2 at
// batch 1 (which takes the former; the line is kUpColsMinElems).
constexpr int kUpColsRows = 32;

inline size_t up_cols_lds_bytes(int ffn, int waves, int matrices, int B, bool from_mask)
{
    return (from_mask ? (size_t)list_words_alloc(ffn / 64) * 8 : 0) +
           (size_t)waves * 4 * (kColsXFloats + kListPriv + 4 + kUpColsRows * matrices * cols_red_floats(B));
}

template <int B, int ACT, bool FROM_MASK, bool GLUE, int CPW, int R, bool SEQ = (CPW * B > 3), int GT = B>
__device__ __forceinline__ void up_cols_body(
    char *lds, const int bid, const int nblocks, const bool write_x, const __half *__restrict__ w_up,
    const __half *__restrict__ w_gate, const float *__restrict__ b_up, const float *__restrict__ x, const GlueIn gi,
    float *__restrict__ x_new, const int32_t *__restrict__ idx_in, const int32_t *__restrict__ count_in,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out, int32_t *__restrict__ count_out,
    float *__restrict__ h, int hs, int d, int ffn, float up_floor)
{
    constexpr bool GATED = (ACT == 1);
    constexpr int NM = GATED ? 2 : 1, N = R * NM * B, NP = cols_red_floats(N);
    static_assert(kUpColsRows % R == 0 && NP <= R * NM * cols_red_floats(B), "the sums of a batch of rows fit");
    constexpr int PASSES = kUpColsRows / R;
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6), W = (int)(blockDim.x >> 6);
    const int nwords = ffn / 64;
    uint64_t *words = reinterpret_cast<uint64_t *>(lds);
    float *fl = reinterpret_cast<float *>(lds + (FROM_MASK ? (size_t)list_words_alloc(nwords) * 8 : 0));
    float *xw = fl + wave * kColsXFloats;
    uint32_t *priv = reinterpret_cast<uint32_t *>(fl + W * kColsXFloats) + wave * kListPriv;
    float *ssl = fl + W * (kColsXFloats + kListPriv);  // [W][4]
    float *red = ssl + W * 4;                          // [W][PASSES][NP]

    PF_TSTAMP(2, 0);
    if (FROM_MASK) list_words_issue(words, mask_words, nwords);
    ColX<B> v[CPW];
    int col[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) col[c] = (c * W + wave) * kChunk + lane * 8;
    const rsrc_t xr = make_rsrc(GLUE ? gi.x : x, (uint32_t)B * (uint32_t)d * 4u);
    float ss[B];
#pragma unroll
    for (int b = 0; b < B; ++b) ss[b] = 0.f;
    if constexpr (GLUE) {
        const uint32_t pbytes = (uint32_t)gi.ypstride * 4u;
        const rsrc_t yr = make_rsrc(gi.yp, (uint32_t)(gi.ny - 1) * pbytes + (uint32_t)B * (uint32_t)d * 4u);
        const rsrc_t sr = make_rsrc(gi.sign, (uint32_t)kSignRows * (uint32_t)gi.sstride);
        auto piece = [&](auto nyc) {
            constexpr int NY = decltype(nyc)::value;
            if constexpr (!SEQ) {
                ColGlue<B, NY> g[CPW];
#pragma unroll
                for (int c = 0; c < CPW; ++c)
                    colglue_issue<B, NY>(g[c], xr, yr, sr, (uint32_t)gi.sstride, pbytes, (c * W + wave) * kChunk + lane * 4, d);
#pragma unroll
                for (int c = 0; c < CPW; ++c) colglue_commit(g[c], v[c], ss, lane);
            } else {  // not enough registers for all of them at once
#pragma unroll
                for (int c = 0; c < CPW; ++c)
                    colglue_chunk<B, NY, GT>(v[c], ss, xr, yr, sr, (uint32_t)gi.sstride, pbytes,
                                             (c * W + wave) * kChunk + lane * 4, d, lane);
            }
        };
        if (gi.ny == 4) piece(IntC<4>());
        else if (gi.ny == 3) piece(IntC<3>());
        else if (gi.ny == 2) piece(IntC<2>());
        else piece(IntC<1>());
    } else {
#pragma unroll
        for (int c = 0; c < CPW; ++c) colx_load<B>(v[c], xr, (c * W + wave) * kChunk + lane * 4, d);
    }
    int n;
    if (FROM_MASK) {
        __syncthreads();
        n = list_scan(words, nwords, priv, lane);
        if (bid == 0 && threadIdx.x == 0) *count_out = n;
    } else {
        n = min(max(*count_in, 0), ffn);
    }
    const int j_begin = (int)((long long)n * bid / nblocks), j_end = (int)((long long)n * (bid + 1) / nblocks);
    if (j_begin == j_end && !(GLUE && write_x)) return;  // uniform over the block
    PF_TSTAMP(2, 1);
    bool have_x = false;
    const rsrc_t br = bias_rsrc(b_up, ffn);

    for (int jb = j_begin; jb < j_end || !have_x; jb += kUpColsRows) {
        const int rows = min(kUpColsRows, j_end - jb);
        // lane l: the neuron of slot jb + l, and its bias
        int id = -1;
        if (FROM_MASK) {
            id = list_select(words, nwords, priv, lane < rows ? jb + lane : n, n);
            if (wave == 0 && id >= 0) idx_out[jb + lane] = id;
        } else if (lane < rows) {
            id = idx_in[jb + lane];
        }
        if ((unsigned)id >= (unsigned)ffn) id = -1;
        PF_TSTAMP(2, 5);
        uint4 wa[R][NM][CPW], wb[R][NM][CPW];
        auto load_row = [&](uint4 (&w)[NM][CPW], int row) {
            const int i = __builtin_amdgcn_readlane(id, row);
            const rsrc_t ru = row_rsrc(w_up, max(i, 0), d, i >= 0), rg = row_rsrc(GATED ? w_gate : w_up, max(i, 0), d, i >= 0);
#pragma unroll
            for (int c = 0; c < CPW; ++c) {
                w[0][c] = ld16_stream(ru, (uint32_t)col[c] * 2u);
                if (GATED) w[NM - 1][c] = ld16_stream(rg, (uint32_t)col[c] * 2u);
            }
        };
        auto multiply = [&](const uint4 (&w)[R][NM][CPW], int pass) {
            float acc[N];
#pragma unroll
            for (int q = 0; q < R; ++q)
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int b = 0; b < B; ++b) {
                        float a = 0.f;
#pragma unroll
                        for (int c = 0; c < CPW; ++c) a = dot8(w[q][m][c], v[c].lo[b], v[c].hi[b], a);
                        acc[(q * NM + m) * B + b] = a;
                    }
            float s[NP / 4];
            wave_sums<N>(acc, s);
            if ((lane & 15) == 0) {
#pragma unroll
                for (int i = 0; i < NP / 4; ++i)
                    red[(wave * PASSES + pass) * NP + 4 * i + wave_sums_value(lane >> 4)] = s[i];
            }
        };
        const int full = max(rows, 0) / R, tail = max(rows, 0) % R;
        if (full > 0) {
#pragma unroll
            for (int q = 0; q < R; ++q) load_row(wa[q], q);
        }
        const float bias = ld4_f32(br, id >= 0 ? (uint32_t)id * 4u : kOobOffset);
        if (!have_x) {
            if (GLUE) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const float s = wave_sum(ss[b]);
                    if (lane == 0) ssl[wave * 4 + b] = s;
                }
            }
#pragma unroll
            for (int c = 0; c < CPW; ++c)
#pragma unroll
                for (int b = 0; b < B; ++b) cols_exchange(xw, v[c].lo[b], v[c].hi[b], lane);
            have_x = true;
        }
        PF_TSTAMP(2, 2);
        int p = 0;
        for (; p + 1 < full; ++p) {
#pragma unroll
            for (int q = 0; q < R; ++q) load_row(wb[q], (p + 1) * R + q);
            multiply(wa, p);
#pragma unroll
            for (int q = 0; q < R; ++q)
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int c = 0; c < CPW; ++c) wa[q][m][c] = wb[q][m][c];
        }
        if (tail > 0) {  // (rows that are not there are not asked for: a padded load costs as much as any)
#pragma unroll
            for (int q = 0; q < R; ++q) {
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int c = 0; c < CPW; ++c) wb[q][m][c] = make_uint4(0u, 0u, 0u, 0u);
                if (q < tail) load_row(wb[q], full * R + q);
            }
        }
        if (full > 0) multiply(wa, full - 1);
        if (tail > 0) multiply(wb, full);
        PF_TSTAMP(2, 3);
        __syncthreads();
        for (int e = threadIdx.x; e < kUpColsRows * B; e += blockDim.x) {
            const int row = e % kUpColsRows, b = e / kUpColsRows;  // a wave: lanes row, row + 32
            const float bv = __shfl(bias, row, 64);
            const int iv = __shfl(id, row, 64);
            if (row < rows) {
                const int at = (row / R) * NP + (row % R) * NM * B + b;
                float su = cols_total(red + at, PASSES * NP, W);
                float sg = GATED ? cols_total(red + at + B, PASSES * NP, W) : 0.f;
                if (GLUE) {
                    const float sq = cols_total(ssl + b, 4, W), sc = sq > 0.f ? sqrtf((float)d / sq) : 0.f;
                    su *= sc;
                    sg *= sc;
                }
                const float o = GATED ? fmaxf(sg + bv, 0.f) * fmaxf(su, up_floor) : fmaxf(su + bv, 0.f);
                h[(size_t)(jb + row) * hs + b] = iv >= 0 ? o : 0.f;
            }
        }
        if (jb + kUpColsRows < j_end) __syncthreads();
    }
    if (GLUE && write_x) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float sq = cols_total(ssl + b, 4, W), sc = sq > 0.f ? sqrtf((float)d / sq) : 0.f;
#pragma unroll
            for (int c = 0; c < CPW; ++c) {
                if (col[c] >= d) continue;
                float4 *to = reinterpret_cast<float4 *>(x_new + (size_t)b * d + col[c]);
                const float4 a = v[c].lo[b], e = v[c].hi[b];
                to[0] = make_float4(a.x * sc, a.y * sc, a.z * sc, a.w * sc);
                to[1] = make_float4(e.x * sc, e.y * sc, e.z * sc, e.w * sc);
            }
        }
    }
    PF_TSTAMP(2, 4);
}

// Rows of a pass: two passes are in flight.
template <int B, int ACT, int CPW>
struct UpColsR {
    static constexpr int value = (ACT + 1) * CPW * B >= 4 ? 2 : 4;
};

template <int B, int ACT, bool FROM_MASK, int CPW>
__global__ __launch_bounds__(64 * kColsMaxWaves) __attribute__((amdgpu_waves_per_eu(2, 4))) void k_up_cols(
    const __half *__restrict__ w_up, const __half *__restrict__ w_gate, const float *__restrict__ b_up,
    const float *__restrict__ x, const int32_t *__restrict__ idx_in, const int32_t *__restrict__ count_in,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out, int32_t *__restrict__ count_out,
    float *__restrict__ h, int hs, int d, int ffn, float up_floor)
{
    extern __shared__ __align__(16) char cols_lds[];
    up_cols_body<B, ACT, FROM_MASK, false, CPW, UpColsR<B, ACT, CPW>::value>(
        cols_lds, (int)blockIdx.x, (int)gridDim.x, false, w_up, w_gate, b_up, x, GlueIn(), nullptr, idx_in, count_in,
        mask_words, idx_out, count_out, h, hs, d, ffn, up_floor);
}

// ---------------------------------------------------------------------------------------
// FC2 over the listed neurons, row-split.  The vector memory path of a CU handles gathered
// rows at a few nanoseconds per distinct 128-byte line, so a tiling in which every workgroup
// walks the whole list over a narrow column strip is bound by k lines per CU, not by HBM
// (measured: 16-column strips took 8.7 us where this form takes 5.6 us at d = 4096, k = 1300).
// Here a workgroup owns 64 output columns (one full line per row: 8 lanes x 16 bytes) and
// only every P-th list slot (slot = P * row + g for row group g), so a CU touches
// k * d / (64 * CUs) lines.  idx and h loads of the first pass are issued before the count
// has arrived (both arrays have capacity ffn), so they overlap with it.  The P
// partial sums of a column tile are NOT combined here: partial g goes to part[g][b][d]
// (group 0 adds b_down) and the consumer adds the P partials in the fixed order
// g = 0 .. P-1 -- the next layer's predictor kernel inside a stack, k_combine otherwise.
// grid = (d / 64 tiles, P), block = 512: 64 list slots per load of the block.
// Batches of 4 and more whose FC1 runs on the matrix cores take k_down2_mfma instead (in the two-launch
// look-ahead form of the matrix-core kernels also batch 3).
constexpr int kDown2Threads = 512;
constexpr int kDown2Waves = kDown2Threads / kWave;
constexpr int kDown2Cols = 64;
constexpr int kDown2RowsPerLoad = kDown2Threads / 8;
constexpr int kDown2MaxSplit = 4;

// Rows of a round that a lane loads (U), and the tokens padded to a power of two for the halving
// butterfly of the epilogue (BP): token b, column e of the lane -> acc[8 b + e].
template <int B>
struct Down2Shape {
    static constexpr int U = (B <= 2) ? 8 : 4;
    static constexpr int BP = B <= 1 ? 1 : B <= 2 ? 2 : B <= 4 ? 4 : 8;
};
template <int B>
struct Down2Round {
    float h[Down2Shape<B>::U][B];
    int iv[Down2Shape<B>::U];
};

// Loads of the round from r0 on that depend on the slot number only.
template <int B>
__device__ __forceinline__ void down2_request(Down2Round<B> &r, int r0, int rslot, int g, int P,
                                              const float *__restrict__ h, const int32_t *__restrict__ idx, int ffn)
{
#pragma unroll
    for (int u = 0; u < Down2Shape<B>::U; ++u) {
        const int jc = min((r0 + u * kDown2RowsPerLoad + rslot) * P + g, ffn - 1);
        r.iv[u] = idx[jc];
        load_h_slot<B>(h, jc, r.h[u]);
    }
}

// The rows of a round of a list of n, into acc.
template <int B>
__device__ __forceinline__ void down2_round(float (&acc)[Down2Shape<B>::BP * 8], Down2Round<B> &r, rsrc_t wd, int r0,
                                            int rslot, int g, int P, int col, int n, int d, int ffn)
{
    constexpr int U = Down2Shape<B>::U;
    uint4 w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int jj = (r0 + u * kDown2RowsPerLoad + rslot) * P + g;
        const bool ok = jj < n && (unsigned)r.iv[u] < (unsigned)ffn;
        w[u] = ld16_stream(wd, (ok && col < d) ? ((uint32_t)r.iv[u] * (uint32_t)d + (uint32_t)col) * 2u
                                               : kOobOffset);
#pragma unroll
        for (int b = 0; b < B; ++b) r.h[u][b] = ok ? r.h[u][b] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float f0 = h_lo(w[u].x), f1 = h_hi(w[u].x), f2 = h_lo(w[u].y), f3 = h_hi(w[u].y);
        const float f4 = h_lo(w[u].z), f5 = h_hi(w[u].z), f6 = h_lo(w[u].w), f7 = h_hi(w[u].w);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float s = r.h[u][b];
            acc[8 * b + 0] = fmaf(s, f0, acc[8 * b + 0]);
            acc[8 * b + 1] = fmaf(s, f1, acc[8 * b + 1]);
            acc[8 * b + 2] = fmaf(s, f2, acc[8 * b + 2]);
            acc[8 * b + 3] = fmaf(s, f3, acc[8 * b + 3]);
            acc[8 * b + 4] = fmaf(s, f4, acc[8 * b + 4]);
            acc[8 * b + 5] = fmaf(s, f5, acc[8 * b + 5]);
            acc[8 * b + 6] = fmaf(s, f6, acc[8 * b + 6]);
            acc[8 * b + 7] = fmaf(s, f7, acc[8 * b + 7]);
        }
    }
}

// The bias of the output column that a thread finishes: row group 0 adds it.
__device__ __forceinline__ float down2_bias(const float *__restrict__ b_down, int tile, int g, int d)
{
    return ld4_f32(bias_rsrc(b_down, d),
                   g == 0 ? (uint32_t)(tile * kDown2Cols + (int)threadIdx.x % kDown2Cols) * 4u : kOobOffset);
}

// Sums over the 8 row slots of each wave (lane bits 5, 4, 3) with a halving butterfly -- a lane ends
// with BP of its 8 BP values, flat indices [BP * slot, BP * (slot + 1)) --, then over the 8 waves
// through LDS, to part[g].  bpre = down2_bias of the thread.
template <int B>
__device__ __forceinline__ void down2_finish(float (&acc)[Down2Shape<B>::BP * 8], float (*red)[B][kDown2Cols],
                                             int tile, int g, float bpre, float *__restrict__ part, int d)
{
    constexpr int BP = Down2Shape<B>::BP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cl = lane & 7;
    butterfly_halve<32, BP * 4>(acc, lane);
    butterfly_halve<16, BP * 2>(acc, lane);
    butterfly_halve<8, BP>(acc, lane);
    {
        const int slot = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
#pragma unroll
        for (int k = 0; k < BP; ++k) {
            const int f = BP * slot + k, b = f >> 3, e = f & 7;
            if (b < B) red[wave][b][cl * 8 + e] = acc[k];
        }
    }
    __syncthreads();
    PF_TSTAMP(3, 4);
    if (threadIdx.x < B * kDown2Cols) {
        const int b = threadIdx.x / kDown2Cols, c = threadIdx.x % kDown2Cols;
        const int oc = tile * kDown2Cols + c;
        if (oc < d) {
            float s = bpre;
#pragma unroll
            for (int wv = 0; wv < kDown2Waves; ++wv) s += red[wv][b][c];
            part[((size_t)g * B + b) * d + oc] = s;
        }
    }
}

template <int B>
__device__ __forceinline__ void down2_body(
    float (*red)[B][kDown2Cols], const int tile, const int g, const int P,
    const __half *__restrict__ w_down, const float *__restrict__ b_down,
    const float *__restrict__ h, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ count_p, float *__restrict__ part, int d, int ffn)
{
    constexpr int U = Down2Shape<B>::U, BP = Down2Shape<B>::BP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rslot = wave * 8 + (lane >> 3);             // row slot of this lane inside a load
    const int col = tile * kDown2Cols + (lane & 7) * 8;   // its 16 bytes of the row's 128-byte line
    const rsrc_t wd = make_rsrc(w_down, (uint32_t)ffn * (uint32_t)d * 2u);

    PF_TSTAMP(3, 0);
    float acc[BP * 8];
#pragma unroll
    for (int f = 0; f < BP * 8; ++f) acc[f] = 0.f;

    int n = 0;
    bool have_n = false;
    for (int r0 = 0; r0 == 0 || r0 * P < n; r0 += kDown2RowsPerLoad * U) {
        Down2Round<B> r;
        down2_request<B>(r, r0, rslot, g, P, h, idx, ffn);
        if (!have_n) {
            n = min(max(*count_p, 0), ffn);
            have_n = true;
            PF_TSTAMP(3, 1);
        }
        down2_round<B>(acc, r, wd, r0, rslot, g, P, col, n, d, ffn);
        if (r0 == 0) PF_TSTAMP(3, 2);
    }
    PF_TSTAMP(3, 3);
    // requested here, under the lane sums: held through the loop it cost lists of several rounds 7 % (2056 x 6528 dense
    // batch 4, 15.2 / 16.4 us)
    const float bpre = down2_bias(b_down, tile, g, d);
    down2_finish<B>(acc, red, tile, g, bpre, part, d);
    PF_TSTAMP(3, 5);
}

template <int B>
__global__ __launch_bounds__(kDown2Threads) void k_down2(
    const __half *__restrict__ w_down, const float *__restrict__ b_down,
    const float *__restrict__ h, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ count_p, float *__restrict__ part, int d, int ffn)
{
    __shared__ float red[kDown2Waves][B][kDown2Cols];
    down2_body<B>(red, (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.y, w_down, b_down, h, idx, count_p,
                  part, d, ffn);
}

// y[b][c] = sum of the P partials in order (for callers that need FC2's output itself).
__global__ __launch_bounds__(256) void k_combine(const float *__restrict__ part, int P, int n,
                                                 float *__restrict__ y)
{
    const int e = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (e >= n) return;
    float4 s = *reinterpret_cast<const float4 *>(part + e);
    for (int p = 1; p < P; ++p) {
        const float4 v = *reinterpret_cast<const float4 *>(part + (size_t)p * n + e);
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    }
    *reinterpret_cast<float4 *>(y + e) = s;
}

// ---------------------------------------------------------------------------------------
// Stack glue: x_next[b] = sign(b, .) * (x[b] + y[b]) * sqrt(d) / ||x[b] + y[b]||_2.  grid = B.
constexpr int kGlueThreads = 1024;

// The activations of a batch as fp16 hi + lo halves in the order in which the matrix-core kernels
// take them: element c of token b's hi half is at half split_at(hs, b, c), hs = h_stride(B), its
// lo half hs * 8 halfs further.  8 consecutive elements of one token's half are contiguous, then
// come the other tokens' hi and lo halves of the same 8 elements: the operand of one matrix
// instruction (32 elements, all tokens, both halves) is one run of 128 hs bytes.  (Planes of
// [B][d] halfs cost the consumers two loads per step of 64-byte pieces from every token's row:
// at the OPT-30B shape, batch 8, the hidden layer's 192 workgroups touched four times as many
// lines for activations as for weights.)  The writers pay for it, as the workgroups of 8 tokens, on
// different XCDs, each write 16 bytes of every 128-byte line: k_glue takes 0.7 us more than
// for planes (that shape, batch 8; batch 4 0.5), with 8-byte and with 16-byte stores alike.
// The consumers gain 4.1 (hidden layer), 2.6 (FC1) and 0.9 us (output layer) a layer.
__device__ __forceinline__ size_t split_at(int hs, int b, int c)
{
    return (size_t)(c >> 3) * (size_t)(16 * hs) + (size_t)(b * 8 + (c & 7));
}

// Elements c .. c + 3 (c % 4 == 0) of token b.
__device__ __forceinline__ void store_split4(__half *xs, int hs, int b, int c, const float4 &o)
{
    _Float16 hi[4], lo[4];
    split_f32(o.x, hi[0], lo[0]);
    split_f32(o.y, hi[1], lo[1]);
    split_f32(o.z, hi[2], lo[2]);
    split_f32(o.w, hi[3], lo[3]);
    typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
    _Float16 *to = reinterpret_cast<_Float16 *>(xs) + split_at(hs, b, c);
    *reinterpret_cast<half4_t *>(to) = (half4_t){hi[0], hi[1], hi[2], hi[3]};
    *reinterpret_cast<half4_t *>(to + hs * 8) = (half4_t){lo[0], lo[1], lo[2], lo[3]};
}

// x_next may alias x: every element is read and written by the same thread.
// y comes as NY partial sums [NY][B][d] (see k_down2): they are added in order.
// block = glue_threads(d), d <= kGlueMaxD: a thread keeps its NP float4 sums in registers, so every load
// of the kernel is issued before the first one is waited for -- one round trip, then the block
// reduction, then the stores.  NP and NY are the launch's own numbers and the block is as wide as d needs: a CU
// takes 16 cycles for a wave's 16-byte load whether or not its lanes are past the end.  (Four passes of 1024
// threads and four partial sums asked for whatever d and ny -> this, a step of the stack, us: 13B-class gated batch
// 4, 20 layers 1073.9 -> 1038.9; 30B-class batch 8, 12 layers 818.6 -> 798.0; the
// kernel alone 5.2 -> 4.8 and 5.8 -> 4.9.)
constexpr int kGlueMaxD = kGlueThreads * 4 * 4;
inline int glue_passes(int d) { return (d + kGlueThreads * 4 - 1) / (kGlueThreads * 4); }
inline int glue_threads(int d)
{
    const int per_wave = 4 * kWave * glue_passes(d);
    return (d + per_wave - 1) / per_wave * kWave;
}

// xs_next (may be null; d % 8 == 0): the same values as fp16 hi and lo halves, see split_at.
template <int NP, int NY>
__global__ __launch_bounds__(kGlueThreads) void k_glue(const float *x, const float *__restrict__ y,
                                                       float *x_next, int d, __half *xs_next)
{
    __shared__ float wsum[kGlueThreads / kWave];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t pbytes = (uint32_t)gridDim.x * (uint32_t)d * 4u;  // between partial sums
    const rsrc_t xr = make_rsrc(x + (size_t)b * d, (uint32_t)d * 4u);
    const rsrc_t yr = make_rsrc(y + (size_t)b * d, (uint32_t)(NY - 1) * pbytes + (uint32_t)d * 4u);
    float4 v[NP], p[NP][NY];
    const int e0 = (int)threadIdx.x * 4, step = (int)blockDim.x * 4;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int e = i * step + e0;
        const uint32_t off = e < d ? (uint32_t)e * 4u : kOobOffset;
        v[i] = ld16_f32(xr, off);
#pragma unroll
        for (int q = 0; q < NY; ++q) p[i][q] = ld16_f32(yr, e < d ? off + (uint32_t)q * pbytes : kOobOffset);
    }
    // the signs while the loads are in flight (two quarter-rate multiplications per element)
    uint32_t sign[NP][4];
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) sign[i][k] = glue_sign_bit((uint32_t)b, (uint32_t)(i * step + e0 + k));
    __builtin_amdgcn_sched_barrier(0);
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        float4 t = p[i][0];
#pragma unroll
        for (int q = 1; q < NY; ++q)
            t = make_float4(t.x + p[i][q].x, t.y + p[i][q].y, t.z + p[i][q].z, t.w + p[i][q].w);
        v[i] = make_float4(__uint_as_float(__float_as_uint(v[i].x + t.x) ^ sign[i][0]),
                           __uint_as_float(__float_as_uint(v[i].y + t.y) ^ sign[i][1]),
                           __uint_as_float(__float_as_uint(v[i].z + t.z) ^ sign[i][2]),
                           __uint_as_float(__float_as_uint(v[i].w + t.w) ^ sign[i][3]));
        ss = fmaf(v[i].x, v[i].x, fmaf(v[i].y, v[i].y, fmaf(v[i].z, v[i].z, fmaf(v[i].w, v[i].w, ss))));
    }
    ss = wave_sum(ss);
    if (lane == 0) wsum[wave] = ss;
    __syncthreads();
    const float tot = wave_sum(lane < (int)(blockDim.x / kWave) ? wsum[lane] : 0.f);
    const float scale = tot > 0.f ? sqrtf((float)d / tot) : 0.f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int e = i * step + e0;
        if (e < d) {
            const float4 o = make_float4(v[i].x * scale, v[i].y * scale, v[i].z * scale, v[i].w * scale);
            *reinterpret_cast<float4 *>(x_next + (size_t)b * d + e) = o;
            if (xs_next != nullptr) store_split4(xs_next, h_stride((int)gridDim.x), b, e, o);
        }
    }
}

// The signs of the glue as bits: bit e of sign[b][i] is set where column 8 i + e of batch row b changes sign.
// grid = (ceil(stride / 256), kSignRows).
__global__ __launch_bounds__(256) void k_sign_table(uint8_t *__restrict__ sign, int stride)
{
    const int i = (int)blockIdx.x * 256 + (int)threadIdx.x, b = (int)blockIdx.y;
    if (i >= stride) return;
    uint32_t bits = 0;
    for (int e = 0; e < 8; ++e) bits |= (glue_sign_bit((uint32_t)b, (uint32_t)(8 * i + e)) >> 31) << e;
    sign[(size_t)b * stride + i] = (uint8_t)bits;
}

// The same for any d (two passes over the inputs).
__global__ __launch_bounds__(kGlueThreads) void k_glue_long(const float *x, const float *__restrict__ y,
                                                            int ny, float *x_next, int d, __half *xs_next)
{
    __shared__ float wsum[kGlueThreads / kWave];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t pstride = (size_t)gridDim.x * d;
    const float *xb = x + (size_t)b * d, *yb = y + (size_t)b * d;
    auto ysum = [&](int c) {
        float t = yb[c];
        for (int p = 1; p < ny; ++p) t += yb[p * pstride + c];
        return t;
    };
    float ss = 0.f;
    for (int c = threadIdx.x; c < d; c += kGlueThreads) {
        const float v = xb[c] + ysum(c);
        ss = fmaf(v, v, ss);
    }
    ss = wave_sum(ss);
    if (lane == 0) wsum[wave] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < kGlueThreads / kWave; ++k) tot += wsum[k];
    const float scale = tot > 0.f ? sqrtf((float)d / tot) : 0.f;
    for (int c = threadIdx.x; c < d; c += kGlueThreads) {
        const float v = (xb[c] + ysum(c)) * scale;
        const float o = __uint_as_float(__float_as_uint(v) ^ glue_sign_bit((uint32_t)b, (uint32_t)c));
        x_next[(size_t)b * d + c] = o;
        if (xs_next != nullptr) {
            _Float16 hi, lo;
            split_f32(o, hi, lo);
            const int hs = h_stride((int)gridDim.x);
            _Float16 *to = reinterpret_cast<_Float16 *>(xs_next) + split_at(hs, b, c);
            to[0] = hi;
            to[hs * 8] = lo;
        }
    }
}

// The split halves of a caller's activations x[B][d] (d % 8 == 0).  grid = ceil(B * d / 1024),
// block = 256.
__global__ __launch_bounds__(256) void k_split(const float *__restrict__ x, __half *__restrict__ xs, int B, int d)
{
    const int e = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4;
    if (e < B * d) store_split4(xs, h_stride(B), e / d, e % d, *reinterpret_cast<const float4 *>(x + e));
}

}  // namespace pf
