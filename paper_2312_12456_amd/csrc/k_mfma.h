// FC1 over the listed neurons for a batch of tokens as a matrix-core contraction
// (PowerInfer Sec. 8.2, batching: the active set is the union over the batch, so the gathered
// rows form a dense [k x d] block that multiplies [d x B]).  At batch 1 the row-sparse GEMV is
// pure HBM streaming; from a few tokens on, B FMAs and B LDS reads per weight make the vector
// path the limiter before HBM saturates, and v_mfma_f32_16x16x32_f16 does the same work in a
// fraction of the issue slots.  M = 16 gathered rows, N = 16 columns (one per half of each token;
// the others read as zero), K = 32 elements of d per instruction.
// Operand layout (verified on the device): lane l supplies A[row l%16][8 halfs from k = 8*(l/16)]
// and B[same 8 k][col l%16]; it receives C[rows 4*(l/16) .. +3][col l%16].
// x enters as fp16 hi + fp16 lo (split_f32: to 2^-24 of x).  Where the halves come ready-made (XS),
// both ride in one MFMA, as a batch has at most 8 tokens: with hs = h_stride(B) column b multiplies
// the hi half of token b and column hs + b its lo half.  Where a kernel splits fp32 activations itself, each step issues two MFMAs into two tiles (lanes of both
// column ranges splitting the same values measured 2 - 6 % slower: OPT-6.7B shape with every neuron
// listed, batch 8, 54.4 -> 57.7 us).  Each wave's two sums are added first, then the waves' (see
// put_tile): both forms give the same bits.
//
// Weights do not go to the registers in operand order: a load in which each quarter-wave
// touches 16 different rows costs the memory pipeline 16 line look-ups for 256 bytes.
// Instead they go global -> LDS (buffer_load ... lds) in instructions that read 512
// contiguous bytes of each of two rows, and the A operands are read back from LDS.
#pragma once
#include "dev_util.h"
#include "k_predict.h"
#include "k_sparse.h"

namespace pf {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4v_t __attribute__((ext_vector_type(4)));

constexpr int kMfmaThreads = 512;
constexpr int kMfmaWaves = kMfmaThreads / kWave;  // the waves of a block split K between them
// LDS image of one chunk of one matrix in a wave's slot: R rows x KC halfs = 8 KB, for
// R = 32 rows (two MFMA tiles) x 128 elements or R = 16 rows x 256 elements.  The fewer rows a
// block has, the longer its chunks: the bytes in flight per wave stay the same.
constexpr int kMfmaSlotBytes = 8192;

// dynamic LDS of k_up_mfma: [mask words | each wave's prefixes] when compacting itself, then one slot per
// wave and matrix
__host__ __device__ constexpr size_t up_mfma_mask_bytes(int ffn, bool from_mask)
{
    return from_mask ? (size_t)list_words_alloc(ffn / 64) * 8 + (size_t)kMfmaWaves * kListPriv * 4 : 0;
}
inline size_t up_mfma_lds_bytes(int ffn, bool from_mask, bool gated)
{
    // At least 12 bytes a mask word: where this passes the LDS of a CU (gated, ffn from 174784 on) a lane would
    // scan 43 words and more, and the vector form is taken.
    const size_t mask = from_mask ? std::max(up_mfma_mask_bytes(ffn, true), (size_t)ffn / 64 * 12 + 64) : 0;
    return mask / 64 * 64 + (size_t)kMfmaWaves * (gated ? 2 : 1) * kMfmaSlotBytes;
}

union Half8Bits {
    uint4 u;
    half8_t h;
};

// The B operand (activations) of one K step for a lane, as loaded.  From split halves (XS; written
// by the glue kernels, k_split or the hidden layer): the 8 halfs of the lane's column as they are,
// stored in operand order (split_at), so that a wave's load of a K step reads one run of 128 hs
// bytes.  From fp32 activations: elements 0-3 and 4-7 of the lane's token, split into fp16 hi
// (rounded) + lo (residual) when used.
struct XRaw {
    uint4 a, b;
};

// Whether this lane supplies a column, and its first element for the step that starts at element
// k: elem + per_k * k.
struct XLane {
    bool ok;
    int k0;  // of the lane's 8 elements in a step
    uint32_t elem, per_k;
};
template <bool XS>
__device__ __forceinline__ XLane x_lane(int row16, int kg, int B, int K)
{
    const int hs = h_stride(B);
    XLane x;
    x.k0 = kg * 8;
    x.ok = XS ? row16 < 2 * hs && (row16 & (hs - 1)) < B : row16 < B;
    x.elem = XS ? (uint32_t)(kg * 2 * hs + row16) * 8u : (uint32_t)row16 * (uint32_t)K + (uint32_t)kg * 8u;
    x.per_k = XS ? 2u * (uint32_t)hs : 1u;
    return x;
}
// Bytes of the activations of a batch.
template <bool XS>
__device__ __forceinline__ uint32_t x_bytes(int B, int K)
{
    return 4u * (uint32_t)(XS ? h_stride(B) : B) * (uint32_t)K;
}

template <bool XS>
__device__ __forceinline__ XRaw load_xraw(rsrc_t xr, const XLane &x, int k, int K)
{
    XRaw r;
    const bool ok = x.ok && k + (XS ? 0 : x.k0) < K;  // (halves past the end lie past the buffer)
    const uint32_t at = (x.elem + x.per_k * (uint32_t)k) * (XS ? 2u : 4u);
    r.a = ld16_cached(xr, ok ? at : kOobOffset);
    if (!XS) r.b = ld16_cached(xr, ok ? at + 16u : kOobOffset);
    return r;
}

// XS: hi = the column's operand, lo unused.
template <bool XS>
__device__ __forceinline__ void finish_x(const XRaw &r, half8_t &hi, half8_t &lo)
{
    if (XS) {
        Half8Bits h;
        h.u = r.a;
        hi = h.h;
    } else {
        const float v[8] = {__uint_as_float(r.a.x), __uint_as_float(r.a.y), __uint_as_float(r.a.z),
                            __uint_as_float(r.a.w), __uint_as_float(r.b.x), __uint_as_float(r.b.y),
                            __uint_as_float(r.b.z), __uint_as_float(r.b.w)};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            _Float16 h, l;
            split_f32(v[e], h, l);
            hi[e] = h;
            lo[e] = l;
        }
    }
}

// The waves' sums over a tile meet in LDS, [16 rows][16 columns] each.  XS: the lo half of column b is
// column hs + b, and the two are added as they are read.  Else the lo halves are a tile of their own
// and are added first, which keeps the traffic that of one tile and gives the same bits.
template <bool XS>
__device__ __forceinline__ void put_tile(float *ct, float4v_t hi, const float4v_t &lo, int kg, int row16, int hs)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (!XS) hi[e] = fmaf(lo[e], kSplitLo, hi[e]);
        if (XS || row16 < hs) ct[(kg * 4 + e) * 16 + row16] = hi[e];
    }
}
template <bool XS>
__device__ __forceinline__ float get_tile(const float *ct, int e, int el)  // el: of the lo column
{
    return XS ? fmaf(ct[el], kSplitLo, ct[e]) : ct[e];
}

// One row of w (at byte row_off) times token b of the fp32 activations x, by a wave.  For sums that came out NaN
// on the matrix cores: an infinite weight has met a half that is zero, or halves of both signs, where x itself
// gives an infinite sum.  (Where x gives NaN too, this does.)  Never taken with finite weights and activations.
__device__ __forceinline__ float row_sum_f32(rsrc_t w, uint32_t row_off, rsrc_t x, int b, int K, int lane)
{
    float s = 0.f;
#pragma unroll 1
    for (int k0 = 0; k0 < K; k0 += kChunk) {
        const int k = k0 + lane * 8;
        const uint32_t at = k < K ? (uint32_t)(b * K + k) * 4u : kOobOffset;
        const uint4 q = ld16_cached(w, k < K ? row_off + (uint32_t)k * 2u : kOobOffset);
        s = dot8(q, ld16_f32(x, at), ld16_f32(x, k < K ? at + 16u : kOobOffset), s);
    }
    return wave_sum(s);
}

// Put chunk `c` (KC = 4096 / R elements) of the R rows of a pass in flight towards `slot`.  One
// instruction moves 1 KB: 2 KC bytes (whole lines) of each of 512 / KC rows.  Row r stores
// 16-byte piece p at position p ^ (r & 7), so that the 8 rows a group of 8 lanes reads together
// (same piece) fall into 8 different 16-byte bank groups.  rowoff[i] = byte offset of this
// lane's row of instruction i in the matrix (kOobOffset: no row).
template <int R>
__device__ __forceinline__ void mfma_issue_chunk(rsrc_t w, char *slot, const uint32_t (&rowoff)[8],
                                                 int c, int d, int lane)
{
    constexpr int KC = kMfmaSlotBytes / 2 / R;
    constexpr int RPI = 512 / KC, LPR = 64 / RPI;  // rows per instruction, lanes per row
    const int rin = lane / LPR, p = lane % LPR;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int piece = p ^ ((RPI * i + rin) & 7);
        const int k = c * KC + piece * 8;
        const uint32_t off = (k < d && rowoff[i] != kOobOffset) ? rowoff[i] + (uint32_t)k * 2u : kOobOffset;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w, (lds_ptr_t)(slot + i * 1024), 16, (int)off, 0, 0, 0);
    }
}

// What the passes of a block need from the kernel around them.
struct UpMfmaArgs {
    rsrc_t wu, wg, xr, xf;  // xr: the activations as the matrix cores take them; xf: in fp32
    const float *b_up;
    const int32_t *idx_in;
    int32_t *idx_out;
    float *h;
    const uint64_t *words_lds;
    const uint32_t *priv;  // this wave's prefixes
    char *slots;
    int *irow;
    float *brow;
    int B, hs, d, ffn, n, nwords, j_begin, j_end;
    float up_floor;  // gated forms: lower clamp of the up branch (-infinity, or 0 for dReLU)
};

// The list slots [j_begin, j_end) of a block in passes of R rows (R / 16 MFMA tiles).
// PARTS: 4 steps from zero, then into the running sums by ordinary additions, as in rows_mfma_body's hidden
// layer: all steps in one running sum, whose every addition is cut towards minus infinity, were less accurate
// than the vector form wherever a wave has more than a few of them.  Error of FC1 alone against 64 bits, vector
// form / one running sum / parts, 10^-7, batch 5, lists of up to 16 rows a workgroup: ungated d 520 0.80 / 1.04 /
// 0.89, 1032 0.92 / 1.07 / 0.94, 1544 0.99 / 1.07 / 0.93, 2056 1.09 / 1.08 / 0.95, 7176 1.70 / 1.70 / 1.02; gated
// 2056 1.66 / 1.68 / 1.45, 3080 1.91 / 1.99 / 1.49, 7176 2.65 / 2.67 / 1.57.  Parts cost a list's step nothing.
// Longer lists (32 rows a pass, 4 steps a chunk) keep the running sum where d is a multiple of 32: pf_dense_ffn of
// 4096 x 16384 at batch 8 would take 0.8 % longer with parts, gated 5120 x 13824 at batch 4 0.7 %.
template <int R, int ACT, bool FROM_MASK, bool XS, bool PARTS>
__device__ __forceinline__ void up_mfma_passes(const UpMfmaArgs &a)
{
    constexpr bool GATED = (ACT == 1);
    constexpr int NM = GATED ? 2 : 1;
    constexpr int T = R / 16;                      // tiles per pass
    constexpr int KC = kMfmaSlotBytes / 2 / R;     // elements of d per chunk
    constexpr int STEPS = KC / 32;                 // MFMA K steps per chunk
    constexpr int PART = PARTS ? 4 : STEPS;        // ... summed at a time
    constexpr int RPI = 512 / KC, LPR = 64 / RPI;
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    const int row16 = lane & 15, kg = lane >> 4;
    char *slot = a.slots + (size_t)wave * NM * kMfmaSlotBytes;  // this wave's: up, then gate
    const int d = a.d, n = a.n;
    const XLane xl = x_lane<XS>(row16, kg, a.B, d);
    const int nchunks = (d + KC - 1) / KC;

    for (int j0 = a.j_begin; j0 < a.j_end; j0 += R) {
        // list slot -> neuron id: lane l looks row l % R of the pass up
        const int jl = j0 + (lane & (R - 1));
        int id = -1;
        if (FROM_MASK) {
            id = list_select(a.words_lds, a.nwords, a.priv, jl < a.j_end ? jl : n, n);
        } else if (jl < a.j_end) {
            id = a.idx_in[jl];
            if ((unsigned)id >= (unsigned)a.ffn) id = -1;
        }
        // the rows' biases are fetched here and parked in LDS only after the chunk loop, so that
        // wave 0 does not wait for them before it puts its first chunk in flight
        float bpre = 0.f;
        if (wave == 0 && lane < R) {
            a.irow[lane] = id;
            if (a.b_up != nullptr && id >= 0) bpre = a.b_up[id];
            if (FROM_MASK && id >= 0) a.idx_out[jl] = id;
        }
        // byte offsets of the rows this lane fetches: instruction i -> row RPI * i + lane / LPR
        uint32_t rowoff[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int rid = __shfl(id, RPI * i + lane / LPR, 64);
            rowoff[i] = rid >= 0 ? (uint32_t)rid * (uint32_t)d * 2u : kOobOffset;
        }
        if (j0 == a.j_begin) PF_TSTAMP(2, 2);

        float4v_t cu[T], cg[T], lu[T], lg[T];  // lu, lg: lo halves, where the kernel splits
#pragma unroll
        for (int t = 0; t < T; ++t) {
            cu[t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
            cg[t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
            lu[t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
            lg[t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
        }
        const int ntile = min(T, (a.j_end - j0 + 15) >> 4);  // block-uniform: tiles with rows
        int c = wave;
        if (c < nchunks) {
            mfma_issue_chunk<R>(a.wu, slot, rowoff, c, d, lane);
            if (GATED) mfma_issue_chunk<R>(a.wg, slot + kMfmaSlotBytes, rowoff, c, d, lane);
        }
        while (c < nchunks) {  // wave-uniform
            XRaw xv[STEPS];
#pragma unroll
            for (int s = 0; s < STEPS; ++s) xv[s] = load_xraw<XS>(a.xr, xl, c * KC + s * 32, d);
            Half8Bits au[T][STEPS], ag[T][STEPS];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (t >= ntile) break;
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    const int row = 16 * t + row16;
                    const int at = row * (KC * 2) + ((4 * s + kg) ^ (row & 7)) * 16;
                    au[t][s].u = *reinterpret_cast<const uint4 *>(slot + at);
                    if (GATED) ag[t][s].u = *reinterpret_cast<const uint4 *>(slot + kMfmaSlotBytes + at);
                }
            }
            const int cn = c + kMfmaWaves;
            if (cn < nchunks) {  // refill the slot once its contents are in the registers
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
                mfma_issue_chunk<R>(a.wu, slot, rowoff, cn, d, lane);
                if (GATED) mfma_issue_chunk<R>(a.wg, slot + kMfmaSlotBytes, rowoff, cn, d, lane);
            }
#pragma unroll
            for (int s0 = 0; s0 < STEPS; s0 += PART) {
                float4v_t part[4][T];
                if (PARTS) {
#pragma unroll
                    for (int t = 0; t < T; ++t) part[0][t] = part[1][t] = part[2][t] = part[3][t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
                }
                float4v_t(&pu)[T] = PARTS ? part[0] : cu, (&pg)[T] = PARTS ? part[1] : cg;
                float4v_t(&qu)[T] = PARTS ? part[2] : lu, (&qg)[T] = PARTS ? part[3] : lg;
#pragma unroll
                for (int s = s0; s < s0 + PART; ++s) {
                    half8_t hi, lo;
                    finish_x<XS>(xv[s], hi, lo);
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        if (t >= ntile) break;
                        pu[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(au[t][s].h, hi, pu[t], 0, 0, 0);
                        if (!XS) qu[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(au[t][s].h, lo, qu[t], 0, 0, 0);
                        if (GATED) {
                            pg[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ag[t][s].h, hi, pg[t], 0, 0, 0);
                            if (!XS) qg[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ag[t][s].h, lo, qg[t], 0, 0, 0);
                        }
                    }
                }
                if (PARTS) {
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        if (t >= ntile) break;
                        cu[t] += pu[t];
                        if (!XS) lu[t] += qu[t];
                        if (GATED) cg[t] += pg[t];
                        if (GATED && !XS) lg[t] += qg[t];
                    }
                }
            }
            c = cn;
        }
        if (j0 == a.j_begin) PF_TSTAMP(2, 3);
        // this lane holds C[row 4*kg + e][col row16] of its chunks, per tile; the wave's slot
        // is free now: [tile][up | gate][256]
        float *ctile = reinterpret_cast<float *>(slot);
        if (wave == 0 && lane < R) a.brow[lane] = bpre;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            put_tile<XS>(ctile + (t * 2) * 256, cu[t], lu[t], kg, row16, a.hs);
            if (GATED) put_tile<XS>(ctile + (t * 2 + 1) * 256, cg[t], lg[t], kg, row16, a.hs);
        }
        __syncthreads();
        if ((int)threadIdx.x < T * 256) {
            const int t = threadIdx.x >> 8, e = threadIdx.x & 255;
            const int row = 16 * t + (e >> 4), colb = e & 15;
            const int el = (e & ~15) + ((colb + a.hs) & 15);  // the same token's lo column
            float pu[kMfmaWaves], pg[kMfmaWaves];  // added in pairs
#pragma unroll
            for (int wv = 0; wv < kMfmaWaves; ++wv) {
                const float *ct = reinterpret_cast<const float *>(a.slots + (size_t)wv * NM * kMfmaSlotBytes);
                pu[wv] = get_tile<XS>(ct + (t * 2) * 256, e, el);
                pg[wv] = GATED ? get_tile<XS>(ct + (t * 2 + 1) * 256, e, el) : 0.f;
            }
#pragma unroll
            for (int o = kMfmaWaves / 2; o >= 1; o /= 2)
#pragma unroll
                for (int wv = 0; wv < o; ++wv) {
                    pu[wv] += pu[wv + o];
                    pg[wv] += pg[wv + o];
                }
            float su = pu[0], sg = pg[0];
            const int i = a.irow[row];
            const int j = j0 + row;
            // wave by wave (T * 256 is whole waves)
            uint64_t again = __ballot(colb < a.B && j < a.j_end && i >= 0 && (su != su || sg != sg));
            for (; __builtin_expect(again != 0, 0); again &= again - 1) {
                const int l = (int)__builtin_ctzll(again);
                const uint32_t off = (uint32_t)__builtin_amdgcn_readlane(i, l) * (uint32_t)d * 2u;
                const int b = __builtin_amdgcn_readlane(colb, l);
                const float u = row_sum_f32(a.wu, off, a.xf, b, d, lane);
                const float g = GATED ? row_sum_f32(a.wg, off, a.xf, b, d, lane) : 0.f;
                if (lane == l) {
                    su = u;
                    sg = g;
                }
            }
            const float bias = a.brow[row];  // fetched when the row was selected
            const float v = GATED ? fmaxf(sg + bias, 0.f) * fmaxf(su, a.up_floor) : fmaxf(su + bias, 0.f);
            if (colb < a.B && j < a.j_end) a.h[(size_t)j * a.hs + colb] = i >= 0 ? v : 0.f;
        }
        __syncthreads();
        if (j0 == a.j_begin) PF_TSTAMP(2, 4);
    }
}

// grid = G blocks; block b owns the list slots [b * rpb, (b + 1) * rpb), rpb = ceil(n / G): an
// even share of the rows for every block (with whole tiles dealt round-robin the CUs that get
// one tile more than the others set the kernel's time).  A share of at most 16 rows is done
// as one 16-row tile with 256-element chunks, a larger one in passes of 32 rows (two tiles)
// with 128-element chunks.  The 8 waves of a block take the chunks round-robin (wave w:
// chunks w, w + 8, ...) for the same rows and their C tiles are added in LDS in wave order.
// d % 8 == 0, B <= 8: both halves of every token have a column.
// Every wave scans the mask words for itself behind one barrier and looks the pass's rows up one per lane (list_scan,
// list_select).  Block-wide prefix with three barriers and a binary search per row -> this, a step of the stack, us:
// 13B-class gated batch 4, 20 layers 1038.5 -> 1026.0, 30B-class batch 8, 12 layers 797.9 -> 790.4, batch 4 with look-ahead
// 595.0 -> 594.5; the same results.
// The body takes its block number and the number of blocks of its role explicitly, so that a
// launch can run it in a range of its blocks beside another role.  Its pointer parameters carry
// no restrict qualifier on purpose: a wave reads back from LDS what its own global -> LDS loads
// wrote, and the wait between the two is the compiler's, which places it only while it takes
// the two accesses to alias.  Inlining a function with restrict parameters tags its accesses
// with no-alias scopes, and with those the waits were dropped (wrong sums on the device).
// XS: x points at the split halves of the activations (see XRaw) instead of fp32 values.  xf: the fp32 values.
template <int ACT, bool FROM_MASK, bool XS>
__device__ __forceinline__ void up_mfma_body(
    uint64_t *dyn_lds64, int *irow, float *brow, const int bid, const int nblocks,
    const __half *w_up, const __half *w_gate,
    const float *b_up, const void *x, const float *xf, int B,
    const int32_t *idx_in, const int32_t *count_in,
    const uint64_t *mask_words, int32_t *idx_out,
    int32_t *count_out, float *h, int hs, int d, int ffn, float up_floor)
{
    constexpr bool GATED = (ACT == 1);
    const int nwords = ffn / 64;
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    uint64_t *words_lds = dyn_lds64;
    uint32_t *priv = reinterpret_cast<uint32_t *>(words_lds + (FROM_MASK ? list_words_alloc(nwords) : 0)) +
                     (FROM_MASK ? wave * kListPriv : 0);

    PF_TSTAMP(2, 0);
    int n;
    if (FROM_MASK) {
        list_words_issue(words_lds, mask_words, nwords);
        __syncthreads();
        n = list_scan(words_lds, nwords, priv, lane);
        if (bid == 0 && threadIdx.x == 0) *count_out = n;
    } else {
        n = min(max(*count_in, 0), ffn);
    }
    UpMfmaArgs a;
    a.wu = make_rsrc(w_up, (uint32_t)ffn * (uint32_t)d * 2u);
    a.wg = make_rsrc(GATED ? w_gate : w_up, (uint32_t)ffn * (uint32_t)d * 2u);
    a.xr = make_rsrc(x, x_bytes<XS>(B, d));
    a.xf = make_rsrc(xf, x_bytes<false>(B, d));
    a.b_up = b_up;
    a.idx_in = idx_in;
    a.idx_out = idx_out;
    a.h = h;
    a.words_lds = words_lds;
    a.priv = priv;
    a.slots = reinterpret_cast<char *>(dyn_lds64) + up_mfma_mask_bytes(ffn, FROM_MASK);
    a.irow = irow;
    a.brow = brow;
    a.B = B;
    a.hs = hs;
    a.d = d;
    a.ffn = ffn;
    a.n = n;
    a.nwords = nwords;
    a.up_floor = up_floor;
    const int rpb = (n + nblocks - 1) / nblocks;
    a.j_begin = min(n, bid * rpb);
    a.j_end = min(n, a.j_begin + rpb);
    PF_TSTAMP(2, 1);
    if (rpb <= 16)
        up_mfma_passes<16, ACT, FROM_MASK, XS, true>(a);
    else if (d % 32 != 0)
        up_mfma_passes<32, ACT, FROM_MASK, XS, true>(a);
    else
        up_mfma_passes<32, ACT, FROM_MASK, XS, false>(a);
    PF_TSTAMP(2, 5);
}

template <int ACT, bool FROM_MASK, bool XS>
__global__ __launch_bounds__(kMfmaThreads) void k_up_mfma(
    const __half *__restrict__ w_up, const __half *__restrict__ w_gate,
    const float *__restrict__ b_up, const void *__restrict__ x, int B,
    const int32_t *__restrict__ idx_in, const int32_t *__restrict__ count_in,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d, int ffn, float up_floor,
    const float *__restrict__ xf)
{
    extern __shared__ uint64_t dyn_lds64[];
    __shared__ int irow[32];
    __shared__ float brow[32];
    up_mfma_body<ACT, FROM_MASK, XS>(dyn_lds64, irow, brow, (int)blockIdx.x, (int)gridDim.x, w_up, w_gate,
                                 b_up, x, xf, B, idx_in, count_in, mask_words, idx_out, count_out, h, hs, d,
                                 ffn, up_floor);
}

// ---------------------------------------------------------------------------------------
// The predictor's two layers for a batch on the matrix cores (PowerInfer Sec. 5.1): dense
// rows, so no list and no row gather.  Block b owns rows [R b, R (b + 1)); its 8 waves take
// the chunks of KC elements of the row length K round-robin, each through its own 8 KB LDS
// slot of R rows x KC halfs filled by global -> LDS loads that read 2 KC bytes of each of
// 512 / KC rows per instruction (whole lines).  Row r keeps 16-byte piece p at position
// p ^ (r & 7): the 8 rows a group of 8 lanes reads together (same piece) then fall into 8
// different bank groups.  v[B][K] are the activations (fp32 or split halves).
//   EPI 0 (hidden layer, R = 8, KC = 512: few rows, so few and long chunks; rows 8..15 of
//          the MFMA tile are zeros):               out[b][row] = ReLU(sum)          out = t
//   EPI 1 (output layer, R = 64 = one mask word, KC = 64): logit = sum + p_bias[row];
//          scores[b][row] = sigmoid(logit) if asked; bit `row` of mask word b = any_b(logit > thr)
constexpr int kRowsMfmaSlotBytes = 8192;  // R rows x 2 KC bytes

template <int R, int KC>
__device__ __forceinline__ void rows_mfma_issue(rsrc_t w, char *slot, uint32_t row0_off, uint32_t row_bytes,
                                                int nrows_left, int c, int K, int lane)
{
    constexpr int RPI = 512 / KC;  // rows per instruction
    constexpr int LPR = 64 / RPI;  // lanes (16-byte pieces) per row
    constexpr int NI = R / RPI;    // instructions per chunk
    const int rin = lane / LPR, p = lane % LPR;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int row = RPI * i + rin;
        const int piece = p ^ (row & 7);
        const int k = c * KC + piece * 8;
        const uint32_t off = (k < K && row < nrows_left) ? row0_off + (uint32_t)row * row_bytes + (uint32_t)k * 2u
                                                         : kOobOffset;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w, (lds_ptr_t)(slot + i * 1024), 16, (int)off, 0, 0, 0);
    }
}

// Body: bid0 = the block's number within its role, logit_s = [16][16 * tiles] floats of LDS.
// No restrict qualifiers, for the same reason as in up_mfma_body.
// XS: v points at the split halves of the activations (see XRaw) instead of fp32 values.  vf (EPI 0): the fp32 values.
// out_split (EPI 0; may be null): the hidden vector goes there as split halves, the form in which
// the output layer's matrix-core kernel takes it, instead of to out.
template <int R, int KC, int EPI, bool XS>
__device__ __forceinline__ void rows_mfma_body(
    uint64_t *dyn_lds64, float (*logit_s)[16 * ((R + 15) / 16)], const int bid0,
    const __half *w, const void *v, const float *vf, int B, int K, int nrows,
    const float *p_bias, float thr_logit, float *out,
    uint64_t *mask_words, int first_word, __half *out_split = nullptr)
{
    constexpr int T = (R + 15) / 16;  // MFMA tiles per block
    static_assert(R * KC * 2 == kRowsMfmaSlotBytes, "slot size");
    static_assert(EPI == 0 || R == 64, "the output layer writes one mask word per block");
    constexpr int STEPS = KC / 32;                // MFMA K steps per chunk
    constexpr int SB = STEPS < 4 ? STEPS : 4;     // ... of which this many share a round of loads
    const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
    const int row16 = lane & 15, kg = lane >> 4;
    char *slots = reinterpret_cast<char *>(dyn_lds64);
    char *slot = slots + (size_t)wave * kRowsMfmaSlotBytes;
    // EPI 1: the launch covers the rows from 64 * first_word on (always-on prefix skipped)
    const int blk = bid0 + (EPI == 1 ? first_word : 0);
    const int r0 = blk * R;
    const int nleft = nrows - r0;  // rows of this block that exist (>= 1)
    if (EPI == 1 && bid0 == 0 && first_word > 0) {
        for (int w = threadIdx.x; w < first_word; w += kMfmaThreads) mask_words[w] = ~0ull;
        if (out != nullptr)
            for (int e = threadIdx.x; e < B * first_word * 64; e += kMfmaThreads)
                out[(size_t)(e / (first_word * 64)) * nrows + e % (first_word * 64)] = 1.f;
    }
    const rsrc_t wr = make_rsrc(w, (uint32_t)nrows * (uint32_t)K * 2u);
    const rsrc_t vr = make_rsrc(v, x_bytes<XS>(B, K));
    const uint32_t row_bytes = (uint32_t)K * 2u, row0_off = (uint32_t)r0 * row_bytes;
    const XLane xl = x_lane<XS>(row16, kg, B, K);
    const int nchunks = (K + KC - 1) / KC, hs = h_stride(B);

    PF_TSTAMP(EPI, 0);
    float4v_t acc[T], acc_lo[T];  // acc_lo: lo halves, where the kernel splits
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = acc_lo[t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
    // activations of sub-block j (SB K steps) of chunk ch into one of two register buffers: they
    // are fetched one sub-block ahead of their use, so that their L2 round trip overlaps the
    // matrix work of the sub-block before
    constexpr int NSB = STEPS / SB;
    XRaw xv[2][SB];
    auto load_x = [&](int ch, int j, XRaw (&px)[SB]) {
#pragma unroll
        for (int s = 0; s < SB; ++s) px[s] = load_xraw<XS>(vr, xl, ch * KC + (j * SB + s) * 32, K);
    };
    int c = wave;
    if (c < nchunks) {
        rows_mfma_issue<R, KC>(wr, slot, row0_off, row_bytes, nleft, c, K, lane);
        load_x(c, 0, xv[0]);
    }
    // output layer: the biases of the rows this thread finishes, fetched behind the first chunk
    // (read only after the chunk loop: their latency is off the block's tail)
    constexpr int NE = (T * 256 + kMfmaThreads - 1) / kMfmaThreads;
    float bias_pre[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = (int)threadIdx.x + i * kMfmaThreads;
        const int row = (e >> 8) * 16 + ((e >> 4) & 15);
        bias_pre[i] = (EPI == 1 && p_bias != nullptr && e < T * 256) ? p_bias[r0 + row] : 0.f;
    }
    while (c < nchunks) {  // wave-uniform
        const int cn = c + kMfmaWaves;
#pragma unroll
        for (int j = 0; j < NSB; ++j) {
            const int cur = j & 1, nxt = cur ^ 1;
            Half8Bits a[T][SB];
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int s = 0; s < SB; ++s) {
                    const int row = 16 * t + row16;
                    a[t][s].u = make_uint4(0u, 0u, 0u, 0u);
                    if (R >= 16 || row < R)
                        a[t][s].u = *reinterpret_cast<const uint4 *>(
                            slot + row * (KC * 2) + ((4 * (j * SB + s) + kg) ^ (row & 7)) * 16);
                }
            if (j + 1 < NSB) {
                load_x(c, j + 1, xv[nxt]);
            } else if (cn < nchunks) {  // last sub-block: refill the slot, fetch the next chunk's x
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the slot is all in registers
                rows_mfma_issue<R, KC>(wr, slot, row0_off, row_bytes, nleft, cn, K, lane);
                load_x(cn, 0, xv[nxt]);
            }
            // EPI 0: SB steps from zero, then into the running sums by ordinary additions.  (The matrix
            // cores round after every 8 products and cut the running sum towards minus infinity.)
            // Error of the scores against 64 bits, vector hidden layer / all steps in one running sum
            // / this: 4 x 4096, r 1024 1.10 / 1.13 / 0.93 * 10^-7; 8 x 2048, r 512 0.92 / 1.07 / 0.85.
            // Every step from zero is no better and 0.3 us slower.
            float4v_t part[T], part_lo[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                part[t] = EPI == 0 ? (float4v_t){0.f, 0.f, 0.f, 0.f} : acc[t];
                part_lo[t] = EPI == 0 ? (float4v_t){0.f, 0.f, 0.f, 0.f} : acc_lo[t];
            }
#pragma unroll
            for (int s = 0; s < SB; ++s) {
                half8_t hi, lo;
                finish_x<XS>(xv[cur][s], hi, lo);
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    part[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t][s].h, hi, part[t], 0, 0, 0);
                    if (!XS) part_lo[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t][s].h, lo, part_lo[t], 0, 0, 0);
                }
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                acc[t] = EPI == 0 ? acc[t] + part[t] : part[t];
                acc_lo[t] = EPI == 0 ? acc_lo[t] + part_lo[t] : part_lo[t];
            }
        }
        if (NSB & 1) {  // the next chunk starts from buffer 0 again
#pragma unroll
            for (int s = 0; s < SB; ++s) xv[0][s] = xv[1][s];
        }
        c = cn;
    }
    PF_TSTAMP(EPI, 1);
    // this lane holds C[tile t][row 4*kg + e][col row16] of its chunks; the slot is free now
    float *ctile = reinterpret_cast<float *>(slot);
#pragma unroll
    for (int t = 0; t < T; ++t) put_tile<XS>(ctile + t * 256, acc[t], acc_lo[t], kg, row16, hs);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = (int)threadIdx.x + i * kMfmaThreads;
        if (e >= T * 256) break;
        const int row = (e >> 8) * 16 + ((e >> 4) & 15), col = e & 15;
        const int el = (e & ~15) + ((col + hs) & 15);  // the same token's lo column
        float s[kMfmaWaves];  // added in pairs: the error of a chain of 8 is a third larger
#pragma unroll
        for (int wv = 0; wv < kMfmaWaves; ++wv)
            s[wv] = get_tile<XS>(reinterpret_cast<const float *>(slots + (size_t)wv * kRowsMfmaSlotBytes), e, el);
#pragma unroll
        for (int o = kMfmaWaves / 2; o >= 1; o /= 2)
#pragma unroll
            for (int wv = 0; wv < o; ++wv) s[wv] += s[wv + o];
        float sum = s[0];
        if (EPI == 0) {
            const rsrc_t fr = make_rsrc(vf, x_bytes<false>(B, K));
            uint64_t again = __ballot(col < B && row < R && row < nleft && sum != sum);
            for (; __builtin_expect(again != 0, 0); again &= again - 1) {  // wave by wave (T * 256 is whole waves)
                const int l = (int)__builtin_ctzll(again);
                const float u = row_sum_f32(wr, row0_off + (uint32_t)__builtin_amdgcn_readlane(row, l) * row_bytes, fr,
                                            __builtin_amdgcn_readlane(col, l), K, lane);
                if (lane == l) sum = u;
            }
            if (col < B && row < R && row < nleft) {
                const float o = fmaxf(sum, 0.f);
                if (out_split != nullptr) {
                    _Float16 hi, lo;
                    split_f32(o, hi, lo);
                    _Float16 *to = reinterpret_cast<_Float16 *>(out_split) + split_at(hs, col, r0 + row);
                    to[0] = hi;
                    to[hs * 8] = lo;
                } else {
                    out[(size_t)col * nrows + r0 + row] = o;
                }
            }
        } else {
            const float lg = sum + bias_pre[i];
            logit_s[col][row] = lg;
            if (out != nullptr && col < B) out[(size_t)col * nrows + r0 + row] = 1.f / (1.f + __expf(-lg));
        }
    }
    if (EPI == 1) {
        __syncthreads();
        if (wave == 0) {
            bool on = false;
            for (int b = 0; b < B; ++b) on = on || logit_s[b][lane] > thr_logit;
            const uint64_t word = __ballot(on);
            if (lane == 0) mask_words[blk] = word;
        }
    }
    PF_TSTAMP(EPI, 2);
}

// (vf, and xf of FC1's kernels, come last: in front they pushed arguments that are needed at once into another line,
// 0.3 us a launch.)
template <int R, int KC, int EPI, bool XS>
__global__ __launch_bounds__(kMfmaThreads) void k_rows_mfma(
    const __half *__restrict__ w, const void *__restrict__ v, int B, int K, int nrows,
    const float *__restrict__ p_bias, float thr_logit, float *__restrict__ out,
    uint64_t *__restrict__ mask_words, int first_word, const int32_t *__restrict__ skip,
    __half *__restrict__ out_split, const float *__restrict__ vf)
{
    extern __shared__ uint64_t dyn_lds64[];
    constexpr int T = (R + 15) / 16;
    __shared__ float logit_s[16][16 * T];
    // adaptive layer step: a set flag means this step runs dense (no prediction; all marked)
    if (skip != nullptr && *skip != 0) {
        if (EPI == 1) {
            if (threadIdx.x == 0) mask_words[first_word + (int)blockIdx.x] = ~0ull;
            if (blockIdx.x == 0)
                for (int w = threadIdx.x; w < first_word; w += kMfmaThreads) mask_words[w] = ~0ull;
        }
        return;
    }
    rows_mfma_body<R, KC, EPI, XS>(dyn_lds64, logit_s, (int)blockIdx.x, w, v, vf, B, K, nrows, p_bias, thr_logit,
                               out, mask_words, first_word, out_split);
}

// ---------------------------------------------------------------------------------------
// FC2 over the listed neurons for a batch, on the matrix cores: y^T[column][token] =
// sum over slots of W_down^T[row][column] * h[slot][token].  The vector form (down2_body) issues
// 8 B + 12 vector instructions per 16-byte load; here it is about 35 whatever the batch.
// Tiling of down2_body: a workgroup owns 64 columns (a whole 128-byte line per row) and every
// P-th chunk of 64 list slots of each wave, and a lane loads 16 bytes (columns 8 cl .. 8 cl + 7,
// cl = lane % 8) of each of 8 rows.  No LDS and no cross-lane step stands between these loads and
// the matrix cores: for column t of its eight a lane collects the t-th halfs of its 8 rows (4
// byte permutes) and has one MFMA operand -- M row lane % 16 = (row slot parity, column group
// cl), K = the 8 rows in each of 4 lane groups.  The two row-slot parities share M and N: rows
// m < 8 belong to even row slots and need tokens n < 8, rows m >= 8 to odd ones and n >= 8, so
// B's columns carry h of the even slots' rows for tokens 0..7, then of the odd slots' rows.
// The two off-diagonal 8 x 8 blocks of the result are not used (the matrix cores have room:
// 24 MFMAs per 8 KB of weights).  A lane's B operand is then h of exactly the rows that it loads.
// h enters with all of its 24 bits, as three fp16 parts of 8 bits each: h * 2^s = p1 + p2 / 2^8 +
// p3 / 2^16, s per chunk, token and slot parity such that the largest |h| lands in [2^14, 2^15).
// The split is exact down to 2^-31 of that largest value; a wave that meets a smaller h other than
// zero forms its sums without the matrix cores, so that a column in which the large values have no
// weight is as accurate as any other.
// Precision: a matrix instruction takes its products in four groups of 8 (k = 0..7, 8..15, ...; all
// of this measured on the device).  In each group it cuts the products, towards zero, and the sum so
// far, towards minus infinity, at 2^-26 of (a bound on) the largest product, adds, and rounds to
// nearest.  So each part's products are summed from zero and added to the running sum by ordinary
// operations, 8-bit parts leave the products 5 bits before the cut reaches them, and the rows of odd
// slots enter negated, which turns the bias of the second cut round (without: -1 to -6 * 10^-8 of the
// rms).  Error of this kernel alone against 64 bits (2-norm, 1e-8; list length x d, batch 4), in
// front the vector form, behind it two 11-bit halves under a running scale with the 16 partial sums
// added in a chain: 1500 x 2048 9.3 / 10.4 -> 8.0; 2600 x 4096 9.6 / 11.4 -> 8.3; 5000 x 5120 10.6 /
// 11.6 -> 8.7; 28672 x 7168 15.9 / 13.4 -> 10.8.
// Bound by memory: ids and h of the next chunk are requested in front of the rows of this one, so
// a wave waits for one round trip per 8 KB.  126 registers leave room for two workgroups per CU
// (the second launch of the look-ahead form needs that).
// Vector form -> this one, us: OPT-30B shape batch 8 (65 MB) 21.0 -> 16.6, LLaMA-13B shape batch 4
// (44 MB) 14.8 -> 12.0, all 16384 neurons of an OPT-6.7B layer at batch 4 (134 MB) 35.3 -> 25.7.
// (With two halves of h: 0.4 us less at most.)
constexpr int kDown2mRows = 64;                       // list slots per chunk (one wave)
constexpr int kDown2mPitch = kDown2Cols + 4;          // floats per token row of the partial sums
constexpr int kDown2mRedFloats = 2 * kDown2Waves * 8 * kDown2mPitch;

struct Down2mIds {
    int iv;       // list entry of slot lane of the chunk
    float h[8];   // h of this lane's token (lane % 8) and rows
};
struct Down2mOps {
    half8_t p1, p2, p3;  // B operand: h * scale = p1 + p2 / 2^8 + p3 / 2^16
};

// a, b cut to their 8 leading bits as fp16 halves (subnormal halves to multiples of 2^-21).
__device__ __forceinline__ uint32_t top8_halves(float a, float b)
{
    const auto h = __builtin_amdgcn_cvt_pkrtz(a, b);
    uint32_t u;
    __builtin_memcpy(&u, &h, 4);
    return u & 0xFFF8FFF8u;
}
__device__ __forceinline__ float half_f32(uint32_t pair, int i)
{
    const uint16_t u = (uint16_t)(pair >> (16 * i));
    _Float16 h;
    __builtin_memcpy(&h, &u, 2);
    return (float)h;
}

template <bool SHORT = false>
__device__ __forceinline__ void down2_mfma_body(
    float *red, const int tile, const int g, const int P, const __half *w_down, const float *b_down,
    const float *h, const int32_t *idx, const int32_t *count_p, float *part, int B, int hs, int d, int ffn)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cl = lane & 7, rs = lane >> 3;
    const bool colok = tile * kDown2Cols + cl * 8 < d;
    const rsrc_t wd = make_rsrc(w_down, (uint32_t)ffn * (uint32_t)d * 2u);
    const rsrc_t ir = make_rsrc(idx, (uint32_t)ffn * 4u);
    const rsrc_t hr = make_rsrc(h, (uint32_t)ffn * (uint32_t)hs * 4u);
    const uint32_t colbyte = (uint32_t)(tile * kDown2Cols + cl * 8) * 2u;

    // ids and h of chunk c: addresses depend on the slot number only (slots past the arrays' end
    // read zeros)
    auto request = [&](Down2mIds &r, int c) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = c * kDown2mRows + u * 8 + rs;
            r.h[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                hr, cl < B && j < ffn ? (int)((uint32_t)(j * hs + cl) * 4u) : (int)kOobOffset, 0, 0));
        }
        const int j = c * kDown2mRows + lane;
        r.iv = (int)__builtin_amdgcn_raw_buffer_load_b32(ir, j < ffn ? j * 4 : (int)kOobOffset, 0, 0);
    };
    // weight rows of chunk c; h of slots without a row becomes 0
    auto load_rows = [&](uint4 (&w)[8], Down2mIds &r, int c, int n) {
        const bool ok = c * kDown2mRows + lane < n && (unsigned)r.iv < (unsigned)ffn;
        const uint32_t row = ok ? (uint32_t)r.iv * (uint32_t)d * 2u : kOobOffset;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t ro = (uint32_t)__shfl((int)row, u * 8 + rs, 64);
            w[u] = ld16_stream(wd, colok && ro != kOobOffset ? ro + colbyte : kOobOffset);
            r.h[u] = ro != kOobOffset ? r.h[u] : 0.f;
        }
    };
    float4v_t acc[8];  // [t][i]: column 8 (m % 8) + t of m = 4 (lane / 16) + i
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = (float4v_t){0.f, 0.f, 0.f, 0.f};
    // The operand of a chunk, and in f what takes its products back to h's units.  True where the
    // three parts do not hold every bit of every h.
    auto operands = [&](Down2mOps &o, float &f, const Down2mIds &r) {
        float m = 0.f;
        uint32_t least = ~0u;  // of 2 bits(|h|) - 1: zero counts as the largest
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            m = fmaxf(m, fabsf(r.h[u]));
            least = min(least, (__float_as_uint(r.h[u]) << 1) - 1u);
        }
        m = fmaxf(m, __shfl_xor(m, 16, 64));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        const int e = max((int)(__float_as_uint(m) >> 23), 15);  // 15 .. 255: both scales are normal
        const uint32_t sign = (uint32_t)(lane & 8) << 28;        // odd row slots
        const float scale = __uint_as_float(sign | (uint32_t)(268 - e) << 23);
        f = __uint_as_float(sign | (uint32_t)(e - 14) << 23);
        uint32_t p1[4], p2[4], p3[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {  // every step but the last conversion is exact
            const float v0 = r.h[2 * k] * scale, v1 = r.h[2 * k + 1] * scale;
            p1[k] = top8_halves(v0, v1);
            const float a0 = fmaf(-256.f, half_f32(p1[k], 0), 256.f * v0);
            const float a1 = fmaf(-256.f, half_f32(p1[k], 1), 256.f * v1);
            p2[k] = top8_halves(a0, a1);
            const auto h = __builtin_amdgcn_cvt_pkrtz(fmaf(-256.f, half_f32(p2[k], 0), 256.f * a0),
                                                      fmaf(-256.f, half_f32(p2[k], 1), 256.f * a1));
            __builtin_memcpy(&p3[k], &h, 4);
        }
        Half8Bits b;
        b.u = make_uint4(p1[0], p1[1], p1[2], p1[3]);
        o.p1 = b.h;
        b.u = make_uint4(p2[0], p2[1], p2[2], p2[3]);
        o.p2 = b.h;
        b.u = make_uint4(p3[0], p3[1], p3[2], p3[3]);
        o.p3 = b.h;
        return least < (uint32_t)max(e - 31, 0) << 24;  // some 0 < |h * scale| < 2^-17
    };
    auto multiply = [&](const uint4 (&w)[8], const Down2mOps &o, float f) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t sel = (t & 1) ? 0x07060302u : 0x05040100u;
            auto dw = [&](int u) { return t < 2 ? w[u].x : t < 4 ? w[u].y : t < 6 ? w[u].z : w[u].w; };
            Half8Bits a;
            a.u = make_uint4(__builtin_amdgcn_perm(dw(1), dw(0), sel), __builtin_amdgcn_perm(dw(3), dw(2), sel),
                             __builtin_amdgcn_perm(dw(5), dw(4), sel), __builtin_amdgcn_perm(dw(7), dw(6), sel));
            // each part's products from zero, then into the running sum by ordinary operations
            const float4v_t z = {0.f, 0.f, 0.f, 0.f};
            const float4v_t s3 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, o.p3, z, 0, 0, 0);
            const float4v_t s2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, o.p2, z, 0, 0, 0);
            const float4v_t s1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, o.p1, z, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[t][i] = fmaf(fmaf(fmaf(s3[i], 0x1p-8f, s2[i]), 0x1p-8f, s1[i]), f, acc[t][i]);
            __builtin_amdgcn_sched_barrier(0);  // bounds the registers of the chunk's sums
        }
    };
    // Lane l holds C[m = 4 (l / 16) + i][n = l % 16]; on the diagonal blocks that is row-slot parity
    // l / 32, columns 32 (l / 16 % 2) + 8 i + t, token l % 8.
    const int par = lane >> 5, chalf = (lane >> 4) & 1;
    const bool mine = par == ((lane >> 3) & 1);
    const int step = kDown2Waves * P;
    int c = wave * P + g;
    Down2mIds ra, rb;
    uint4 w[8];
    Down2mOps o;
    float f;
    Down2Round<4> rs4;
    if (SHORT) down2_request<4>(rs4, 0, wave * 8 + rs, g, P, h, idx, ffn);
    request(ra, c);
    const int n = min(max(wave_uniform(*count_p), 0), ffn);
    if (SHORT && n <= kDown2RowsPerLoad * Down2Shape<4>::U * P) {  // the same in all workgroups
        const float bpre = down2_bias(b_down, tile, g, d);
        float a4[32];
#pragma unroll
        for (int e = 0; e < 32; ++e) a4[e] = 0.f;
        down2_round<4>(a4, rs4, wd, 0, wave * 8 + rs, g, P, tile * kDown2Cols + cl * 8, n, d, ffn);
        down2_finish<4>(a4, reinterpret_cast<float(*)[4][kDown2Cols]>(red), tile, g, bpre, part, d);
        return;
    }
    const int nc = (n + kDown2mRows - 1) / kDown2mRows;
    bool again = false;
    for (; c < nc; c += step) {
        request(rb, c + step);  // ahead of the rows, so that the next chunk's do not wait for it
        load_rows(w, ra, c, n);
        again |= operands(o, f, ra);
        multiply(w, o, f);
        ra = rb;
    }
    const float bpre = down2_bias(b_down, tile, g, d);  // there is no register for it before
    // An infinite weight or h may have met a part of h that is zero, or another of the other sign.
    float nan = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) nan = fmaf(acc[t][i], 0.f, nan);
    again |= mine && nan != 0.f;

    float *to = red + ((wave * 2 + par) * 8 + cl) * kDown2mPitch + 32 * chalf;
    if (__ballot(again) == 0) {
        if (mine) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *reinterpret_cast<float4 *>(to + 8 * i) = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
                *reinterpret_cast<float4 *>(to + 8 * i + 4) = make_float4(acc[4][i], acc[5][i], acc[6][i], acc[7][i]);
            }
        }
    } else {
        // Sums that the parts do not hold, or that are not finite: all of the wave's once more in fp32,
        // row by row.  Hardly ever taken, so it is kept small and out of the loop: one copy of it in the
        // loop and one behind slowed down the workgroups of the other role in the look-ahead launch
        // (OPT-30B shape, batch 4: 26.5 -> 28.3 us).
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const int col = tile * kDown2Cols + 32 * chalf + 8 * i;
            float tot[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) tot[t] = 0.f;
#pragma unroll 1
            for (c = wave * P + g; c < nc; c += step) {
                const int jl = c * kDown2mRows + lane;
                const int il = (int)__builtin_amdgcn_raw_buffer_load_b32(ir, jl < n ? jl * 4 : (int)kOobOffset, 0, 0);
                const uint32_t row =
                    jl < n && (unsigned)il < (unsigned)ffn ? (uint32_t)il * (uint32_t)d * 2u : kOobOffset;
                float sum[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) sum[t] = 0.f;
#pragma unroll 1
                for (int s = 0; s < kDown2mRows / 2; ++s) {
                    const int slot = 2 * s + par, j = c * kDown2mRows + slot;
                    const uint32_t ro = (uint32_t)__shfl((int)row, slot, 64);
                    const bool ok = mine && cl < B && ro != kOobOffset;  // then j < n
                    const float hv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        hr, ok ? (int)((uint32_t)(j * hs + cl) * 4u) : (int)kOobOffset, 0, 0));
                    const uint4 q = ld16_cached(wd, ok && col < d ? ro + (uint32_t)col * 2u : kOobOffset);
                    const uint32_t qd[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        sum[t] = fmaf(hv, (t & 1) ? h_hi(qd[t / 2]) : h_lo(qd[t / 2]), sum[t]);
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) tot[t] += sum[t];
            }
            if (mine) {
                *reinterpret_cast<float4 *>(to + 8 * i) = make_float4(tot[0], tot[1], tot[2], tot[3]);
                *reinterpret_cast<float4 *>(to + 8 * i + 4) = make_float4(tot[4], tot[5], tot[6], tot[7]);
            }
        }
    }
    __syncthreads();
    const int b = threadIdx.x / kDown2Cols, oc = tile * kDown2Cols + (int)threadIdx.x % kDown2Cols;
    if (b < B && oc < d) {
        // the 16 sums in pairs: a chain of 16 additions would be the largest error of the kernel
        float s[2 * kDown2Waves];
#pragma unroll
        for (int k = 0; k < 2 * kDown2Waves; ++k)
            s[k] = red[(k * 8 + b) * kDown2mPitch + (int)threadIdx.x % kDown2Cols];
#pragma unroll
        for (int o2 = kDown2Waves; o2 >= 1; o2 /= 2)
#pragma unroll
            for (int k = 0; k < o2; ++k) s[k] += s[k + o2];
        part[((size_t)g * B + b) * d + oc] = bpre + s[0];
    }
}

// grid = (d / 64 tiles, P), block = 512.
// SHORT (batch 4): a list that one round of the vector form covers (256 rows per row group) is added up
// by that form's code -- its waves then share the rows evenly, where most waves here would have no
// chunk and the others 0.8 us of work after their rows have arrived.  Both forms' first loads leave
// together, as the length of the list is only known on the device.  A step of 12 layers, us, vector
// kernel / always this form / this rule: 768 x 3072, 15 % active 218 / 225 / 218; 2048 x 5120, 8 %
// 265 / 273 / 265, 15 % (longer lists) 286 / 282 / 279; 768 x 3072, 4 % 211 / 215 / 213.  From batch 5
// on the vector form has no such range.
template <bool SHORT>
__global__ __launch_bounds__(kDown2Threads, 4) void k_down2_mfma(
    const __half *__restrict__ w_down, const float *__restrict__ b_down, const float *__restrict__ h,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ count_p, float *__restrict__ part, int B, int hs,
    int d, int ffn)
{
    __shared__ __align__(16) float red[kDown2mRedFloats];
    down2_mfma_body<SHORT>(red, (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.y, w_down, b_down, h, idx, count_p,
                           part, B, hs, d, ffn);
}

}  // namespace pf
