// Look-ahead prediction with the overlap realised inside the launches (PowerInfer Sec. 2.1: the
// activations of a layer can be predicted from an earlier layer's input).  With the active set
// of layer l+1 taken from its predictor applied to the INPUT of layer l, the predictor of the
// next layer and the sparse kernels of this layer are independent, and a layer becomes two
// launches whose block ranges play two roles each:
//   k_la_up_hidden : blocks [0, n_hid)   hidden layer of predictor l+1 on x_l     (k_predict.h)
//                    blocks [n_hid, ..)  FC1 of layer l over mask_l                (k_sparse.h)
//   k_la_down_out  : blocks [0, n_fc2)   FC2 of layer l over the list FC1 left     (k_sparse.h)
//                    blocks [n_fc2, ..)  output layer of predictor l+1 -> mask_l+1 (k_predict.h)
// The dense predictor rows stream while the dependent chains of the sparse kernels (mask scan,
// list, gathered rows) wait on memory, in the same launch: nothing is gained from a second
// stream on this part (graph branches replay one after the other), but workgroups of two roles
// share the CUs.  Inside a stack both roles of the first launch form the layer input from the
// previous layer's input and FC2 partial sums themselves (GLUE); FC1's first block stores it.
// The role bodies are the stand-alone kernels' own.  Three families: the vector kernels (fp16,
// batch <= 3; below), the matrix-core kernels (fp16, larger batches) and the int4 kernels
// (further down; those two read a layer input that a glue kernel in front has formed).
#pragma once
#include "dev_util.h"
#include "k_predict.h"
#include "k_sparse.h"
#include "k_mfma.h"
#include "k_int4.h"

namespace pf {

static_assert(kUpThreads == kPredThreads, "both roles of the first launch use the same block size");

// grid = n_hid + n_up, block = 256.  Dynamic LDS: staged input [B][dpad] + scrap + mask scan.
template <int B, int ACT, bool GLUE>
__global__ __launch_bounds__(kUpThreads) void k_la_up_hidden(
    int n_hid, const __half *__restrict__ p1, float *__restrict__ t, int r,
    const __half *__restrict__ w_up, const __half *__restrict__ w_gate,
    const float *__restrict__ b_up, const float *__restrict__ x, const float *__restrict__ yp, int ny,
    int ypstride, float *__restrict__ x_new, const uint64_t *__restrict__ mask_words,
    int32_t *__restrict__ idx_out, int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d,
    int ffn, float up_floor, bool up_first)
{
    extern __shared__ float xs[];
    __shared__ uint32_t wave_tot[kUpWaves];
    __shared__ float ss_w[kUpWaves][B];
    // up_first: FC1's blocks take the low block numbers (dispatched first)
    const int n_up = (int)gridDim.x - n_hid;
    const int bid = (int)blockIdx.x;
    const bool is_hid = up_first ? bid >= n_up : bid < n_hid;
    if (is_hid) {  // uniform over the block
        pred_hidden_body<B, GLUE, (B >= 2 ? 1 : 4)>(xs, ss_w, up_first ? bid - n_up : bid, false, p1, x, yp,
                                                    ny, ypstride, x_new, t, d, r, 0);
    } else {
        const int ub = up_first ? bid : bid - n_hid;
        up_body<B, ACT, true, GLUE>(xs, wave_tot, ss_w, ub, n_up, ub == 0, w_up, w_gate, b_up, x, nullptr,
                                    nullptr, mask_words, idx_out, count_out, h, hs, d, ffn, up_floor,
                                    yp, ny, ypstride, x_new);
    }
}

// The same with the activations held by column (up_cols_body, hidden_cols_body; rows of up to 512 CPW chunks
// per wave).  grid = n_up + ceil(r / hid_rows), block = 64 * cols_waves(d): FC1's blocks have the low
// numbers.  Dynamic LDS: up_cols_lds_bytes.  Two workgroups fit a CU, one of either role: at most 128
// registers up to two chunks per wave, and hid_rows (2, 4 or la_hid_rows_max) rows of the hidden layer per block.
// No scratch memory: the glue is formed token by token, the hidden layer's body knows that one pass covers the
// row, and where two tokens meet two chunks a wave there are at most 4 rows of the hidden layer and, gated, one
// row of FC1 at a time.  (All tokens at once, 6 and 2 rows: up to 162 registers in scratch and, us, 8192 x 26176
// batch 2 (4 layers) 242 against 213 now, gated 7168 x 22912 batch 2 (4) 240 / 210, 3072 x 9792, r 1536 batch 3 (12)
// 337 / 261, 4096 x 13056, r 2048 batch 3 (7) 246 / 205.)
// One wave per row with x in LDS -> this, and the second launch with two workgroups per CU, a step of the stack,
// us: 30B-class batch 1 (8 layers) 303 -> 263, batch 2 387 -> 342, 13B-class gated (12) 331 -> 305, 7B-class batch 1
// 563 -> 548, batch 2 (12) 285 -> 255, 3000 x 9600 batch 2 (8) 153 -> 132.
constexpr __host__ __device__ int la_hid_rows_max(int B, int cpw) { return B * cpw >= 3 ? 4 : 6; }

template <int B, int ACT, bool GLUE, int CPW>
__global__ __launch_bounds__(64 * kColsMaxWaves) __attribute__((amdgpu_waves_per_eu(CPW <= 2 ? 4 : 2, 4))) void
k_la_up_hidden_cols(
    int n_up, int hid_rows, const __half *__restrict__ p1, float *__restrict__ t, int r, const __half *__restrict__ w_up,
    const __half *__restrict__ w_gate, const float *__restrict__ b_up, const float *__restrict__ x, GlueIn gi,
    float *__restrict__ x_new, const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d, int ffn, float up_floor)
{
    extern __shared__ __align__(16) char cols_lds[];
    const int bid = (int)blockIdx.x;
    if (bid < n_up) {  // uniform over the block
        constexpr int R = B == 2 && CPW == 2 && ACT == 1 ? 1 : UpColsR<B, ACT, CPW>::value;
        up_cols_body<B, ACT, true, GLUE, CPW, R, (CPW * B > 2), 1>(
            cols_lds, bid, n_up, bid == 0, w_up, w_gate, b_up, x, gi, x_new, nullptr, nullptr, mask_words, idx_out,
            count_out, h, hs, d, ffn, up_floor);
    } else {
        constexpr int RED = kColsMaxWaves * cols_red_floats(7 * B);
        static_assert(RED <= kUpColsRows * kColsMaxWaves, "the hidden layer's sums fit FC1's LDS");
        float *xch = reinterpret_cast<float *>(cols_lds);
        auto hidden = [&](auto rows) {
            hidden_cols_body<B, GLUE, CPW, decltype(rows)::value, (CPW * B > 2), 1, true>(
                xch + (blockDim.x >> 6) * kColsXFloats, xch + (threadIdx.x >> 6) * kColsXFloats, bid - n_up, false, p1,
                x, gi, nullptr, t, d, r);
        };
        if (hid_rows == 2) hidden(IntC<2>());
        else if (hid_rows == 4) hidden(IntC<4>());
        else hidden(IntC<la_hid_rows_max(B, CPW)>());
    }
}

constexpr int kLaOutNeurons = 32;                      // output-layer role: 32 neurons per block,
static_assert(kLaOutNeurons * 16 == kDown2Threads,     // 16 threads per neuron = FC2's block size
              "both roles of the second launch use the same block size");

// grid = tiles * P + ffn_next / 32, block = 512.  C > 0: the output layer holds the hidden vector by column, C =
// chunks of r (dynamic LDS: kColsXFloats floats per wave and its sums); C = 0 (r > 2048): staged in LDS,
// [B][rpad] floats.
constexpr size_t kLaDownOutLds = 54000;  // two workgroups per CU: with four all rows of the output layer were
// asked for at once and FC2's dependent trips queued behind them (us: 7B-class batch 1 565 / 549, batch 2 270 /
// 254, batch 3 358 / 341 for 12 layers; 2048 and less wide layers the same)
template <int B, int C>
__global__ __launch_bounds__(kDown2Threads) void k_la_down_out(
    int tiles, int P, const __half *__restrict__ w_down, const float *__restrict__ b_down,
    const float *__restrict__ h, const int32_t *__restrict__ idx, const int32_t *__restrict__ count_p,
    float *__restrict__ part, int d, int ffn, const __half *__restrict__ p2,
    const float *__restrict__ p_bias, const float *__restrict__ t, int r, int ffn_next, float thr_logit,
    uint64_t *__restrict__ mask_next, int first_word, bool out_first)
{
    extern __shared__ float ts[];
    __shared__ float red[kDown2Waves][B][kDown2Cols];
    __shared__ float logit_s[B][kLaOutNeurons];
    const int bid = (int)blockIdx.x, n_fc2 = tiles * P, n_out = (int)gridDim.x - n_fc2;
    const bool is_fc2 = out_first ? bid >= n_out : bid < n_fc2;
    if (is_fc2) {  // uniform over the block
        const int fb = out_first ? bid - n_out : bid;
        down2_body<B>(red, fb % tiles, fb / tiles, P, w_down, b_down, h, idx, count_p, part, d, ffn);
    } else {
        const int ob = out_first ? bid : bid - n_fc2;
        if constexpr (C > 0)
            pred_out_cols_body<B, kLaOutNeurons, C>(ts + kDown2Waves * kColsXFloats, ts, ob, p2, p_bias, t, r, ffn_next,
                                                    thr_logit, nullptr, mask_next, first_word);
        else
            pred_out_body<B, kLaOutNeurons>(ts, logit_s, ob, p2, p_bias, t, r, ffn_next, thr_logit, nullptr, mask_next,
                                            first_word);
    }
}

// ---------------------------------------------------------------------------------------
// The same two launches for batches on the matrix cores (batch >= 4, or 3 with long rows),
// from the matrix-core kernels' bodies.  These read the layer input from memory, as split
// fp16 halves, so a glue kernel of its own (or k_split for the first layer) runs in front of
// the first launch.  Ungated layers: two workgroups of
// either role fit a CU.  The gated FC1 needs 128 KB of LDS per workgroup, so there a CU holds
// one workgroup at a time and the hidden-layer role follows FC1 rather than sharing the CUs.
static_assert(kMfmaThreads == kDown2Threads, "all roles of these launches use 512 threads");

// grid = n_up + n_hid, block = 512: [FC1 of layer l on the matrix cores | hidden layer of
// predictor l+1 on the matrix cores].  Dynamic LDS: FC1's mask scan + slots (>= the hidden
// layer's 64 KB of slots).
template <int ACT>
__global__ __launch_bounds__(kMfmaThreads) void k_la_up_hidden_mfma(
    int n_hid, const __half *__restrict__ p1, __half *__restrict__ t_split, int r,
    const __half *__restrict__ w_up, const __half *__restrict__ w_gate,
    const float *__restrict__ b_up, const void *__restrict__ xs, int B,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d, int ffn, float up_floor,
    const float *__restrict__ x)
{
    extern __shared__ uint64_t dyn_lds64[];
    __shared__ int irow[32];
    __shared__ float brow[32];
    __shared__ float logit_s[16][16];
    const int n_up = (int)gridDim.x - n_hid, bid = (int)blockIdx.x;
    if (bid < n_up) {  // uniform over the block
        up_mfma_body<ACT, true, true>(dyn_lds64, irow, brow, bid, n_up, w_up, w_gate, b_up, xs, x, B,
                                      nullptr, nullptr, mask_words, idx_out, count_out, h, hs, d, ffn, up_floor);
    } else {
        rows_mfma_body<8, 512, 0, true>(dyn_lds64, logit_s, bid - n_up, p1, xs, x, B, d, r, nullptr, 0.f, nullptr,
                                        nullptr, 0, t_split);
    }
}

// grid = tiles * P + (ffn_next - always-on prefix) / 64, block = 512: [FC2 of layer l | output
// layer of predictor l+1 on the matrix cores].  Dynamic LDS: the output layer's 64 KB of slots;
// FC2's cross-wave sums live in the same region (a workgroup plays one role), so that two
// workgroups fit a CU.
__global__ __launch_bounds__(kMfmaThreads, 4) void k_la_down_out_mfma(
    int B, int hs, int tiles, int P, const __half *__restrict__ w_down, const float *__restrict__ b_down,
    const float *__restrict__ h, const int32_t *__restrict__ idx, const int32_t *__restrict__ count_p,
    float *__restrict__ part, int d, int ffn, const __half *__restrict__ p2,
    const float *__restrict__ p_bias, const __half *__restrict__ t_split, int r, int ffn_next, float thr_logit,
    uint64_t *__restrict__ mask_next, int first_word)
{
    extern __shared__ uint64_t dyn_lds64[];
    __shared__ float logit_s[16][64];
    static_assert(sizeof(float) * kDown2mRedFloats <= (size_t)kMfmaWaves * kRowsMfmaSlotBytes,
                  "FC2's sums fit the slots");
    const int bid = (int)blockIdx.x, n_fc2 = tiles * P;
    if (bid < n_fc2) {  // uniform over the block
        down2_mfma_body(reinterpret_cast<float *>(dyn_lds64), bid % tiles, bid / tiles, P, w_down, b_down,
                        h, idx, count_p, part, B, hs, d, ffn);
    } else {
        rows_mfma_body<64, 64, 1, true>(dyn_lds64, logit_s, bid - n_fc2, p2, t_split, nullptr, B, r, ffn_next, p_bias,
                                        thr_logit, nullptr, mask_next, first_word);
    }
}

// ---------------------------------------------------------------------------------------
// The same two launches over int4 weights (the predictor stays fp16).  FC1's int4 kernel reads
// the layer input from memory, so a glue kernel of its own runs in front of the first launch.
static_assert(kUpI4Threads == kDown2I4Threads && kDown2I4Threads == kDown2Threads, "512 threads in all roles");

// grid = n_up + n_hid, block = 512: [FC1 of layer l over int4 rows | hidden layer of predictor
// l+1, 8 rows per block].  Dynamic LDS: FC1's staged input + scrap + mask scan (>= the hidden
// layer's staged input).
template <int B, int ACT>
__global__ __launch_bounds__(kUpI4Threads) void k_la_up_hidden_i4(
    int n_hid, const __half *__restrict__ p1, float *__restrict__ t, int r,
    const uint8_t *__restrict__ q_up, const __half *__restrict__ s_up,
    const uint8_t *__restrict__ q_gate, const __half *__restrict__ s_gate,
    const float *__restrict__ b_up, const float *__restrict__ x,
    const uint64_t *__restrict__ mask_words, int32_t *__restrict__ idx_out,
    int32_t *__restrict__ count_out, float *__restrict__ h, int hs, int d, int ffn, float up_floor)
{
    extern __shared__ float xs[];
    __shared__ uint32_t wave_tot[kUpI4Waves];
    __shared__ float ss_w[kUpI4Waves][B];
    const int n_up = (int)gridDim.x - n_hid, bid = (int)blockIdx.x;
    if (bid < n_up) {  // uniform over the block
        up_i4_body<B, ACT, true>(xs, wave_tot, bid, n_up, q_up, s_up, q_gate, s_gate, b_up, x, nullptr, nullptr,
                                 mask_words, idx_out, count_out, h, hs, d, ffn, up_floor);
    } else {
        pred_hidden_body<B, false, 1, kUpI4Threads>(xs, ss_w, bid - n_up, false, p1, x, nullptr, 0, 0, nullptr, t,
                                                    d, r, 0);
    }
}

// grid = tiles * P + (ffn_next - always-on prefix) / 32, block = 512: [FC2 of layer l over int4
// rows | output layer of predictor l+1].  Dynamic LDS: staged hidden vector [B][rpad].
template <int B>
__global__ __launch_bounds__(kDown2I4Threads) void k_la_down_out_i4(
    int tiles, int P, const uint8_t *__restrict__ q_down, const __half *__restrict__ s_down,
    const float *__restrict__ b_down, const float *__restrict__ h, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ count_p, float *__restrict__ part, int d, int ffn,
    const __half *__restrict__ p2, const float *__restrict__ p_bias, const float *__restrict__ t, int r,
    int ffn_next, float thr_logit, uint64_t *__restrict__ mask_next, int first_word)
{
    extern __shared__ float ts[];
    __shared__ float red[kDown2I4Waves][B][kDown2I4Cols];
    __shared__ float logit_s[B][kLaOutNeurons];
    const int bid = (int)blockIdx.x, n_fc2 = tiles * P;
    if (bid < n_fc2) {  // uniform over the block
        down2_i4_body<B>(red, bid % tiles, tiles, bid / tiles, P, q_down, s_down, b_down, h, idx, count_p, part,
                         d, ffn);
    } else {
        pred_out_body<B, kLaOutNeurons>(ts, logit_s, bid - n_fc2, p2, p_bias, t, r, ffn_next, thr_logit, nullptr,
                                        mask_next, first_word);
    }
}

}  // namespace pf
