// The dense block around the routed layer (Algorithm 1, steps 1, 3 and 4):
//   X~ = LN_1(X);  (Q, K, V) = QKV(X~) with the 2D rotary encoding of the
//   token positions applied to Q and K;  [routed attention: Y];
//   X_attn = X + LS_1 (Y W_O^T + b_O);
//   X_out  = X_attn + LS_2 (W_fc2 GELU(W_fc1 LN_2(X_attn) + b_fc1) + b_fc2).
// Two kinds of kernel: a LayerNorm (one wave per row, HBM-bound) and a bf16
// GEMM on MFMA whose epilogue applies the bias and then the step's own
// elementwise work (rotary encoding and the split into Q, K, V; GELU; or
// LayerScale plus residuals), so no projection output makes an extra trip
// through HBM.  The residual stream is never rounded in between: the W_O
// step stores only the attention update A = LS_1 (Y W_O^T + b_O), and LN_2
// and the last step form X_attn = X + A in fp32 from X and A.
#include "vp_device.hpp"
#include "vp_internal.hpp"

namespace vp {

constexpr int kDm = 1024;   // model width D = 16 heads x 64

// ------------------------------------------------------------------------
// B1: LayerNorm over the D = 1024 features of each row of X (+ X2 when given,
// added in fp32): mean and biased variance in fp32 (two passes over
// registers), y = (x - mean) r g + b, r = 1 / sqrt(var + eps), rounded to
// bf16.  One wave per kLnRows consecutive rows, g and b held in registers;
// lane l holds features 8 l ... 8 l + 7 and 512 + 8 l ... 512 + 8 l + 7, so
// each 16-byte load or store of a wave covers 1 KB of the row contiguously.
// The next row's loads are issued before the current row is normalised.
// ------------------------------------------------------------------------
constexpr int kLnRows = 2;

template <bool kAdd>
__global__ __launch_bounds__(256) void k_layernorm(const bf16* __restrict__ X,
                                                   const bf16* __restrict__ X2, int64_t T,
                                                   const float* __restrict__ g,
                                                   const float* __restrict__ b, float eps,
                                                   bf16* __restrict__ Y) {
    const int64_t row0 =
        ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kLnRows;
    if (row0 >= T) return;
    const int lane = threadIdx.x & 63, c0 = 8 * lane, c1 = kDm / 2 + 8 * lane;
    float gg[16], bv[16];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        gg[j] = g[c0 + j];
        gg[8 + j] = g[c1 + j];
        bv[j] = b[c0 + j];
        bv[8 + j] = b[c1 + j];
    }
    const int nr = T - row0 < kLnRows ? (int)(T - row0) : kLnRows;
    constexpr int kV = kAdd ? 4 : 2;
    auto load = [&](int64_t row, bf16x8 (&v)[kV]) {
        const bf16* xr = X + row * kDm;
        v[0] = load_bf16x8(xr + c0);
        v[1] = load_bf16x8(xr + c1);
        if constexpr (kAdd) {
            const bf16* x2 = X2 + row * kDm;
            v[2] = load_bf16x8(x2 + c0);
            v[3] = load_bf16x8(x2 + c1);
        }
    };
    auto norm = [&](int64_t row, const bf16x8 (&v)[kV]) {
        float x[16];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = bf16_to_f32(v[0][j]);
            x[8 + j] = bf16_to_f32(v[1][j]);
            if constexpr (kAdd) {
                x[j] += bf16_to_f32(v[2][j]);
                x[8 + j] += bf16_to_f32(v[3][j]);
            }
        }
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) s += x[j];
        const float mean = wave_sum(s) * (1.f / kDm);
        float q = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) q = fmaf(x[j] - mean, x[j] - mean, q);
        const float r = rsqrtf(wave_sum(q) * (1.f / kDm) + eps);
        float y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = fmaf((x[j] - mean) * r, gg[j], bv[j]);
        bf16* yr = Y + row * kDm;
        *reinterpret_cast<bf16x8*>(yr + c0) =
            pack_bf16x8(y[0], y[1], y[2], y[3], y[4], y[5], y[6], y[7]);
        *reinterpret_cast<bf16x8*>(yr + c1) =
            pack_bf16x8(y[8], y[9], y[10], y[11], y[12], y[13], y[14], y[15]);
    };
    // Straight-line over kLnRows rows with two register sets, each row's loads
    // issued one row ahead of its use.  Rows past the last are the last row
    // again (the same values stored twice; Y never aliases X or X2), so no
    // branch sits around the loads and each wait covers only the row in use.
    auto rowi = [&](int i) { return row0 + (i < nr ? i : nr - 1); };
    bf16x8 v[2][kV];
    load(rowi(0), v[0]);
#pragma unroll
    for (int i = 0; i < kLnRows; ++i) {
        if (i + 1 < kLnRows) load(rowi(i + 1), v[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of the row's arithmetic
        norm(rowi(i), v[i & 1]);
    }
}

// ------------------------------------------------------------------------
// B2: D^T = W X^T for W [F, Kd] (weights as stored, [out, in]) and X [T, Kd]
// (token rows), bf16 operands, fp32 accumulation: both operands are
// Kd-contiguous, as the MFMA wants them.  Workgroup tile 256 features x 256
// tokens, Kd in stages of 64.  Output features are the MFMA rows, so lane l
// holds token l % 32 of a block and features 8 (r / 4) + 4 (l / 32) + r % 4 in
// its register r, and the rotary pair (j, j + 16) of a 32-feature half in
// registers r and r + 8 of one lane.
// ------------------------------------------------------------------------
constexpr int kGM = 256, kGN = 256, kGK = 64;
constexpr int kGemmWG = 256;               // persistent workgroups: one per CU
constexpr uint32_t kGStage = 32768;        // bytes of one operand's stage: 256 rows of 128
constexpr uint32_t kGLdsX = 2 * kGStage;   // two W stages, then three X stages

// EPI_SCALE: ls (acc + bias); EPI_RESID2: ls (acc + bias) + res + res2.
enum { EPI_QKV = 0, EPI_GELU = 1, EPI_SCALE = 2, EPI_RESID2 = 3 };

struct GemmArgs {
    const bf16* W;        // [F, Kd]
    const bf16* X;        // [T, Kd]
    const float* bias;    // [F]
    int64_t T;
    int F, Kd;
    bf16* out;            // GELU, SCALE, RESID2: [T, F]
    const bf16 *res, *res2;   // RESID2: residuals [T, F]
    const float* ls;      // SCALE, RESID2: LayerScale [F]
    bf16 *q, *k, *v;      // QKV: [T, D] each
    const int32_t* pos;   // QKV: [T, 2] (row, column)
    float log2_base;      // QKV: log2 of the rotary base
};

// Epilogue of a wave's 128 features f0 + 128 wm .. x 64 tokens t0 + 64 wn ..
// The outputs pass through 4 KB of LDS that only this wave uses at that time
// (32 rows of 128 bytes, row r at scratch + 8192 (r / 8) + 128 (r % 8), 16-byte
// chunks at position chunk ^ (r / 2 % 8)), so that every store writes whole
// 128-byte lines.  Loads and stores complete in issue order, so a load issued
// after a store waits for it: bias and LayerScale go to LDS first (1 KB at
// `vecs`, this wave's too) and the residuals of a block are read before the
// previous block is stored.
template <int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, f32x16 (&acc)[4][2], int f0,
                                              int64_t t0, int wm, int wn, int lane0,
                                              uint32_t scratch, uint32_t vecs) {
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
    typedef __attribute__((address_space(3))) f32x2 lds_f32x2;
    constexpr bool kScale = EPI == EPI_SCALE || EPI == EPI_RESID2;
    // (an opaque copy, so that nothing of the epilogue's addresses is kept in
    // registers over the main loop)
    int lane = lane0;
    asm volatile("" : "+v"(lane));
    const int n = lane & 31, hh = lane >> 5;
    const int fw = f0 + 128 * wm;
    const int64_t tw = t0 + 64 * wn;
    // chunk c of row n, for the writes (c = 4 f2 + 2 p + hh: flips bits 5-6)
    const uint32_t wr = scratch + 8192u * (n >> 3) + 128u * (n & 7) +
                        (uint32_t)((hh ^ ((n >> 1) & 7)) << 4);
    // chunk lane % 8 of row 8 i + lane / 8, for the reads (i: + 8192, flips bit 6)
    const uint32_t rd = scratch + 128u * (lane >> 3) +
                        (uint32_t)(((lane & 7) ^ (lane >> 4)) << 4);
    // All of a wave's features lie in one of Q, K, V (f0 is a multiple of
    // 256); Q and K are rotated, the first 32 features of each 64 by the row
    // coordinate and the next 32 by the column coordinate.
    const int which = EPI == EPI_QKV ? __builtin_amdgcn_readfirstlane(fw / kDm) : 0;
    const bool rotate = EPI == EPI_QKV && which < 2;
    bf16* const qkv_out = which == 0 ? g.q : (which == 1 ? g.k : g.v);
    bf16* const dst0 = EPI == EPI_QKV ? qkv_out + (fw - which * kDm) : g.out + fw;
    const int64_t ldo = EPI == EPI_QKV ? kDm : g.F;
    // Rows of the lane's tokens in the MFMA layout (past T - 1: row T - 1, not stored).
    int64_t tn[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
        tn[tb] = tw + 32 * tb + n < g.T ? tw + 32 * tb + n : g.T - 1;
    int2 pos[2];
    if (rotate) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) pos[tb] = *reinterpret_cast<const int2*>(g.pos + 2 * tn[tb]);
    }
    // Residuals of a 32 x 32 block in the 16-byte layout of the exchanged registers.
    u32x4 r1[2][2], r2[2][2];
    auto load_res = [&](int blk, int set) {
        const int64_t at = tn[blk >> 2] * ldo + fw + 32 * (blk & 3) + 8 * hh;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            r1[set][p] = *reinterpret_cast<const u32x4*>(g.res + at + 16 * p);
            r2[set][p] = *reinterpret_cast<const u32x4*>(g.res2 + at + 16 * p);
        }
    };
    {
        // (the caller's vectors are aligned to 4 bytes)
        typedef float f32x2_at4 __attribute__((__vector_size__(8), aligned(4)));
        const f32x2 bv = *reinterpret_cast<const f32x2_at4*>(g.bias + fw + 2 * lane);
        f32x2 lv = {0.f, 0.f};
        if constexpr (kScale) lv = *reinterpret_cast<const f32x2_at4*>(g.ls + fw + 2 * lane);
        if constexpr (EPI == EPI_RESID2) load_res(0, 0);
        *(lds_f32x2*)(uintptr_t)(vecs + 8u * lane) = bv;
        if constexpr (kScale) *(lds_f32x2*)(uintptr_t)(vecs + 512u + 8u * lane) = lv;
    }
    float omega[8];   // rotary frequencies of features j = 8 (r / 4) + 4 hh + r % 4, r < 8
    if (rotate) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
            omega[r] = exp2f(-(float)(8 * (r >> 2) + 4 * hh + (r & 3)) * (1.f / 16.f) * g.log2_base);
    }
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        // (sin, cos) of the token's angles: half 0 takes the row coordinate,
        // half 1 the column coordinate.
        float rs[2][8], rc[2][8];
        if (rotate) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                __sincosf((float)pos[tb].x * omega[r], &rs[0][r], &rc[0][r]);
                __sincosf((float)pos[tb].y * omega[r], &rs[1][r], &rc[1][r]);
            }
        }
#pragma unroll
        for (int fp = 0; fp < 2; ++fp) {
#pragma unroll
            for (int f2 = 0; f2 < 2; ++f2) {
                const int fb = 2 * fp + f2, blk = 4 * tb + fb;
                if constexpr (EPI == EPI_RESID2) {
                    if (blk + 1 < 8) load_res(blk + 1, (blk + 1) & 1);
                }
                float v[16];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 bias = *(const lds_f32x4*)(uintptr_t)(vecs + 4u * (32 * fb + 8 * q + 4 * hh));
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[4 * q + i] = acc[fb][tb][4 * q + i] + bias[i];
                }
                if (EPI == EPI_QKV) {
                    if (rotate) {   // the planes (j, j + 16) of this half
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const float sn = rs[f2][r], cs = rc[f2][r];
                            const float u = v[r], w = v[r + 8];
                            v[r] = u * cs - w * sn;
                            v[r + 8] = u * sn + w * cs;
                        }
                    }
                } else if (EPI == EPI_GELU) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = gelu(v[r]);
                } else {
                    float base[16];
                    if constexpr (EPI == EPI_RESID2) {
#pragma unroll
                        for (int p = 0; p < 2; ++p)
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                uint32_t a1 = r1[blk & 1][p][k], b1 = r1[blk & 1][p][2 + k];
                                uint32_t a2 = r2[blk & 1][p][k], b2 = r2[blk & 1][p][2 + k];
                                swap_halves(a1, b1);
                                swap_halves(a2, b2);
                                const bf16x2 x1 = __builtin_bit_cast(bf16x2, a1);
                                const bf16x2 y1 = __builtin_bit_cast(bf16x2, b1);
                                const bf16x2 x2 = __builtin_bit_cast(bf16x2, a2);
                                const bf16x2 y2 = __builtin_bit_cast(bf16x2, b2);
#pragma unroll
                                for (int i = 0; i < 2; ++i) {
                                    base[8 * p + 2 * k + i] = (float)x1[i] + (float)x2[i];
                                    base[8 * p + 4 + 2 * k + i] = (float)y1[i] + (float)y2[i];
                                }
                            }
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 ls = *(const lds_f32x4*)(uintptr_t)(vecs + 512u + 4u * (32 * fb + 8 * q + 4 * hh));
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = 4 * q + i;
                            v[r] = EPI == EPI_RESID2 ? fmaf(ls[i], v[r], base[r]) : ls[i] * v[r];
                        }
                    }
                }
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    u32x4 o;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int ra = 8 * p + 2 * k;
                        const bf16x2 x = {(bf16)v[ra], (bf16)v[ra + 1]};
                        const bf16x2 y = {(bf16)v[ra + 4], (bf16)v[ra + 5]};
                        uint32_t a = __builtin_bit_cast(uint32_t, x);
                        uint32_t b = __builtin_bit_cast(uint32_t, y);
                        swap_halves(a, b);
                        o[k] = a;
                        o[2 + k] = b;
                    }
                    *(lds_u32x4*)(uintptr_t)(wr ^ (uint32_t)((4 * f2 + 2 * p) << 4)) = o;
                }
            }
            // (one wave's LDS operations execute in order: no wait between the
            // writes and these reads, nor before the next block's writes)
            u32x4 o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o[i] = *(const lds_u32x4*)(uintptr_t)((rd ^ (uint32_t)((i & 1) << 6)) + 8192u * i);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t t = tw + 32 * tb + 8 * i + (lane >> 3);
                if (t < g.T)
                    *reinterpret_cast<u32x4*>(dst0 + t * ldo + 64 * fp + 8 * (lane & 7)) = o[i];
            }
        }
    }
}

// Persistent, one workgroup of 8 waves per CU (two per SIMD), each wave a block of 128
// features x 64 tokens.  Waves 0-3 (features 0-127) and 4-7 (features 128-255)
// alternate, one phase apart, with one barrier per phase: while one group
// issues a stage's 32 MFMAs per wave, the other reads its next stage's 24
// fragments from LDS into registers.
//   phase 2 s:     group 0 reads stage s,      group 1 multiplies stage s - 1
//   phase 2 s + 1: group 0 multiplies stage s, group 1 reads stage s
// Stages are copied straight from global memory to LDS (no registers), 128-byte
// rows whose 16-byte chunks are stored at position chunk ^ (row / 2 % 8), so that
// the fragment reads of sixteen consecutive rows hit all 64 banks once.  Group 0's
// half of a W stage is dead after phase 2 s, the other half and the X stage after phase
// 2 s + 1; with two W and three X buffers the copies are issued
//   phase 2 s:     W half 1 of stage s + 1, X of stage s + 2
//   phase 2 s + 1: W half 0 of stage s + 2
// i.e. three to four phases before they are read, and the waits (12 and 8 copies
// still in flight, by issue order) never drain them.  The copies run ahead over
// tile boundaries; past the last stage they repeat the last tile's.  Token rows
// past T - 1 read row T - 1 and are not stored.  Both groups run their epilogue
// in the same phase.  The multiplying group runs at raised priority (2-3 %).
//
// What bounds it: matrix issue and power together.  At 137,400 tokens the four
// projections take 0.28 (W_O), 0.80 (QKV), 1.11 (FFN 1) and 1.05 ms (FFN 2), 1.0-1.1 PF/s
// over the last three (0.39, 1.14, 1.52 and 1.27 ms for the register-staged kernels
// before it); the matrix pipe is busy 49-54 % of the cycles at 1.6-1.75 GHz, and what
// takes idle cycles out lowers the clock.  Without any copies the FFN kernels
// took 12-14 % fewer cycles, without the epilogue 15-25 %.
template <int EPI>
__global__ __launch_bounds__(512, 1) void k_gemm(GemmArgs g) {
    const int nft = g.F / kGM;
    const int ntt = (int)((g.T + kGN - 1) / kGN);
    const int total = nft * ntt;
    const int nk = g.Kd / kGK;
    const int G = gridDim.x;
    const int slot = xcd_remap(blockIdx.x, G);
    const int ntile = slot < total ? (total - 1 - slot) / G + 1 : 0;
    if (ntile == 0) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 31, hh = lane >> 5;
    const int grp = wave >> 2, wn = wave & 3;

    __shared__ __attribute__((aligned(1024))) char smem[5 * kGStage];
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(3))) const bf16x8 lds_frag;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

    // Groups of `gft` feature tiles per token tile, consecutive tiles on one
    // XCD, whose L2 serves a token tile to all its feature tiles at once.  All
    // feature tiles in one group, but FFN 1's 16 in two of 8: an XCD's 32
    // tiles then are 4 x 8 instead of 2 x 16 (token x feature) tiles, 6 instead
    // of 9 MB (output stage at 137,400 tokens 2712 -> 2682 us; QKV's 12 in
    // groups of 4 or 6 were 1 % slower than in one).
    const int gft = nft % 8 == 0 ? 8 : nft;
    auto tile_of = [&](int i, int& f0, int64_t& t0) {
        const int L = i * G + slot;
        const int gi = L / (gft * ntt), in = L - gi * gft * ntt;
        f0 = (gi * gft + in % gft) * kGM;
        t0 = (int64_t)(in / gft) * kGN;
    };

    // Copies: wave w, instruction i moves rows 64 i + 8 w + lane / 8, lane
    // l's 16 bytes are chunk (l % 8) ^ (row / 2 % 8) of the row's 128.
    const uint32_t rstride = (uint32_t)g.Kd * 2u;
    const int crow = 8 * wave + (lane >> 3);
    const uint32_t ccol = (uint32_t)((lane & 7) ^ ((crow >> 1) & 7)) * 16u;
    const uint32_t woff = (uint32_t)crow * rstride + ccol;
    uint32_t xoff[4];
    const char *wb, *xb;              // stage being copied, of W and of X
    int wi = 0, wkt = -1, xi = 0, xkt = -1;
    uint32_t wbuf = kGStage, xbuf = 2 * kGStage;   // its LDS buffer (byte offset)
    int tf0;
    int64_t tt0;
    auto x_tile = [&](int i) {
        tile_of(i, tf0, tt0);
        xb = reinterpret_cast<const char*>(g.X + tt0 * g.Kd);
        const int last = (int)(g.T - 1 - tt0 < kGN - 1 ? g.T - 1 - tt0 : kGN - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            xoff[j] = (uint32_t)min(64 * j + crow, last) * rstride + ccol;
    };
    auto next_w = [&]() {
        wbuf ^= kGStage;
        wb += kGK * 2;
        if (++wkt == nk) {
            wkt = 0;
            if (wi + 1 < ntile) ++wi;
            tile_of(wi, tf0, tt0);
            wb = reinterpret_cast<const char*>(g.W + (int64_t)tf0 * g.Kd);
        }
    };
    auto next_x = [&]() {
        xbuf = xbuf == 2 * kGStage ? 0 : xbuf + kGStage;
        xb += kGK * 2;
        if (++xkt == nk) {
            xkt = 0;
            if (xi + 1 < ntile) ++xi;
            x_tile(xi);
        }
    };
    auto copy_w = [&](int half) {
#pragma unroll
        for (int j = 2 * half; j < 2 * half + 2; ++j)
            copy_to_lds(lds0 + wbuf + (64 * j + 8 * wave) * 128, wb + (int64_t)(64 * j) * rstride,
                        woff);
    };
    auto copy_x = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            copy_to_lds(lds0 + kGLdsX + xbuf + (64 * j + 8 * wave) * 128, xb, xoff[j]);
    };
    auto issue_even = [&]() { copy_w(1); next_x(); copy_x(); };
    auto issue_odd = [&]() { next_w(); copy_w(0); };
    auto wait_even = [&]() { asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); };
    auto wait_odd = [&]() { asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); };
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    // Prologue: X(0), W(0) half 0, then what phases -2 and -1 would issue.
    tile_of(0, tf0, tt0);
    wb = reinterpret_cast<const char*>(g.W + (int64_t)tf0 * g.Kd) - kGK * 2;
    x_tile(0);
    xb -= kGK * 2;
    next_x();
    copy_x();
    issue_odd();
    issue_even();
    issue_odd();
    wait_odd();
    barrier();
    if (grp) {   // phase 0 of group 1
        issue_even();
        wait_even();
        barrier();
    }

    f32x16 acc[4][2];
    // Fragment addresses of k-step 0 (buffer 0); k-step ks flips bits 5-6.
    const uint32_t a0 = lds0 + (uint32_t)(128 * grp + n) * 128u + (uint32_t)((hh ^ ((n >> 1) & 7)) << 4);
    const uint32_t x0 = lds0 + kGLdsX + (uint32_t)(64 * wn + n) * 128u +
                        (uint32_t)((hh ^ ((n >> 1) & 7)) << 4);
    uint32_t arb = 0, xrb = 0;
    for (int i = 0; i < ntile; ++i) {
        for (int kt = 0; kt < nk; ++kt) {
            bf16x8 a[4][4], x[4][2];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const uint32_t ap = (a0 + arb) ^ (uint32_t)(ks << 5);
                const uint32_t xp = (x0 + xrb) ^ (uint32_t)(ks << 5);
#pragma unroll
                for (int fb = 0; fb < 4; ++fb) a[ks][fb] = *(lds_frag*)(uintptr_t)(ap + 4096u * fb);
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) x[ks][tb] = *(lds_frag*)(uintptr_t)(xp + 4096u * tb);
            }
            arb ^= kGStage;
            xrb = xrb == 2 * kGStage ? 0 : xrb + kGStage;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (grp)
                issue_odd();
            else
                issue_even();
            if (grp)
                wait_odd();
            else
                wait_even();
            barrier();
            __builtin_amdgcn_s_setprio(1);
            // The phase's copies go behind the first MFMAs, which keep the
            // matrix pipe busy meanwhile.
            if (kt == 0) {
#pragma unroll
                for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb)
                        acc[fb][tb] = mfma_bf16(a[0][fb], x[0][tb], zero_f32x16());
            } else {
#pragma unroll
                for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb)
                        acc[fb][tb] = mfma_bf16(a[0][fb], x[0][tb], acc[fb][tb]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (grp == 0)
                issue_odd();
            else if (kt + 1 < nk)
                issue_even();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 1; ks < 4; ++ks)
#pragma unroll
                for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb)
                        acc[fb][tb] = mfma_bf16(a[ks][fb], x[ks][tb], acc[fb][tb]);
            __builtin_amdgcn_s_setprio(0);
            if (grp == 0) {
                wait_odd();
                barrier();
            } else if (kt + 1 < nk) {
                wait_even();
                barrier();
            }
        }
        int f0;
        int64_t t0;
        tile_of(i, f0, t0);
        // The wave's scratch is those parts of the next X stage's and of the
        // next W half's buffer that its own copies fill, which it issues only
        // afterwards.
        const uint32_t xnext = xbuf == 2 * kGStage ? 0 : xbuf + kGStage;
        gemm_epilogue<EPI>(g, acc, f0, t0, grp, wn, lane, lds0 + kGLdsX + xnext + 1024u * wave,
                           lds0 + wbuf + kGStage / 2 + 1024u * wave);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (grp) {
            issue_even();
            wait_even();
            barrier();
        }
    }
    if (grp == 0) barrier();
    // (no copy may land after the workgroup's LDS is given back)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// ------------------------------------------------------------------ launchers

// F a multiple of 256, Kd of 64 and at least 128.
template <int EPI>
static void gemm(const GemmArgs& a, hipStream_t st) {
    const int total = (a.F / kGM) * (int)((a.T + kGN - 1) / kGN);
    hipLaunchKernelGGL(k_gemm<EPI>, dim3(total < kGemmWG ? total : kGemmWG), dim3(512), 0, st, a);
}

static void layernorm(const bf16* X, const bf16* X2, int64_t T, const float* g, const float* b,
                      float eps, bf16* Y, hipStream_t st) {
    const dim3 grid((unsigned)((T + 4 * kLnRows - 1) / (4 * kLnRows)));
    if (X2)
        hipLaunchKernelGGL(k_layernorm<true>, grid, dim3(256), 0, st, X, X2, T, g, b, eps, Y);
    else
        hipLaunchKernelGGL(k_layernorm<false>, grid, dim3(256), 0, st, X, X2, T, g, b, eps, Y);
}

void launch_block_qkv(const BlockArgs& a, hipStream_t st) {
    layernorm(a.X, nullptr, a.T, a.ln1_w, a.ln1_b, a.eps, a.ln, st);
    GemmArgs g = {};
    g.W = a.w_qkv; g.X = a.ln; g.bias = a.b_qkv; g.T = a.T; g.F = 3 * kDm; g.Kd = kDm;
    g.q = a.Q; g.k = a.K; g.v = a.V; g.pos = a.pos; g.log2_base = log2f(a.rope_base);
    gemm<EPI_QKV>(g, st);
}

void launch_block_out(const BlockArgs& a, hipStream_t st) {
    GemmArgs g = {};
    g.T = a.T;
    // A = LS_1 (Y W_O^T + b_O), the attention update (X_attn = X + A)
    g.W = a.w_o; g.X = a.Y; g.bias = a.b_o; g.F = kDm; g.Kd = kDm;
    g.ls = a.ls1; g.out = a.xa;
    gemm<EPI_SCALE>(g, st);
    layernorm(a.X, a.xa, a.T, a.ln2_w, a.ln2_b, a.eps, a.ln, st);
    // H = GELU(LN_2(X + A) W_fc1^T + b_fc1)
    g.W = a.w_fc1; g.X = a.ln; g.bias = a.b_fc1; g.F = 4 * kDm; g.Kd = kDm; g.out = a.hid;
    gemm<EPI_GELU>(g, st);
    // X_out = X + A + LS_2 (H W_fc2^T + b_fc2)
    g.W = a.w_fc2; g.X = a.hid; g.bias = a.b_fc2; g.F = kDm; g.Kd = 4 * kDm;
    g.res = a.X; g.res2 = a.xa; g.ls = a.ls2; g.out = a.Xout;
    gemm<EPI_RESID2>(g, st);
}

}  // namespace vp
