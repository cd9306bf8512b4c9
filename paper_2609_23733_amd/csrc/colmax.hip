// D2 of the distillation targets: column maxima of the teacher's attention
// (Eq.8), see distill.hip.  A file of its own because it is compiled with
// -fno-honor-nans: otherwise every three-way maximum comes with a
// canonicalising move per operand (three times the vector work).  A NaN
// logit still never wins a maximum (v_max returns the other operand).
#include "vp_device.hpp"
#include "vp_internal.hpp"

namespace vp {

constexpr int kDL = 72;   // bf16 LDS row stride (144 B)

// ------------------------------------------------------------------------
// D2: 8 waves x 128 keys of one head per workgroup, the keys held in registers
// as the MFMA's B operand.  Tiles of 64 queries (Q rows and -o_q / c) stream
// through three LDS buffers shared by the waves; queries are the MFMA's rows,
// so a lane's 16 results of a 32 x 32 block are 16 queries of one key and keep
// one running maximum (half a three-way max per score).  The accumulator
// input of a query block, -o_q / c of its 16 rows per lane half, is read from
// LDS as it is (four 16-byte reads per 32 queries instead of register moves),
// the MFMA returns (x_qk - o_q) / c, and c > 0 carries the maximum over to
// x - o.  Two 32-key blocks are multiplied together (two MFMA chains) while
// the previous two blocks' maxima are taken, and a tile's first operands are
// read before the barrier that ends the tile before it.  Queries past N carry
// -inf; keys past N read row 0 and are not written.
//
// The work is one sequence of (head, 1024 keys, query tile) steps split evenly
// over the workgroups, whatever N and H are (with one workgroup per 1024 keys,
// 24,744 tokens filled 400 of 512 places in two rounds); parts of a key's
// queries meet in an integer atomic maximum of the non-negative results'
// bits, whose outcome does not depend on the order.  colmax starts at 0.
//
// Bound by the matrix pipe and the clock it leaves: 24,744 tokens, 16 heads
// 1450 -> 960 us (1.3 PF/s; pipe 74 % busy at 1.65 GHz, was 41-50 % at 1.95-2.2
// with 16 running maxima per 32 keys and register moves for the accumulator
// inputs).
// ------------------------------------------------------------------------
constexpr int kCmWaves = 8;
constexpr int kCmKB = 4;                            // 32-key blocks per wave
constexpr int kCmKeys = 32 * kCmKB * kCmWaves;      // keys per workgroup
constexpr int kCmQ = 64;                            // queries per LDS tile
constexpr int kCmWG = 256;                          // workgroups: one per CU

__global__ __launch_bounds__(64 * kCmWaves, 1) void k_colmax(const bf16* __restrict__ Q,
                                                             const bf16* __restrict__ K,
                                                             const float* __restrict__ off,
                                                             int64_t N, int H, float c,
                                                             uint32_t* __restrict__ colmax) {
    static_assert(64 * kCmWaves == kCmQ * 8, "one 16-byte tile segment per thread");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
    __shared__ __attribute__((aligned(16))) bf16 sQ[3][kCmQ * kDL];
    __shared__ __attribute__((aligned(16))) float sO[3][kCmQ];
    const float ninv = -1.f / c;
    // (Token indices fit int32: N is at most 2^28.)
    const int Ni = (int)N;
    const int64_t qstride = (int64_t)H * kD;
    const int lr = threadIdx.x >> 3, lc = (threadIdx.x & 7) * 8;
    const int nt = (Ni + kCmQ - 1) / kCmQ, nkb = (Ni + kCmKeys - 1) / kCmKeys;
    const int64_t total = (int64_t)H * nkb * nt, G = gridDim.x;
    const int w = xcd_remap(blockIdx.x, (int)G);
    int64_t x = total * w / G;
    const int64_t end = total * (w + 1) / G;
    while (x < end) {
        const int64_t item = x / nt;
        const int t0 = (int)(x - item * nt);
        const int t1 = (int)(end - x < nt - t0 ? t0 + (end - x) : nt);
        x += t1 - t0;
        const int h = (int)(item / nkb);
        const int64_t k0 = (item - (int64_t)h * nkb) * kCmKeys + wave * 32 * kCmKB;
        const float* oh = off + (int64_t)h * N;
        const bf16* qh = Q + (int64_t)h * kD;
        bf16x8 Kb[kCmKB][4];
#pragma unroll
        for (int kb = 0; kb < kCmKB; ++kb) {
            const int64_t key = k0 + 32 * kb + n;
            const bf16* kp = K + ((key < N ? key : 0) * H + h) * kD + 8 * hh;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) Kb[kb][ks] = load_bf16x8(kp + 16 * ks);
        }
        bf16x8 gq;
        float go = 0.f;
        auto gload = [&](int t) {   // (clamped to the last tile)
            t = t < t1 ? t : t1 - 1;
            gq = load_bf16x8(qh + (int64_t)min(t * kCmQ + lr, Ni - 1) * qstride + lc);
            // (scaled at the store, so that nothing waits for the load here)
            if (threadIdx.x < kCmQ) go = oh[min(t * kCmQ + (int)threadIdx.x, Ni - 1)];
        };
        auto lstore = [&](int t, int b) {
            *reinterpret_cast<bf16x8*>(&sQ[b][lr * kDL + lc]) = gq;
            if (threadIdx.x < kCmQ)
                sO[b][threadIdx.x] = t * kCmQ + (int)threadIdx.x < Ni ? go * ninv : -INFINITY;
        };
        bf16x8 qv[2][4];
        f32x16 ci[2];   // accumulator inputs: rows 8 g + 4 hh + i in registers 4 g + i
        auto lread = [&](int b, int qb) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                qv[qb][ks] = *reinterpret_cast<const bf16x8*>(
                    &sQ[b][(32 * qb + n) * kDL + 16 * ks + 8 * hh]);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 o = *reinterpret_cast<const f32x4*>(&sO[b][32 * qb + 8 * g + 4 * hh]);
#pragma unroll
                for (int i = 0; i < 4; ++i) ci[qb][4 * g + i] = o[i];
            }
        };
        float acc[kCmKB];
        f32x16 Sa[2], Sb[2];   // the blocks being multiplied, and the two before them
#pragma unroll
        for (int kb = 0; kb < kCmKB; ++kb) acc[kb] = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) Sb[0][r] = Sb[1][r] = -INFINITY;
        // S = blocks (qb, 2 kp and 2 kp + 1); maxima of T, the pair before them.
        auto step = [&](int qb, int kp, f32x16 (&S)[2], const f32x16 (&T)[2]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) S[u] = mfma_bf16(qv[qb][0], Kb[2 * kp + u][0], ci[qb]);
#pragma unroll
            for (int ks = 1; ks < 4; ++ks)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    S[u] = mfma_bf16(qv[qb][ks], Kb[2 * kp + u][ks], S[u]);
            const int tp = kp ^ 1;
#pragma unroll
            for (int r = 0; r < 16; r += 2)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[2 * tp + u] = fmaxf(fmaxf(acc[2 * tp + u], T[u][r]), T[u][r + 1]);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            }
        };
        __syncthreads();   // the previous segment's reads are done
        gload(t0);
        lstore(t0, 0);
        gload(t0 + 1);
        lstore(t0 + 1, 1);
        gload(t0 + 2);
        __syncthreads();
        lread(0, 0);
        int b0 = 0, b1 = 1, b2 = 2;   // buffers of tiles t, t + 1, t + 2
        for (int t = t0; t < t1; ++t) {
            lread(b0, 1);
            step(0, 0, Sa, Sb);
            lstore(t + 2, b2);
            gload(t + 3);
            step(0, 1, Sb, Sa);
            step(1, 0, Sa, Sb);
            lread(b1, 0);
            step(1, 1, Sb, Sa);
            __syncthreads();
            const int b = b0;
            b0 = b1;
            b1 = b2;
            b2 = b;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[2 + u] = fmaxf(acc[2 + u], Sb[u][r]);
        // Maximum over the two lane halves (the other queries of the same
        // key), then 2^(c max).
#pragma unroll
        for (int kb = 0; kb < kCmKB; ++kb) {
            const float v = fmaxf(acc[kb], __shfl_xor(acc[kb], 32));
            const int64_t key = k0 + 32 * kb + n;
            if (hh == 0 && key < N)
                atomicMax(&colmax[(int64_t)h * N + key], __float_as_uint(exp2f(c * v)));
        }
    }
}

// colmax [H, N] (zero on entry).
void launch_colmax(const __bf16* Q, const __bf16* K, const float* off, int64_t N, int H, float c,
                   float* colmax, hipStream_t st) {
    const int64_t steps = H * ((N + kCmKeys - 1) / kCmKeys) * ((N + kCmQ - 1) / kCmQ);
    hipLaunchKernelGGL(k_colmax, dim3((unsigned)(steps < kCmWG ? steps : kCmWG)),
                       dim3(64 * kCmWaves), 0, st, Q, K, off, N, H, c, (uint32_t*)colmax);
}

}  // namespace vp
