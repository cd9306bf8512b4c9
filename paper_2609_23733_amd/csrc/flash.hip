// FULL-mode heads (Algorithm 1, first branch): exact softmax attention of a
// head's queries over all N = S * P keys of all views, Y_h =
// softmax(Q_h K_h^T / sqrt(d)) V_h, on MFMA with an online softmax over
// 64-key tiles that are double-buffered through LDS.
//
// Work is taken from the FULL bucket that the mode assignment wrote on the
// device: a grid sized for every head exits early past n_full * q_tiles, so
// no mode is ever copied to the host.
#include <type_traits>

#include "vp_device.hpp"
#include "vp_internal.hpp"

namespace vp {

constexpr int kBK = 64;       // keys per tile

// Number of FULL heads in the bucket array written by the mode assignment,
// 0 if the counts are inconsistent with H (never index past the head list).
__device__ __forceinline__ int full_count(const int32_t* buckets, int H) {
    const int c0 = buckets[0], c1 = buckets[1], c2 = buckets[2];
    if (c0 < 0 || c1 < 0 || c2 < 0 || c0 + c1 + c2 != H) return 0;
    return c2;
}

// Head id of FULL slot `slot` (< full_count), or -1 if out of range.
__device__ __forceinline__ int full_head(const int32_t* buckets, int H, int slot) {
    const int h = buckets[3 + buckets[0] + buckets[1] + slot];
    return (h >= 0 && h < H) ? h : -1;
}
constexpr int kLdsRow = 72;   // bf16 LDS row stride (144 B: 16-B aligned, bank-staggered)

// ------------------------------------------------------------------------
// K5a: the scale of each FULL head's packed values.  The attention
// kernels multiply fp16 weights with fp16 values; the gather stores
// V_h 2^-e_h, with e_h chosen so that the head's largest |v| lies in
// [2^14, 2^15), and the kernels multiply O by 2^e_h at the end (both scalings
// exact).  Every bf16 value then fits fp16's range; values more than 2^29
// below the head's largest land in fp16's subnormals (absolute error at most
// 2^-40 of that largest value).
// K5a: per (group of kVmaxTiles key tiles, FULL slot), max |v|; the gather
// (K5) reduces those per slot and records vsc[slot] = (2^-e_h, 2^e_h).
// ------------------------------------------------------------------------
constexpr int kVmaxTiles = 16;

__device__ __forceinline__ float block_max256(float m, float* red) {
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__global__ __launch_bounds__(256) void k_vmax_partial(const bf16* __restrict__ V,
                                                      const int32_t* __restrict__ buckets,
                                                      int64_t N, int H,
                                                      float* __restrict__ vpart) {
    const int slot = blockIdx.y;
    if (slot >= full_count(buckets, H)) return;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    const int64_t r0 = (int64_t)blockIdx.x * kVmaxTiles * kBK;
    const int64_t r1 = (r0 + kVmaxTiles * kBK < N) ? r0 + kVmaxTiles * kBK : N;
    const int seg = (threadIdx.x & 7) * 8;
    float m = 0.f;
    // Four rows per thread and iteration, their loads issued together.
    for (int64_t row = r0 + (threadIdx.x >> 3); row < r1; row += 128) {
        bf16x8 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t rr = row + 32 * u;
            v[u] = rr < r1 ? load_bf16x8(V + (rr * H + h) * kD + seg) : zero_bf16x8();
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(bf16_to_f32(v[u][j])));
    }
    __shared__ float red[4];
    m = block_max256(m, red);
    if (threadIdx.x == 0) vpart[(int64_t)slot * gridDim.x + blockIdx.x] = m;
}

// Exponent e_h of the head's V scale 2^-e_h from its largest |v| (so that
// max |v| 2^-e_h lies in [2^14, 2^15)).  An all-zero head keeps scale 1; an
// infinite value (NaN never wins fmaxf) keeps scale 1 too and reaches the
// output as it would in exact arithmetic.
__device__ __forceinline__ int vscale_exponent(float m) {
    int e = 0;
    if (m > 0.f && m <= 3.4028235e38f) e = ilogbf(m) - 14;
    return e < -126 ? -126 : (e > 126 ? 126 : e);
}

// ------------------------------------------------------------------------
// K5: bucket gather.  For each FULL head (slot s of the FULL bucket), copy
// V_h 2^-e_h into a packed, tile-transposed fp16 buffer Vt[s][tile][d][64
// keys], K_h into packed fp16 tiles Kh[s][tile][64 keys][d] (key rows in
// swap23 order; bf16 values convert exactly while |k| stays in fp16's normal
// range), keys past N zero in both, and record kmax[s][tile] = max |k_j| over
// the tile's keys.  The attention kernels read the tiles as contiguous 8 KB
// blocks whose rows feed the MFMA operands directly, and use kmax to bound
// the logits.
// ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gather_vt(const bf16* __restrict__ K,
                                                   const bf16* __restrict__ V,
                                                   const int32_t* __restrict__ buckets, int64_t N,
                                                   int H, int nkt, const float* __restrict__ vpart,
                                                   int nvp, float* __restrict__ vsc,
                                                   f16* __restrict__ Vt, f16* __restrict__ Kh,
                                                   float* __restrict__ kmax) {
    const int slot = blockIdx.y, tile = blockIdx.x;
    const int nfull = full_count(buckets, H);
    if (slot >= nfull) return;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    __shared__ __attribute__((aligned(16))) f16 s[kD * kLdsRow];
    __shared__ float s_norm[4];
    const int t = threadIdx.x;
    const int key = t >> 2, dseg = (t & 3) * 16;
    const int64_t row = (int64_t)tile * kBK + key;
    const bool ok = row < N;
    const int64_t off = ((ok ? row : 0) * H + h) * kD + dseg;
    bf16x8 a = load_bf16x8(V + off), b = load_bf16x8(V + off + 8);
    bf16x8 ka = load_bf16x8(K + off), kb = load_bf16x8(K + off + 8);
    if (!ok) a = b = ka = kb = zero_bf16x8();
    // The head's V scale from the partial maxima (every workgroup of the
    // head reduces the same values in the same order; the tile-0 one
    // records the scale and its inverse for the attention kernels).
    float vm = 0.f;
    for (int i = t; i < nvp; i += 256) vm = fmaxf(vm, vpart[(int64_t)slot * nvp + i]);
    vm = block_max256(vm, s_norm);
    const int e = vscale_exponent(vm);
    const float down = ldexpf(1.f, -e);
    if (tile == 0 && t == 0) {
        vsc[2 * slot] = down;
        vsc[2 * slot + 1] = ldexpf(1.f, e);
    }
    __syncthreads();   // s_norm is reused below
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        s[(dseg + j) * kLdsRow + key] = (f16)(bf16_to_f32(a[j]) * down);
        s[(dseg + 8 + j) * kLdsRow + key] = (f16)(bf16_to_f32(b[j]) * down);
    }
    float n2 = 0.f;
    f16x8 ha, hb;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float x = bf16_to_f32(ka[j]), y = bf16_to_f32(kb[j]);
        ha[j] = (f16)x;
        hb[j] = (f16)y;
        n2 = fmaf(x, x, fmaf(y, y, n2));
    }
    f16* kd = Kh + (((int64_t)slot * nkt + tile) * kBK + swap23(key)) * kD + dseg;
    *reinterpret_cast<f16x8*>(kd) = ha;
    *reinterpret_cast<f16x8*>(kd + 8) = hb;
    n2 += __shfl_xor(n2, 1);
    n2 += __shfl_xor(n2, 2);
    n2 = wave_max(n2);
    if ((t & 63) == 0) s_norm[t >> 6] = n2;
    __syncthreads();
    if (t == 0)
        kmax[(int64_t)slot * nkt + tile] =
            sqrtf(fmaxf(fmaxf(s_norm[0], s_norm[1]), fmaxf(s_norm[2], s_norm[3])));
    const int d = t >> 2, kseg = (t & 3) * 16;
    f16* dst = Vt + (((int64_t)slot * nkt + tile) * kD + d) * kBK + kseg;
    *reinterpret_cast<f16x8*>(dst) = *reinterpret_cast<const f16x8*>(&s[d * kLdsRow + kseg]);
    *reinterpret_cast<f16x8*>(dst + 8) =
        *reinterpret_cast<const f16x8*>(&s[d * kLdsRow + kseg + 8]);
}

// ------------------------------------------------------------------------
// K6 (bf16): FULL-head attention.  Per 64-key tile and wave of 64 queries:
// S^T = K Q^T (keys x queries, 2 x 2 blocks of 32x32, 16 MFMAs), softmax
// weights in registers, O^T += V^T P^T (d x queries, 16 MFMAs).  Each lane
// owns one query column of every block, so softmax row statistics stay in
// the lane plus one exchange with lane ^ 32.  K rows sit in LDS with index
// bits 2 and 3 swapped so that the S^T registers hold eight consecutive keys
// per lane-half: they become the B operand of the PV MFMA without any data
// movement.  Operands are fp16: K as packed by the gather (bf16 values in
// fp16's range convert exactly), V^T scaled by 2^-e_h, P rounded to nearest
// (relative error at most 2^-11).
//
// Softmax is invariant to the reference point subtracted from the logits
// before exponentiation.  A work item (512 queries of one head) runs in one
// of three modes, chosen from Cauchy-Schwarz bounds (|q . k| <= |q| max_j
// |k_j|) before its first tile:
//  - FAST: every logit of the item lies within +-kFastBound in log2 units.
//    The scale c = log2(e) / sqrt(d) is folded into Q (rounded to fp16,
//    relative error 2^-11), S comes out of the MFMA in log2 units and the
//    reference point is 0: p = 2^S lies in [2^-10, 2^10], fp16's normal range,
//    and a score costs one exp2 and half a pack.
//  - EXT: every logit lies within +-kExtBound.  Q and S as in FAST mode, and
//    the reference point m of a query stays 0 unless the segment's first
//    tile's maximum lies below kExtLow (then m is that maximum) or a weight
//    or a lane's fp16 row sum overflows (then m moves to the tile maximum,
//    O and l are rescaled and the tile's weights taken again).  While m = 0
//    for every query of a wave's 32-query block, its scores cost what they
//    cost in FAST mode; otherwise one subtraction more.  The fp16 rounding
//    of c q moves a logit by at most 2^-11 kExtBound.
//  - WIDE: Q keeps its bf16 value (exact in fp16), logits are scaled in fp32
//    and a running reference point m moves with the logits.  The segment's
//    first tile sets m to its maximum; every later tile is exponentiated
//    against m as it comes, and only if a weight or a lane's fp16 row sum
//    overflows (some logit more than ~15 above m) is the tile maximum taken,
//    m moved to it (O and l rescaled) and the tile's weights taken again.
//    A score costs one FMA more than in FAST mode.  (Teacher instances keep
//    the earlier test before the weights: a tile whose logits provably stay
//    below m + kSlack, by its largest key norm, is exponentiated against m
//    directly; otherwise the tile maximum is taken and m moves when the tile
//    exceeds m + kSlack.)
// In EXT and WIDE modes one wave-wide vote per tile, after both of a wave's
// 32-query blocks are packed and summed, decides whether any of them
// overflowed.
// Row sums: the packed fp16 weights of a lane's 32 keys per tile are added
// as a tree of packed fp16 adds (at most 32 weights of at most 2^10: no
// overflow; relative error at most 5 * 2^-11), then into l in fp32.  The
// numerator uses the same rounded weights.  Teacher instances (which also
// write each query's log2 sum_k 2^x) run every item in WIDE mode, whose
// logits are exact, and add the unrounded fp32 weights with a compensated
// sum instead.  Items whose Q or K values exceed fp16's range are flagged
// and left to K6b, which keeps bf16 operands.
// ------------------------------------------------------------------------
constexpr int kBQ16 = 256;
constexpr float kFastBound = 10.f;   // |logit| bound (log2 units) of FAST mode
constexpr float kSlack = 10.f;       // WIDE: log2 headroom above the running reference
constexpr float kF16Safe = 4096.f;   // FAST: |c q|, |k| limit for the fp16 operands
constexpr float kF16Max = 65504.f;   // WIDE: largest finite fp16
constexpr float kExtBound = 24.f;    // EXT: |logit| bound (log2 units)
constexpr float kExtLow = -4.f;      // EXT: lowest first-tile maximum kept at reference 0

// Kahan step: adds x to the sum s with compensation e (the sum is s - e).
__device__ __forceinline__ void kahan_add(float& s, float& e, float x) {
    const float y = x - e;
    const float t = s + y;
    e = (t - s) - y;
    s = t;
}

__device__ __forceinline__ float dot2_ones(uint32_t pair, float acc) {
    const f16x2 v = __builtin_bit_cast(f16x2, pair);
    const f16x2 one = {(f16)1.0f, (f16)1.0f};
    return __builtin_amdgcn_fdot2(v, one, acc, false);
}

// Sum of the 32 packed fp16 weights of one query block (16 registers of two
// weights) as a tree of packed fp16 adds, added to acc in fp32.
__device__ __forceinline__ float tree_sum(const f16x8 (&P)[2][2], float acc) {
    f16x2 t[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        t[2 * i] = f16x2{P[0][0][2 * i], P[0][0][2 * i + 1]} +
                   f16x2{P[0][1][2 * i], P[0][1][2 * i + 1]};
        t[2 * i + 1] = f16x2{P[1][0][2 * i], P[1][0][2 * i + 1]} +
                       f16x2{P[1][1][2 * i], P[1][1][2 * i + 1]};
    }
#pragma unroll
    for (int w = 4; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) t[i] = t[i] + t[i + w];
    return dot2_ones(__builtin_bit_cast(uint32_t, t[0]), acc);
}

// Y[q, h, d] = O up / l for the wave's two 32-query blocks (up = 2^e_h, the
// inverse of the packed values' scale); lane holds d = 32 db + 8 g + 4 hh + i
// for i = 0..3.
__device__ __forceinline__ void store_rows(const f32x16 (&O)[2][2], const float (&l)[2],
                                           const int64_t (&qidx)[2], int64_t N, int H, int h,
                                           int hh, float up, void* __restrict__ Y, int ydt) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const float lt = l[qb] + __shfl_xor(l[qb], 32);
        const float inv = up / lt;
        const int64_t qi = qidx[qb];
        if (qi < N) {
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int64_t off = (qi * H + h) * kD + db * 32 + 8 * g + 4 * hh;
                    const float y0 = O[qb][db][4 * g] * inv, y1 = O[qb][db][4 * g + 1] * inv;
                    const float y2 = O[qb][db][4 * g + 2] * inv, y3 = O[qb][db][4 * g + 3] * inv;
                    if (ydt == DT_BF16) {
                        bf16x4 v;
                        v[0] = (bf16)y0; v[1] = (bf16)y1; v[2] = (bf16)y2; v[3] = (bf16)y3;
                        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Y) + off) = v;
                    } else {
                        *reinterpret_cast<float4*>(reinterpret_cast<float*>(Y) + off) =
                            make_float4(y0, y1, y2, y3);
                    }
                }
        }
    }
}

// o_q = m + log2 l per query of the wave's two blocks (teacher instances).
// (m is the same in both lane halves.)
__device__ __forceinline__ void store_offsets(const float (&l)[2], const float (&m)[2],
                                              const int64_t (&qidx)[2], int64_t N, int h, int hh,
                                              float* __restrict__ off) {
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const float lt = l[qb] + __shfl_xor(l[qb], 32);
        if (hh == 0 && qidx[qb] < N) off[(int64_t)h * N + qidx[qb]] = m[qb] + __log2f(lt);
    }
}

// K6a: one workgroup = 8 waves x 64 queries of one FULL head, two waves per
// SIMD (waves w and w + 4).  Ping-pong: waves 0-3 (group A) and 4-7 (group
// B) run the same sequence of phases, matrix(0), vector(0), matrix(1), ...,
// group B one phase behind, with one workgroup barrier per phase, so that in
// every phase one wave of each SIMD issues MFMAs while the other issues the
// softmax's vector instructions:
//   matrix(t): O += V(t-1) P(t-1)  then  S(t) = K(t) Q^T   (32 MFMAs)
//   vector(t): P(t) = fp16 weights of S(t), l += their row sums
// LDS slot t % 2 holds K(t) and V(t-1).
//
// Balanced tail: the work is n_full x q-tiles items of nkt key tiles.  A
// fixed grid of G workgroups (one per CU) takes the items in rounds,
// workgroup w item r G + w, so that in every round the workgroups of an XCD
// stream the same key tiles of one head through its L2.  The R < G items of
// the last, partial round are cut into one flat sequence of R nkt item-tile
// steps, split evenly over the workgroups (at least kMinPartTiles steps
// each), so the tail takes R / G of a round instead of a whole one.  Results
// over key ranges combine exactly: a workgroup that covers only part of an
// item writes its unnormalized O, l and reference point m to one of its two
// partial slots (0 for the first item of its range, 1 for the last), and K6c
// combines the parts of each split item in workgroup order.  The part
// holding tile 0 writes exact_items[L] (1 = left to K6b), so flags never
// carry over.
constexpr int kBQf = 512;
constexpr int kStreamWG = 256;      // grid: one workgroup per CU
constexpr int kPartFloats = kBQf * kD + 2 * kBQf;   // partial slot: O[512][64], l[512], m[512]

// Fewest key tiles per workgroup in the tail: one.  A workgroup's chain of tiles (2-3
// us each) is what a short layer waits for; a part costs its 131 KB once more in
// K6c.  Layer, 4 FULL heads, with at least 8, 4, 2 and 1: 300 tokens 79.0, 81.4, 80.5,
// 73.5 us; 600 84.3, 80.9, 71.7, 70.5; 1,000 78.2, 76.2, 74.2, 72.7; 1,374 91.2, 88.0,
// 75.5, 77.4; 16 heads of 300 90.8, 79.7, 77.2, 69.5.  From 2,048 steps on all are the
// same (256 workgroups).
constexpr int kMinPartTiles = 1;
constexpr int64_t kRotateTiles = 4096;   // 64 MB of K and V^T tiles (16 KB each)

// Workgroups used for T tail steps (at most G, at least `least` steps each), the first step of workgroup w, and the workgroup holding step x.
__host__ __device__ inline int tail_groups(int64_t T, int G, int least = kMinPartTiles) {
    const int64_t g = T / least;
    return g < 1 ? 1 : (g < G ? (int)g : G);
}
__device__ __forceinline__ int64_t tail_start(int w, int64_t T, int G) {
    return (int64_t)w * T / G;
}
__device__ __forceinline__ int tail_owner(int64_t x, int64_t T, int G) {
    return (int)(((x + 1) * G + T - 1) / T) - 1;
}

enum { ITEM_FAST = 0, ITEM_WIDE = 1, ITEM_EXACT = 2, ITEM_EXT = 3 };

template <bool kTeach>
__global__ __launch_bounds__(512, 1) void k_flash_bf16(const bf16* __restrict__ Q,
                                                       const f16* __restrict__ Kh,
                                                       const f16* __restrict__ Vt,
                                                       const float* __restrict__ kmax,
                                                       const float* __restrict__ vsc,
                                                       const int32_t* __restrict__ buckets,
                                                       int64_t N, int H, int nqt, int nkt, float c,
                                                       int32_t* __restrict__ exact_items,
                                                       float* __restrict__ part, int G,
                                                       void* __restrict__ Y, int ydt,
                                                       float* __restrict__ off) {
    const int nfull = full_count(buckets, H);
    const int active = nfull * nqt;
    if (active == 0) return;
    const int w = xcd_remap(blockIdx.x, G);
    const int full = active / G * G, R = active - full;
    // The wave index is uniform within a wave: say so, so that the group
    // choice and everything derived from it stay scalar.
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 31, hh = lane >> 5;
    const bool groupB = wave >= 4;

    __shared__ __attribute__((aligned(16))) f16 sK[2][kBK * kLdsRow];
    __shared__ __attribute__((aligned(16))) f16 sV[2][kD * kLdsRow];
    __shared__ float sKmax[8], sQmax[8];

    // One segment: key tiles [t0, t1) of item L; written to partial slot
    // pslot of this workgroup if the segment is not the whole item.
    auto segment = [&](int L, int t0, int t1, int pslot) __attribute__((always_inline)) {
        const int slot = L / nqt, qt = L - slot * nqt;
        const int h = full_head(buckets, H, slot);
        if (h < 0) return;

        // max_j |k_j| over the head, from the per-tile maxima.
        const float* kmx = kmax + (int64_t)slot * nkt;
        {
            float km = 0.f;
            for (int i = threadIdx.x; i < nkt; i += 512) km = fmaxf(km, kmx[i]);
            km = wave_max(km);
            if (lane == 0) sKmax[wave] = km;
        }

        // This wave's two 32-query blocks (bf16) and |q| per query.
        bf16x8 qraw[2][4];
        int64_t qidx[2];
        float qn[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            const int64_t qi = (int64_t)qt * kBQf + wave * 64 + qb * 32 + n;
            qidx[qb] = qi;
            const bool ok = qi < N;
            const bf16* qp = Q + ((ok ? qi : 0) * H + h) * kD + 8 * hh;
            float n2 = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                qraw[qb][ks] = ok ? load_bf16x8(qp + 16 * ks) : zero_bf16x8();
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float x = bf16_to_f32(qraw[qb][ks][j]);
                    n2 = fmaf(x, x, n2);
                }
            }
            n2 += __shfl_xor(n2, 32);
            qn[qb] = sqrtf(n2);
        }
        {
            const float qm = wave_max(fmaxf(qn[0], qn[1]));
            if (lane == 0) sQmax[wave] = qm;
        }
        __syncthreads();
        int mode;
        {
            float km = sKmax[0], qm = sQmax[0];
#pragma unroll
            for (int v = 1; v < 8; ++v) {
                km = fmaxf(km, sKmax[v]);
                qm = fmaxf(qm, sQmax[v]);
            }
            // Conditions written as "within" so that a NaN norm goes to K6b.
            const bool safe = !kTeach && qm * c <= kF16Safe && km <= kF16Safe;
            const bool fast = safe && qm * c * km <= kFastBound;
            const bool ext = safe && qm * c * km <= kExtBound;
            const bool wide = qm <= kF16Max && km <= kF16Max;
            mode = fast ? ITEM_FAST : (ext ? ITEM_EXT : (wide ? ITEM_WIDE : ITEM_EXACT));
        }
        if (t0 == 0 && threadIdx.x == 0) exact_items[L] = mode == ITEM_EXACT;
        if (mode == ITEM_EXACT) return;   // uniform over the workgroup

        // Q^T operands, kept in registers: fp16 c q (FAST, EXT) or fp16 q
        // (WIDE).
        f16x8 Qop[2][4];
        const float qs = mode == ITEM_WIDE ? 1.f : c;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    Qop[qb][ks][j] = (f16)(bf16_to_f32(qraw[qb][ks][j]) * qs);

        // Tile copies: group A (threads 0-255) copies K tiles, group B V^T
        // tiles, each a contiguous 8 KB block: 64 rows x 4 segments of 16
        // elements.  r counts tiles from t0.
        const int ns = t1 - t0;
        const int tl = threadIdx.x & 255, lr = tl >> 2, lc = (tl & 3) * 16;
        const f16* Khh = Kh + ((int64_t)slot * nkt + t0) * kBK * kD;
        const f16* Vth = Vt + ((int64_t)slot * nkt + t0) * kD * kBK;
        u32x4 g0, g1;
        // While all FULL heads' tiles fit in 64 MB (a quarter of the
        // last-level cache), the segment's tiles are taken in a rotated
        // order, starting at a different tile in each of the 32 workgroups of
        // an XCD, so that they do not all read the same tile at the same time
        // (larger sets are read in step, so that the workgroups of an XCD
        // share what its L2 holds).
        const int rot = (int64_t)nfull * nkt <= kRotateTiles
                            ? (int)(((int64_t)(w & 31) * ns) >> 5) : 0;
        auto tile_of = [&](int r) {   // r < ns
            const int t = r + rot;
            return t >= ns ? t - ns : t;
        };
        auto fetch = [&](int r) {   // tile r (clamped to the last one) into registers
            r = tile_of(r < ns ? r : ns - 1);
            const u32x4* src = groupB
                ? reinterpret_cast<const u32x4*>(Vth + ((int64_t)r * kD + lr) * kBK + lc)
                : reinterpret_cast<const u32x4*>(Khh + ((int64_t)r * kBK + lr) * kD + lc);
            g0 = src[0];
            g1 = src[1];
        };
        auto stash = [&](int sl) {   // ... into LDS slot sl
            u32x4* dst = groupB ? reinterpret_cast<u32x4*>(&sV[sl][lr * kLdsRow + lc])
                                : reinterpret_cast<u32x4*>(&sK[sl][lr * kLdsRow + lc]);
            dst[0] = g0;
            dst[1] = g1;
        };

        f32x16 O[2][2], S[2][2];
        f16x8 P[2][2][2];
        float l[2], le[2], m[2];   // le: Kahan compensation of l (teacher instances)
        const float qnc[2] = {qn[0] * c, qn[1] * c};
        const f16x8 zp = {};
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            O[qb][0] = O[qb][1] = zero_f32x16();
            l[qb] = le[qb] = 0.f;
            m[qb] = mode == ITEM_WIDE ? -INFINITY : 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) P[qb][kb][0] = P[qb][kb][1] = zp;
        }

        // Matrix phase of tile r: O += V(r-1) P(r-1), then S(r) = K(r) Q^T
        // from sK[r%2].  The V operands were read into registers at the end of
        // the wave's previous vector phase, so the 16 PV MFMAs start at once
        // and hide the latency of the K reads.  (PV first: P(r-1) is dead
        // before S(r) is written, so the two can share registers.  r = 0: P
        // and the V operands are zero, so the PV adds exactly nothing.)
        f16x8 va[2][2][2];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) va[db][kb][0] = va[db][kb][1] = zp;
        auto prefetch_v = [&](int sl) {   // V operands of the next PV product
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        va[db][kb][b] = *reinterpret_cast<const f16x8*>(
                            &sV[sl][(db * 32 + n) * kLdsRow + kb * 32 + 16 * b + 8 * hh]);
        };
        auto pv = [&] {
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        O[0][db] = mfma_f16(va[db][kb][b], P[0][kb][b], O[0][db]);
                        O[1][db] = mfma_f16(va[db][kb][b], P[1][kb][b], O[1][db]);
                    }
        };
        auto mma_phase = [&](int r) {
            const int sl = r & 1;
            f16x8 ka[2][4];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    ka[kb][ks] = *reinterpret_cast<const f16x8*>(
                        &sK[sl][(kb * 32 + n) * kLdsRow + 16 * ks + 8 * hh]);
            pv();
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    if (ks == 0) S[0][kb] = S[1][kb] = zero_f32x16();
                    S[0][kb] = mfma_f16(ka[kb][ks], Qop[0][ks], S[0][kb]);
                    S[1][kb] = mfma_f16(ka[kb][ks], Qop[1][ks], S[1][kb]);
                }
            // K operands first, then the PV and S products.
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 32, 0);
        };
        // Vector phase of tile r: S(r) -> P(r), l += row sums.  The segment's
        // last tile masks keys >= N to weight 0 (a separate instance, so that
        // no other tile pays for the test).
        auto tile_max = [&](int qb) {   // largest S of the tile, per query
            float mx = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[qb][kb][i]);
            return fmaxf(mx, __shfl_xor(mx, 32));
        };
        auto valu_phase = [&](int r, auto last_tag, auto mode_tag, auto mid) {
            constexpr bool kWide = decltype(mode_tag)::value == ITEM_WIDE;
            constexpr bool kExt = decltype(mode_tag)::value == ITEM_EXT;
            (void)last_tag;
            const int tr = t0 + tile_of(r);
            if ((N & (kBK - 1)) && tr == nkt - 1) {
                const int64_t k0 = (int64_t)tr * kBK;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int64_t key = k0 + kb * 32 + 16 * (i >> 3) + 8 * hh + (i & 7);
                        if (key >= N) S[0][kb][i] = S[1][kb][i] = -INFINITY;
                    }
            }
            const float kbt = kTeach ? kmx[tr] : 0.f;
            if (kExt) {
                // Exponentials in place (S <= kExtBound - m: finite in fp32),
                // then fp16 packs and row sums; a query block whose weights
                // or row sums overflow fp16 moves its reference point to the
                // tile maximum, log2 of its largest exponential.
                bool sh[2];
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    if (r == 0) {
                        const float mx = tile_max(qb);
                        m[qb] = mx < kExtLow ? mx : 0.f;   // O, l are still 0
                    }
                    sh[qb] = __builtin_amdgcn_ballot_w64(m[qb] != 0.f) != 0;
                }
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    const float nm = -m[qb];
                    if (sh[qb]) {
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int i = 0; i < 16; ++i)
                                S[qb][kb][i] = exp2f_fast(S[qb][kb][i] + nm);
                    } else {
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) S[qb][kb][i] = exp2f_fast(S[qb][kb][i]);
                    }
                }
                auto pack = [&](int qb, float sc) {   // P = fp16 (sc * e)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            u32x4 pk;
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                f32x2 e = {S[qb][kb][8 * b + 2 * j], S[qb][kb][8 * b + 2 * j + 1]};
                                if (sc != 1.f) e = e * sc;
                                pk[j] = __builtin_bit_cast(uint32_t,
                                                           __builtin_convertvector(e, f16x2));
                            }
                            P[qb][kb][b] = __builtin_bit_cast(f16x8, pk);
                        }
                };
                // Both blocks packed and summed, then one overflow test for
                // the two (a branch per block would keep the second block's
                // work from overlapping the first one's dependent sums).
                float ln[2];
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) pack(qb, 1.f);
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) ln[qb] = tree_sum(P[qb], l[qb]);
                if (__builtin_amdgcn_ballot_w64(!(ln[0] < INFINITY) || !(ln[1] < INFINITY)) != 0) {
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) {
                        if (__builtin_amdgcn_ballot_w64(!(ln[qb] < INFINITY)) != 0) {
                            const float mn = fmaxf(m[qb], m[qb] + __log2f(tile_max(qb)));
                            const float al = exp2f_fast(m[qb] - mn);
                            m[qb] = mn;
                            l[qb] *= al;
#pragma unroll
                            for (int db = 0; db < 2; ++db)
#pragma unroll
                                for (int i = 0; i < 16; ++i) O[qb][db][i] *= al;
                            pack(qb, al);
                            ln[qb] = tree_sum(P[qb], l[qb]);
                        }
                    }
                }
                l[0] = ln[0];
                l[1] = ln[1];
                // (S is dead: the next V operands' LDS reads)
                mid();
                return;
            }
            if (!kWide && !kTeach) {
                // FAST: all exponentials first (in place), then the packs and
                // row sums.
#pragma unroll
                for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) S[qb][kb][i] = exp2f_fast(S[qb][kb][i]);
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            u32x4 pk;
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const f32x2 e = {S[qb][kb][8 * b + 2 * j],
                                                 S[qb][kb][8 * b + 2 * j + 1]};
                                pk[j] = __builtin_bit_cast(uint32_t,
                                                           __builtin_convertvector(e, f16x2));
                            }
                            P[qb][kb][b] = __builtin_bit_cast(f16x8, pk);
                        }
                }
                // (S is dead: the next V operands' LDS reads go here, so that
                // they complete under the row sums rather than at the barrier.)
                mid();
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) l[qb] = tree_sum(P[qb], l[qb]);
                return;
            }
            // WIDE items and teacher instances from here on.  WIDE (not
            // teacher): the segment's first tile sets m to its maximum before
            // the weights; later tiles are taken against m and redone only on
            // fp16 overflow (below).
            auto reset_m = [&](int qb) {
                float mx = -INFINITY;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[qb][kb][i]);
                mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
                const float mn = fmaxf(m[qb], mx);
                const float al = exp2f_fast(m[qb] - mn);
                m[qb] = mn;
                l[qb] *= al;
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) O[qb][db][i] *= al;
            };
            if (!kTeach && r == 0) {
                reset_m(0);
                reset_m(1);
            }
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                if (kTeach) {
                    // Keep m unless the bound cannot rule out a logit above
                    // m + kSlack for some query of this block.
                    if (__builtin_amdgcn_ballot_w64(qnc[qb] * kbt > m[qb] + kSlack) != 0) {
                        float mx = -INFINITY;
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[qb][kb][i]);
                        mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
                        const bool move = mx > m[qb] + kSlack;
                        const float mn = move ? mx : m[qb];
                        const float al = move ? exp2f_fast(m[qb] - mn) : 1.f;
                        m[qb] = mn;
                        l[qb] *= al;
                        le[qb] *= al;
#pragma unroll
                        for (int db = 0; db < 2; ++db)
#pragma unroll
                            for (int i = 0; i < 16; ++i) O[qb][db][i] *= al;
                    }
                }
                const float nm = -m[qb];
                float ls0 = 0.f, ls1 = 0.f;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        u32x4 pk;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            f32x2 e;
                            e[0] = exp2f_fast(fmaf(S[qb][kb][8 * b + 2 * j], c, nm));
                            e[1] = exp2f_fast(fmaf(S[qb][kb][8 * b + 2 * j + 1], c, nm));
                            pk[j] = __builtin_bit_cast(uint32_t,
                                                       __builtin_convertvector(e, f16x2));
                            if (kTeach) {
                                ls0 += e[0];
                                ls1 += e[1];
                            }
                        }
                        P[qb][kb][b] = __builtin_bit_cast(f16x8, pk);
                    }
                if (kTeach) {
                    kahan_add(l[qb], le[qb], ls0 + ls1);
                    if (qb == 0) mid();   // (the first block's S is dead)
                }
            }
            if (kTeach) return;
            // WIDE: both blocks' fp16 row sums, then one overflow vote for
            // the two (as in EXT mode); a block that overflowed moves m to
            // its tile maximum and is taken again from its fp32 logits.
            float ln[2];
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) ln[qb] = tree_sum(P[qb], l[qb]);
            if (__builtin_amdgcn_ballot_w64(!(ln[0] < INFINITY) || !(ln[1] < INFINITY)) != 0) {
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    if (__builtin_amdgcn_ballot_w64(!(ln[qb] < INFINITY)) == 0) continue;
                    reset_m(qb);
                    const float nm2 = -m[qb];
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            u32x4 pk;
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                f32x2 e;
                                e[0] = exp2f_fast(fmaf(S[qb][kb][8 * b + 2 * j], c, nm2));
                                e[1] = exp2f_fast(fmaf(S[qb][kb][8 * b + 2 * j + 1], c, nm2));
                                pk[j] = __builtin_bit_cast(uint32_t,
                                                           __builtin_convertvector(e, f16x2));
                            }
                            P[qb][kb][b] = __builtin_bit_cast(f16x8, pk);
                        }
                    ln[qb] = tree_sum(P[qb], l[qb]);
                }
            }
            l[0] = ln[0];
            l[1] = ln[1];
            mid();   // (S is dead)
        };
        const std::false_type body{};
        const std::true_type tail{};
        // End of a phase: a workgroup barrier that the compiler may not
        // schedule any instruction across (it would otherwise hoist the next
        // phase's register-only work above it and undo the alternation).
        auto phase_end = [] {
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
        };

        // Phases, one workgroup barrier each (2 ns + 2 in both groups, counting
        // the prologue's):
        //   group A:  M(0) V(0) M(1) V(1) ... M(ns-1) V(ns-1) -
        //   group B:  -    M(0) V(0) M(1) ... V(ns-2) M(ns-1) V(ns-1)
        // A wave issues its 32 MFMAs in a few dozen cycles and then waits for
        // the other wave's vector phase, so the tile copies live in the
        // matrix phases: a group loads a tile from global memory during its
        // vector phase and stores it to LDS after issuing the MFMAs of its
        // next matrix phase.  Group A stores K(r+1) to sK[(r+1) % 2] during
        // M(r); group B stores V(r+1) to sV[r % 2] during M(r) (V(0) to sV[1]
        // in the first phase), two phases before group A reads those V
        // operands at the end of its V(r+1) for M(r+2), and group B at the end
        // of its own V(r+1).  A slot is rewritten only after both groups'
        // last reads.
        auto mma_then = [&](int r, int store_slot) {
            mma_phase(r);
            __builtin_amdgcn_sched_barrier(0);
            if (store_slot >= 0) stash(store_slot);
        };
        auto run = [&](auto mode_tag) {
            if (!groupB) {
                fetch(0);
                stash(0);
                fetch(1);
                phase_end();
                for (int r = 0; r < ns - 1; ++r) {
                    mma_then(r, (r + 1) & 1);
                    phase_end();
                    fetch(r + 2);
                    valu_phase(r, body, mode_tag, [&] { prefetch_v((r + 1) & 1); });
                    phase_end();
                }
                mma_then(ns - 1, -1);
                phase_end();
                valu_phase(ns - 1, tail, mode_tag, [&] { prefetch_v(ns & 1); });
                phase_end();
                phase_end();
            } else {
                fetch(0);
                phase_end();
                stash(1);
                fetch(1);
                phase_end();
                for (int r = 0; r < ns - 1; ++r) {
                    mma_then(r, r & 1);
                    phase_end();
                    fetch(r + 2);
                    valu_phase(r, body, mode_tag, [&] { prefetch_v((r + 1) & 1); });
                    phase_end();
                }
                mma_then(ns - 1, -1);
                phase_end();
                valu_phase(ns - 1, tail, mode_tag, [&] { prefetch_v(ns & 1); });
                phase_end();
            }
            pv();   // O += V(ns-1) P(ns-1)
        };
        if (kTeach || mode == ITEM_WIDE)
            run(std::integral_constant<int, ITEM_WIDE>{});
        else if (!kTeach && mode == ITEM_EXT)
            run(std::integral_constant<int, ITEM_EXT>{});
        else
            run(std::integral_constant<int, ITEM_FAST>{});

        if (kTeach) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) l[qb] -= le[qb];
        }
        if (t0 == 0 && t1 == nkt) {
            store_rows(O, l, qidx, N, H, h, hh, vsc[2 * slot + 1], Y, ydt);
            if (kTeach) store_offsets(l, m, qidx, N, h, hh, off);
        } else {
            // Partial slot: O[q][d] unnormalized, then l[q], then m[q]
            // (q = row in item).
            float* ps = part + (int64_t)(w * 2 + pslot) * kPartFloats;
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                const int qr = wave * 64 + qb * 32 + n;
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *reinterpret_cast<float4*>(ps + qr * kD + db * 32 + 8 * g + 4 * hh) =
                            make_float4(O[qb][db][4 * g], O[qb][db][4 * g + 1],
                                        O[qb][db][4 * g + 2], O[qb][db][4 * g + 3]);
                const float lt = l[qb] + __shfl_xor(l[qb], 32);
                if (hh == 0) {
                    ps[kBQf * kD + qr] = lt;
                    ps[kBQf * kD + kBQf + qr] = m[qb];
                }
            }
        }
    };

    for (int L = w; L < full; L += G) {
        segment(L, 0, nkt, 0);
        __syncthreads();   // LDS is reused by the next segment
    }
    if (R > 0) {
        const int64_t T = (int64_t)R * nkt;
        const int Gt = tail_groups(T, G);
        if (w < Gt) {
            const int64_t start = tail_start(w, T, Gt), end = tail_start(w + 1, T, Gt);
            for (int64_t x = start; x < end;) {
                const int i = (int)(x / nkt);
                const int t0 = (int)(x - (int64_t)i * nkt);
                const int64_t left = end - x;
                const int t1 = (int64_t)(nkt - t0) < left ? nkt : (int)(t0 + left);
                segment(full + i, t0, t1, x == start ? 0 : 1);
                x += t1 - t0;
                __syncthreads();
            }
        }
    }
}

// K6c: Y of the tail items that K6a split over workgroups: the parts' O and
// l, each relative to its part's reference point m, scaled to the largest m
// and added in a fixed order (so results are deterministic), then O 2^e_h / l.
// Items that K6a finished whole or left to K6b are passed over.
//
// Bound by reading the parts, 131 KB each, at most two per workgroup of K6a,
// and by the latency of a unit's loads.  The number of tail items R is known
// only on the device (0 .. G - 1), with Gt / R parts or one more each.  With
// few parts an item has 8 units of 64 queries (4 threads per query, one group).
// With 8 parts or more it has 64 units of 8 queries (16 threads per query, two
// groups of threads share the parts, 8 parts in flight): few items then still
// give enough workgroups, and no thread adds up more than half of the parts.
// 3 heads of 43,968 tokens (2 items of 128 parts) 87 us with 8 units an item,
// 14 us with 64; 4 heads of 34,350 tokens (16 items of 16 parts) 20 -> 10 us;
// 8 heads of 10,992 tokens (176 items of 2 parts) 14 us with 8 units, 30 us
// with 64 in a persistent loop.  Lines at 8 and 16 parts measured the same.
constexpr int kCombUnits = 8;   // workgroups per workgroup of K6a
constexpr int kCombFew = 8;     // fewer than this many parts per item

// One unit: the parts wf .. wl of ROWS queries of an item, dealt to GROUPS
// groups of threads whose sums are added in order.
template <int ROWS, int GROUPS>
__device__ __forceinline__ void combine_parts(const float* __restrict__ part, int wf, int wl,
                                              int vbase, int qr0, int qt, int64_t N, int H, int h,
                                              const float* __restrict__ vsc, int slot,
                                              void* __restrict__ Y, int ydt,
                                              float* __restrict__ off, float4* s_acc) {
    constexpr int TPR = 256 / (ROWS * GROUPS), NV = kD / TPR / 4;   // threads, float4s per query
    const int grp = threadIdx.x / (ROWS * TPR), rl = threadIdx.x % (ROWS * TPR);
    const int lr = rl % TPR, qr = qr0 + rl / TPR, d0 = lr * 4 * NV;
    const int64_t qi = (int64_t)qt * kBQf + qr;
    // Workgroup v's partial slot for this item: its first, unless v began
    // with an earlier item (only the item's first workgroup can).
    auto pslot = [&](int v) {
        return part + (int64_t)(v * 2 + (v == wf ? vbase : 0)) * kPartFloats;
    };
    // largest reference point and the sum of l, over the lanes of a query
    float mt = -INFINITY;
    for (int v = wf + lr; v <= wl; v += TPR) mt = fmaxf(mt, pslot(v)[kBQf * kD + kBQf + qr]);
#pragma unroll
    for (int o = TPR / 2; o >= 1; o >>= 1) mt = fmaxf(mt, __shfl_xor(mt, o));
    // 2^(m_v - max m): exactly 1 for parts at the largest reference point
    // (every part of a FAST item has m = 0).
    float lt = 0.f;
    for (int v = wf + lr; v <= wl; v += TPR) {
        const float* ps = pslot(v) + kBQf * kD + qr;
        lt = fmaf(ps[0], exp2f_fast(ps[kBQf] - mt), lt);
    }
#pragma unroll
    for (int o = TPR / 2; o >= 1; o >>= 1) lt += __shfl_xor(lt, o);
    float4 acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int kInFlight = NV == 1 ? 8 : 1;
#pragma unroll kInFlight
    for (int v = wf + grp; v <= wl; v += GROUPS) {
        const float* ps = pslot(v);
        const float sc = exp2f_fast(ps[kBQf * kD + kBQf + qr] - mt);
        const float4* src = reinterpret_cast<const float4*>(ps + qr * kD + d0);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const float4 a = src[k];
            acc[k].x = fmaf(a.x, sc, acc[k].x);
            acc[k].y = fmaf(a.y, sc, acc[k].y);
            acc[k].z = fmaf(a.z, sc, acc[k].z);
            acc[k].w = fmaf(a.w, sc, acc[k].w);
        }
    }
    if (GROUPS > 1) {
        static_assert(GROUPS == 1 || NV == 1, "one float4 per thread goes through s_acc");
        if (grp) s_acc[(grp - 1) * ROWS * TPR + rl] = acc[0];
        __syncthreads();
        if (grp) return;
#pragma unroll
        for (int g = 0; g < GROUPS - 1; ++g) {
            const float4 b = s_acc[g * ROWS * TPR + rl];
            acc[0].x += b.x; acc[0].y += b.y; acc[0].z += b.z; acc[0].w += b.w;
        }
    }
    if (qi >= N) return;
    if (off && lr == 0) off[(int64_t)h * N + qi] = mt + __log2f(lt);
    const float inv = vsc[2 * slot + 1] / lt;
    const int64_t yo = (qi * H + h) * kD + d0;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const float4 a = make_float4(acc[k].x * inv, acc[k].y * inv, acc[k].z * inv,
                                     acc[k].w * inv);
        if (ydt == DT_BF16) {
            bf16x4 o;
            o[0] = (bf16)a.x; o[1] = (bf16)a.y; o[2] = (bf16)a.z; o[3] = (bf16)a.w;
            *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Y) + yo + 4 * k) = o;
        } else {
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(Y) + yo + 4 * k) = a;
        }
    }
}

__global__ __launch_bounds__(256) void k_flash_combine(const int32_t* __restrict__ buckets,
                                                       int64_t N, int H, int nqt, int nkt,
                                                       const int32_t* __restrict__ exact_items,
                                                       const float* __restrict__ part,
                                                       const float* __restrict__ vsc, int G,
                                                       void* __restrict__ Y, int ydt,
                                                       float* __restrict__ off) {
    __shared__ float4 s_acc[128];
    const int nfull = full_count(buckets, H);
    const int active = nfull * nqt;
    const int full = active / G * G, R = active - full;
    if (R == 0) return;
    const int64_t T = (int64_t)R * nkt;
    const int Gt = tail_groups(T, G);
    // Few parts per item: 8 units of 64 queries.  Many: 64 units of 8 queries,
    // at most kCombUnits * G in all, since R <= Gt / kCombFew <= G / 8.
    const bool few = Gt < kCombFew * R;
    const int units = few ? 8 : 64;
    const int i = blockIdx.x / units, rb = blockIdx.x % units;
    if (i >= R) return;
    const int L = full + i;
    const int wf = tail_owner((int64_t)i * nkt, T, Gt);
    const int wl = tail_owner((int64_t)(i + 1) * nkt - 1, T, Gt);
    if (wf == wl || exact_items[L]) return;
    const int slot = L / nqt, qt = L - slot * nqt;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    const int vbase = tail_start(wf, T, Gt) == (int64_t)i * nkt ? 0 : 1;
    if (few)
        combine_parts<64, 1>(part, wf, wl, vbase, rb * 64, qt, N, H, h, vsc, slot, Y, ydt, off,
                             s_acc);
    else
        combine_parts<8, 2>(part, wf, wl, vbase, rb * 8, qt, N, H, h, vsc, slot, Y, ydt, off,
                            s_acc);
}
static_assert(kBQf == 512 && kCombUnits * kCombFew == 64, "units of k_flash_combine");

// ------------------------------------------------------------------------
// K6b (bf16, wide logit range): one workgroup = 4 waves x 64 queries of one
// FULL head; runs only the work items that K6a flagged.
// Per 64-key tile and wave:  S^T = K Q^T  (keys x queries, 2 x 2 blocks of
// 32x32, 16 MFMAs), online softmax in registers, O^T += V^T P^T (d x queries,
// 16 MFMAs).  Each lane owns one query column of every block, so softmax row
// statistics stay in the lane plus one exchange with lane ^ 32.  K rows are
// stored in LDS with index bits 2 and 3 swapped so that the S^T registers
// hold eight consecutive keys per lane-half: they become the B operand of the
// PV MFMA without any data movement.
//
// Softmax work per score is one FMA, one exp2, half an fp16 pack and half a
// dot2 (row sums of the packed P).  The running maximum m is a reference
// point, not necessarily the exact maximum: a tile whose logits provably stay
// below m + 8 (in log2 units; Cauchy-Schwarz, |q . k| c <= |q| c max|k|) is
// exponentiated against m directly, so p <= 2^8 fits fp16.  Only otherwise is
// the tile maximum computed, and m moves (rescaling O and l) only when the
// tile exceeds m + 8; the key that set m has p = 1, so l >= 1 and weights
// below fp16's normal range add at most 2^-25 each.  O / l is unchanged by
// the choice of reference point.
// ------------------------------------------------------------------------
template <bool kTeach>
__global__ __launch_bounds__(256, 2) void k_flash_bf16_wide(const bf16* __restrict__ Q,
                                                       const bf16* __restrict__ K,
                                                       const f16* __restrict__ Vt,
                                                       const float* __restrict__ kmax,
                                                       const float* __restrict__ vsc,
                                                       const int32_t* __restrict__ buckets,
                                                       int64_t N, int H, int nqt, int nkt, float c,
                                                       const int32_t* __restrict__ wide_items,
                                                       int nqt_fast, void* __restrict__ Y, int ydt,
                                                       float* __restrict__ off) {
    const int nfull = full_count(buckets, H);
    const int active = nfull * nqt;
    if ((int)blockIdx.x >= active) return;
    const int L = xcd_remap(blockIdx.x, active);
    const int slot = L / nqt, qt = L - slot * nqt;
    const int h = full_head(buckets, H, slot);
    if (h < 0 || wide_items[slot * nqt_fast + qt / (kBQf / kBQ16)] == 0) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = lane & 31, hh = lane >> 5;

    __shared__ __attribute__((aligned(16))) bf16 sK[2][kBK * kLdsRow];
    __shared__ __attribute__((aligned(16))) f16 sV[2][kD * kLdsRow];

    // Q^T operands of this wave's two 32-query blocks, kept in registers,
    // and |q| * c per query for the logit bound.
    bf16x8 Qop[2][4];
    int64_t qidx[2];
    float qnc[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const int64_t qi = (int64_t)qt * kBQ16 + wave * 64 + qb * 32 + n;
        qidx[qb] = qi;
        const bool ok = qi < N;
        const bf16* qp = Q + ((ok ? qi : 0) * H + h) * kD + 8 * hh;
        float n2 = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            Qop[qb][ks] = load_bf16x8(qp + 16 * ks);
            if (!ok) Qop[qb][ks] = zero_bf16x8();
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x = bf16_to_f32(Qop[qb][ks][j]);
                n2 = fmaf(x, x, n2);
            }
        }
        n2 += __shfl_xor(n2, 32);
        qnc[qb] = sqrtf(n2) * c;
    }

    // Global -> LDS copy assignment: 64 rows x 4 segments of 16 elements.
    const int lr = threadIdx.x >> 2, lc = (threadIdx.x & 3) * 16;
    const f16* Vth = Vt + (int64_t)slot * nkt * kD * kBK;
    const float* kmx = kmax + (int64_t)slot * nkt;
    bf16x8 pk0, pk1;
    f16x8 pv0, pv1;
    // Keys past N read row 0 instead (always in bounds); their logits are
    // masked to -inf in the last tile, so their values never matter.  (No
    // select on the loaded data: it would stall on the prefetch.)
    auto gload = [&](int t) {
        const int64_t key = (int64_t)t * kBK + lr;
        const bf16* kp = K + ((key < N ? key : 0) * H + h) * kD + lc;
        pk0 = load_bf16x8(kp);
        pk1 = load_bf16x8(kp + 8);
        const f16* vp = Vth + ((int64_t)t * kD + lr) * kBK + lc;
        pv0 = *reinterpret_cast<const f16x8*>(vp);
        pv1 = *reinterpret_cast<const f16x8*>(vp + 8);
    };
    auto lstore = [&](int buf) {
        bf16* kd = &sK[buf][swap23(lr) * kLdsRow + lc];
        *reinterpret_cast<bf16x8*>(kd) = pk0;
        *reinterpret_cast<bf16x8*>(kd + 8) = pk1;
        f16* vd = &sV[buf][lr * kLdsRow + lc];
        *reinterpret_cast<f16x8*>(vd) = pv0;
        *reinterpret_cast<f16x8*>(vd + 8) = pv1;
    };

    f32x16 O[2][2];
    float m[2], l[2], le[2];   // le: Kahan compensation of l (teacher instances)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        O[qb][0] = O[qb][1] = zero_f32x16();
        m[qb] = -INFINITY;
        l[qb] = le[qb] = 0.f;
    }

    gload(0);
    lstore(0);
    __syncthreads();

    for (int t = 0; t < nkt; ++t) {
        const int buf = t & 1;
        const float kbound = kmx[t];
        if (t + 1 < nkt) gload(t + 1);

        // Per 32-query block: S^T = K Q^T, then its probabilities.  Blocks are
        // done one after the other to keep one S^T live (the K operand is
        // re-read from LDS for the second block).
        const bool last = (int64_t)(t + 1) * kBK > N;
        f16x8 P[2][2][2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            f32x16 S[2];
            S[0] = S[1] = zero_f32x16();
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const bf16x8 a = *reinterpret_cast<const bf16x8*>(
                        &sK[buf][(kb * 32 + n) * kLdsRow + 16 * ks + 8 * hh]);
                    S[kb] = mfma_bf16(a, Qop[qb][ks], S[kb]);
                }
            if (last) {   // ragged last tile: mask keys >= N
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int64_t key =
                            (int64_t)t * kBK + kb * 32 + 16 * (r >> 3) + 8 * hh + (r & 7);
                        if (key >= N) S[kb][r] = -INFINITY;
                    }
            }
            // Reference point: keep m unless the bound cannot rule out a
            // logit above m + kSlack for some query of this block.
            if (__builtin_amdgcn_ballot_w64(qnc[qb] * kbound > m[qb] + kSlack) != 0) {
                float mx = -INFINITY;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[kb][r]);
                mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
                const bool move = mx > m[qb] + kSlack;
                const float mn = move ? mx : m[qb];
                const float al = move ? exp2f_fast(m[qb] - mn) : 1.f;
                m[qb] = mn;
                l[qb] *= al;
                le[qb] *= al;
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) O[qb][db][r] *= al;
            }
            // p = 2^(s c - m), packed to fp16; row sums per tile from zero, then
            // added to l: from the packed values, or in teacher instances from
            // the fp32 values with a compensated add.
            const float nm = -m[qb];
            float ls = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    u32x4 pk;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        f32x2 e;
                        e[0] = exp2f_fast(fmaf(S[kb][8 * b + 2 * j], c, nm));
                        e[1] = exp2f_fast(fmaf(S[kb][8 * b + 2 * j + 1], c, nm));
                        pk[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(e, f16x2));
                        if (kTeach)
                            ls += e[0] + e[1];
                        else
                            ls = dot2_ones(pk[j], ls);
                    }
                    P[qb][kb][b] = __builtin_bit_cast(f16x8, pk);
                }
            if (kTeach)
                kahan_add(l[qb], le[qb], ls);
            else
                l[qb] += ls;
        }

        // O^T += V^T P^T
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const f16x8 a = *reinterpret_cast<const f16x8*>(
                        &sV[buf][(db * 32 + n) * kLdsRow + kb * 32 + 16 * b + 8 * hh]);
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) O[qb][db] = mfma_f16(a, P[qb][kb][b], O[qb][db]);
                }

        if (t + 1 < nkt) lstore(buf ^ 1);
        __syncthreads();
    }

    if (kTeach) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) l[qb] -= le[qb];
    }
    store_rows(O, l, qidx, N, H, h, hh, vsc[2 * slot + 1], Y, ydt);
    if (kTeach) store_offsets(l, m, qidx, N, h, hh, off);
}

// ------------------------------------------------------------------------
// K6 (fp32): one workgroup = 4 waves x 32 queries; 32x32x2 fp32 MFMA.  S^T
// output register r of lane-half hh holds key 8 (r / 4) + 4 hh + (r % 4) of
// its 32-key block; the PV MFMA consumes one register per step, reading the
// matching V row from LDS.  Small layers (few work items for the chip) split
// each item's key tiles into two halves run by separate workgroups; each
// half writes O (unnormalized, relative to its reference point m), l and m
// per query, and K6d combines the two halves in order.  Longer layers run K6e,
// and K6's loop there for the segments that K6e does not split.
// ------------------------------------------------------------------------
constexpr int kBQ32 = 128;
constexpr int kKRow32 = 65;   // odd stride: column reads are bank-conflict free
constexpr int kRec32 = kD + 4;   // part record: O[64], l, m, 2 pad (16-byte aligned)

// Key tiles t0 .. t1 - 1 for the lane's query (row qp of Q; zeros unless qok): O and l
// relative to m, l this lane half's share.  kLean: fewer LDS reads in flight, for K6e,
// whose registers would spill otherwise.
constexpr int kLds32 = 2 * kBK * (kKRow32 + kD);   // floats: two buffers of K and V rows
template <bool kLean>
__device__ __forceinline__ void f32_tiles(const float* __restrict__ qp, bool qok,
                                          const float* __restrict__ K,
                                          const float* __restrict__ V, int64_t N, int H, int h,
                                          int t0, int t1, float c, float* __restrict__ sK,
                                          float* __restrict__ sV, f32x16 (&O)[2], float& m,
                                          float& l) {
    const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
    float Qf[32];
#pragma unroll
    for (int ks = 0; ks < 32; ++ks) Qf[ks] = qok ? qp[2 * ks + hh] : 0.f;

    const int lr = threadIdx.x >> 2, lc = (threadIdx.x & 3) * 16;
    // Keys past N read row 0 (in bounds); their logits are masked to -inf,
    // so they get weight exactly 0 (inputs are finite).
    float4 pk0, pk1, pk2, pk3, pv0, pv1, pv2, pv3;
    auto gload = [&](int t) {
        const int64_t key = (int64_t)t * kBK + lr;
        const int64_t row = key < N ? key : 0;
        const float4* kp = reinterpret_cast<const float4*>(K + (row * H + h) * kD + lc);
        const float4* vp = reinterpret_cast<const float4*>(V + (row * H + h) * kD + lc);
        pk0 = kp[0]; pk1 = kp[1]; pk2 = kp[2]; pk3 = kp[3];
        pv0 = vp[0]; pv1 = vp[1]; pv2 = vp[2]; pv3 = vp[3];
    };
    auto put4 = [](float* d, float4 v) {
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    };
    auto lstore = [&](int buf) {
        float* kd = sK + buf * kBK * kKRow32 + lr * kKRow32 + lc;
        put4(kd, pk0); put4(kd + 4, pk1); put4(kd + 8, pk2); put4(kd + 12, pk3);
        float4* vd = reinterpret_cast<float4*>(sV + buf * kBK * kD + lr * kD + lc);
        vd[0] = pv0; vd[1] = pv1; vd[2] = pv2; vd[3] = pv3;
    };

    O[0] = O[1] = zero_f32x16();
    m = -INFINITY;
    l = 0.f;
    gload(t0);
    lstore(0);
    __syncthreads();

    for (int t = t0; t < t1; ++t) {
        const int buf = (t - t0) & 1;
        if (t + 1 < t1) gload(t + 1);
        f32x16 S[2] = {zero_f32x16(), zero_f32x16()};
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int ks = 0; ks < 32; ++ks)
            {
                S[kb] = mfma_f32(sK[buf * kBK * kKRow32 + (kb * 32 + n) * kKRow32 + 2 * ks + hh],
                                 Qf[ks], S[kb]);
                if (kLean && ks % 8 == 7) __builtin_amdgcn_sched_barrier(0);
            }
        if ((int64_t)(t + 1) * kBK > N) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t key = (int64_t)t * kBK + kb * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                    if (key >= N) S[kb][r] = -INFINITY;
                }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[kb][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mn = fmaxf(m, mx * c);
        const float al = exp2f_fast(m - mn);
        m = mn;
        // Two-level sums: the tile's weights and its PV product are summed
        // from zero, then added to the running l and O, so that rounding
        // grows with the tile count rather than the key count.
        float ls = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = exp2f_fast(fmaf(S[kb][r], c, -mn));
                S[kb][r] = p;
                ls += p;
            }
        l = fmaf(l, al, ls);
        f32x16 Ot[2] = {zero_f32x16(), zero_f32x16()};
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kb * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                    Ot[db] = mfma_f32(sV[buf * kBK * kD + key * kD + db * 32 + n], S[kb][r], Ot[db]);
                    if (kLean && r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[db][r] = fmaf(O[db][r], al, Ot[db][r]);
        if (t + 1 < t1) lstore(buf ^ 1);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256, 2) void k_flash_f32(const float* __restrict__ Q,
                                                      const float* __restrict__ K,
                                                      const float* __restrict__ V,
                                                      const int32_t* __restrict__ buckets,
                                                      int64_t N, int H, int nqt, int nkt, float c,
                                                      int splits, float* __restrict__ part,
                                                      void* __restrict__ Y, int ydt) {
    const int nfull = full_count(buckets, H);
    const int active = nfull * nqt;
    if ((int)blockIdx.x >= active * splits) return;
    const int Lx = xcd_remap(blockIdx.x, active * splits);
    const int L = Lx / splits, half = Lx - L * splits;
    const int slot = L / nqt, qt = L - slot * nqt;
    // key tiles [t0, t1) of the item (all of them unless split)
    const int t0 = (int)((int64_t)half * nkt / splits);
    const int t1 = (int)((int64_t)(half + 1) * nkt / splits);
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = lane & 31, hh = lane >> 5;

    __shared__ __attribute__((aligned(16))) float smem[kLds32];

    const int64_t qi = (int64_t)qt * kBQ32 + wave * 32 + n;
    const bool qok = qi < N;
    f32x16 O[2];
    float m, l;
    f32_tiles<false>(Q + ((qok ? qi : 0) * H + h) * kD, qok, K, V, N, H, h, t0, t1, c,
              smem + 2 * kBK * kD, smem, O, m, l);

    const float lt = l + __shfl_xor(l, 32);
    if (splits > 1) {
        float* pr = part + ((int64_t)(L * 2 + half) * kBQ32 + wave * 32 + n) * kRec32;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(pr + db * 32 + 8 * g + 4 * hh) =
                    make_float4(O[db][4 * g], O[db][4 * g + 1], O[db][4 * g + 2],
                                O[db][4 * g + 3]);
        if (hh == 0) {
            pr[kD] = lt;
            pr[kD + 1] = m;
        }
        return;
    }
    const float inv = 1.f / lt;
    if (qok) {
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int64_t off = (qi * H + h) * kD + db * 32 + 8 * g + 4 * hh;
                const float y0 = O[db][4 * g] * inv, y1 = O[db][4 * g + 1] * inv;
                const float y2 = O[db][4 * g + 2] * inv, y3 = O[db][4 * g + 3] * inv;
                if (ydt == DT_BF16) {
                    bf16x4 v;
                    v[0] = (bf16)y0; v[1] = (bf16)y1; v[2] = (bf16)y2; v[3] = (bf16)y3;
                    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Y) + off) = v;
                } else {
                    *reinterpret_cast<float4*>(reinterpret_cast<float*>(Y) + off) =
                        make_float4(y0, y1, y2, y3);
                }
            }
    }
}

// K6d: Y of the fp32 items that K6 split into two key halves: the halves' O
// and l scaled to the larger reference point and added (half 0, then half
// 1), then O / l.  Two workgroups of 256 threads per item, 4 threads per
// query and 16 of its values each.
__global__ __launch_bounds__(256) void k_flash_f32_combine(const int32_t* __restrict__ buckets,
                                                           int64_t N, int H, int nqt,
                                                           const float* __restrict__ part,
                                                           void* __restrict__ Y, int ydt) {
    const int nfull = full_count(buckets, H);
    const int L = blockIdx.x >> 1;
    if (L >= nfull * nqt) return;
    const int slot = L / nqt, qt = L - slot * nqt;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    const int qr = (blockIdx.x & 1) * 64 + (threadIdx.x >> 2), d0 = (threadIdx.x & 3) * 16;
    const int64_t qi = (int64_t)qt * kBQ32 + qr;
    if (qi >= N) return;
    const float* r0 = part + ((int64_t)(L * 2) * kBQ32 + qr) * kRec32;
    const float* r1 = r0 + (int64_t)kBQ32 * kRec32;
    const float m0 = r0[kD + 1], m1 = r1[kD + 1];
    const float mt = fmaxf(m0, m1);
    const float w0 = exp2f_fast(m0 - mt), w1 = exp2f_fast(m1 - mt);
    const float inv = 1.f / fmaf(r1[kD], w1, r0[kD] * w0);
    float y[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 a = *reinterpret_cast<const float4*>(r0 + d0 + 4 * k);
        const float4 b = *reinterpret_cast<const float4*>(r1 + d0 + 4 * k);
        y[4 * k] = fmaf(b.x, w1, a.x * w0) * inv;
        y[4 * k + 1] = fmaf(b.y, w1, a.y * w0) * inv;
        y[4 * k + 2] = fmaf(b.z, w1, a.z * w0) * inv;
        y[4 * k + 3] = fmaf(b.w, w1, a.w * w0) * inv;
    }
    const int64_t yo = (qi * H + h) * kD + d0;
    if (ydt == DT_BF16) {
#pragma unroll
        for (int k8 = 0; k8 < 2; ++k8) {
            bf16x8 o;
#pragma unroll
            for (int k = 0; k < 8; ++k) o[k] = (bf16)y[8 * k8 + k];
            *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16*>(Y) + yo + 8 * k8) = o;
        }
    } else {
        float* yp = reinterpret_cast<float*>(Y) + yo;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<float4*>(yp + 4 * k) =
                make_float4(y[4 * k], y[4 * k + 1], y[4 * k + 2], y[4 * k + 3]);
    }
}

// ------------------------------------------------------------------------
// K6e (fp32, longer layers).  Every operand is a power of two times hi + 2^-11 lo, two
// fp16 values (both rounded to nearest: the remainder is at most 2^-23 |x|, and 2^-49 of
// the largest value of its group where lo is subnormal; lo is held times 2^11, so that
// it is as far from that as hi), and a product takes three 32x32x16 fp16 MFMAs,
// 2^-11 (lo hi + hi lo) + hi hi (2^-22 lo lo is at most 2^-22 of it), 96 cycles per 16
// values against 512 for the 32x32x2 fp32 MFMA; all sums stay fp32.  The bounds are
// wider than fp32's rounding of a value (2^-24), but on random values the error
// against float64 is smaller than with fp32 MFMAs, whose 64 products per sum are added
// one by one (of the output norm, 2,748 tokens: 1.4e-7 against 1.9e-7; sharp
// heads 2.2e-7 against 3.5e-7, Q x 3 4.3e-7 against 9.6e-7).
// K is scaled per head, V per head and feature (undone at the end, so that
// every feature keeps its own precision), Q per query.  The segments of these run K6's
// loop instead, on the same split of the work (2,748 tokens, 8 such heads: FULL stage
// 175 us; 229 us with a K6 launch of their own after this one, a workgroup per item; 201 us
// with K6 alone in two halves.  1,374 tokens 76, 128 and 63 us; 5,496 tokens 539, 761
// and 724 us):
//   - heads and items with a value that is not finite or whose largest magnitude lies
//     outside [2^-60, 2^60] (zero aside);
//   - heads with a row of V all of whose features lie below 2^-20 of their largest: small
//     weights (held to 2^-50 of the largest) on the other rows could outweigh it;
//   - items whose logits may reach 2^24 (64 |q| |k| c, the largest magnitudes of the query
//     and of the head's K): a query's reference point is a rounded logit, by up to half an
//     ulp, and its weights, then as large as 2 to the power of that, must stay in fp16's
//     range times 2^14.
//   k_absmax_f32: per group of token rows, largest |k| and per feature |v|, as
//   integer bits (a NaN is larger than any number);
//   k_pack_f32: scales, and per 64-key tile K hi, K lo (rows in swap23 order),
//   V^T hi, V^T lo: 4 x 8 KB, 128-byte rows with 16-byte chunks at position
//   chunk ^ (row / 2 % 8), copied to LDS as they are.
// ------------------------------------------------------------------------
constexpr int kWG32 = 512;       // workgroups: two per CU
constexpr int kMinTiles32 = 4;   // fewest key tiles per workgroup in the tail
constexpr uint32_t kTile32 = 32768;    // bytes of a packed key tile
constexpr int kMax32 = kD + 1;         // |v| per feature, |k|
constexpr int kScale32 = kD + 4;       // per slot: 2^e_d of V, 2^e of K, exact flag, |k|, 1 pad
constexpr float kMaxProduct32 = 0x1p18f;   // |q| |k| c of the items that K6e computes
constexpr int kMaxGroups32 = 64;

__host__ __device__ inline int64_t f32_group_rows(int64_t N) {   // rows per maximum group
    const int64_t r = (N + kMaxGroups32 - 1) / kMaxGroups32;
    return r < 128 ? 128 : (r + 31) / 32 * 32;
}

__global__ __launch_bounds__(256) void k_absmax_f32(const float* __restrict__ K,
                                                    const float* __restrict__ V,
                                                    const int32_t* __restrict__ buckets, int64_t N,
                                                    int H, uint32_t* __restrict__ part,
                                                    float* __restrict__ scales) {
    const int slot = blockIdx.y;
    if (slot >= full_count(buckets, H)) return;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    __shared__ uint32_t s[kMax32];
    if (threadIdx.x < kMax32) s[threadIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) scales[slot * kScale32 + kD + 1] = 0.f;
    __syncthreads();
    const int64_t rows = f32_group_rows(N), r0 = (int64_t)blockIdx.x * rows;
    const int64_t r1 = r0 + rows < N ? r0 + rows : N;
    const int seg = (threadIdx.x & 15) * 4;
    uint32_t mk = 0, mv[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int64_t row = r0 + (threadIdx.x >> 4); row < r1; row += 16) {
        const int64_t o = (row * H + h) * kD + seg;
        const u32x4 k = *reinterpret_cast<const u32x4*>(K + o);
        const u32x4 v = *reinterpret_cast<const u32x4*>(V + o);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            mk = max(mk, k[j] & 0x7fffffffu);
            mv[j] = max(mv[j], v[j] & 0x7fffffffu);
        }
    }
    atomicMax(&s[kD], mk);
#pragma unroll
    for (int j = 0; j < 4; ++j) atomicMax(&s[seg + j], mv[j]);
    __syncthreads();
    if (threadIdx.x < kMax32)
        part[((int64_t)slot * gridDim.x + blockIdx.x) * kMax32 + threadIdx.x] = s[threadIdx.x];
}

// Exponent e with |x| 2^-e < 2^14 for all |x| up to the one with bits m, and
// whether it is in the split's range.
__device__ __forceinline__ int f32_exponent(uint32_t m) {
    return m == 0 ? 0 : (int)(m >> 23) - 127 - 13;
}
__device__ __forceinline__ bool f32_in_range(uint32_t m) {
    return m == 0 || (m >= (uint32_t)(127 - 60) << 23 && m < (uint32_t)(127 + 60) << 23);
}
__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }

// x = hi + 2^-11 lo (x already scaled, at most 2^15: |lo| is at most 2^14).
constexpr float kLow32 = 0x1p-11f;
__device__ __forceinline__ void split16(float x, f16& hi, f16& lo) {
    hi = (f16)x;
    lo = (f16)((x - (float)hi) * (1.f / kLow32));
}

__global__ __launch_bounds__(256) void k_pack_f32(const float* __restrict__ K,
                                                  const float* __restrict__ V,
                                                  const int32_t* __restrict__ buckets, int64_t N,
                                                  int H, int nkt, const uint32_t* __restrict__ part,
                                                  int ng, float* __restrict__ scales,
                                                  char* __restrict__ tiles) {
    const int slot = blockIdx.y, tile = blockIdx.x;
    if (slot >= full_count(buckets, H)) return;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    __shared__ uint32_t smax[kMax32];
    __shared__ __attribute__((aligned(16))) f16 sT[2][kD * kLdsRow];
    const int t = threadIdx.x;
    const int key = t >> 2, dseg = (t & 3) * 16;
    const int64_t row = (int64_t)tile * kBK + key;
    const bool ok = row < N;
    const int64_t o = ((ok ? row : 0) * H + h) * kD + dseg;
    f32x4 kv[4], vv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        kv[i] = *reinterpret_cast<const f32x4*>(K + o + 4 * i);
        vv[i] = *reinterpret_cast<const f32x4*>(V + o + 4 * i);
    }
    if (t < kMax32) {
        uint32_t m = 0;
        for (int g = 0; g < ng; ++g) m = max(m, part[((int64_t)slot * ng + g) * kMax32 + t]);
        smax[t] = m;
    }
    __syncthreads();
    const int ek = f32_exponent(smax[kD]);
    bool bad = false;
    if (tile == 0) {
        bad = t < kMax32 && !f32_in_range(smax[t]);
        if (t < kD) scales[slot * kScale32 + t] = f32_in_range(smax[t]) ? pow2(f32_exponent(smax[t])) : 1.f;
        if (t == kD) scales[slot * kScale32 + kD] = f32_in_range(smax[kD]) ? pow2(ek) : 1.f;
        if (t == kD + 2) scales[slot * kScale32 + kD + 2] = __uint_as_float(smax[kD]);
    }
    // (out of range: any scale, the tiles are not used)
    const float dk = f32_in_range(smax[kD]) ? pow2(-ek) : 1.f;
    char* out = tiles + ((int64_t)slot * nkt + tile) * kTile32;
    const int kr = swap23(key);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        f16x8 hi, lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            f16 a, b;
            split16(ok ? kv[2 * c + (j >> 2)][j & 3] * dk : 0.f, a, b);
            hi[j] = a;
            lo[j] = b;
        }
        char* p = out + kr * 128 + ((((t & 3) * 2 + c) ^ ((kr >> 1) & 7)) << 4);
        *reinterpret_cast<f16x8*>(p) = hi;
        *reinterpret_cast<f16x8*>(p + 8192) = lo;
    }
    float vmax = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t m = smax[dseg + j];
        const float dv = f32_in_range(m) ? pow2(-f32_exponent(m)) : 1.f;
        const float x = ok ? vv[j >> 2][j & 3] * dv : 0.f;
        f16 a, b;
        split16(x, a, b);
        vmax = fmaxf(vmax, fabsf(x));
        sT[0][(dseg + j) * kLdsRow + key] = a;
        sT[1][(dseg + j) * kLdsRow + key] = b;
    }
    // (a feature's largest value is scaled to 2^13 .. 2^14; four lanes hold a row)
    vmax = fmaxf(vmax, __shfl_xor(vmax, 1));
    vmax = fmaxf(vmax, __shfl_xor(vmax, 2));
    bad |= vmax > 0.f && vmax < 0x1p-6f;
    if (__syncthreads_or(bad) && t == 0)
        atomicOr((uint32_t*)&scales[slot * kScale32 + kD + 1], 1u);
    const int d = t >> 2;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int ch = (t & 3) * 2 + c;
            *reinterpret_cast<f16x8*>(out + (2 + p) * 8192 + d * 128 + ((ch ^ ((d >> 1) & 7)) << 4)) =
                *reinterpret_cast<const f16x8*>(&sT[p][d * kLdsRow + ch * 8]);
        }
}

// Work items (128 queries of a FULL head) go to the workgroups as in K6a:
// whole rounds, and the last, partial round cut into one sequence of item-tile
// steps.  One workgroup = 4 waves x 32 queries; two workgroups per CU, so that one
// wave's softmax runs beside another's MFMAs.
__global__ __launch_bounds__(256, 2) void k_flash_f32s(const float* __restrict__ Q,
                                                       const float* __restrict__ K,
                                                       const float* __restrict__ V,
                                                       const int32_t* __restrict__ buckets,
                                                       int64_t N, int H, int nqt, int nkt, float c,
                                                       const float* __restrict__ scales,
                                                       const char* __restrict__ tiles,
                                                       float* __restrict__ part, int G,
                                                       void* __restrict__ Y, int ydt) {
    const int nfull = full_count(buckets, H);
    const int active = nfull * nqt;
    if (active == 0) return;
    const int w = xcd_remap(blockIdx.x, G);
    const int full = active / G * G, R = active - full;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 31, hh = lane >> 5;
    __shared__ __attribute__((aligned(1024))) char smem[kLds32 * 4];
    static_assert(kLds32 * 4 >= 2 * kTile32, "both loops' buffers");
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(3))) const f16x8 lds_frag;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

    auto segment = [&](int L, int t0, int t1, int pslot) __attribute__((always_inline)) {
        const int slot = L / nqt, qt = L - slot * nqt;
        const int h = full_head(buckets, H, slot);
        if (h < 0) return;
        const int64_t qi = (int64_t)qt * kBQ32 + wave * 32 + n;
        const bool qok = qi < N;
        const float* sc = scales + slot * kScale32;
        const float* qrow = Q + ((qok ? qi : 0) * H + h) * kD;
        f32x16 O[2] = {zero_f32x16(), zero_f32x16()};
        float m = -INFINITY, l = 0.f;

        // Q: features 16 ks + 8 hh .. + 7 of the lane's query, and its scale.
        f32x4 q[8];
        {
            const float* qp = qrow + 8 * hh;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                q[i] = *reinterpret_cast<const f32x4*>(qp + 16 * (i >> 1) + 4 * (i & 1));
                if (!qok) q[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        uint32_t mq = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) mq = max(mq, __float_as_uint(q[i][j]) & 0x7fffffffu);
        mq = max(mq, (uint32_t)__shfl_xor(mq, 32));
        // (also the barrier between one segment's LDS reads and the next's writes)
        const bool exact = __syncthreads_or(!f32_in_range(mq) || __float_as_uint(sc[kD + 1]) ||
                                            !(__uint_as_float(mq) * sc[kD + 2] * c <
                                              kMaxProduct32)) != 0;
        if (exact) {   // uniform over the workgroup, and the same for every part of an item
            float* sf = reinterpret_cast<float*>(smem);
            f32_tiles<true>(qrow, qok, K, V, N, H, h, t0, t1, c, sf + 2 * kBK * kD, sf, O, m, l);
        } else {
            const int eq = f32_exponent(mq);
            const float dq = pow2(-eq), cs = c * sc[kD] * pow2(eq);
            f16x8 qh[4], ql[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    f16 a, b;
                    split16(q[2 * ks + (j >> 2)][j & 3] * dq, a, b);
                    qh[ks][j] = a;
                    ql[ks][j] = b;
                }
            const char* tb = tiles + (int64_t)slot * nkt * kTile32;
            auto copy = [&](int t, int buf) {   // 8 KB per wave, as it lies
                const char* src = tb + (int64_t)t * kTile32 + wave * 8192;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    copy_to_lds(lds0 + buf * kTile32 + wave * 8192 + i * 1024, src + i * 1024,
                                (uint32_t)lane * 16u);
            };
            const uint32_t f0 = lds0 + (uint32_t)n * 128u + (uint32_t)((hh ^ ((n >> 1) & 7)) << 4);
            // chunk 2 k + hh of row 32 blk + n of matrix `mat` (K hi, K lo, V hi, V lo)
            auto frag = [&](int buf, int mat, int blk, int k) {
                return *(lds_frag*)(uintptr_t)((f0 ^ (uint32_t)(k << 5)) + buf * kTile32 +
                                               8192u * mat + 4096u * blk);
            };
            copy(t0, 0);
            for (int t = t0; t < t1; ++t) {
                const int buf = (t - t0) & 1;
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();   // tile t is there; the other buffer's reads are done
                if (t + 1 < t1) copy(t + 1, buf ^ 1);
                f32x16 S[2] = {zero_f32x16(), zero_f32x16()};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
                        S[kb] = mfma_f16(frag(buf, 1, kb, ks), qh[ks], S[kb]);
                f16x8 kh[4][2];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) {
                        kh[ks][kb] = frag(buf, 0, kb, ks);
                        S[kb] = mfma_f16(kh[ks][kb], ql[ks], S[kb]);
                    }
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) S[kb][i] *= kLow32;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) S[kb] = mfma_f16(kh[ks][kb], qh[ks], S[kb]);
                if ((int64_t)(t + 1) * kBK > N) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int64_t key =
                                (int64_t)t * kBK + kb * 32 + 16 * (i >> 3) + 8 * hh + (i & 7);
                            if (key >= N) S[kb][i] = -INFINITY;
                        }
                }
                float mx = -INFINITY;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[kb][i]);
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float mn = fmaxf(m, mx * cs);
                const float al = exp2f_fast(m - mn);
                m = mn;
                // The weights are split times 2^14, a factor that O keeps until the end.
                // (Added to the exponent it would cost the precision of an argument
                // near 14.)
                float ls = 0.f;
                f16x8 ph[2][2], pl[2][2];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        u32x4 h4, l4;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const f32x2 e = {exp2f_fast(fmaf(S[kb][8 * b + 2 * j], cs, -mn)),
                                             exp2f_fast(fmaf(S[kb][8 * b + 2 * j + 1], cs, -mn))};
                            ls += e[0];
                            ls += e[1];
                            const f32x2 es = {e[0] * 16384.f, e[1] * 16384.f};
                            const f16x2 eh = __builtin_convertvector(es, f16x2);
                            const f32x2 er = {(es[0] - (float)eh[0]) * (1.f / kLow32),
                                              (es[1] - (float)eh[1]) * (1.f / kLow32)};
                            h4[j] = __builtin_bit_cast(uint32_t, eh);
                            l4[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(er, f16x2));
                        }
                        ph[kb][b] = __builtin_bit_cast(f16x8, h4);
                        pl[kb][b] = __builtin_bit_cast(f16x8, l4);
                    }
                l = fmaf(l, al, ls);
                // Two-level sums: the tile's product is summed from zero,
                // then added to the running O, so that rounding grows with the
                // tile count rather than the key count.
                f32x16 Ot[2] = {zero_f32x16(), zero_f32x16()};
#pragma unroll
                for (int kc = 0; kc < 4; ++kc)
#pragma unroll
                    for (int db = 0; db < 2; ++db)
                        Ot[db] = mfma_f16(frag(buf, 3, db, kc), ph[kc >> 1][kc & 1], Ot[db]);
                f16x8 vh[4][2];
#pragma unroll
                for (int kc = 0; kc < 4; ++kc)
#pragma unroll
                    for (int db = 0; db < 2; ++db) {
                        vh[kc][db] = frag(buf, 2, db, kc);
                        Ot[db] = mfma_f16(vh[kc][db], pl[kc >> 1][kc & 1], Ot[db]);
                    }
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) Ot[db][r] *= kLow32;
#pragma unroll
                for (int kc = 0; kc < 4; ++kc)
#pragma unroll
                    for (int db = 0; db < 2; ++db)
                        Ot[db] = mfma_f16(vh[kc][db], ph[kc >> 1][kc & 1], Ot[db]);
#pragma unroll
                for (int db = 0; db < 2; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) O[db][r] = fmaf(O[db][r], al, Ot[db][r]);
            }
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 up = *reinterpret_cast<const f32x4*>(sc + db * 32 + 8 * g + 4 * hh);
#pragma unroll
                    for (int i = 0; i < 4; ++i) O[db][4 * g + i] *= up[i] * 0x1p-14f;
                }
        }

        const float lt = l + __shfl_xor(l, 32);
        if (t0 != 0 || t1 != nkt) {
            float* pr = part + ((int64_t)(w * 2 + pslot) * kBQ32 + wave * 32 + n) * kRec32;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<float4*>(pr + db * 32 + 8 * g + 4 * hh) =
                        make_float4(O[db][4 * g], O[db][4 * g + 1], O[db][4 * g + 2],
                                    O[db][4 * g + 3]);
            if (hh == 0) {
                pr[kD] = lt;
                pr[kD + 1] = m;
            }
            return;
        }
        const float inv = 1.f / lt;
        if (qok) {
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int64_t off = (qi * H + h) * kD + db * 32 + 8 * g + 4 * hh;
                    const float y0 = O[db][4 * g] * inv, y1 = O[db][4 * g + 1] * inv;
                    const float y2 = O[db][4 * g + 2] * inv, y3 = O[db][4 * g + 3] * inv;
                    if (ydt == DT_BF16) {
                        bf16x4 v;
                        v[0] = (bf16)y0; v[1] = (bf16)y1; v[2] = (bf16)y2; v[3] = (bf16)y3;
                        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Y) + off) = v;
                    } else {
                        *reinterpret_cast<float4*>(reinterpret_cast<float*>(Y) + off) =
                            make_float4(y0, y1, y2, y3);
                    }
                }
        }
    };

    for (int L = w; L < full; L += G) segment(L, 0, nkt, 0);
    if (R > 0) {
        const int64_t T = (int64_t)R * nkt;
        const int Gt = tail_groups(T, G, kMinTiles32);
        if (w < Gt) {
            const int64_t start = tail_start(w, T, Gt), end = tail_start(w + 1, T, Gt);
            for (int64_t x = start; x < end;) {
                const int i = (int)(x / nkt);
                const int t0 = (int)(x - (int64_t)i * nkt);
                const int64_t left = end - x;
                const int t1 = (int64_t)(nkt - t0) < left ? nkt : (int)(t0 + left);
                segment(full + i, t0, t1, x == start ? 0 : 1);
                x += t1 - t0;
            }
        }
    }
}

// K6f: Y of the items that K6e split over workgroups: the parts' O and l scaled to the
// largest reference point and added in workgroup order (deterministic), then O
// / l.  Two workgroups of 256 threads per tail item, 4 threads per query and 16 of
// its values each.
__global__ __launch_bounds__(256) void k_flash_f32s_combine(const int32_t* __restrict__ buckets,
                                                            int64_t N, int H, int nqt, int nkt,
                                                            const float* __restrict__ part, int G,
                                                            void* __restrict__ Y, int ydt) {
    const int nfull = full_count(buckets, H);
    const int active = nfull * nqt, full = active / G * G, R = active - full;
    const int i = blockIdx.x >> 1;
    if (i >= R) return;
    const int64_t T = (int64_t)R * nkt;
    const int Gt = tail_groups(T, G, kMinTiles32);
    const int wf = tail_owner((int64_t)i * nkt, T, Gt);
    const int wl = tail_owner((int64_t)(i + 1) * nkt - 1, T, Gt);
    if (wf == wl) return;
    const int L = full + i, slot = L / nqt, qt = L - slot * nqt;
    const int h = full_head(buckets, H, slot);
    if (h < 0) return;
    const int qr = (blockIdx.x & 1) * 64 + (threadIdx.x >> 2), d0 = (threadIdx.x & 3) * 16;
    const int64_t qi = (int64_t)qt * kBQ32 + qr;
    if (qi >= N) return;
    auto rec = [&](int v) {
        const int k = i == (int)(tail_start(v, T, Gt) / nkt) ? 0 : 1;
        return part + ((int64_t)(v * 2 + k) * kBQ32 + qr) * kRec32;
    };
    float mt = -INFINITY;
    for (int v = wf; v <= wl; ++v) mt = fmaxf(mt, rec(v)[kD + 1]);
    float y[16], lt = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) y[k] = 0.f;
    for (int v = wf; v <= wl; ++v) {
        const float* r = rec(v);
        const float wt = exp2f_fast(r[kD + 1] - mt);
        lt = fmaf(r[kD], wt, lt);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const f32x4 a = *reinterpret_cast<const f32x4*>(r + d0 + 4 * k);
#pragma unroll
            for (int j = 0; j < 4; ++j) y[4 * k + j] = fmaf(a[j], wt, y[4 * k + j]);
        }
    }
    const float inv = 1.f / lt;
#pragma unroll
    for (int k = 0; k < 16; ++k) y[k] *= inv;
    const int64_t yo = (qi * H + h) * kD + d0;
    if (ydt == DT_BF16) {
#pragma unroll
        for (int k8 = 0; k8 < 2; ++k8) {
            bf16x8 o;
#pragma unroll
            for (int k = 0; k < 8; ++k) o[k] = (bf16)y[8 * k8 + k];
            *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16*>(Y) + yo + 8 * k8) = o;
        }
    } else {
        float* yp = reinterpret_cast<float*>(Y) + yo;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<float4*>(yp + 4 * k) =
                make_float4(y[4 * k], y[4 * k + 1], y[4 * k + 2], y[4 * k + 3]);
    }
}

// ------------------------------------------------------------------ launchers

int flash_q_tile(int dtype) { return dtype == DT_BF16 ? kBQ16 : kBQ32; }

int flash_stream_groups(int64_t N, int H) {
    (void)N;
    (void)H;
    return kStreamWG;
}

size_t flash_part_bytes(int64_t N, int H) {
    return (size_t)2 * flash_stream_groups(N, H) * kPartFloats * sizeof(float);
}

// fp32 layers.  Up to kSplit32 tokens: K6, with two key halves per work item while
// the items alone would leave the chip short of waves (at most 2 workgroups
// per CU of them).  Longer ones: K6e, whose packing and combine launches cost more than
// it gains on short ones.  FULL stage, us, K6 and K6e with 1, 2, 4, 8 and 16 of 16 heads:
//   640 tokens   32.3 32.0   32.4 32.9   32.8 39.9   33.7 42.3   35.7 44.4
//   896          41.1 33.8   41.4 40.6   41.9 42.5   43.4 45.3   46.1 46.4
//   1,024        45.7 32.0   46.0 39.8   46.5 41.7   48.3 45.1   51.9 45.0
// 1,374 tokens, 8 heads 63 and 50; 2,748 201 and 90; 5,496 724 and 242.  With no FULL head
// the launches alone are 11 us (K6, two) and 19 us (K6e, four).
constexpr int64_t kSplit32 = 1024;
static bool f32_split(int64_t N) { return N > kSplit32; }
static int flash_f32_halves(int64_t N, int H) {
    const int64_t nqt = (N + kBQ32 - 1) / kBQ32, nkt = (N + kBK - 1) / kBK;
    return nqt * H <= 2 * kStreamWG && nkt >= 2 ? 2 : 1;
}
// Bytes of the partial results (K6's halves, or two part slots per workgroup
// that K6e's tail can use), of K6e's maxima and scales, and of its tiles.
size_t flash_f32_part_bytes(int64_t N, int H) {
    const int64_t nqt = (N + kBQ32 - 1) / kBQ32, nkt = (N + kBK - 1) / kBK;
    if (!f32_split(N))
        return flash_f32_halves(N, H) == 1
                   ? 0 : (size_t)H * nqt * 2 * kBQ32 * kRec32 * sizeof(float);
    const int64_t most = nqt * H < kWG32 ? nqt * H : kWG32 - 1;   // tail items
    return (size_t)2 * tail_groups(most * nkt, kWG32, kMinTiles32) * kBQ32 * kRec32 * sizeof(float);
}
static int flash_f32_groups(int64_t N) { return (int)((N + f32_group_rows(N) - 1) / f32_group_rows(N)); }
size_t flash_f32_max_bytes(int64_t N, int H) {
    if (!f32_split(N)) return 0;
    return (size_t)H * (flash_f32_groups(N) * kMax32 + kScale32) * 4;
}
size_t flash_f32_tile_bytes(int64_t N, int H) {
    if (!f32_split(N)) return 0;
    return (size_t)H * ((N + kBK - 1) / kBK) * kTile32;
}

int64_t flash_vmax_parts(int64_t N) {
    const int64_t nkt = (N + kBK - 1) / kBK;
    return (nkt + kVmaxTiles - 1) / kVmaxTiles;
}

void launch_gather(const AttnArgs& a, hipStream_t st) {
    const int nkt = (int)((a.N + kBK - 1) / kBK);
    const int nvp = (int)flash_vmax_parts(a.N);
    hipLaunchKernelGGL(k_vmax_partial, dim3(nvp, a.H), dim3(256), 0, st, (const bf16*)a.V,
                       a.buckets, a.N, a.H, a.vpart);
    hipLaunchKernelGGL(k_gather_vt, dim3(nkt, a.H), dim3(256), 0, st, (const bf16*)a.K,
                       (const bf16*)a.V, a.buckets, a.N, a.H, nkt, (const float*)a.vpart, nvp,
                       a.vsc, (f16*)a.vt, (f16*)a.kh, a.kmax);
}

void launch_flash(const AttnArgs& a, hipStream_t st) {
    const int nkt = (int)((a.N + kBK - 1) / kBK);
    const float c = kLog2e / sqrtf((float)kD);
    const int bq = flash_q_tile(a.dtype);
    const int nqt = (int)((a.N + bq - 1) / bq);
    if (a.dtype == DT_BF16) {
        const int nqf = (int)((a.N + kBQf - 1) / kBQf);
        const int G = flash_stream_groups(a.N, a.H);
        hipLaunchKernelGGL(a.off ? k_flash_bf16<true> : k_flash_bf16<false>, dim3(G), dim3(512),
                           0, st, (const bf16*)a.Q, (const f16*)a.kh, (const f16*)a.vt,
                           (const float*)a.kmax, (const float*)a.vsc, a.buckets, a.N, a.H, nqf,
                           nkt, c, a.qflag, a.part, G, a.Y, a.ydt, a.off);
        hipLaunchKernelGGL(k_flash_combine, dim3(G * kCombUnits), dim3(256), 0, st,
                           a.buckets, a.N, a.H, nqf,
                           nkt, (const int32_t*)a.qflag, (const float*)a.part,
                           (const float*)a.vsc, G, a.Y, a.ydt, a.off);
        hipLaunchKernelGGL(a.off ? k_flash_bf16_wide<true> : k_flash_bf16_wide<false>,
                           dim3(nqt * a.H), dim3(256), 0, st, (const bf16*)a.Q, (const bf16*)a.K,
                           (const f16*)a.vt, (const float*)a.kmax, (const float*)a.vsc, a.buckets,
                           a.N, a.H, nqt, nkt, c, a.qflag, nqf, a.Y, a.ydt, a.off);
    } else if (!f32_split(a.N)) {
        const int splits = flash_f32_halves(a.N, a.H);
        hipLaunchKernelGGL(k_flash_f32, dim3(nqt * a.H * splits), dim3(256), 0, st,
                           (const float*)a.Q, (const float*)a.K, (const float*)a.V, a.buckets,
                           a.N, a.H, nqt, nkt, c, splits, a.part, a.Y, a.ydt);
        if (splits > 1)
            hipLaunchKernelGGL(k_flash_f32_combine, dim3(nqt * a.H * 2), dim3(256), 0, st,
                               a.buckets, a.N, a.H, nqt, (const float*)a.part, a.Y, a.ydt);
    } else {
        const int ng = flash_f32_groups(a.N);
        float* scales = a.fmax;   // (first: read 16 bytes at a time)
        uint32_t* mx = (uint32_t*)(scales + (size_t)a.H * kScale32);
        static_assert(kScale32 % 4 == 0, "16-byte alignment of every slot's scales");
        hipLaunchKernelGGL(k_absmax_f32, dim3(ng, a.H), dim3(256), 0, st, (const float*)a.K,
                           (const float*)a.V, a.buckets, a.N, a.H, mx, scales);
        hipLaunchKernelGGL(k_pack_f32, dim3(nkt, a.H), dim3(256), 0, st, (const float*)a.K,
                           (const float*)a.V, a.buckets, a.N, a.H, nkt, (const uint32_t*)mx, ng,
                           scales, (char*)a.ftiles);
        hipLaunchKernelGGL(k_flash_f32s, dim3(kWG32), dim3(256), 0, st, (const float*)a.Q,
                           (const float*)a.K, (const float*)a.V, a.buckets, a.N, a.H, nqt, nkt, c,
                           (const float*)scales, (const char*)a.ftiles, a.part, kWG32, a.Y, a.ydt);
        hipLaunchKernelGGL(k_flash_f32s_combine, dim3(2 * (nqt * a.H < kWG32 ? nqt * a.H : kWG32)),
                           dim3(256), 0, st, a.buckets, a.N, a.H, nqt, nkt,
                           (const float*)a.part, kWG32, a.Y, a.ydt);
    }
}

}  // namespace vp
