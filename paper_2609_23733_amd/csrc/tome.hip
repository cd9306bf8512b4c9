// Token merging before the routed attention: ToMe's bipartite soft matching
// (the paper combines its layer with ToMe and gives no steps of its own):
//   T1  metric m_i = bf16(sum over heads of K_{i,h}) (fp32, head order) and
//       1 / |m_i|;
//   T2  for every source, the most similar destination by cosine similarity
//       (MFMA over source x destination tiles, running argmax in registers);
//   T3  the M most similar sources: radix select on unique 64-bit keys
//       (similarity, then the lower token index);
//   T4  rows of the merged sequence (kept tokens in token order), and for
//       each row its tokens: own token first, then its merged sources in
//       token order (stable radix sort of the merged sources by destination);
//   T5  merge = mean of a row's tokens (fp32 sums in member order, one
//       rounding), unmerge = copy of a row's output to each of its tokens.
// Every reduction has a fixed order: results are bitwise reproducible.
#include "vp_device.hpp"
#include "vp_internal.hpp"

namespace vp {

namespace {

constexpr int kRow = 72;           // bf16 LDS row stride (144 B)
constexpr int kScanBlock = 1024;   // elements per scan block (256 threads x 4)
constexpr int kSortBlock = 1024;   // items per radix-sort block (1024 threads x 1)

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Lanes of the wave holding the same digit of BITS bits (for an active lane).
template <int BITS>
__device__ __forceinline__ uint64_t wave_match(uint32_t d, bool active) {
    uint64_t m = __builtin_amdgcn_ballot_w64(active);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __builtin_amdgcn_ballot_w64(active && bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

__device__ __forceinline__ uint32_t float_order(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float float_unorder(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}
// Matching key of a source without a destination yet: (-inf, slot 0).
constexpr uint64_t kNoMatch = 0x007fffffffffffffull;

// ---------------------------------------------------------------- T1
// 8 threads per token, 8 features each.
__global__ __launch_bounds__(256) void k_tome_metric(const bf16* __restrict__ K, int64_t N, int H,
                                                     bf16* __restrict__ m,
                                                     float* __restrict__ invn) {
    const int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 3;
    const int f = (threadIdx.x & 7) * 8;
    const bool ok = t < N;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (ok)
        for (int h = 0; h < H; ++h) {
            const bf16x8 v = load_bf16x8(K + (t * H + h) * kD + f);
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += bf16_to_f32(v[j]);
        }
    bf16x8 o;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        o[j] = (bf16)s[j];
        const float x = bf16_to_f32(o[j]);
        q = fmaf(x, x, q);
    }
    q += __shfl_xor(q, 1);
    q += __shfl_xor(q, 2);
    q += __shfl_xor(q, 4);
    if (ok) {
        *reinterpret_cast<bf16x8*>(m + t * kD + f) = o;
        if (f == 0) invn[t] = q > 0.f ? 1.f / sqrtf(q) : 0.f;
    }
}

// ---------------------------------------------------------------- T2
// 8 waves x 128 sources per workgroup, the sources' metric rows in registers as
// the MFMA's B operand.  Tiles of 64 destinations stream through three LDS
// buffers; destinations are the MFMA's rows, so a lane's 16 results of a 32 x
// 32 block are 16 destinations of one source, in increasing slot order.  The
// similarity up to the source's own norm is v = fl(m_s . m_d fl(1 / |m_d|)); a
// lane keeps its source's first largest v.
// Most blocks raise no lane's maximum, so a block is first bounded: every v is
// at most max(m_s . m_d, 0) times the largest 1 / |m_d| of the lane's 16 rows
// (rounding is monotone, so the bound holds for the rounded products, too), and
// only if that passes some lane's maximum are the products formed and, if one
// is larger, its slot found: eight integer maxima (non-negative floats order like
// integers), a multiplication and a compare per 16 scores instead of 64
// instructions.  A NaN product makes the bound NaN, which takes the exact path,
// where it never wins.  Rows past the last destination repeat it.
//
// The work is one sequence of (1024 sources, destination tile) steps split evenly
// over the workgroups; the parts of a source meet in an atomic maximum of
// (ordered v, complement of the slot), so the lower slot wins on equal values
// whatever the order.  Every 16 tiles a part publishes what it has found and
// takes a value below the source's maximum so far (the next one, but past -0)
// as its own lower bound: that leaves out only destinations that are strictly
// worse than a published one, so the outcome does not depend on when it is read.
// 108,405 sources x 28,995 destinations (S = 100, 75 %): 911 -> 475 us, 325 of
// them without a block past its bound (the products alone would take 160).
// Screening on rows scaled beforehand (a tighter bound, the products taken
// again past it) was slower (549 us): the blocks that pass are mostly real
// improvements.
constexpr int kTmWaves = 8;
constexpr int kTmKB = 4;                           // 32-source blocks per wave
constexpr int kTmSrc = 32 * kTmKB * kTmWaves;      // sources per workgroup
constexpr int kTmWG = 256;                         // workgroups: one per CU

// Destination slot -> token in 32 bits (N is at most 2^28).
__device__ __forceinline__ uint32_t dst_token32(uint32_t j, uint32_t P, uint32_t per, uint32_t nsp,
                                                uint32_t g) {
    if (j < P) return j;
    const uint32_t q = (j - P) / per, w = j - P - q * per;
    return (1 + q) * P + (w < nsp ? w : nsp + (w - nsp) * g);
}

__global__ __launch_bounds__(64 * kTmWaves, 1) void k_tome_match(const bf16* __restrict__ m,
                                                                 const float* __restrict__ invn,
                                                                 TomeGeom G,
                                                                 unsigned long long* __restrict__ best) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
    __shared__ __attribute__((aligned(16))) bf16 sD[3][64 * kRow];
    __shared__ __attribute__((aligned(16))) float sInv[3][64];   // 1 / |m_d|
    __shared__ float sTop[3][4];   // the largest of the 16 rows (block, lane half)
    const int nD = (int)G.nD;
    const uint32_t P = (uint32_t)G.P, per = (uint32_t)(G.nsp + G.ndp), nsp = (uint32_t)G.nsp,
                   gs = (uint32_t)G.g;
    const int nt = (nD + 63) / 64;
    const int64_t nsb = (G.nA + kTmSrc - 1) / kTmSrc;
    const int64_t total = nsb * nt, W = gridDim.x;
    const int w = xcd_remap(blockIdx.x, (int)W);
    int64_t x = total * w / W;
    const int64_t end = total * (w + 1) / W;
    while (x < end) {
        const int64_t item = x / nt;
        const int t0 = (int)(x - item * nt);
        const int t1 = (int)(end - x < nt - t0 ? t0 + (end - x) : nt);
        x += t1 - t0;
        const int64_t i0 = item * kTmSrc + wave * 32 * kTmKB;
        bf16x8 B[kTmKB][4];
#pragma unroll
        for (int kb = 0; kb < kTmKB; ++kb) {
            const int64_t i = i0 + 32 * kb + n;
            const int64_t tok = i < G.nA ? tome_src_token(G, i) : 0;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) B[kb][ks] = load_bf16x8(m + tok * kD + 16 * ks + 8 * hh);
        }
        bf16x8 gq;
        float gi = 0.f;
        const int lr = threadIdx.x >> 3, lc = (threadIdx.x & 7) * 8;
        auto gload = [&](int t) {   // (clamped to the last tile and destination)
            t = t < t1 ? t : t1 - 1;
            gq = load_bf16x8(m + (int64_t)dst_token32(min(t * 64 + lr, nD - 1), P, per, nsp, gs) * kD +
                             lc);
            if (wave == 0)
                gi = invn[dst_token32(min(t * 64 + lane, nD - 1), P, per, nsp, gs)];
        };
        auto lstore = [&](int b) {
            *reinterpret_cast<bf16x8*>(&sD[b][lr * kRow + lc]) = gq;
            if (wave == 0) {
                sInv[b][lane] = gi;
                // rows 8 g + 4 hh + i of a block: the same bits 2 and 5
                float top = gi;
                top = fmaxf(top, __shfl_xor(top, 1));
                top = fmaxf(top, __shfl_xor(top, 2));
                top = fmaxf(top, __shfl_xor(top, 8));
                top = fmaxf(top, __shfl_xor(top, 16));
                if ((lane & 27) == 0) sTop[b][2 * (lane >> 5) + ((lane >> 2) & 1)] = top;
            }
        };
        bf16x8 qv[2][4];
        auto lread = [&](int b, int qb) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                qv[qb][ks] = *reinterpret_cast<const bf16x8*>(
                    &sD[b][(32 * qb + n) * kRow + 16 * ks + 8 * hh]);
        };
        float acc[kTmKB];
        int idx[kTmKB];
#pragma unroll
        for (int kb = 0; kb < kTmKB; ++kb) {
            acc[kb] = -INFINITY;
            idx[kb] = -1;   // none of this part's, or one already published
        }
        // Publish the part's finds; known = the sources' maxima so far (lane half 0).
        unsigned long long known[kTmKB];
        auto publish = [&]() {
#pragma unroll
            for (int kb = 0; kb < kTmKB; ++kb) {
                const float v = acc[kb] + 0.f;   // (no -0)
                unsigned long long k =
                    idx[kb] < 0 ? 0
                                : ((unsigned long long)float_order(v) << 32) |
                                      (uint32_t)~(uint32_t)idx[kb];
                const unsigned long long o = __shfl_xor(k, 32);   // the source's other rows
                k = o > k ? o : k;
                const int64_t i = i0 + 32 * kb + n;
                known[kb] = 0;
                if (hh == 0 && i < G.nA) known[kb] = max(k, atomicMax(&best[i], k));
            }
        };
        auto raise = [&]() {
#pragma unroll
            for (int kb = 0; kb < kTmKB; ++kb) {
                const uint32_t u = __shfl((uint32_t)(known[kb] >> 32), n);
                // (-0 is ordered just below +0 but equals it: below a maximum of 0 comes
                // the largest negative value, here the largest normal one)
                const float low = u == 0x80000000u ? -0x1p-126f
                                  : u > 0x007fffffu ? float_unorder(u - 1) : -INFINITY;
                if (low > acc[kb]) {
                    acc[kb] = low;
                    idx[kb] = -1;
                }
            }
        };
        f32x16 Sa[2], Sb[2];   // the blocks being multiplied, and the two before them
        // S = blocks (qb, 2 kp and 2 kp + 1)
        auto mul = [&](int qb, int kp, f32x16 (&S)[2]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) S[u] = mfma_bf16(qv[qb][0], B[2 * kp + u][0], zero_f32x16());
#pragma unroll
            for (int ks = 1; ks < 4; ++ks)
#pragma unroll
                for (int u = 0; u < 2; ++u) S[u] = mfma_bf16(qv[qb][ks], B[2 * kp + u][ks], S[u]);
        };
        // Blocks T of sources 2 kp, 2 kp + 1 and the 32 destinations from slot j0, whose
        // 1 / |m| start at inv (LDS; the largest of the lane half's 16: top).
        auto take = [&](int kp, const f32x16 (&T)[2], const float* inv, float top, int j0) {
            bool over[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                int mx = 0;
#pragma unroll
                for (int r = 0; r < 16; r += 2)
                    mx = max(max(mx, __float_as_int(T[u][r])), __float_as_int(T[u][r + 1]));
                over[u] = !(__int_as_float(mx) * top <= acc[2 * kp + u]);
            }
            if (__builtin_amdgcn_ballot_w64(over[0] || over[1]) == 0) return;
            f32x4 iv[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) iv[g] = *reinterpret_cast<const f32x4*>(inv + 8 * g + 4 * hh);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (__builtin_amdgcn_ballot_w64(over[u]) == 0) continue;
                float v[16], mx = -INFINITY;
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = T[u][r] * iv[r >> 2][r & 3];
#pragma unroll
                for (int r = 0; r < 16; r += 2) mx = fmaxf(fmaxf(mx, v[r]), v[r + 1]);
                const bool up = mx > acc[2 * kp + u];
                if (__builtin_amdgcn_ballot_w64(up) == 0) continue;
                int at = 0;   // the first row with that value
#pragma unroll
                for (int r = 15; r >= 0; --r) at = v[r] == mx ? 8 * (r >> 2) + (r & 3) : at;
                acc[2 * kp + u] = up ? mx : acc[2 * kp + u];
                idx[2 * kp + u] = up ? min(j0 + 4 * hh + at, nD - 1) : idx[2 * kp + u];
            }
        };
        __syncthreads();   // the previous segment's reads are done
        gload(t0);
        lstore(0);
        gload(t0 + 1);
        lstore(1);
        gload(t0 + 2);
        __syncthreads();
        lread(0, 0);
        mul(0, 0, Sa);
        int b0 = 0, b1 = 1, b2 = 2;   // buffers of tiles t, t + 1, t + 2
        for (int t = t0; t < t1; ++t) {
            const float* inv = sInv[b0];
            const float top0 = sTop[b0][hh], top1 = sTop[b0][2 + hh];
            lread(b0, 1);
            mul(0, 1, Sb);
            lstore(b2);
            gload(t + 3);
            if (((t - t0) & 15) == 8) publish();
            if (((t - t0) & 15) == 10) raise();
            take(0, Sa, inv, top0, 64 * t);
            mul(1, 0, Sa);
            take(1, Sb, inv, top0, 64 * t);
            lread(b1, 0);
            mul(1, 1, Sb);
            take(0, Sa, inv + 32, top1, 64 * t + 32);
            mul(0, 0, Sa);   // (past the last tile: a block that is not taken)
            take(1, Sb, inv + 32, top1, 64 * t + 32);
            __syncthreads();
            const int b = b0;
            b0 = b1;
            b1 = b2;
            b2 = b;
        }
        publish();
    }
}

// Exclusive prefix sum of one value per thread (256 threads); *total: the sum.
__device__ __forceinline__ int block_scan_excl(int v, int* total) {
    __shared__ int ws[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    int off = 0;
    for (int w = 0; w < wave; ++w) off += ws[w];
    *total = ws[0] + ws[1] + ws[2] + ws[3];
    __syncthreads();
    return off + x - v;
}

// ---------------------------------------------------------------- T3
// Radix select of the M largest keys (similarity, then the lower token): the
// ordered 32 bits of the score above tb bits of the token's complement, N <=
// 2^tb, so that a key has only the bits that can differ.  11 bits per pass from
// the top, one histogram of 2,048 counts per pass.  State before pass p: [2 p]
// prefix, [2 p + 1] keys still to take.  The digit of pass p - 1 is found by every
// workgroup of pass p for itself (a scan of 2,048 counts; the first one records
// it), and the last digit by the workgroups of k_tome_flags; pass 0 counts as
// k_tome_match_final makes the keys.
// Bound by launches and the latency of a pass: 108,405 keys in 8 passes of 8
// bits, each a histogram (27 workgroups of 4,096 keys) and a kernel for the
// digit, 126 us; in 5 passes of 1,024 keys a workgroup, 25 us.
constexpr int kSelBits = 11, kSelBins = 1 << kSelBits, kSelPasses = 6;   // 32 + 28 bits at most
constexpr int kSelBlock = 1024;   // keys per workgroup (256 threads x 4)

__device__ __forceinline__ uint64_t sel_key(float score, int64_t tok, int tb) {
    return ((uint64_t)float_order(score) << tb) | (((uint64_t)1 << tb) - 1 - (uint64_t)tok);
}

// The digit of a pass: the largest d with as many keys of digits >= d as are still to
// take.  256 threads; prefix and rem in and out.
__device__ __forceinline__ void sel_pick(const uint32_t* __restrict__ ghist, int shift,
                                         uint64_t& prefix, uint64_t& rem) {
    constexpr int kPer = kSelBins / 256;
    __shared__ uint32_t s_d, s_rem;
    uint32_t c[kPer];   // digits from kSelBins - 1 - kPer t down
    const u32x4* g = reinterpret_cast<const u32x4*>(ghist + kSelBins - kPer * (threadIdx.x + 1));
    const u32x4 lo = g[0], hi = g[1];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = hi[3 - k];
        c[4 + k] = lo[3 - k];
    }
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) sum += (int)c[k];
    if (threadIdx.x == 0) {
        s_d = 0;
        s_rem = (uint32_t)rem;
    }
    int tot;
    uint32_t above = (uint32_t)block_scan_excl(sum, &tot);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (above < rem && above + c[k] >= rem) {
            s_d = kSelBins - 1 - kPer * threadIdx.x - k;
            s_rem = (uint32_t)rem - above;
        }
        above += c[k];
    }
    __syncthreads();
    prefix |= (uint64_t)s_d << shift;
    rem = s_rem;
}

// Count of a workgroup's digits into the histogram h (LDS, zeroed), then ghist.
__device__ __forceinline__ void sel_count(uint32_t* h, uint32_t d, bool act) {
    const uint64_t mt = wave_match<kSelBits>(d, act);
    if (act && (mt & lanemask_lt()) == 0) atomicAdd(&h[d], (uint32_t)__popcll(mt));
}
__device__ __forceinline__ void sel_flush(const uint32_t* h, uint32_t* __restrict__ ghist) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSelBins; k += 256)
        if (h[k + threadIdx.x]) atomicAdd(&ghist[k + threadIdx.x], h[k + threadIdx.x]);
}

__global__ __launch_bounds__(256) void k_tome_init(uint64_t* __restrict__ st,
                                                   uint32_t* __restrict__ ghist, int64_t M,
                                                   int32_t* __restrict__ cnt, int64_t nD,
                                                   uint64_t* __restrict__ top, int64_t nA) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t k = i; k < kSelPasses * kSelBins; k += (int64_t)gridDim.x * 256) ghist[k] = 0;
    if (i == 0) {
        st[0] = 0;
        st[1] = (uint64_t)M;
    }
    if (i < nD) cnt[i] = 0;    // merged sources per destination
    if (i < nA) top[i] = kNoMatch;   // matching: maxima so far
}

// Per source: its destination slot, the cosine similarity and the selection key;
// the histogram of the keys' first digits.
__global__ __launch_bounds__(256) void k_tome_match_final(TomeGeom G, int tb, int shift,
                                                          const uint64_t* __restrict__ top,
                                                          const float* __restrict__ invn,
                                                          int32_t* __restrict__ best,
                                                          float* __restrict__ score,
                                                          uint64_t* __restrict__ key,
                                                          uint32_t* __restrict__ ghist) {
    __shared__ uint32_t h[kSelBins];
#pragma unroll
    for (int k = 0; k < kSelBins; k += 256) h[k + threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSelBlock + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kSelBlock / 256; ++k) {
        const int64_t i = base + 256 * k;
        uint32_t d = 0;
        if (i < G.nA) {
            const float v = float_unorder((uint32_t)(top[i] >> 32));
            const int64_t tok = tome_src_token(G, i);
            const float sc = v * invn[tok] + 0.f;   // + 0: no -0
            best[i] = (int32_t)~(uint32_t)top[i];
            score[i] = sc;
            const uint64_t ky = sel_key(sc, tok, tb);
            key[i] = ky;
            d = (uint32_t)(ky >> shift);
        }
        sel_count(h, d, i < G.nA);
    }
    sel_flush(h, ghist);
}

// Pass p > 0 at `shift`: counts of the next digit among the keys with the prefix so far.
__global__ __launch_bounds__(256) void k_rsel_hist(const uint64_t* __restrict__ key, int64_t n,
                                                   int p, int shift, uint64_t* __restrict__ st,
                                                   uint32_t* __restrict__ ghist) {
    __shared__ uint32_t h[kSelBins];
#pragma unroll
    for (int k = 0; k < kSelBins; k += 256) h[k + threadIdx.x] = 0;
    uint64_t v[kSelBlock / 256];
    const int64_t base = (int64_t)blockIdx.x * kSelBlock + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kSelBlock / 256; ++k) {
        const int64_t i = base + 256 * k;
        v[k] = i < n ? key[i] : ~0ull;   // (no key: it has at most 60 bits)
    }
    uint64_t prefix = st[2 * p - 2], rem = st[2 * p - 1];
    sel_pick(ghist + (p - 1) * kSelBins, shift + kSelBits, prefix, rem);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st[2 * p] = prefix;
        st[2 * p + 1] = rem;
    }
#pragma unroll
    for (int k = 0; k < kSelBlock / 256; ++k)
        sel_count(h, (uint32_t)(v[k] >> shift) & (kSelBins - 1),
                  ((v[k] ^ prefix) >> (shift + kSelBits)) == 0);
    sel_flush(h, ghist + p * kSelBins);
}

// ---------------------------------------------------------------- scans
// Exclusive scans of non-negative int32, up to two arrays at once (blockIdx.y):
// block sums, then per-block scans plus the sums before them (in == out
// allowed).  Up to kScanFew blocks each block adds those up itself; beyond,
// a one-workgroup scan of the sums comes between.  At 137,400 tokens a kernel
// of this size takes 4 us, nearly all of it latency: six scans of three kernels
// 72 us, three (two of them on two arrays) of two kernels 28 us.  The whole plan
// of 5,496 tokens is 110 us shorter (merged layer 314 -> 204 us), that of 137,400
// tokens 130 us (2293 -> 2161 us).
constexpr int kScanFew = 1024;
struct ScanJob {
    const int32_t* in;
    int32_t* out;
    int64_t n;
    int32_t* bsum;
};

__global__ __launch_bounds__(256) void k_scan_sums(ScanJob a, ScanJob b) {
    const ScanJob j = blockIdx.y ? b : a;
    if ((int64_t)blockIdx.x * kScanBlock >= j.n) return;
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * 4;
    int s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) s += (i + k < j.n) ? j.in[i + k] : 0;
    int tot;
    block_scan_excl(s, &tot);
    if (threadIdx.x == 0) j.bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_scan_top(ScanJob a, ScanJob b) {
    const ScanJob j = blockIdx.y ? b : a;
    const int64_t nb = (j.n + kScanBlock - 1) / kScanBlock;
    int carry = 0;
    for (int64_t c = 0; c < nb; c += kScanBlock) {
        const int64_t i = c + threadIdx.x * 4;
        int v[4], s = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = (i + k < nb) ? j.bsum[i + k] : 0;
            s += v[k];
        }
        int tot;
        int run = carry + block_scan_excl(s, &tot);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k < nb) {
                j.bsum[i + k] = run;
                run += v[k];
            }
        carry += tot;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_scan_apply(ScanJob a, ScanJob b, int scanned) {
    const ScanJob j = blockIdx.y ? b : a;
    if ((int64_t)blockIdx.x * kScanBlock >= j.n) return;
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * 4;
    int v[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = (i + k < j.n) ? j.in[i + k] : 0;
        s += v[k];
    }
    int before;
    if (scanned) {
        before = j.bsum[blockIdx.x];
    } else {
        int pre = 0;
#pragma unroll
        for (int k = 0; k < kScanFew / 256; ++k) {
            const unsigned q = threadIdx.x + 256 * k;
            pre += q < blockIdx.x ? j.bsum[q] : 0;
        }
        block_scan_excl(pre, &before);
    }
    int tot;
    int run = before + block_scan_excl(s, &tot);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i + k < j.n) {
            j.out[i + k] = run;
            run += v[k];
        }
}

void scan_excl(ScanJob a, ScanJob b, hipStream_t st) {
    const int64_t n = a.n > b.n ? a.n : b.n;
    if (n <= 0) return;
    const dim3 grid((unsigned)((n + kScanBlock - 1) / kScanBlock), b.n > 0 ? 2 : 1);
    const int scanned = grid.x > kScanFew;
    hipLaunchKernelGGL(k_scan_sums, grid, dim3(256), 0, st, a, b);
    if (scanned) hipLaunchKernelGGL(k_scan_top, dim3(1, grid.y), dim3(256), 0, st, a, b);
    hipLaunchKernelGGL(k_scan_apply, grid, dim3(256), 0, st, a, b, scanned);
}

// ---------------------------------------------------------------- sort
// Stable LSD radix sort of (key, value) pairs by 8-bit digits.
__global__ __launch_bounds__(kSortBlock) void k_rs_hist(const uint32_t* __restrict__ key,
                                                        int64_t n, int shift, int64_t nb,
                                                        int32_t* __restrict__ hist) {
    __shared__ int32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kSortBlock + threadIdx.x;
    const bool act = i < n;
    const uint32_t d = act ? (key[i] >> shift) & 255u : 0u;
    const uint64_t mt = wave_match<8>(d, act);
    if (act && (mt & lanemask_lt()) == 0) atomicAdd(&h[d], (int32_t)__popcll(mt));
    __syncthreads();
    if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(kSortBlock) void k_rs_scatter(const uint32_t* __restrict__ key,
                                                           const int32_t* __restrict__ val,
                                                           int64_t n, int shift, int64_t nb,
                                                           const int32_t* __restrict__ off,
                                                           uint32_t* __restrict__ key_out,
                                                           int32_t* __restrict__ val_out) {
    constexpr int kWaves = kSortBlock / 64;
    __shared__ int32_t wc[kWaves][256];
    for (int k = threadIdx.x; k < kWaves * 256; k += kSortBlock) (&wc[0][0])[k] = 0;
    __syncthreads();
    const int wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * kSortBlock + threadIdx.x;
    const bool act = i < n;
    const uint32_t k = act ? key[i] : 0u;
    const uint32_t d = (k >> shift) & 255u;
    const uint64_t mt = wave_match<8>(d, act);
    const int rank = __popcll(mt & lanemask_lt());
    if (act && rank == 0) wc[wave][d] = __popcll(mt);
    __syncthreads();
    if (act) {
        int64_t pos = off[(int64_t)d * nb + blockIdx.x] + rank;
        for (int w = 0; w < wave; ++w) pos += wc[w][d];
        key_out[pos] = k;
        val_out[pos] = val[i];
    }
}

// ---------------------------------------------------------------- T4
// Per token: kept flag; merged count per destination; the optional best /
// score outputs.  The threshold of the merged sources' keys is the prefix
// before the last pass (shift 0) and that pass's digit.
__global__ __launch_bounds__(256) void k_tome_flags(TomeGeom G, int passes,
                                                    const uint64_t* __restrict__ key,
                                                    const uint64_t* __restrict__ st,
                                                    const uint32_t* __restrict__ ghist,
                                                    const int32_t* __restrict__ bslot,
                                                    const float* __restrict__ score,
                                                    int32_t* __restrict__ kept,
                                                    int32_t* __restrict__ cnt,
                                                    int32_t* __restrict__ best_out,
                                                    float* __restrict__ score_out) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint64_t least = 0, rem = 0;
    if (G.nA > 0) {
        least = st[2 * passes - 2];
        rem = st[2 * passes - 1];
        sel_pick(ghist + (passes - 1) * kSelBins, 0, least, rem);
    }
    if (t >= G.N) return;
    const int64_t s = tome_slot(G, t);
    int k = 1;
    if (s < 0) {
        const int64_t i = -1 - s;
        const int merged = key[i] >= least ? 1 : 0;
        k = 1 - merged;
        if (merged) atomicAdd(&cnt[bslot[i]], 1);
        if (best_out) best_out[t] = (int32_t)tome_dst_token(G, bslot[i]);
        if (score_out) score_out[t] = score[i];
    } else {
        if (best_out) best_out[t] = -1;
        if (score_out) score_out[t] = 0.f;
    }
    kept[t] = k;
}

// Row sizes of kept tokens (1 + the sources merged into a destination); for
// merged sources, of which t - row[t] come before token t (row: the scan of
// the kept flags), their place in the list of (destination slot, token) in
// token order, and their row, the destination's.
__global__ __launch_bounds__(256) void k_tome_rows(TomeGeom G, int64_t M,
                                                   const int32_t* __restrict__ kept,
                                                   const int32_t* __restrict__ bslot,
                                                   const int32_t* __restrict__ cnt,
                                                   int32_t* __restrict__ row,
                                                   int32_t* __restrict__ size,
                                                   uint32_t* __restrict__ lkey,
                                                   int32_t* __restrict__ lval,
                                                   int32_t* __restrict__ row_start) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t == 0) row_start[G.N - M] = (int32_t)G.N;
    if (t >= G.N) return;
    const int64_t s = tome_slot(G, t), r = row[t];
    if (kept[t]) {
        if (r >= 0 && r < G.N) size[r] = 1 + (s >= 0 ? cnt[s] : 0);
    } else {
        const int32_t j = bslot[-1 - s];
        const int64_t p = t - r;
        if (p >= 0 && p < M) {
            lkey[p] = (uint32_t)j;
            lval[p] = (int32_t)t;
        }
        // a kept destination's row is final (it came from the scan)
        row[t] = row[tome_dst_token(G, j)];
    }
}

// (Every index is checked against its array, so an inconsistent plan cannot
// write outside the caller's buffers.)
__global__ __launch_bounds__(256) void k_tome_members(TomeGeom G, int64_t M, int64_t nrows,
                                                      const int32_t* __restrict__ kept,
                                                      const int32_t* __restrict__ row,
                                                      const int32_t* __restrict__ row_start,
                                                      const uint32_t* __restrict__ skey,
                                                      const int32_t* __restrict__ sval,
                                                      const int32_t* __restrict__ off,
                                                      int32_t* __restrict__ members) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < G.N && kept[i]) {
        const int64_t r = row[i];
        if (r >= 0 && r < nrows) {
            const int64_t p = row_start[r];
            if (p >= 0 && p < G.N) members[p] = (int32_t)i;
        }
    }
    if (i < M) {
        const uint32_t j = skey[i];
        if ((int64_t)j >= G.nD) return;
        const int64_t r = row[tome_dst_token(G, j)];
        if (r < 0 || r >= nrows) return;
        const int64_t p = (int64_t)row_start[r] + 1 + (i - off[j]);
        if (p >= 0 && p < G.N) members[p] = sval[i];
    }
}

// ---------------------------------------------------------------- T5
template <int DT>
__global__ __launch_bounds__(256) void k_tome_merge(const void* __restrict__ X, int64_t N, int F,
                                                    const int32_t* __restrict__ row_start,
                                                    const int32_t* __restrict__ members,
                                                    void* __restrict__ Xm) {
    const int64_t r = blockIdx.x;
    int64_t b = row_start[r], e = row_start[r + 1];
    b = b < 0 ? 0 : (b > N ? N : b);
    e = e < b ? b : (e > N ? N : e);
    for (int f0 = threadIdx.x * 4; f0 < F; f0 += 1024) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        int c = 0;
        for (int64_t p = b; p < e; ++p) {
            const int64_t t = members[p];
            if (t < 0 || t >= N) continue;
            if (DT == DT_BF16) {
                const bf16x4 v = *reinterpret_cast<const bf16x4*>(
                    reinterpret_cast<const bf16*>(X) + t * F + f0);
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] += bf16_to_f32(v[k]);
            } else {
                const float4 v = *reinterpret_cast<const float4*>(
                    reinterpret_cast<const float*>(X) + t * F + f0);
                acc[0] += v.x;
                acc[1] += v.y;
                acc[2] += v.z;
                acc[3] += v.w;
            }
            ++c;
        }
        const float cf = c > 0 ? (float)c : 1.f;
        if (DT == DT_BF16) {
            bf16x4 o;
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = (bf16)(acc[k] / cf);
            *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(Xm) + r * F + f0) = o;
        } else {
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(Xm) + r * F + f0) =
                make_float4(acc[0] / cf, acc[1] / cf, acc[2] / cf, acc[3] / cf);
        }
    }
}

// Q, K and V of a row at once (bf16, F = 1024 or less): the row's member
// indices are staged in LDS first (256 per pass), so the loads of the three
// tensors do not wait on one index each; sums in member order, as above.
__global__ __launch_bounds__(256) void k_tome_merge_qkv(const bf16* __restrict__ Q,
                                                        const bf16* __restrict__ K,
                                                        const bf16* __restrict__ V, int64_t N,
                                                        int F, const int32_t* __restrict__ row_start,
                                                        const int32_t* __restrict__ members,
                                                        bf16* __restrict__ Qm, bf16* __restrict__ Km,
                                                        bf16* __restrict__ Vm) {
    __shared__ int32_t sm[256];
    const int64_t r = blockIdx.x;
    int64_t b = row_start[r], e = row_start[r + 1];
    b = b < 0 ? 0 : (b > N ? N : b);
    e = e < b ? b : (e > N ? N : e);
    const int f0 = threadIdx.x * 4;
    const bool act = f0 < F;
    float aq[4] = {0.f, 0.f, 0.f, 0.f}, ak[4] = {0.f, 0.f, 0.f, 0.f}, av[4] = {0.f, 0.f, 0.f, 0.f};
    int c = 0;
    for (int64_t p0 = b; p0 < e; p0 += 256) {
        const int cnt = (int)((e - p0) < 256 ? (e - p0) : 256);
        __syncthreads();
        if ((int)threadIdx.x < cnt) sm[threadIdx.x] = members[p0 + threadIdx.x];
        __syncthreads();
        for (int j = 0; j < cnt; ++j) {
            const int64_t t = sm[j];
            if (t < 0 || t >= N) continue;
            ++c;
            if (!act) continue;
            const bf16x4 q = *reinterpret_cast<const bf16x4*>(Q + t * F + f0);
            const bf16x4 k = *reinterpret_cast<const bf16x4*>(K + t * F + f0);
            const bf16x4 v = *reinterpret_cast<const bf16x4*>(V + t * F + f0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                aq[i] += bf16_to_f32(q[i]);
                ak[i] += bf16_to_f32(k[i]);
                av[i] += bf16_to_f32(v[i]);
            }
        }
    }
    if (!act) return;
    const float cf = c > 0 ? (float)c : 1.f;
    bf16x4 oq, ok, ov;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        oq[i] = (bf16)(aq[i] / cf);
        ok[i] = (bf16)(ak[i] / cf);
        ov[i] = (bf16)(av[i] / cf);
    }
    *reinterpret_cast<bf16x4*>(Qm + r * F + f0) = oq;
    *reinterpret_cast<bf16x4*>(Km + r * F + f0) = ok;
    *reinterpret_cast<bf16x4*>(Vm + r * F + f0) = ov;
}

// 16-byte chunks: Y[t] = Ym[row[t]] (zero for a row outside [0, nrows)).
__global__ __launch_bounds__(256) void k_tome_unmerge(const u32x4* __restrict__ Ym, int64_t nrows,
                                                      const int32_t* __restrict__ row, int64_t N,
                                                      int cpr, u32x4* __restrict__ Y) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N * cpr) return;
    const int64_t t = i / cpr, c = i - t * cpr;
    const int64_t r = row[t];
    const u32x4 z = {0u, 0u, 0u, 0u};
    Y[i] = (r >= 0 && r < nrows) ? Ym[r * cpr + c] : z;
}

// Workspace of the plan for N tokens.
struct TomeWs {
    size_t m, invn, bslot, score, key, st, ghist, kept, cnt, off, size, lk0, lv0, lk1, lv1,
        bsum0, bsum1, hist, top, total;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

TomeWs tome_ws(int64_t N) {
    TomeWs w;
    const size_t n = (size_t)(N > 0 ? N : 1);
    const size_t nbr = (n + kSortBlock - 1) / kSortBlock;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align256(o + bytes);
        return at;
    };
    w.m = take(n * kD * 2);
    w.invn = take(n * 4);
    w.bslot = take(n * 4);
    w.score = take(n * 4);
    w.key = take(n * 8);
    w.st = take(kSelPasses * 16);
    w.ghist = take(kSelPasses * kSelBins * 4);
    w.kept = take(n * 4);
    w.cnt = take(n * 4);
    w.off = take(n * 4);
    w.size = take(n * 4);
    w.lk0 = take(n * 4);
    w.lv0 = take(n * 4);
    w.lk1 = take(n * 4);
    w.lv1 = take(n * 4);
    w.bsum0 = take(((256 * nbr > n ? 256 * nbr : n) / kScanBlock + 1) * 4);
    w.bsum1 = take((n / kScanBlock + 1) * 4);
    w.hist = take(256 * nbr * 4);
    w.top = take(n * 8);
    w.total = o;
    return w;
}

unsigned grid256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

size_t tome_workspace_bytes(int64_t N) { return tome_ws(N).total; }

void launch_tome_plan(const TomeArgs& a, hipStream_t st) {
    const TomeGeom& G = a.G;
    const TomeWs w = tome_ws(G.N);
    char* ws = (char*)a.ws;
    bf16* m = (bf16*)(ws + w.m);
    float* invn = (float*)(ws + w.invn);
    int32_t* bslot = (int32_t*)(ws + w.bslot);
    float* score = (float*)(ws + w.score);
    uint64_t* key = (uint64_t*)(ws + w.key);
    uint64_t* sel = (uint64_t*)(ws + w.st);
    uint32_t* ghist = (uint32_t*)(ws + w.ghist);
    int32_t *kept = (int32_t*)(ws + w.kept), *cnt = (int32_t*)(ws + w.cnt);
    int32_t *off = (int32_t*)(ws + w.off), *size = (int32_t*)(ws + w.size);
    uint32_t *lk0 = (uint32_t*)(ws + w.lk0), *lk1 = (uint32_t*)(ws + w.lk1);
    int32_t *lv0 = (int32_t*)(ws + w.lv0), *lv1 = (int32_t*)(ws + w.lv1);
    int32_t *bsum0 = (int32_t*)(ws + w.bsum0), *bsum1 = (int32_t*)(ws + w.bsum1);
    int32_t* hist = (int32_t*)(ws + w.hist);
    uint64_t* top = (uint64_t*)(ws + w.top);
    const int64_t N = G.N, M = a.M, nrows = N - M;
    int tb = 1;   // bits of a token
    while (tb < 28 && ((int64_t)1 << tb) < N) ++tb;
    const int passes = (32 + tb + kSelBits - 1) / kSelBits;

    hipLaunchKernelGGL(k_tome_init, dim3(grid256(N)), dim3(256), 0, st, sel, ghist, M, cnt, G.nD,
                       top, G.nA);
    if (G.nA > 0) {
        hipLaunchKernelGGL(k_tome_metric, dim3(grid256(N * 8)), dim3(256), 0, st, a.K, N, a.H, m,
                           invn);
        const int64_t steps = ((G.nA + kTmSrc - 1) / kTmSrc) * ((G.nD + 63) / 64);
        hipLaunchKernelGGL(k_tome_match, dim3((unsigned)(steps < kTmWG ? steps : kTmWG)),
                           dim3(64 * kTmWaves), 0, st, (const bf16*)m, (const float*)invn, G,
                           (unsigned long long*)top);
        const unsigned gs = (unsigned)((G.nA + kSelBlock - 1) / kSelBlock);
        int shift = (passes - 1) * kSelBits;
        hipLaunchKernelGGL(k_tome_match_final, dim3(gs), dim3(256), 0, st, G, tb, shift,
                           (const uint64_t*)top, (const float*)invn, bslot, score, key, ghist);
        // (M > 0 here: M = 0 leaves stride 1, hence no sources)
        for (int p = 1; p < passes; ++p) {
            shift -= kSelBits;
            hipLaunchKernelGGL(k_rsel_hist, dim3(gs), dim3(256), 0, st, (const uint64_t*)key, G.nA,
                               p, shift, sel, ghist);
        }
    }
    hipLaunchKernelGGL(k_tome_flags, dim3(grid256(N)), dim3(256), 0, st, G, passes,
                       (const uint64_t*)key, (const uint64_t*)sel, (const uint32_t*)ghist,
                       (const int32_t*)bslot, (const float*)score, kept, cnt, a.best, a.score);
    // rows of kept tokens; merged sources before each destination's
    const ScanJob none = {nullptr, nullptr, 0, nullptr};
    scan_excl({kept, a.row, N, bsum0}, M > 0 ? ScanJob{cnt, off, G.nD, bsum1} : none, st);
    hipLaunchKernelGGL(k_tome_rows, dim3(grid256(N)), dim3(256), 0, st, G, M, (const int32_t*)kept,
                       (const int32_t*)bslot, (const int32_t*)cnt, a.row, size, lk0, lv0,
                       a.row_start);
    if (M > 0) {
        // stable sort of the merged sources by destination slot
        int bits = 1;
        while (bits < 31 && ((int64_t)1 << bits) < G.nD) ++bits;
        const int64_t nb = (M + kSortBlock - 1) / kSortBlock;
        uint32_t *ki = lk0, *ko = lk1;
        int32_t *vi = lv0, *vo = lv1;
        for (int shift = 0; shift < bits; shift += 8) {
            hipLaunchKernelGGL(k_rs_hist, dim3((unsigned)nb), dim3(kSortBlock), 0, st,
                               (const uint32_t*)ki, M, shift, nb, hist);
            // (the rows' starts ride along with the first pass)
            scan_excl({hist, hist, 256 * nb, bsum0},
                      shift == 0 ? ScanJob{size, a.row_start, nrows, bsum1} : none, st);
            hipLaunchKernelGGL(k_rs_scatter, dim3((unsigned)nb), dim3(kSortBlock), 0, st,
                               (const uint32_t*)ki, (const int32_t*)vi, M, shift, nb,
                               (const int32_t*)hist, ko, vo);
            uint32_t* tk = ki;
            ki = ko;
            ko = tk;
            int32_t* tv = vi;
            vi = vo;
            vo = tv;
        }
        lk0 = ki;
        lv0 = vi;
    } else {
        scan_excl({size, a.row_start, nrows, bsum0}, none, st);
    }
    hipLaunchKernelGGL(k_tome_members, dim3(grid256(N)), dim3(256), 0, st, G, M, nrows,
                       (const int32_t*)kept, (const int32_t*)a.row, (const int32_t*)a.row_start,
                       (const uint32_t*)lk0, (const int32_t*)lv0, (const int32_t*)off,
                       a.members);
}

void launch_tome_merge(int dt, const void* X, int64_t N, int F, int64_t nrows,
                       const int32_t* row_start, const int32_t* members, void* Xm,
                       hipStream_t st) {
    if (nrows <= 0) return;
    if (dt == DT_BF16)
        hipLaunchKernelGGL(k_tome_merge<DT_BF16>, dim3((unsigned)nrows), dim3(256), 0, st, X, N, F,
                           row_start, members, Xm);
    else
        hipLaunchKernelGGL(k_tome_merge<DT_F32>, dim3((unsigned)nrows), dim3(256), 0, st, X, N, F,
                           row_start, members, Xm);
}

void launch_tome_merge_qkv(const void* Q, const void* K, const void* V, int64_t N, int F,
                           int64_t nrows, const int32_t* row_start, const int32_t* members,
                           void* Qm, void* Km, void* Vm, hipStream_t st) {
    if (nrows <= 0) return;
    hipLaunchKernelGGL(k_tome_merge_qkv, dim3((unsigned)nrows), dim3(256), 0, st, (const bf16*)Q,
                       (const bf16*)K, (const bf16*)V, N, F, row_start, members, (bf16*)Qm,
                       (bf16*)Km, (bf16*)Vm);
}

void launch_tome_unmerge(int dt, const void* Ym, int64_t nrows, const int32_t* row, int64_t N,
                         int F, void* Y, hipStream_t st) {
    const int cpr = F * (dt == DT_BF16 ? 2 : 4) / 16;
    if (N <= 0) return;
    hipLaunchKernelGGL(k_tome_unmerge, dim3(grid256(N * cpr)), dim3(256), 0, st,
                       (const u32x4*)Ym, nrows, row, N, cpr, (u32x4*)Y);
}

}  // namespace vp
