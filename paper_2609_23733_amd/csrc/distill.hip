// Distillation targets and losses (Section 4.4, Eq.8-11), bf16 layers.
//   Eq.8  p^T_{h,k} = max over queries q of A_{h,k,q}, A_h the teacher's
//         post-softmax attention (every query attends all N keys);
//         s^attn_h = max_k p^T_{h,k};
//   Eq.10 Delta^T_h = (A_h - I) V_h;
//   Eq.9  router loss  KL(p_bar || r_bar) + lambda |max p^T - max r|;
//   Eq.11 latent loss  ||D_hat - D^T|| + lambda (1 - cos(D_hat, D^T)).
// The column maxima take two passes over all (query, key) pairs:
//   D1  per query, o_q = log2 sum_k 2^x_qk (x the logit in log2 units), its
//       softmax normaliser: written by the teacher instances of the FULL-head
//       kernels, which compute Delta^T's attention in the same pass;
//   D2  per key, max over queries of x_qk - o_q, exponentiated once at the
//       end (exp2 is monotone, so the maximum can be taken before it), on the
//       bf16 MFMA (bf16 products are exact in fp32): colmax.hip.
#include "vp_device.hpp"
#include "vp_internal.hpp"

namespace vp {

// s^attn_h = max_k colmax[h][k]; one workgroup of 16 waves per head, 16 loads
// in flight per thread (bound by their latency: 4 N bytes a head).
// 24,744 tokens: 25.5 us with 4 waves and one load in flight, 5.4 us so.
__global__ __launch_bounds__(1024) void k_colmax_max(const float* __restrict__ colmax, int64_t N,
                                                     float* __restrict__ smax) {
    const int h = blockIdx.x;
    const float* row = colmax + (int64_t)h * N;
    float m = 0.f;
    int64_t k = threadIdx.x;
    for (; k + 15 * 1024 < N; k += 16 * 1024) {
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = row[k + 1024 * i];
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, v[i]);
    }
#pragma unroll 4
    for (; k < N; k += 1024) m = fmaxf(m, row[k]);
    m = wave_max(m);
    __shared__ float s[16];
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 1; i < 16; ++i) m = fmaxf(m, s[i]);
        smax[h] = m;
    }
}

// Bucket array with every head FULL (the teacher): counts (0, 0, H), ids
// 0 .. H-1, no flags; and colmax [n] = 0 for k_colmax's maxima.
__global__ __launch_bounds__(256) void k_teacher_init(int H, int32_t* __restrict__ buckets,
                                                      float* __restrict__ colmax, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < kBucketsLen) {
        int v = 0;
        if (i == 2) v = H;
        else if (i >= 3 && i < 3 + kMaxHeads) v = ((int)i - 3 < H) ? (int)i - 3 : 0;
        buckets[i] = v;
    }
    for (int64_t k = i; k < n; k += (int64_t)gridDim.x * 256) colmax[k] = 0.f;
}

// delta = Y - V (Y fp32, V bf16), rounded once to the output type.
__global__ __launch_bounds__(256) void k_sub_v(const float* __restrict__ Y,
                                               const bf16* __restrict__ V, int64_t n,
                                               void* __restrict__ out, int odt) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    const float4 a = *reinterpret_cast<const float4*>(Y + i);
    const float4 b = *reinterpret_cast<const float4*>(Y + i + 4);
    const bf16x8 v = load_bf16x8(V + i);
    float d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] -= bf16_to_f32(v[j]);
    if (odt == DT_BF16) {
        *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16*>(out) + i) =
            pack_bf16x8(d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7]);
    } else {
        float* o = reinterpret_cast<float*>(out) + i;
        *reinterpret_cast<float4*>(o) = make_float4(d[0], d[1], d[2], d[3]);
        *reinterpret_cast<float4*>(o + 4) = make_float4(d[4], d[5], d[6], d[7]);
    }
}

// ------------------------------------------------------------------------
// Eq.9 per head, one pass over the keys: with t_k = scale q_pool . k_k,
// log r_k = t_k - m - log l (router stats), p_k the column maxima and
// P = sum p, the loss is sum p log p / P - log P - sum p log r / P
// + lambda |max p - 1/l|.  Partial sums (P, sum p log p, sum p log r) per
// (key chunk, head), then a fixed-order combine.  8 lanes per key.
// ------------------------------------------------------------------------
constexpr int kLossChunks = 128;
static_assert(kLossChunks == 128, "sum_partials takes two per lane");

__global__ __launch_bounds__(256) void k_router_loss_partial(
    const bf16* __restrict__ K, const float* __restrict__ q_pool, const float* __restrict__ stats,
    float scale, const float* __restrict__ colmax, int64_t N, int H, float* __restrict__ part) {
    const int h = blockIdx.y, cnk = blockIdx.x;
    const int64_t chunk = (N + kLossChunks - 1) / kLossChunks;
    const int64_t t0 = cnk * chunk, t1 = (t0 + chunk < N) ? t0 + chunk : N;
    const int seg = (threadIdx.x & 7) * 8, rr = threadIdx.x >> 3;
    float qp[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) qp[j] = q_pool[h * kD + seg + j];
    const float m = stats[2 * h], lnl = logf(stats[2 * h + 1]);
    float P = 0.f, Ppp = 0.f, Ppr = 0.f;
    for (int64_t k = t0 + rr; k < t1; k += 32) {
        const bf16x8 kv = load_bf16x8(K + (k * H + h) * kD + seg);
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) dot = fmaf(qp[j], bf16_to_f32(kv[j]), dot);
        dot += __shfl_xor(dot, 1);
        dot += __shfl_xor(dot, 2);
        dot += __shfl_xor(dot, 4);
        if ((threadIdx.x & 7) == 0) {
            const float p = colmax[(int64_t)h * N + k];
            const float logr = dot * scale - m - lnl;
            P += p;
            Ppp += p > 0.f ? p * logf(p) : 0.f;
            Ppr += p * logr;
        }
    }
    P = wave_sum(P);
    Ppp = wave_sum(Ppp);
    Ppr = wave_sum(Ppr);
    __shared__ float s[4][3];
    if ((threadIdx.x & 63) == 0) {
        s[threadIdx.x >> 6][0] = P;
        s[threadIdx.x >> 6][1] = Ppp;
        s[threadIdx.x >> 6][2] = Ppr;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int j = threadIdx.x;
        part[((int64_t)h * kLossChunks + cnk) * 3 + j] = (s[0][j] + s[1][j]) + (s[2][j] + s[3][j]);
    }
}

// The kLossChunks = 128 partials of sum j of one head, in double: one wave,
// two per lane, then a butterfly (the order is fixed).
template <int NS>
__device__ __forceinline__ void sum_partials(const float* __restrict__ part, double (&s)[NS]) {
    const float* a = part + (threadIdx.x & 63) * NS;
#pragma unroll
    for (int j = 0; j < NS; ++j) s[j] = (double)a[j] + (double)a[64 * NS + j];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
        for (int j = 0; j < NS; ++j) s[j] += __shfl_xor(s[j], o);
}

// One wave per head (one lane per head, 128 partials in series: 7.2 us here and
// 9.7 us for the latent loss; 4.6 us each so, most of it the launch).
__global__ __launch_bounds__(64) void k_router_loss_combine(const float* __restrict__ part,
                                                            const float* __restrict__ stats,
                                                            const float* __restrict__ smax,
                                                            float lambda,
                                                            float* __restrict__ loss) {
    const int h = blockIdx.x;
    double s[3];
    sum_partials<3>(part + (int64_t)h * kLossChunks * 3, s);
    if (threadIdx.x) return;
    const double P = s[0], A = s[1], B = s[2];
    const double kl = A / P - log(P) - B / P;
    loss[h] = (float)(kl + (double)lambda * fabs((double)smax[h] - 1.0 / (double)stats[2 * h + 1]));
}

// Eq.11 per head: sums of (a - b)^2, a b, a^2, b^2 over the head's N x d
// entries; partials per (row chunk, head), then a fixed-order combine.
template <int DT>
__global__ __launch_bounds__(256) void k_latent_loss_partial(const void* __restrict__ A,
                                                             const void* __restrict__ B,
                                                             int64_t N, int H,
                                                             float* __restrict__ part) {
    const int h = blockIdx.y, cnk = blockIdx.x;
    const int64_t chunk = (N + kLossChunks - 1) / kLossChunks;
    const int64_t t0 = cnk * chunk, t1 = (t0 + chunk < N) ? t0 + chunk : N;
    const int seg = (threadIdx.x & 7) * 8, rr = threadIdx.x >> 3;
    float sdd = 0.f, sab = 0.f, saa = 0.f, sbb = 0.f;
    for (int64_t t = t0 + rr; t < t1; t += 32) {
        const int64_t o = (t * H + h) * kD + seg;
        float a[8], b[8];
        if (DT == DT_BF16) {
            const bf16x8 x = load_bf16x8(reinterpret_cast<const bf16*>(A) + o);
            const bf16x8 y = load_bf16x8(reinterpret_cast<const bf16*>(B) + o);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                a[j] = bf16_to_f32(x[j]);
                b[j] = bf16_to_f32(y[j]);
            }
        } else {
            const float* x = reinterpret_cast<const float*>(A) + o;
            const float* y = reinterpret_cast<const float*>(B) + o;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                a[j] = x[j];
                b[j] = y[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float d = a[j] - b[j];
            sdd = fmaf(d, d, sdd);
            sab = fmaf(a[j], b[j], sab);
            saa = fmaf(a[j], a[j], saa);
            sbb = fmaf(b[j], b[j], sbb);
        }
    }
    float v[4] = {wave_sum(sdd), wave_sum(sab), wave_sum(saa), wave_sum(sbb)};
    __shared__ float s[4][4];
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[threadIdx.x >> 6][j] = v[j];
    __syncthreads();
    if (threadIdx.x < 4) {
        const int j = threadIdx.x;
        part[((int64_t)h * kLossChunks + cnk) * 4 + j] = (s[0][j] + s[1][j]) + (s[2][j] + s[3][j]);
    }
}

__global__ __launch_bounds__(64) void k_latent_loss_combine(const float* __restrict__ part,
                                                            float lambda,
                                                            float* __restrict__ loss) {
    const int h = blockIdx.x;
    double s[4];
    sum_partials<4>(part + (int64_t)h * kLossChunks * 4, s);
    if (threadIdx.x) return;
    const double cosv = s[1] / (sqrt(s[2]) * sqrt(s[3]));
    loss[h] = (float)(sqrt(s[0]) + (double)lambda * (1.0 - cosv));
}

// ------------------------------------------------------------------ launchers

size_t distill_part_bytes(int H) { return (size_t)H * kLossChunks * 4 * sizeof(float); }

void launch_teacher_targets(const TeacherArgs& a, hipStream_t st) {
    const float c = kLog2e / sqrtf((float)kD);
    const bf16 *Q = (const bf16*)a.attn.Q, *K = (const bf16*)a.attn.K;
    // D1 with Delta^T's attention: every head FULL into fp32 Y, offsets into
    // attn.off.
    const int64_t nc = a.attn.N * a.attn.H;
    hipLaunchKernelGGL(k_teacher_init, dim3((unsigned)(nc < 262144 ? (nc + 255) / 256 : 1024)),
                       dim3(256), 0, st, a.attn.H, const_cast<int32_t*>(a.attn.buckets), a.colmax,
                       nc);
    launch_gather(a.attn, st);
    launch_flash(a.attn, st);
    launch_colmax(Q, K, a.attn.off, a.attn.N, a.attn.H, c, a.colmax, st);
    hipLaunchKernelGGL(k_colmax_max, dim3(a.attn.H), dim3(1024), 0, st, (const float*)a.colmax,
                       a.attn.N, a.smax);
    // Delta^T = Y - V.
    const int64_t n = a.attn.N * a.attn.H * kD;
    hipLaunchKernelGGL(k_sub_v, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, st,
                       (const float*)a.attn.Y, (const bf16*)a.attn.V, n, a.delta, a.delta_dt);
}

void launch_router_loss(const LossArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(k_router_loss_partial, dim3(kLossChunks, a.H), dim3(256), 0, st,
                       (const bf16*)a.A, a.q_pool, a.stats, a.scale, a.colmax, a.N, a.H, a.part);
    hipLaunchKernelGGL(k_router_loss_combine, dim3(a.H), dim3(64), 0, st, (const float*)a.part,
                       a.stats, a.smax, a.lambda, a.loss);
}

void launch_latent_loss(const LossArgs& a, hipStream_t st) {
    if (a.dtype == DT_BF16)
        hipLaunchKernelGGL(k_latent_loss_partial<DT_BF16>, dim3(kLossChunks, a.H), dim3(256), 0,
                           st, a.A, a.B, a.N, a.H, a.part);
    else
        hipLaunchKernelGGL(k_latent_loss_partial<DT_F32>, dim3(kLossChunks, a.H), dim3(256), 0,
                           st, a.A, a.B, a.N, a.H, a.part);
    hipLaunchKernelGGL(k_latent_loss_combine, dim3(a.H), dim3(64), 0, st, (const float*)a.part,
                       a.lambda, a.loss);
}

}  // namespace vp
