// Attention form of power attention in float32 on the matrix cores (v_mfma_f32_16x16x4_f32: float32 operands, products and
// sums), d = v in {16, 32, 64, 128}, degrees 1 .. 4, without gates, any sequence length.
//
//     O_i = sum_{j <= i} a_ij v_j / Z_i,  a_ij = s_ij^p,  s_ij = scale q_i . k_j,  Z_i = sum_{j <= i} a_ij
//     e_ij = (dO_i . v_j - delta_i) / Z_i,  delta_i = dO_i . O_i          (un-normalised: Z = 1, delta = 0)
//     dQ_i = p scale sum_j e_ij s_ij^(p-1) k_j,  dK_j = p scale sum_i e_ij s_ij^(p-1) q_i,  dV_j = sum_i a_ij dO_i / Z_i
//
// What bounds such calls is latency: they are short (a few thousand tokens at most), and the chunked float32 kernels walk
// a serial chain of state updates on a handful of workgroups.  So a workgroup owns only 16 N rows (queries for the forward
// pass and dQ, keys for dK / dV), its four waves take every fourth tile of 16 rows of the other side, and their sums meet
// in LDS at the end, in a fixed order.  The waves share nothing on the way: no staging, no barrier; operands come straight
// from L2 with 16-byte loads, and the other waves of the SIMD cover their latency.
//
// MFMA 16x16x4 (lane l, m = l % 16, g = l / 16): A row m, k-slot g;  B column m, k-slot g;  C column m, rows 4 g + r.
//   * First contraction (over the features): four consecutive MFMAs take features 16 f + 4 g + 0 .. 3, so an operand row is
//     one 16-byte load per 16 features.
//   * Second contraction (over the streamed rows): MFMA r takes the rows 4 g + r, which is where the first one's
//     accumulator r lies: it is the B operand as it stands.  Output column 16 x NV is dealt out as NV m + vb, so that a
//     lane's A operands of one row are NV consecutive floats, and so are the results it stores.
//
// MI355X, before (chunked, vector ALU) and after: 1 head of 256 tokens, d = 16, forward 132 -> 17 us a call (6.7 in the
// kernel); B2 H4 T1024 d32 forward + backward 2368 -> 62 us.
#include "common.hpp"

namespace pa {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ float sum_over_g(float x) {   // over the lanes with the same m, in every lane
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}
template <int P>
__device__ __forceinline__ float power(float s) {
    if (P == 0) return 1.f;
    if (P == 1) return s;
    if (P == 2) return s * s;
    if (P == 3) return s * s * s;
    const float s2 = s * s;
    return s2 * s2;
}

// a row's features 16 f + 4 g .. + 3
template <int HD>
struct RowFrag {
    f32x4 v[HD / 16];
};
template <int HD>
__device__ __forceinline__ RowFrag<HD> row_frag(const float* __restrict__ row, int g) {
    RowFrag<HD> f;
#pragma unroll
    for (int i = 0; i < HD / 16; ++i) f.v[i] = *(const f32x4*)(row + 16 * i + 4 * g);
    return f;
}
// rows row0 + 4 g + r (clamped to the sequence), columns NV m .. + NV - 1
template <int HD>
struct ColFrag {
    float v[4][HD / 16];
};
template <int HD>
__device__ __forceinline__ ColFrag<HD> col_frag(const float* __restrict__ head, int row0, int T, int m, int g) {
    constexpr int NV = HD / 16;
    ColFrag<HD> f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float* p = head + (size_t)min(row0 + 4 * g + r, T - 1) * HD + NV * m;
        if constexpr (NV >= 4) {
#pragma unroll
            for (int i = 0; i < NV; i += 4) {
                const f32x4 q = *(const f32x4*)(p + i);
#pragma unroll
                for (int k = 0; k < 4; ++k) f.v[r][i + k] = q[k];
            }
        } else if constexpr (NV == 2) {
            const float2 q = *(const float2*)p;
            f.v[r][0] = q.x;
            f.v[r][1] = q.y;
        } else {
            f.v[r][0] = *p;
        }
    }
    return f;
}
template <int HD>
__device__ __forceinline__ f32x4 dot(const RowFrag<HD>& a, const RowFrag<HD>& b, f32x4 c) {
#pragma unroll
    for (int i = 0; i < HD / 16; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) c = mfma4(a.v[i][k], b.v[i][k], c);
    return c;
}
// acc[vb] += the columns' sums weighted by w[r] (one weight per streamed row and lane)
template <int HD>
__device__ __forceinline__ void accumulate(f32x4 (&acc)[HD / 16], const ColFrag<HD>& c, const float (&w)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int vb = 0; vb < HD / 16; ++vb) acc[vb] = mfma4(c.v[r][vb], w[r], acc[vb]);
}
// acc[vb][r] is column NV (4 g + r) + vb of the lane's row: 4 NV consecutive floats
template <int HD>
__device__ __forceinline__ void store_row(float* __restrict__ row, const f32x4 (&acc)[HD / 16], float f, int g) {
    constexpr int NV = HD / 16;
    float* p = row + 4 * NV * g;
#pragma unroll
    for (int i = 0; i < 4 * NV; i += 4) {
        f32x4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = f * acc[(i + k) % NV][(i + k) / NV];
        *(f32x4*)(p + i) = o;
    }
}
// the four waves' sums of `n` registers, complete in wave 0
template <int N>
__device__ __forceinline__ void sum_waves(f32x4 (&x)[N], f32x4 (*red)[64], int w, int lane) {
    __syncthreads();
    if (w != 0)
#pragma unroll
        for (int i = 0; i < N; ++i) red[(w - 1) * N + i][lane] = x[i];
    __syncthreads();
    if (w == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = (x[i] + red[i][lane]) + (red[N + i][lane] + red[2 * N + i][lane]);
}

// grid (heads, blocks of 16 N queries, the longest walks of every head first)
template <int P, int HD, int N>
__global__ __launch_bounds__(256) void k_f32_attn_fwd(const float* __restrict__ Q, const float* __restrict__ K,
                                                      const float* __restrict__ V, float* __restrict__ O, float* __restrict__ Z,
                                                      int T, float scale, int normalize) {
    constexpr int NV = HD / 16;
    __shared__ f32x4 red[3 * NV][64];
    __shared__ float zred[N][3][64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, m = lane & 15, g = lane >> 4;
    const int i0 = (int)(gridDim.y - 1 - blockIdx.y) * 16 * N;
    const size_t head = (size_t)blockIdx.x * T;
    const float *Kh = K + head * HD, *Vh = V + head * HD;
    RowFrag<HD> q[N];
    f32x4 acc[N][NV];
    float z[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        q[n] = row_frag<HD>(Q + (head + min(i0 + 16 * n + m, T - 1)) * HD, g);
#pragma unroll
        for (int i = 0; i < NV; ++i) q[n].v[i] *= scale;
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[n][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        z[n] = 0.f;
    }
    const int key_end = min(i0 + 16 * N, T);
    for (int key0 = 16 * w; key0 < key_end; key0 += 64) {
        const RowFrag<HD> k = row_frag<HD>(Kh + (size_t)min(key0 + m, T - 1) * HD, g);
        const ColFrag<HD> v = col_frag<HD>(Vh, key0, T, m, g);
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const f32x4 s = dot<HD>(k, q[n], (f32x4){0.f, 0.f, 0.f, 0.f});     // key 4 g + r, query m
            float a[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                a[r] = key0 + 4 * g + r <= i0 + 16 * n + m ? power<P>(s[r]) : 0.f;
                z[n] += a[r];
            }
            accumulate<HD>(acc[n], v, a);
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
        if (w != 0) zred[n][w - 1][lane] = z[n];
#pragma unroll
    for (int n = 0; n < N; ++n) sum_waves<NV>(acc[n], red, w, lane);
    if (w != 0) return;
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const float zz = sum_over_g((z[n] + zred[n][0][lane]) + (zred[n][1][lane] + zred[n][2][lane]));
        const int i = i0 + 16 * n + m;
        if (i >= T) continue;
        store_row<HD>(O + (head + i) * HD, acc[n], normalize ? (zz != 0.f ? 1.f / zz : 0.f) : 1.f, g);
        if (Z != nullptr && g == 0) Z[head + i] = zz;
    }
}

// also leaves delta[head][i] (normalised) for the dK / dV kernel
template <int P, int HD, int N>
__global__ __launch_bounds__(256) void k_f32_attn_dq(const float* __restrict__ Q, const float* __restrict__ K,
                                                     const float* __restrict__ V, const float* __restrict__ O,
                                                     const float* __restrict__ Z, const float* __restrict__ dO,
                                                     float* __restrict__ delta, float* __restrict__ dQ, int T, float scale,
                                                     int normalize) {
    constexpr int NV = HD / 16;
    __shared__ f32x4 red[3 * NV][64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, m = lane & 15, g = lane >> 4;
    const int i0 = (int)(gridDim.y - 1 - blockIdx.y) * 16 * N;
    const size_t head = (size_t)blockIdx.x * T;
    const float *Kh = K + head * HD, *Vh = V + head * HD;
    RowFrag<HD> q[N], go[N];
    f32x4 acc[N][NV];
    float dl[N], iz[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const size_t row = head + min(i0 + 16 * n + m, T - 1);
        q[n] = row_frag<HD>(Q + row * HD, g);
        go[n] = row_frag<HD>(dO + row * HD, g);
        dl[n] = 0.f;
        iz[n] = 1.f;
        if (normalize) {
            const RowFrag<HD> o = row_frag<HD>(O + row * HD, g);
#pragma unroll
            for (int i = 0; i < NV; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) dl[n] += go[n].v[i][k] * o.v[i][k];
            dl[n] = sum_over_g(dl[n]);
            const float z = Z[row];
            iz[n] = z != 0.f ? 1.f / z : 0.f;
            if (w == 0 && g == 0 && i0 + 16 * n + m < T) delta[row] = dl[n];
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) q[n].v[i] *= scale;
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[n][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const int key_end = min(i0 + 16 * N, T);
    for (int key0 = 16 * w; key0 < key_end; key0 += 64) {
        const size_t row = (size_t)min(key0 + m, T - 1) * HD;
        const RowFrag<HD> k = row_frag<HD>(Kh + row, g), v = row_frag<HD>(Vh + row, g);
        const ColFrag<HD> kc = col_frag<HD>(Kh, key0, T, m, g);
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const f32x4 s = dot<HD>(k, q[n], (f32x4){0.f, 0.f, 0.f, 0.f});
            const f32x4 e = dot<HD>(v, go[n], (f32x4){-dl[n], -dl[n], -dl[n], -dl[n]});
            float t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                t[r] = key0 + 4 * g + r <= i0 + 16 * n + m ? iz[n] * e[r] * power<P - 1>(s[r]) : 0.f;
            accumulate<HD>(acc[n], kc, t);
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) sum_waves<NV>(acc[n], red, w, lane);
    if (w != 0) return;
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int i = i0 + 16 * n + m;
        if (i < T) store_row<HD>(dQ + (head + i) * HD, acc[n], (float)P * scale, g);
    }
}

// grid (heads, blocks of 16 N keys)
template <int P, int HD, int N>
__global__ __launch_bounds__(256) void k_f32_attn_dkdv(const float* __restrict__ Q, const float* __restrict__ K,
                                                       const float* __restrict__ V, const float* __restrict__ Z,
                                                       const float* __restrict__ dO, const float* __restrict__ delta,
                                                       float* __restrict__ dK, float* __restrict__ dV, int T, float scale,
                                                       int normalize) {
    constexpr int NV = HD / 16;
    __shared__ f32x4 red[3 * NV][64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, m = lane & 15, g = lane >> 4;
    const int j0 = (int)blockIdx.y * 16 * N;
    const size_t head = (size_t)blockIdx.x * T;
    const float *Qh = Q + head * HD, *Gh = dO + head * HD;
    RowFrag<HD> k[N], v[N];
    f32x4 dk[N][NV], dv[N][NV];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const size_t row = (head + min(j0 + 16 * n + m, T - 1)) * HD;
        k[n] = row_frag<HD>(K + row, g);
        v[n] = row_frag<HD>(V + row, g);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            k[n].v[i] *= scale;
            dk[n][i] = dv[n][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    }
    for (int q0 = j0 + 16 * w; q0 < T; q0 += 64) {
        const size_t row = (size_t)min(q0 + m, T - 1) * HD;
        const RowFrag<HD> q = row_frag<HD>(Qh + row, g), go = row_frag<HD>(Gh + row, g);
        const ColFrag<HD> gc = col_frag<HD>(Gh, q0, T, m, g), qc = col_frag<HD>(Qh, q0, T, m, g);
        f32x4 nd = (f32x4){0.f, 0.f, 0.f, 0.f};
        float iz[4] = {1.f, 1.f, 1.f, 1.f};
        if (normalize) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const size_t i = head + min(q0 + 4 * g + r, T - 1);
                const float z = Z[i];
                iz[r] = z != 0.f ? 1.f / z : 0.f;
                nd[r] = -delta[i];
            }
        }
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const f32x4 s = dot<HD>(q, k[n], (f32x4){0.f, 0.f, 0.f, 0.f});     // query 4 g + r, key m
            const f32x4 e = dot<HD>(go, v[n], nd);
            float a[4], t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = q0 + 4 * g + r;
                const bool in = i < T && i >= j0 + 16 * n + m;
                const float pw = power<P - 1>(s[r]);
                a[r] = in ? iz[r] * (pw * s[r]) : 0.f;
                t[r] = in ? iz[r] * e[r] * pw : 0.f;
            }
            accumulate<HD>(dv[n], gc, a);
            accumulate<HD>(dk[n], qc, t);
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        sum_waves<NV>(dk[n], red, w, lane);
        sum_waves<NV>(dv[n], red, w, lane);
    }
    if (w != 0) return;
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int j = j0 + 16 * n + m;
        if (j >= T) continue;
        store_row<HD>(dK + (head + j) * HD, dk[n], (float)P * scale, g);
        store_row<HD>(dV + (head + j) * HD, dv[n], 1.f, g);
    }
}

// Rows per workgroup: 32 read half the bytes per pair, 16 give twice the workgroups.  32 where that still leaves two
// workgroups per CU.
bool wide_blocks(int BH, int T) { return (long long)BH * ((T + 31) / 32) >= 512; }

template <int P, int HD>
bool fwd_t(const Ctx& c, const float* Q, const float* K, const float* V, float* O, float* Z) {
    const pa_problem& pr = c.prob;
    const int BH = pr.B * pr.H;
    LaunchScope ls("f32_attn_fwd", c.stream);
    if (wide_blocks(BH, pr.T))
        hipLaunchKernelGGL((k_f32_attn_fwd<P, HD, 2>), dim3(BH, (pr.T + 31) / 32), dim3(256), 0, c.stream, Q, K, V, O, Z, pr.T,
                           pr.scale, pr.normalize);
    else
        hipLaunchKernelGGL((k_f32_attn_fwd<P, HD, 1>), dim3(BH, (pr.T + 15) / 16), dim3(256), 0, c.stream, Q, K, V, O, Z, pr.T,
                           pr.scale, pr.normalize);
    return launch_ok();
}
template <int P, int HD, int N>
bool bwd_n(const Ctx& c, const float* Q, const float* K, const float* V, const float* O, const float* Z, const float* dO, float* dQ,
           float* dK, float* dV) {
    const pa_problem& pr = c.prob;
    const dim3 grid(pr.B * pr.H, (pr.T + 16 * N - 1) / (16 * N));
    float* delta = (float*)c.ws;
    {
        LaunchScope ls("f32_attn_dq", c.stream);
        hipLaunchKernelGGL((k_f32_attn_dq<P, HD, N>), grid, dim3(256), 0, c.stream, Q, K, V, O, Z, dO, delta, dQ, pr.T, pr.scale,
                           pr.normalize);
        if (!launch_ok()) return false;
    }
    LaunchScope ls("f32_attn_dkdv", c.stream);
    hipLaunchKernelGGL((k_f32_attn_dkdv<P, HD, N>), grid, dim3(256), 0, c.stream, Q, K, V, Z, dO, delta, dK, dV, pr.T, pr.scale,
                       pr.normalize);
    return launch_ok();
}
template <int P, int HD>
bool bwd_t(const Ctx& c, const float* Q, const float* K, const float* V, const float* O, const float* Z, const float* dO, float* dQ,
           float* dK, float* dV) {
    // at d = 128 one block of operands and accumulators already fills the registers of a wave (dK / dV: 288, one wave per SIMD)
    if constexpr (HD < 128)
        if (wide_blocks(c.prob.B * c.prob.H, c.prob.T)) return bwd_n<P, HD, 2>(c, Q, K, V, O, Z, dO, dQ, dK, dV);
    return bwd_n<P, HD, 1>(c, Q, K, V, O, Z, dO, dQ, dK, dV);
}

}  // namespace

// Where the line lies (forward / backward, ms, chunked float32 kernels at chunk 64 -> these, p = 2): up to 4096 tokens these
// are ahead whatever the number of heads (128 heads of 4096, d = 16: 1.70 -> 0.74 / 5.5 -> 2.7; p = 1: 1.32 -> 0.76 /
// 3.1 -> 1.9; 1 head of 1024, d = 32: 0.67 -> 0.02 / 1.66 -> 0.05).  Beyond, the chunked kernels' serial walk leaves most of
// the chip idle as long as the heads are few (16 of 16384, d = 16: 5.1 -> 1.5 / 11.3 -> 5.1; p = 1, d = 64: 13 -> 5 /
// 28 -> 13), but with many they meet (128 heads of 8192, d = 16: 3.5 -> 2.8 / 11.0 -> 10.8; p = 1: 2.7 -> 2.8 / 6.4 -> 7.5).
// At 16 heads of 4096 tokens, d = 64, the backward pass runs at 110 TFLOP/s of float32 (a large matrix product: 153).
bool f32_attn_applies(const pa_problem& pr) {
    if (pr.impl != PA_IMPL_AUTO || pr.dtype != PA_DTYPE_F32 || pr.gated || pr.d != pr.v) return false;
    if (pr.d != 16 && pr.d != 32 && pr.d != 64 && pr.d != 128) return false;
    return pr.p >= 1 && pr.p <= 4 && (pr.T <= 4096 || (pr.T <= 16384 && (long long)pr.B * pr.H * pr.T <= 262144));
}

#define PA_DISPATCH(FN, ...)                          \
    switch (8 * pr.d + pr.p) {                        \
        case 8 * 16 + 1: return FN<1, 16>(__VA_ARGS__);   \
        case 8 * 16 + 2: return FN<2, 16>(__VA_ARGS__);   \
        case 8 * 16 + 3: return FN<3, 16>(__VA_ARGS__);   \
        case 8 * 16 + 4: return FN<4, 16>(__VA_ARGS__);   \
        case 8 * 32 + 1: return FN<1, 32>(__VA_ARGS__);   \
        case 8 * 32 + 2: return FN<2, 32>(__VA_ARGS__);   \
        case 8 * 32 + 3: return FN<3, 32>(__VA_ARGS__);   \
        case 8 * 32 + 4: return FN<4, 32>(__VA_ARGS__);   \
        case 8 * 64 + 1: return FN<1, 64>(__VA_ARGS__);   \
        case 8 * 64 + 2: return FN<2, 64>(__VA_ARGS__);   \
        case 8 * 64 + 3: return FN<3, 64>(__VA_ARGS__);   \
        case 8 * 64 + 4: return FN<4, 64>(__VA_ARGS__);   \
        case 8 * 128 + 1: return FN<1, 128>(__VA_ARGS__); \
        case 8 * 128 + 2: return FN<2, 128>(__VA_ARGS__); \
        case 8 * 128 + 3: return FN<3, 128>(__VA_ARGS__); \
        case 8 * 128 + 4: return FN<4, 128>(__VA_ARGS__); \
    }

bool f32_attn_fwd(const Ctx& c, const float* Q, const float* K, const float* V, float* O, float* Z) {
    const pa_problem& pr = c.prob;
    PA_DISPATCH(fwd_t, c, Q, K, V, O, Z)
    return false;
}

bool f32_attn_bwd(const Ctx& c, const float* Q, const float* K, const float* V, const float* O, const float* Z, const float* dO,
                  float* dQ, float* dK, float* dV) {
    const pa_problem& pr = c.prob;
    PA_DISPATCH(bwd_t, c, Q, K, V, O, Z, dO, dQ, dK, dV)
    return false;
}
#undef PA_DISPATCH

}  // namespace pa
