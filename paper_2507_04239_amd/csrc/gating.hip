// Gating (arXiv 2507.04239 Sec. 2 "Gating"; gated update-state of App. E.2, discounted
// cumulative sum of App. E.3): the kernels every kernel family shares.  The paper states the
// operation at chunk granularity; the per-timestep definition behind it is
//     a_ij = s_ij^p exp(b_i - b_j),   b_i = sum_{t<=i} log g_t,   j <= i.
// In the chunked form only sums of log-gates inside one chunk are ever needed (every factor is
// then a decay <= 1): see GateBuf in common.hpp.  The gradient of the log-gates follows from the
// homogeneity of the scores: dL/db_i = (q_i . dq_i - k_i . dk_i) / p, dL/dlog g_t = sum_{i>=t} dL/db_i.
#include "common.hpp"

namespace pa {
namespace {

constexpr int GT = 256;

// Log-gates below this are a factor of zero in float32 all the same; clamped to it, a gate that closes for good (the start of a
// document: -1e4, or minus infinity) leaves the digits of the sums it goes into to the gates beside it.
constexpr float GATE_FLOOR = -104.f;

// the value of another lane of the wave by DPP; lanes without a source, or whose row of 16 is not in ROWS, get 0
template <int CTRL, int ROWS>
__device__ __forceinline__ double lane_move(double x) {
    union {
        double d;
        int i[2];
    } u, v;
    u.d = x;
#pragma unroll
    for (int k = 0; k < 2; ++k) v.i[k] = __builtin_amdgcn_update_dpp(0, u.i[k], CTRL, ROWS, 0xf, false);
    return v.d;
}
__device__ __forceinline__ double wave_scan(double x) {      // inclusive, over the wave: in each row of 16 lanes, then across the rows
    x += lane_move<0x111, 0xf>(x);
    x += lane_move<0x112, 0xf>(x);
    x += lane_move<0x114, 0xf>(x);
    x += lane_move<0x118, 0xf>(x);
    x += lane_move<0x142, 0xa>(x);      // lane 15 of rows 0 and 2 to the row after
    x += lane_move<0x143, 0xc>(x);      // lane 31 to rows 2 and 3
    return x;
}

// One workgroup per (chunk, head): running sums of the chunk's log-gates, then the factors.  A pair's decay is a difference of two
// sums, so a sum kept in one float32 from a distant start loses what the pair's own gates contribute: at 5120 tokens of mean
// -0.02 the decays are off by 5e-5, with a gate of -1e4 every 300 tokens by 9e-2.  So sums run in float64 and are kept
// relative to blocks of GATE_BLOCK tokens, as decays from blocks this short are when nothing is added to them.
// A wave scans a block, two tokens per lane, and holds GB blocks at a time; the workgroup's blocks meet in LDS.
__global__ __launch_bounds__(GT) void k_gate_prep(const float* __restrict__ log_g, float* __restrict__ bl, double* __restrict__ blk,
                                                  float* __restrict__ qfac, float* __restrict__ kfac,
                                                  float* __restrict__ lam, int T, int chunk, int head_blocks, int in_blocks) {
    constexpr int WAVES = GT / 64, GB = 4, STEP = WAVES * GB;
    static_assert(GATE_BLOCK == 128, "two tokens per lane");
    __shared__ double sums[2][STEP];
    const int n = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const size_t base = (size_t)bh * T + (size_t)n * chunk;
    const int len = min(chunk, T - n * chunk);    // (the last chunk may be shorter)
    const int nblk = (len + GATE_BLOCK - 1) / GATE_BLOCK;
    double* blk_out = blk + (size_t)bh * head_blocks + (size_t)n * ((chunk + GATE_BLOCK - 1) / GATE_BLOCK);
    auto gate = [&](int i) {
        const float g = i < len ? log_g[base + i] : 0.f;
        return g < GATE_FLOOR ? GATE_FLOOR : g;   // (a NaN stays one)
    };
    float g[GB][2];
    double incl[GB];
    // the blocks b0 + WAVES u + w; their sums to sums[buf]
    auto scan = [&](int b0, int buf) {
#pragma unroll
        for (int u = 0; u < GB; ++u) {
            const int i = (b0 + WAVES * u + w) * GATE_BLOCK + 2 * lane;
            g[u][0] = gate(i);
            g[u][1] = gate(i + 1);
        }
#pragma unroll
        for (int u = 0; u < GB; ++u) {
            incl[u] = wave_scan((double)g[u][0] + (double)g[u][1]);
            if (lane == 63) sums[buf][WAVES * u + w] = incl[u];
        }
        __syncthreads();
    };
    double total = 0.;
    int buf = 0;
    for (int b0 = 0; b0 < nblk; b0 += STEP, buf ^= 1) {
        scan(b0, buf);
        for (int k = 0; k < min(STEP, nblk - b0); ++k) total += sums[buf][k];
    }
    if (tid == 0) lam[(size_t)bh * gridDim.x + n] = __expf((float)total);
    double before = 0.;
    for (int b0 = 0; b0 < nblk; b0 += STEP, buf ^= 1) {
        if (nblk > STEP) scan(b0, buf);           // (else the blocks are still here, and their sums in the other buffer)
        const double* in = nblk > STEP ? sums[buf] : sums[buf ^ 1];
        for (int k = 0; k < min(STEP, nblk - b0); ++k) {
            const int u = k / WAVES;
            if (k % WAVES == w) {
                const int i = (b0 + k) * GATE_BLOCK + 2 * lane;
                double x = 0., pair = 0.;
#pragma unroll
                for (int v = 0; v < GB; ++v)
                    if (v == u) {
                        x = lane_move<0x138, 0xf>(incl[v]) + (double)g[v][0];      // (from the lane before)
                        pair = incl[v];
                    }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float rel = (float)(e == 0 ? x : pair);
                    const double run = before + rel;
                    if (i + e < len) {
                        bl[base + i + e] = in_blocks ? rel : (float)run;
                        qfac[base + i + e] = __expf((float)run);
                        kfac[base + i + e] = __expf((float)(total - run));
                    }
                }
                if (lane == 0) blk_out[b0 + k] = before;
            }
            before += in[k];
        }
    }
}

// dlog_g[t] = sum_{i >= t} dL/db_i.  A running sum over the whole sequence would pile up the
// rounding noise of tens of thousands of terms on a result that is local (only pairs within a few
// decay lengths of t matter).  Instead: the part of the sum beyond the end of t's chunk m equals
//     X_m = sum_{j <= end_m < i} e_ij a_ij = < R_m , S_{m+1} >,
// the inner product of the two states that meet at that chunk boundary, which each kernel family
// computes from its states (xb); only the part inside the chunk is summed here.
// dotk (may be null): the states' share of db2.  xb is then the pairs that straddle the whole chunk, and
//     X_m = xb_m + sum_{j in m} dotk_j / p.
// As the terms of db2 and of X_m cancel but for the keys before t, both have to be of one rounding: with X_m from the states and
// db2 from products with them, the difference of the two is in every token of the chunk, and it is what a chunk of 1280 tokens is
// long for (gates of mean -0.5: relative error of dlog_g 1.03e-2 that way, 3.6e-3 this way, as in the attention form).
// db holds q_i . dq_i and db2 k_i . dk_i: dL/db_i = (db[i] - db2[i]) / p.
__device__ __forceinline__ float gate_term(const float* __restrict__ db, const float* __restrict__ db2, float inv_p,
                                           size_t i) {
    return (db[i] - db2[i]) * inv_p;
}

__global__ __launch_bounds__(GT) void k_gate_finish(const float* __restrict__ db, const float* __restrict__ db2, float inv_p,
                                                    const float* __restrict__ xb, int xparts, const float* __restrict__ dotk,
                                                    float* __restrict__ dlog_g, int T, int chunk) {
    __shared__ float part[GT], past[GT / 64];
    const int n = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
    const size_t base = (size_t)bh * T + (size_t)n * chunk;
    const int len = min(chunk, T - n * chunk);
    const int per = (len + GT - 1) / GT;
    const int lo = min(tid * per, len), hi = min(lo + per, len);
    float s = 0.f;
    for (int i = lo; i < hi; ++i) s += gate_term(db, db2, inv_p, base + i);
    part[tid] = s;
    if (dotk != nullptr) {
        float k = 0.f;
        for (int i = lo; i < hi; ++i) k += dotk[base + i];
        for (int off = 32; off > 0; off >>= 1) k += __shfl_xor(k, off);
        if ((tid & 63) == 0) past[tid >> 6] = k * inv_p;
    }
    __syncthreads();
    for (int off = 1; off < GT; off <<= 1) {      // inclusive suffix scan of the per-thread sums
        const float add = tid + off < GT ? part[tid + off] : 0.f;
        __syncthreads();
        part[tid] += add;
        __syncthreads();
    }
    float run = tid + 1 < GT ? part[tid + 1] : 0.f;
    if (dotk != nullptr) run += past[0] + past[1] + past[2] + past[3];
    for (int k = 0; k < xparts; ++k) run += xb[((size_t)bh * gridDim.x + n) * xparts + k];
    for (int i = hi - 1; i >= lo; --i) {
        run += gate_term(db, db2, inv_p, base + i);
        dlog_g[base + i] = run;
    }
}

}  // namespace

// entries per head of the per-chunk arrays: the boundary sums of the backward pass may be kept per
// 128 tokens when the chunk is longer (the attention form)
static size_t chunk_slots(const pa_problem& pr) {
    const size_t a = (size_t)(pr.T / pr.chunk), b = (size_t)((pr.T + 127) / 128);
    return a > b ? a : b;
}
// ... and of xb, which the chunked matrix-core kernels leave in several terms per chunk of theirs
static size_t xb_bytes(const pa_problem& pr) {
    const size_t a = chunk_slots(pr), b = mfma_gate_slots(pr);
    return align_up((size_t)pr.B * pr.H * (a > b ? a : b) * sizeof(float), 256);
}

// blocks of GATE_BLOCK tokens per head: every chunk starts one
static size_t blocks_of(int T, int chunk) { return (size_t)((T + chunk - 1) / chunk) * ((chunk + GATE_BLOCK - 1) / GATE_BLOCK); }
static size_t blk_bytes(const pa_problem& pr) {
    const size_t a = blocks_of(pr.T, pr.chunk), b = blocks_of(pr.T, GATE_BLOCK);      // (b: see gate_prepare)
    return align_up((size_t)pr.B * pr.H * (a > b ? a : b) * sizeof(double), 256);
}

size_t gate_workspace_bytes(const pa_problem& pr, bool backward) {
    if (!pr.gated) return 0;
    const size_t BH = (size_t)pr.B * pr.H;
    const size_t tok = align_up(BH * pr.T * sizeof(float), 256);
    return blk_bytes(pr) + (backward ? 5 : 3) * tok + align_up(BH * chunk_slots(pr) * sizeof(float), 256) + (backward ? xb_bytes(pr) : 0);
}

GateBuf gate_buffers(const pa_problem& pr, bool backward, char* base) {
    GateBuf g;
    if (!pr.gated) return g;
    const size_t BH = (size_t)pr.B * pr.H;
    const size_t tok = align_up(BH * pr.T * sizeof(float), 256);
    g.blk = (double*)base;
    base += blk_bytes(pr);
    g.bl = (float*)base;
    g.qfac = (float*)(base + tok);
    g.kfac = (float*)(base + 2 * tok);
    g.lam = (float*)(base + 3 * tok);
    if (backward) {
        g.db = (float*)(base + 3 * tok + align_up(BH * chunk_slots(pr) * sizeof(float), 256));
        g.db2 = g.db + tok / sizeof(float);
        g.xb = g.db2 + tok / sizeof(float);
    }
    return g;
}

pa_status gate_prepare(const Ctx& c, const float* log_g, int chunk, bool in_blocks) {
    const pa_problem& pr = c.prob;
    if (in_blocks && chunk != pr.T && chunk % GATE_BLOCK != 0) return PA_ERR_UNSUPPORTED;
    const int head_blocks = (int)(in_blocks ? blocks_of(pr.T, GATE_BLOCK) : blocks_of(pr.T, chunk));   // in blocks: block t / GATE_BLOCK of a head
    LaunchScope ls("gate_prep", c.stream);
    hipLaunchKernelGGL(k_gate_prep, dim3((pr.T + chunk - 1) / chunk, pr.B * pr.H), dim3(GT), 0, c.stream, log_g, c.gate.bl, c.gate.blk,
                       c.gate.qfac, c.gate.kfac, c.gate.lam, pr.T, chunk, head_blocks, in_blocks ? 1 : 0);
    return launch_ok() ? PA_OK : PA_ERR_HIP;
}

pa_status gate_gradient(const Ctx& c, float* dlog_g, int fin_chunk, int xparts, const float* dotk) {
    const pa_problem& pr = c.prob;
    // Under the sum normalisation q_i . dq_i is zero in exact arithmetic, yet the term stays: what the
    // device finds there is dO_i . (O_i - rounded O_i), and the k_j . dk_j of the keys after t contain
    // exactly that with the opposite sign, row by row.  Both dot products come from the kernels' float32
    // accumulators: formed from the rounded bf16 outputs they would carry 2^-9 of terms that cancel.
    // (Measured, bf16, decay 0.5 per step: relative L2 error of dlog_g 1.8e-2 without the row term, 9e-3
    // with it from rounded outputs, 3e-3 from the accumulators; no worse at weak decay.)
    LaunchScope ls("gate_finish", c.stream);
    hipLaunchKernelGGL(k_gate_finish, dim3((pr.T + fin_chunk - 1) / fin_chunk, pr.B * pr.H), dim3(GT), 0, c.stream, (const float*)c.gate.db,
                       (const float*)c.gate.db2, 1.f / pr.p, (const float*)c.gate.xb, xparts, dotk, dlog_g, pr.T, fin_chunk);
    return launch_ok() ? PA_OK : PA_ERR_HIP;
}

}  // namespace pa
