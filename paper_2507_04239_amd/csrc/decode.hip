// Single-token decode step of power attention: the recurrent form of arXiv 2507.04239, Sec. 2
// Eq. (6), one iteration per call with the state resident in device memory between calls
// (the constant-cost inference the paper argues for in App. D):
//     S <- g S + phi(k) [v, 1]^T,      y = S^T phi(scale q),      o = y[:v] / y[v].
//
// Embedding as in the generic kernel family: the monomials psi(x)_r = prod_z x[i_z] over the
// non-decreasing multi-indices of Lemma 4.2, with the integer multiplicity m_r on the state only
// (S_r = sum m_r psi(k)_r [v, 1]), read out with the bare psi(q): the product is (q.k)^p.
//
// The state is float32 and caller-owned; one buffer per problem holds
//     S     [B*H][D][v]     the value part
//     gamma [B*H][D]        the normaliser column
//     idx   [D] uchar4, mult [D] float   the multi-index table (built by decode_init)
//     part  [B*H][nblk][v+1]             partial read-outs of the step in flight
// A step reads and writes S and gamma once: it is bound by HBM bandwidth, 8 bytes per state
// element and token.
#include <type_traits>

#include "mfma_common.hpp"

namespace pa {
namespace {

constexpr int DRB = 128;   // state rows per workgroup
constexpr int DMAX = 128;  // largest head size

template <int P>
__device__ __forceinline__ float monomial(const float* __restrict__ x, uchar4 ix) {
    float c = x[ix.x];
    if (P > 1) c *= x[ix.y];
    if (P > 2) c *= x[ix.z];
    if (P > 3) c *= x[ix.w];
    return c;
}

struct DecodeLayout {
    long long D;
    int nblk;
    size_t off_s, off_gam, off_idx, off_mult, off_part, total;
};

DecodeLayout make_decode_layout(const pa_problem& pr) {
    DecodeLayout L;
    L.D = generic_state_rows(pr);
    L.nblk = (int)((L.D + DRB - 1) / DRB);
    const size_t BH = (size_t)pr.B * pr.H;
    size_t off = 0;
    L.off_s = off;    off = align_up(off + BH * (size_t)L.D * pr.v * sizeof(float), 256);
    L.off_gam = off;  off = align_up(off + BH * (size_t)L.D * sizeof(float), 256);
    L.off_idx = off;  off = align_up(off + (size_t)L.D * sizeof(uchar4), 256);
    L.off_mult = off; off = align_up(off + (size_t)L.D * sizeof(float), 256);
    L.off_part = off; off = align_up(off + BH * (size_t)L.nblk * (pr.v + 1) * sizeof(float), 256);
    L.total = off;
    return L;
}

__global__ __launch_bounds__(256) void k_decode_zero(float4* __restrict__ p, size_t n4) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256)
        p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// grid (nblk, B*H): rows [DRB blk, DRB (blk + 1)) of one head's state.  A wave takes one row at
// a time (its lanes the value columns: 256-byte runs), then the block's rows of the normaliser
// column go one per thread.
template <typename T, int P>
__global__ __launch_bounds__(256) void k_decode_step(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ vin,
                                                     const float* __restrict__ log_g, float* __restrict__ S,
                                                     float* __restrict__ gam, const uchar4* __restrict__ idx,
                                                     const float* __restrict__ mult, float* __restrict__ part, long long D,
                                                     int d, int v, float scale) {
    __shared__ float qs[DMAX], ks[DMAX], vs[DMAX];
    __shared__ float red[4][DMAX + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int blk = blockIdx.x, bh = blockIdx.y, nblk = gridDim.x;
    if (tid < d) {
        qs[tid] = scale * io<T>::ld(q + (size_t)bh * d + tid);
        ks[tid] = io<T>::ld(k + (size_t)bh * d + tid);
    }
    if (tid < v) vs[tid] = io<T>::ld(vin + (size_t)bh * v + tid);
    const float g = log_g != nullptr ? __expf(log_g[bh]) : 1.f;
    __syncthreads();

    const long long r_begin = (long long)blk * DRB;
    const long long r_end = r_begin + DRB < D ? r_begin + DRB : D;
    float y0 = 0.f, y1 = 0.f;
    const float v0 = lane < v ? vs[lane] : 0.f, v1 = lane + 64 < v ? vs[lane + 64] : 0.f;
    for (long long r = r_begin + w; r < r_end; r += 4) {
        const uchar4 ix = idx[r];
        const float ck = mult[r] * monomial<P>(ks, ix), cq = monomial<P>(qs, ix);
        float* row = S + ((size_t)bh * D + r) * v;
        if (lane < v) {
            const float s = g * row[lane] + ck * v0;
            row[lane] = s;
            y0 += cq * s;
        }
        if (lane + 64 < v) {
            const float s = g * row[lane + 64] + ck * v1;
            row[lane + 64] = s;
            y1 += cq * s;
        }
    }
    float zp = 0.f;
    for (long long r = r_begin + tid; r < r_end; r += 256) {
        const uchar4 ix = idx[r];
        const float ck = mult[r] * monomial<P>(ks, ix), cq = monomial<P>(qs, ix);
        const float s = g * gam[(size_t)bh * D + r] + ck;
        gam[(size_t)bh * D + r] = s;
        zp += cq * s;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) zp += __shfl_xor(zp, off);
    red[w][lane] = y0;
    red[w][lane + 64] = y1;
    if (lane == 0) red[w][DMAX] = zp;
    __syncthreads();
    if (tid <= v) {
        const int c = tid < v ? tid : DMAX;
        part[((size_t)bh * nblk + blk) * (v + 1) + tid] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
    }
}

// The same for v in {16, 32, 64, 128}: v / 4 lanes share a row, each with four columns (16-byte accesses).  A call for one
// sequence is a chain of memory latencies, so everything a block reads is asked for at its start, up to eight rows per lane
// before the first of them is used: a block's 128 rows are two or three latencies deep (d = 64, one sequence, 12 heads: 6.2 us
// with two rows in flight, 5.2 now; 64 sequences, at the rate of a large copy either way).
template <typename T, int P, int V>
__global__ __launch_bounds__(256) void k_decode_step_vec(const T* __restrict__ q, const T* __restrict__ k,
                                                         const T* __restrict__ vin, const float* __restrict__ log_g,
                                                         float* __restrict__ S, float* __restrict__ gam,
                                                         const uchar4* __restrict__ idx, const float* __restrict__ mult,
                                                         float* __restrict__ part, long long D, int d, float scale) {
    constexpr int LPR = V / 4, RPW = 64 / LPR, RPB = 4 * RPW;   // lanes per row, rows per wave and per block pass
    constexpr int PASSES = DRB / RPB, GP = PASSES < 8 ? PASSES : 8;
    static_assert(DRB % RPB == 0 && PASSES % GP == 0 && GP % 2 == 0 && DRB <= 256, "whole groups of passes");
    __shared__ float qs[DMAX], ks[DMAX];
    __shared__ __attribute__((aligned(16))) float vs[DMAX];
    __shared__ __attribute__((aligned(16))) float red[4][DMAX + 4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int blk = blockIdx.x, bh = blockIdx.y, nblk = gridDim.x;
    const long long r_begin = (long long)blk * DRB;
    const long long r_end = r_begin + DRB < D ? r_begin + DRB : D;
    const int c4 = lane % LPR, rl = w * RPW + lane / LPR;        // column quad, row inside a block pass
    float4 st[GP];
    uchar4 ix[GP];
    float mu[GP];
    auto row_of = [&](int pass) { return r_begin + (long long)pass * RPB + rl; };
    auto fetch = [&](int p0) {
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            const long long r = row_of(p0 + i), rr = r < r_end ? r : r_begin;
            st[i] = *((const float4*)(S + ((size_t)bh * D + rr) * V) + c4);
            ix[i] = idx[rr];
            mu[i] = mult[rr];
        }
    };
    fetch(0);
    const long long rz = r_begin + tid;                          // the row whose normaliser this thread updates
    const bool okz = rz < r_end;
    const uchar4 iz = idx[okz ? rz : r_begin];
    const float mz = mult[okz ? rz : r_begin], gz = gam[(size_t)bh * D + (okz ? rz : r_begin)];
    if (tid < d) {
        qs[tid] = scale * io<T>::ld(q + (size_t)bh * d + tid);
        ks[tid] = io<T>::ld(k + (size_t)bh * d + tid);
    }
    if (tid < V) vs[tid] = io<T>::ld(vin + (size_t)bh * V + tid);
    const float g = log_g != nullptr ? __expf(log_g[bh]) : 1.f;
    __syncthreads();

    const float4 vv = *(const float4*)&vs[4 * c4];
    float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int p0 = 0; p0 < PASSES; p0 += GP) {
        if (p0 > 0) fetch(p0);
#pragma unroll
        for (int i = 0; i < GP; i += 2) {
            const long long ra = row_of(p0 + i), rb = row_of(p0 + i + 1);
            const bool oka = ra < r_end, okb = rb < r_end;
            const float4 sa = st[i], sb = st[i + 1];
            const float cka = mu[i] * monomial<P>(ks, ix[i]), cqa = oka ? monomial<P>(qs, ix[i]) : 0.f;
            const float ckb = mu[i + 1] * monomial<P>(ks, ix[i + 1]), cqb = okb ? monomial<P>(qs, ix[i + 1]) : 0.f;
            const float4 na = make_float4(g * sa.x + cka * vv.x, g * sa.y + cka * vv.y, g * sa.z + cka * vv.z, g * sa.w + cka * vv.w);
            const float4 nb = make_float4(g * sb.x + ckb * vv.x, g * sb.y + ckb * vv.y, g * sb.z + ckb * vv.z, g * sb.w + ckb * vv.w);
            if (oka) *((float4*)(S + ((size_t)bh * D + ra) * V) + c4) = na;
            if (okb) *((float4*)(S + ((size_t)bh * D + rb) * V) + c4) = nb;
            y.x += cqa * na.x + cqb * nb.x;
            y.y += cqa * na.y + cqb * nb.y;
            y.z += cqa * na.z + cqb * nb.z;
            y.w += cqa * na.w + cqb * nb.w;
        }
    }
    float zp = 0.f;
    if (okz) {
        const float ck = mz * monomial<P>(ks, iz), cq = monomial<P>(qs, iz);
        const float s = g * gz + ck;
        gam[(size_t)bh * D + rz] = s;
        zp = cq * s;
    }
    // rows of a wave: lanes LPR apart hold the same columns
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) {
        y.x += __shfl_xor(y.x, off);
        y.y += __shfl_xor(y.y, off);
        y.z += __shfl_xor(y.z, off);
        y.w += __shfl_xor(y.w, off);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) zp += __shfl_xor(zp, off);
    if (lane < LPR) *(float4*)&red[w][4 * lane] = y;
    if (lane == 0) red[w][DMAX] = zp;
    __syncthreads();
    if (tid <= V) {
        const int c = tid < V ? tid : DMAX;
        part[((size_t)bh * nblk + blk) * (V + 1) + tid] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
    }
}

// ---- absorbing a whole prompt ------------------------------------------------------------------------
// S <- (prod of the prompt's gates) S + sum_t (prod of the gates after t) m_r psi(k_t)_r [v_t, 1], i.e. the
// state after stepping through K, V [B*H][Tlen][.] token by token, without producing outputs (those come
// from power_attn_fwd).  One thread owns a state row and every fourth column, holds them in registers
// and walks the tokens, which are staged through LDS 32 at a time; the decay is applied token by
// token (acc <- g_t acc + ...), which needs no running sums of the log-gates.
constexpr int ART = 32;   // tokens per LDS batch
// NQ: column quads per thread (thread xg of a row's four owns the quads xg, xg + 4, ...: 16-byte LDS
// reads); the normaliser column rides with thread 0 of the four.
template <typename T, int P, int NQ, bool GATED>
__global__ __launch_bounds__(256) void k_decode_absorb(const T* __restrict__ K, const T* __restrict__ V,
                                                       const float* __restrict__ log_g, float* __restrict__ S,
                                                       float* __restrict__ gam, const uchar4* __restrict__ idx,
                                                       const float* __restrict__ mult, long long D, int Tlen, int d, int v) {
    __shared__ float ks[ART][DMAX];
    __shared__ __attribute__((aligned(16))) float vs[ART][DMAX];
    __shared__ float gs[ART];
    const int tid = threadIdx.x, xg = tid & 3, bh = blockIdx.y;
    const long long row = (long long)blockIdx.x * 64 + (tid >> 2);
    const bool live = row < D;
    uchar4 ix = make_uchar4(0, 0, 0, 0);
    float m = 0.f;
    if (live) {
        ix = idx[row];
        m = mult[row];
    }
    float* srow = S + ((size_t)bh * D + (live ? row : 0)) * v;
    float* grow = gam + (size_t)bh * D + (live ? row : 0);
    const int nquad = (v + 3) / 4;
    float4 acc[NQ];
    float accz = live && xg == 0 ? *grow : 0.f;
#pragma unroll
    for (int kk = 0; kk < NQ; ++kk) {
        const int x = 4 * (xg + 4 * kk);
        acc[kk] = make_float4(live && x < v ? srow[x] : 0.f, live && x + 1 < v ? srow[x + 1] : 0.f,
                              live && x + 2 < v ? srow[x + 2] : 0.f, live && x + 3 < v ? srow[x + 3] : 0.f);
    }
    const T* Kb = K + (size_t)bh * Tlen * d;
    const T* Vb = V + (size_t)bh * Tlen * v;
    for (int t0 = 0; t0 < Tlen; t0 += ART) {
        const int nt = min(ART, Tlen - t0);
        __syncthreads();
        for (int e = tid; e < nt * d; e += 256) ks[e / d][e % d] = io<T>::ld(Kb + (size_t)t0 * d + e);
        for (int e = tid; e < nt * 4 * nquad; e += 256) {        // columns past v read as zero
            const int j = e / (4 * nquad), x = e % (4 * nquad);
            vs[j][x] = x < v ? io<T>::ld(Vb + (size_t)(t0 + j) * v + x) : 0.f;
        }
        if (GATED && tid < nt) gs[tid] = __expf(log_g[(size_t)bh * Tlen + t0 + tid]);
        __syncthreads();
#pragma unroll 4
        for (int j = 0; j < nt; ++j) {
            const float coef = m * monomial<P>(ks[j], ix);
            const float g = GATED ? gs[j] : 1.f;
            accz = GATED ? g * accz + coef : accz + coef;
#pragma unroll
            for (int kk = 0; kk < NQ; ++kk) {
                if (xg + 4 * kk < nquad) {
                    const float4 y = *(const float4*)&vs[j][4 * (xg + 4 * kk)];
                    if (GATED) {
                        acc[kk].x *= g; acc[kk].y *= g; acc[kk].z *= g; acc[kk].w *= g;
                    }
                    acc[kk].x += coef * y.x; acc[kk].y += coef * y.y; acc[kk].z += coef * y.z; acc[kk].w += coef * y.w;
                }
            }
        }
    }
    if (!live) return;
#pragma unroll
    for (int kk = 0; kk < NQ; ++kk) {
        const int x = 4 * (xg + 4 * kk);
        if (x < v) srow[x] = acc[kk].x;
        if (x + 1 < v) srow[x + 1] = acc[kk].y;
        if (x + 2 < v) srow[x + 2] = acc[kk].z;
        if (x + 3 < v) srow[x + 3] = acc[kk].w;
    }
    if (xg == 0) *grow = accz;
}

// Rows (i, j0 .. j0 + 7) of a p = 2 state from j = i on, token by token in float32 as above, by one wave: lane = column.
// (Kept small: the matrix-core kernel below reaches it only for sums that are not finite, and shares its registers with it.)
template <int HD, bool GATED, bool GAM = true>      // GAM: the normaliser too
__device__ __forceinline__ void absorb_rows(const bf16_t* __restrict__ Kh, const bf16_t* __restrict__ Vh, const float* __restrict__ lgh,
                                            float* __restrict__ Sh, float* __restrict__ gamh, int Tlen, int i, int j0, int lane) {
    using namespace mfma;
    constexpr int NC = (HD + 63) / 64, NR = 8;
    const int col = lane % HD;      // (d = 32: the upper half of the wave repeats the lower one's columns)
    // row of (i, j0); those of j < i are rows of other pairs, read and dropped
    const int row0 = i * HD - i * (i - 1) / 2 + j0 - i;
    float* S0 = Sh + (size_t)row0 * HD + col;
    float* g0 = gamh + row0;
    float acc[NR][NC], accz[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        accz[r] = GAM ? g0[r] : 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[r][c] = S0[r * HD + 64 * c];
    }
#pragma unroll 1
    for (int t = 0; t < Tlen; ++t) {
        const bf16_t* kt = Kh + (size_t)t * HD;
        const float g = GATED ? __expf(lgh[t]) : 1.f, ki = io<bf16_t>::ld(kt + i);
        Frag kj;
        kj.u = *(const uint4*)(kt + j0);
        float v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = io<bf16_t>::ld(Vh + (size_t)t * HD + 64 * c + col);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const float coef = (j0 + r == i ? 1.f : 2.f) * (ki * ((r & 1) ? bf_hi(kj.q[r / 2]) : bf_lo(kj.q[r / 2])));
            accz[r] = GATED ? g * accz[r] + coef : accz[r] + coef;
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[r][c] = (GATED ? g * acc[r][c] : acc[r][c]) + coef * v[c];
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (j0 + r < i) continue;
        if (GAM && lane == 0) g0[r] = accz[r];
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (lane < HD) S0[r * HD + 64 * c] = acc[r][c];
    }
}

// The same for p = 2, bf16 tokens, d = v in {32, 64, 128} on the matrix cores, with nothing rounded below float32.
// The product k_i k_j of two bf16 numbers has at most 16 significant bits, so it is exactly the sum of two bf16 numbers
// (its upper and its lower half), and the two MFMAs that contract the halves with the values form the float32 sum of exact
// products.  With gates the product carries its token's decay to the end of the 64-token tile, is a float32 number like any
// other and takes three parts; the accumulators decay from tile to tile.  The sum over the prompt joins the state, which
// has decayed across the whole prompt, at the end.  The parts of an infinite product, and of any product beside an infinite
// value, are not the product's (inf - inf, 0 inf): a wave that ends with anything but finite sums forms its rows token by token
// instead (absorb_rows), at the vector kernel's speed.
//
// d = 32: a state row is a pair i <= j.  A wave owns the rows of 16 consecutive j (operand row = j) for 2 consecutive i: k_j for 8
// tokens per lane is formed once per 32 tokens and multiplied by two broadcast k_i.  Eight such waves share the staged tokens.
// Tokens are staged feature-major, so that every operand is one 16-byte LDS read.  Blocks on the diagonal also form the pairs
// j < i and drop them.
constexpr int AXT = 64;         // tokens per tile
constexpr int AXP = AXT + 8;    // pitch of a feature's tokens: 16 rows read 16 bytes each from distinct banks
struct AbsorbTile {
    bf16_t k[32][AXP], v[32][AXP];
    float w[AXT];               // decay of each token to the end of the tile
};
constexpr int ABSORB_UNITS = 2 * 3 * 4;     // (j block, i pair) with the pair not beyond the block's last row
template <bool GATED>
__global__ __launch_bounds__(512, GATED ? 5 : 6) void k_decode_absorb_32(const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
                                                                         const float* __restrict__ log_g, float* __restrict__ S,
                                                                         float* __restrict__ gam, long long D, int Tlen) {
    constexpr int HD = 32;
    using namespace mfma;
    constexpr int NV = HD / 16, NP = GATED ? 3 : 2, NI = 2;
    __shared__ __attribute__((aligned(16))) AbsorbTile tiles[2];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r16 = lane & 15, g = lane >> 4;
    const size_t bh = blockIdx.y;
    int unit = 8 * (int)blockIdx.x + w, jb = 0;       // jb has 8 jb + 8 pairs
    while (unit >= 8 * jb + 8) unit -= 8 * jb++ + 8;
    const int j0 = 16 * jb, i0 = NI * unit;
    const bf16_t *Kh = K + bh * Tlen * HD, *Vh = V + bh * Tlen * HD;

    f32x4 acc[NI][NV], accz[NI];
#pragma unroll
    for (int ii = 0; ii < NI; ++ii) {
        accz[ii] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int vb = 0; vb < NV; ++vb) acc[ii][vb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    Frag ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones.v[e] = (__bf16)1.f;

    // thread: token `lane` of the tile, features 8 w .. 8 w + 7 (the first four waves).  Tokens past the end are zeros (log-gate 0).
    Frag kr, vr;
    float lg = 0.f, decay = 1.f;
    auto load = [&](int t0) {
        const int t = t0 + lane;
        const size_t off = (size_t)min(t, Tlen - 1) * HD + 8 * w;
        if (GATED) lg = t < Tlen ? log_g[bh * Tlen + t] : 0.f;
        if (w >= 4) return;
        kr.u = *(const uint4*)(Kh + off);
        vr.u = *(const uint4*)(Vh + off);
        if (t >= Tlen) kr.u = vr.u = make_uint4(0, 0, 0, 0);
    };
    float tile_decay = 1.f;     // across the tile that `store` was last called for
    auto store = [&](AbsorbTile& dst) {
        if (w < 4)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int f = 8 * w + e;
                dst.k[f][lane] = (bf16_t)(((e & 1) ? kr.q[e / 2] >> 16 : kr.q[e / 2]) & 0xffffu);
                dst.v[f][lane] = (bf16_t)(((e & 1) ? vr.q[e / 2] >> 16 : vr.q[e / 2]) & 0xffffu);
            }
        if (GATED) {
            float s = lg;       // sum of the log-gates of this token and those after it in the tile
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const float o = __shfl_down(s, off);
                if (lane + off < 64) s += o;
            }
            tile_decay = expf(__shfl(s, 0));
            const float after = __shfl_down(s, 1);
            if (w == 0) dst.w[lane] = lane < 63 ? expf(after) : 1.f;
        }
    };

    load(0);
    store(tiles[0]);
    float cur_decay = tile_decay;
    __syncthreads();
    int buf = 0;
    for (int t0 = 0; t0 < Tlen; t0 += AXT, buf ^= 1) {
        const bool more = t0 + AXT < Tlen;
        if (more) load(t0 + AXT);
        const AbsorbTile& tl = tiles[buf];
        if (GATED) {
            decay *= cur_decay;
#pragma unroll
            for (int ii = 0; ii < NI; ++ii) {
                accz[ii] *= cur_decay;
#pragma unroll
                for (int vb = 0; vb < NV; ++vb) acc[ii][vb] *= cur_decay;
            }
        }
#pragma unroll
        for (int ks = 0; ks < AXT; ks += 32) {
            Frag f;
            f.u = *(const uint4*)&tl.k[j0 + r16][ks + 8 * g];
            float kj[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) kj[e] = (e & 1) ? bf_hi(f.q[e / 2]) : bf_lo(f.q[e / 2]);
            if (GATED) {
#pragma unroll
                for (int e = 0; e < 8; ++e) kj[e] *= tl.w[ks + 8 * g + e];
            }
            Frag vf[NV];
#pragma unroll
            for (int vb = 0; vb < NV; ++vb) vf[vb].u = *(const uint4*)&tl.v[16 * vb + r16][ks + 8 * g];
#pragma unroll
            for (int ii = 0; ii < NI; ++ii) {
                Frag fi, part[NP];
                fi.u = *(const uint4*)&tl.k[i0 + ii][ks + 8 * g];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    float x0 = kj[e] * bf_lo(fi.q[e / 2]), x1 = kj[e + 1] * bf_hi(fi.q[e / 2]);
#pragma unroll
                    for (int n = 0; n < NP; ++n) {      // the upper 16 bits of both, then what is left
                        const uint32_t u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
                        part[n].q[e / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
                        if (n + 1 < NP) {
                            x0 -= __uint_as_float(u0 & 0xffff0000u);
                            x1 -= __uint_as_float(u1 & 0xffff0000u);
                        }
                    }
                }
#pragma unroll
                for (int n = 0; n < NP; ++n) {
                    accz[ii] = mfma16(part[n].v, ones.v, accz[ii]);
#pragma unroll
                    for (int vb = 0; vb < NV; ++vb) acc[ii][vb] = mfma16(part[n].v, vf[vb].v, acc[ii][vb]);
                }
            }
        }
        if (more) store(tiles[buf ^ 1]);
        cur_decay = tile_decay;
        __syncthreads();
    }
    // acc[ii][vb][r]: i = i0 + ii, j = j0 + 4 g + r, column 16 vb + r16
    auto each_row = [&](auto&& f) {
#pragma unroll
        for (int ii = 0; ii < NI; ++ii)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + ii, j = j0 + 4 * g + r;
                if (j >= i) f(ii, r, bh * D + (size_t)(i * HD - i * (i - 1) / 2 + j - i), i == j ? 1.f : 2.f);
            }
    };
    f32x4 nought4 = {0.f * decay, 0.f, 0.f, 0.f};       // NaN if any sum is infinite or NaN
#pragma unroll
    for (int ii = 0; ii < NI; ++ii) {
        nought4 += 0.f * accz[ii];
#pragma unroll
        for (int vb = 0; vb < NV; ++vb) nought4 += 0.f * acc[ii][vb];
    }
    float nought = nought4[0] + nought4[1] + nought4[2] + nought4[3];
    if (GATED && decay == 0.f)      // a product of gates that has vanished keeps an infinity in the state, a gate of zero does not
        each_row([&](int, int, size_t row, float) {
            nought += 0.f * gam[row];
#pragma unroll
            for (int vb = 0; vb < NV; ++vb) nought += 0.f * S[row * HD + 16 * vb + r16];
        });
    if (!__all(nought == 0.f)) {
#pragma unroll 1
        for (int n = 0; n < 2 * NI; ++n)
            absorb_rows<HD, GATED>(Kh, Vh, GATED ? log_g + bh * Tlen : nullptr, S + bh * D * HD, gam + bh * D, Tlen,
                                   __builtin_amdgcn_readfirstlane(i0) + n / 2, __builtin_amdgcn_readfirstlane(j0) + 8 * (n & 1), lane);
        return;
    }
    each_row([&](int ii, int r, size_t row, float m) {
#pragma unroll
        for (int vb = 0; vb < NV; ++vb) {
            float* dst = S + row * HD + 16 * vb + r16;
            *dst = decay * *dst + m * acc[ii][vb][r];
        }
        if (r16 == 0) gam[row] = decay * gam[row] + m * accz[ii][r];
    });
}

// d = 64 and 128, in larger blocks (32x32x16).  A wave owns 2 R values i by 16 values j of one state and all columns, at most 128
// accumulators: a row block is 2 i x 16 j, so a lane needs k_i of one token per row block and the multiply fetches the token it
// stands at from its 16-lane row by DPP; k_j for its 8 tokens is read once per 16 tokens and serves R row blocks.  Tokens stay
// row-major in LDS, operands along tokens come through the transposing read.
// Bound by the vector instructions beside the MFMAs: a row block and 16 tokens are 4 MFMAs at d = 64 (32 cycles each) and 8
// products in two parts each (4 instructions; subtracting by v_dot2_f32_bf16 instead takes one fewer and 25 % longer: it gets in
// the MFMAs' way).  So the pieces of the next step's products stand between this step's MFMAs, a pair's one MFMA apart, with no
// result read soon after, and a stage's first operands are read before the barrier that ends the stage before it (three buffers).
// The normaliser is k k^T, whose products the matrix cores form exactly from the bf16 tokens: workgroups of their own with
// 32 x 32 blocks of it (a column of ones beside the values is half a column block more MFMAs at d = 64).
// MI355X, 48 heads of 3000 tokens (16x16x32 in the manner of d = 32 -> this): d = 64 142 -> 97 us, gated 220 -> 156;
// d = 128 1020 -> 568, gated 1332 -> 1007; 12 heads, d = 64: 99 -> 44.
template <int HD, int R>
struct AbsorbBlk {
    static constexpr int AU = 2 * R, NC = HD / 32, PER = 16 / AU;
    static constexpr int G = (HD / 16) * (HD / 16 + 1) / 2 * PER / 4;      // workgroups of 4 waves
    static constexpr int NB = HD / 32, NU = NB * (NB + 1) / 2, GN = (NU + 3) / 4;      // normaliser: waves and workgroups
    static constexpr int XF = HD == 64 ? 64 : 32;      // features staged for the products: all, or a workgroup's 16 i and 16 j
    static constexpr int XP = XF + 16, YP = HD + 16;   // pitches: 8 rows x 32 bytes of a transposing read on distinct banks
    static constexpr int ST = 64;                      // tokens per stage
    static_assert(HD == 64 || PER % 4 == 0, "the waves of a workgroup share their 16 i and 16 j at d = 128");
};
template <int HD, int R>
struct AbsorbSmem {
    bf16_t x[3][AbsorbBlk<HD, R>::ST][AbsorbBlk<HD, R>::XP];
    bf16_t y[3][AbsorbBlk<HD, R>::ST][AbsorbBlk<HD, R>::YP];
    float w[3][AbsorbBlk<HD, R>::ST];      // gates: each token's decay to the end of its stage
    float td[3];                           // ... and across the stage
};
struct AbsorbArgs {
    const bf16_t *K, *V;
    const float* log_g;
    float *S, *gam;
    long long D;
    int T, heads;
};
// x = the sum of bf16 numbers, the upper 16 bits first (two x at a time), what is left stays in x
__device__ __forceinline__ uint32_t upper_halves(const float (&x)[2]) {
    return __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u);
}
__device__ __forceinline__ uint32_t split_pair(float (&x)[2]) {
#pragma clang fp contract(off)      // (a product that is used twice cannot take its factor by DPP)
    const uint32_t u = upper_halves(x);
    x[0] -= __uint_as_float(__float_as_uint(x[0]) & 0xffff0000u);
    x[1] -= __uint_as_float(__float_as_uint(x[1]) & 0xffff0000u);
    return u;
}

template <int N>
__device__ __forceinline__ float row_shl(float x) {     // the value of the lane N further on in this lane's 16-lane row, 0 past its end
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x100 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_value(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

template <int HD, int R_, bool GATED, bool NORM>
__device__ __forceinline__ void absorb_body(const AbsorbArgs& A, AbsorbSmem<HD, R_>& sm, size_t bh, int g) {
    using namespace mfma;
    using C = AbsorbBlk<HD, R_>;
    constexpr int R = NORM ? 1 : R_, NC = NORM ? 1 : C::NC, NP = GATED ? 3 : 2, ST = C::ST;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int hl = lane >> 5, row16 = (lane >> 4) & 1, i16 = lane & 15, T = A.T;
    int J = 0, a0 = 0, nr = 0, nc = 0;      // 16 j from 16 J, AU i from a0; normaliser: rows 32 nr .., columns 32 nc ..
    bool idle = false;
    if (NORM) {
        int u = 4 * g + w;
        idle = u >= C::NU;
        for (u = min(u, C::NU - 1); u > nc; u -= ++nc) {}
        nr = u;
    } else {
        int u = 4 * g + w;
        for (; u >= C::PER * (J + 1); ++J) u -= C::PER * (J + 1);
        a0 = C::AU * u;
    }
    const int I = a0 >> 4;                  // (d = 128: the same for all four waves)
    const bf16_t *Kh = A.K + bh * T * HD, *Vh = A.V + bh * T * HD;
    const bf16_t* Yh = NORM ? Kh : Vh;
    const float* lgh = GATED ? A.log_g + bh * T : nullptr;
    float* Sh = A.S + bh * A.D * HD;
    float* gh = A.gam + bh * A.D;

    // staging: 16-byte pieces of rows.  Tokens past the end are zeros (log-gate 0).
    constexpr int NY = HD / 32, NX = NORM ? 0 : C::XF / 32;
    uint4 xr[NX > 0 ? NX : 1], yr[NY];
    float lg = 0.f, decay = 1.f;
    auto load = [&](int t0) {
#pragma unroll
        for (int q = 0; q < NY; ++q) {
            const int id = tid + 256 * q, row = t0 + id / (HD / 8);
            yr[q] = *(const uint4*)(Yh + (size_t)min(row, T - 1) * HD + 8 * (id % (HD / 8)));
        }
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int id = tid + 256 * q, c8 = id % (C::XF / 8), row = t0 + id / (C::XF / 8);
            const int f = HD == 64 ? 8 * c8 : (c8 < 2 ? 16 * I + 8 * c8 : 16 * J + 8 * (c8 - 2));
            xr[q] = *(const uint4*)(Kh + (size_t)min(row, T - 1) * HD + f);
        }
        if (GATED && tid < ST) lg = t0 + tid < T ? lgh[t0 + tid] : 0.f;
    };
    auto only = [](const uint4& u, bool yes) { return make_uint4(yes ? u.x : 0u, yes ? u.y : 0u, yes ? u.z : 0u, yes ? u.w : 0u); };
    auto put = [&](int buf, int t0) {
#pragma unroll
        for (int q = 0; q < NY; ++q) {
            const int id = tid + 256 * q, row = id / (HD / 8);
            *(uint4*)&sm.y[buf][row][8 * (id % (HD / 8))] = only(yr[q], t0 + row < T);
        }
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int id = tid + 256 * q, row = id / (C::XF / 8);
            *(uint4*)&sm.x[buf][row][8 * (id % (C::XF / 8))] = only(xr[q], t0 + row < T);
        }
        if (GATED && w == 0) {
            // sums of the log-gates from each token on, in its row of 16 lanes, then the rows after it
            float sum = lg;
            sum += row_shl<1>(sum);
            sum += row_shl<2>(sum);
            sum += row_shl<4>(sum);
            sum += row_shl<8>(sum);
            const float t1 = lane_value(sum, 16), t2 = lane_value(sum, 32), t3 = lane_value(sum, 48);
            const float rest = lane < 16 ? t1 + (t2 + t3) : lane < 32 ? t2 + t3 : lane < 48 ? t3 : 0.f;
            sm.w[buf][lane] = expf(row_shl<1>(sum) + rest);
            if (lane == 0) sm.td[buf] = expf(sum + rest);
        }
    };

    f32x16 acc[R][NC];
#pragma unroll
    for (int rb = 0; rb < R; ++rb)
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) acc[rb][cb] = zero16();
    float big = 0.f;            // normaliser: the largest magnitude that goes into a product

    // k-slots of a 16-token step: half hl has tokens 4 hl + 0 .. 3 and 8 + 4 hl + 0 .. 3
    const uint32_t sel = row16 ? 0x07060c0cu : 0x05040c0cu;      // the upper or lower bf16 of a dword as float32
    const int xa_tok = 16 * (i16 >> 3) + 8 * ((i16 >> 2) & 1) + 4 * hl + (i16 & 3);
    const int tr_tok = 4 * hl + (i16 >> 2), tr_col = 16 * row16 + 4 * (i16 & 3);
    const int xa_col = HD == 64 ? a0 : (a0 & 15), xb_col = (HD == 64 ? 16 * J : 16) + 4 * (i16 & 3);
    struct Ops {            // LDS operands of one step; the next step's are read before this one's are used
        Frag v[NC], xb;     // (normaliser: xb holds the rows)
        float4 w0, w1;
    };
    auto read_ops = [&](Ops& o, int buf, int ks) {
        const int t = 16 * ks + tr_tok;
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) o.v[cb] = tr_frag(&sm.y[buf][t][32 * (nc + cb) + tr_col], C::YP);
        o.xb = NORM ? tr_frag(&sm.y[buf][t][32 * nr + tr_col], C::YP) : tr_frag(&sm.x[buf][t][xb_col], C::XP);
        if (GATED) {
            o.w0 = *(const float4*)&sm.w[buf][16 * ks + 4 * hl];
            o.w1 = *(const float4*)&sm.w[buf][16 * ks + 8 + 4 * hl];
        }
    };
    using XaRaw = std::conditional_t<R == 4, uint4, std::conditional_t<R == 2, uint2, uint32_t>>;
    auto read_xa = [&](int buf, int kp) { return *(const XaRaw*)&sm.x[buf][32 * kp + xa_tok][xa_col]; };
    auto elem = [&](const Ops& c, int j) {      // k_j (normaliser: k_i) of the step in c, token j, with its decay
        float x = (j & 1) ? bf_hi(c.xb.q[j / 2]) : bf_lo(c.xb.q[j / 2]);
        if (GATED) x *= j == 0 ? c.w0.x : j == 1 ? c.w0.y : j == 2 ? c.w0.z : j == 3 ? c.w0.w : j == 4 ? c.w1.x : j == 5 ? c.w1.y : j == 6 ? c.w1.z : c.w1.w;
        return x;
    };
    // Stages n and n + 1 are in LDS while n is worked on, n + 2 goes there during it and n + 3 is on its way in registers
    // (stages past the end are zeros: no branches)
    load(0);
    put(0, 0);
    load(ST);
    put(1, ST);
    load(2 * ST);
    lds_barrier();
    int buf = 0, nbuf = 1, pbuf = 2;
    auto ahead = [&](int t0) {
        put(pbuf, t0 + 2 * ST);
        load(t0 + 3 * ST);
    };
    auto turn = [&] {
        lds_barrier();
        const int b = buf;
        buf = nbuf;
        nbuf = pbuf;
        pbuf = b;
    };
    auto scale = [&](int rb, float f) {
#pragma unroll
        for (int cb = 0; cb < NC; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[rb][cb][i] *= f;
    };
    if constexpr (NORM) {
        for (int t0 = 0; t0 < T; t0 += ST) {
            ahead(t0);
            if (GATED) {
                const float f = sm.td[buf];
                decay *= f;
                scale(0, f);
            }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                Ops c;
                read_ops(c, buf, ks);
                Frag part[NP];
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    float x[2] = {elem(c, j), elem(c, j + 1)};
                    big = fmaxf(fmaxf(big, fmaxf(fabsf(x[0]), fabsf(x[1]))), fmaxf(fabsf(bf_lo(c.v[0].q[j / 2])), fabsf(bf_hi(c.v[0].q[j / 2]))));
                    if (GATED) {
#pragma unroll
                        for (int n = 0; n + 1 < NP; ++n) part[n].q[j / 2] = split_pair(x);
                        part[NP - 1].q[j / 2] = upper_halves(x);
                    }
                }
                if (GATED) {
#pragma unroll
                    for (int n = 0; n < NP; ++n) acc[0][0] = mfma32(part[n].v, c.v[0].v, acc[0][0]);
                } else {
                    acc[0][0] = mfma32(c.xb.v, c.v[0].v, acc[0][0]);
                }
            }
            turn();
        }
    } else {
        constexpr int AHEAD = R == 1 ? 2 : 1, NO = 2 * AHEAD;       // steps that operands are read ahead of their products
        Ops o[NO];
        XaRaw xw[2];
        Frag part[2][NP];
        float xb[8], xa[2], x[4][2];
        // Step u (taken modulo a stage's 4 R) in small pieces: its factors k_i, the products 2 p and 2 p + 1, and their parts
        auto factor = [&](int u) {
            const XaRaw& raw = xw[(u / R & 3) >> 1];
            const int rb = u % R;
            uint32_t d;
            if constexpr (R == 4) d = rb == 0 ? raw.x : rb == 1 ? raw.y : rb == 2 ? raw.z : raw.w;
            else if constexpr (R == 2) d = rb == 0 ? raw.x : raw.y;
            else d = raw;
            xa[u & 1] = __uint_as_float(__builtin_amdgcn_perm(d, 0u, sel));
        };
        auto product = [&](int u, int p) {
            const int ks = u / R & 3;
#pragma unroll
            for (int j = 2 * p; j < 2 * p + 2; ++j) {
                if (u % R == 0) xb[j] = elem(o[ks % NO], j);
                float m;
                switch (8 * (ks & 1) + j) {
#define PA_LANE(L_) case L_: m = row_lane<L_>(xa[u & 1]); break;
                    PA_LANE(0) PA_LANE(1) PA_LANE(2) PA_LANE(3) PA_LANE(4) PA_LANE(5) PA_LANE(6) PA_LANE(7)
                    PA_LANE(8) PA_LANE(9) PA_LANE(10) PA_LANE(11) PA_LANE(12) PA_LANE(13) PA_LANE(14)
#undef PA_LANE
                    default: m = row_lane<15>(xa[u & 1]);
                }
                x[p][j & 1] = m * xb[j];
            }
        };
        auto piece = [&](int u, int p, int n) {
            part[u & 1][n].q[p] = n + 1 < NP ? split_pair(x[p]) : upper_halves(x[p]);
        };
#pragma unroll
        for (int n = 0; n < AHEAD; ++n) read_ops(o[n], 0, n);
        xw[0] = read_xa(0, 0);
        factor(0);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            product(0, p);
#pragma unroll
            for (int n = 0; n < NP; ++n) piece(0, p, n);
        }
        factor(1);
        product(1, 0);
        for (int t0 = 0; t0 < T; t0 += ST) {
            float f = 1.f;
            if (GATED) {
                f = sm.td[buf];
                decay *= f;
                scale(0, f);
            }
            // (after the last stage the next one's operands are read from what stands there, and dropped)
#pragma unroll
            for (int i = 0; i < 4 * R; ++i) {
                const int ks = i / R, rb = i % R;
                if (rb == 0) {
                    read_ops(o[(ks + AHEAD) % NO], ks + AHEAD < 4 ? buf : nbuf, (ks + AHEAD) & 3);
                    if (ks == 0) xw[1] = read_xa(buf, 1);
                    if (ks == 2) xw[0] = read_xa(nbuf, 0);
                    if (ks == 1) ahead(t0);
                }
                // Between this step's MFMAs the pieces of the next one, a pair's one MFMA apart: none waits for another's result.
                // Pair p's first part comes with MFMA at(p) of the step before its own, its product one MFMA sooner.
                constexpr int NM = NP * NC;
                auto at = [](int p) { return p * NM / 4; };
#pragma unroll
                for (int n = 0; n < NM; ++n) {
                    acc[rb][n % NC] = mfma32(part[i & 1][n / NC].v, o[ks % NO].v[n % NC].v, acc[rb][n % NC]);
                    if (n == NM - 2) factor(i + 2);
#pragma unroll
                    for (int u = i; u < i + 3; ++u)
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const int rel = n + (i + 1 - u) * NM - at(p);
                            if (rel == -1) product(u, p);
                            if (rel >= 0 && rel < NP) piece(u, p, rel);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (GATED && ks == 0 && rb + 1 < R) scale(rb + 1, f);
            }
            turn();
        }
    }
    if (idle) return;

    float nought = 0.f * decay;         // NaN if any sum is infinite or NaN
#pragma unroll
    for (int rb = 0; rb < R; ++rb)
#pragma unroll
        for (int cb = 0; cb < NC; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) nought += 0.f * acc[rb][cb][i];
    if constexpr (NORM) {
        // element 4 q + r of a lane: row i = 32 nr + 8 q + 4 hl + r, column j = 32 nc + (lane & 31)
        const int j = 32 * nc + (lane & 31);
        float old[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int i = min(32 * nr + 8 * (e >> 2) + 4 * hl + (e & 3), j);
            old[e] = gh[i * HD - i * (i - 1) / 2 + j - i];
            if (GATED && decay == 0.f) nought += 0.f * old[e];      // (a product of gates that has vanished keeps an infinity, a gate of zero does not)
        }
        // Products beyond float32 are infinite one by one, also where the matrix cores would add them to something finite
        const bool plain = __all(nought == 0.f && big < 0x1p63f);
        if (!plain) {
#pragma unroll 1
            for (int t = 0; t < T; ++t) {
                const float gt = GATED ? __expf(lgh[t]) : 1.f, kj = io<bf16_t>::ld(Kh + (size_t)t * HD + j);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int i = min(32 * nr + 8 * (e >> 2) + 4 * hl + (e & 3), j);
                    const float coef = (i == j ? 1.f : 2.f) * (io<bf16_t>::ld(Kh + (size_t)t * HD + i) * kj);
                    old[e] = GATED ? gt * old[e] + coef : old[e] + coef;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int i = 32 * nr + 8 * (e >> 2) + 4 * hl + (e & 3);
            if (i <= j) gh[i * HD - i * (i - 1) / 2 + j - i] = plain ? decay * old[e] + (i == j ? 1.f : 2.f) * acc[0][0][e] : old[e];
        }
    } else {
        // element 4 q + r of row block rb: i = a0 + 2 rb + (q >> 1), j = 16 J + 8 (q & 1) + 4 hl + r, column 32 cb + (lane & 31)
        auto row_of = [&](int rb, int e, int& i, int& j) {
            i = a0 + 2 * rb + (e >> 3);
            j = 16 * J + 8 * ((e >> 2) & 1) + 4 * hl + (e & 3);
            const int jj = max(i, j);
            return (size_t)(i * HD - i * (i - 1) / 2 + jj - i) * HD + (lane & 31);
        };
        if (GATED && decay == 0.f)
#pragma unroll 1
            for (int rb = 0; rb < R; ++rb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
#pragma unroll
                    for (int cb = 0; cb < NC; ++cb) {
                        int i, j;
                        nought += 0.f * Sh[row_of(rb, e, i, j) + 32 * cb];
                    }
        if (!__all(nought == 0.f)) {
#pragma unroll 1
            for (int n = 0; n < 2 * C::AU; ++n)
                absorb_rows<HD, GATED, false>(Kh, Vh, lgh, Sh, gh, T, __builtin_amdgcn_readfirstlane(a0) + n / 2,
                                              __builtin_amdgcn_readfirstlane(16 * J) + 8 * (n & 1), lane);
            return;
        }
#pragma unroll
        for (int rb = 0; rb < R; ++rb)
#pragma unroll
            for (int cb = 0; cb < NC; ++cb) {
                float old[16];
                int i, j;
#pragma unroll
                for (int e = 0; e < 16; ++e) old[e] = Sh[row_of(rb, e, i, j) + 32 * cb];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float* dst = Sh + row_of(rb, e, i, j) + 32 * cb;
                    if (j >= i) *dst = decay * old[e] + (i == j ? 1.f : 2.f) * acc[rb][cb][e];
                }
            }
    }
}

template <int HD, int R, bool GATED>
__global__ __launch_bounds__(256, 2) void k_decode_absorb_blk(AbsorbArgs A) {
    using C = AbsorbBlk<HD, R>;
    __shared__ __attribute__((aligned(16))) AbsorbSmem<HD, R> sm;
    // (the normaliser's workgroups, the shortest, after all others)
    const int first = (int)mfma::xcd_grid(A.heads * C::G);
    if ((int)blockIdx.x < first) {
        const int item = mfma::xcd_item(A.heads * C::G, blockIdx.x);
        if (item >= 0) absorb_body<HD, R, GATED, false>(A, sm, item / C::G, item % C::G);
    } else {
        const int item = mfma::xcd_item(A.heads * C::GN, blockIdx.x - first);
        if (item >= 0) absorb_body<HD, R, GATED, true>(A, sm, item / C::GN, item % C::GN);
    }
}

template <int HD, int R, bool GATED>
bool launch_absorb_blk(const AbsorbArgs& a, hipStream_t s) {
    using C = AbsorbBlk<HD, R>;
    LaunchScope ls("decode_absorb", s);
    const dim3 grid(mfma::xcd_grid(a.heads * C::G) + mfma::xcd_grid(a.heads * C::GN));
    hipLaunchKernelGGL((k_decode_absorb_blk<HD, R, GATED>), grid, dim3(256), 0, s, a);
    return launch_ok();
}
// Large blocks form fewest operands per MFMA, small ones spread few states over the chip.  d = 64: R = 1 while all its workgroups
// run at once, two to a CU (3000 tokens, R = 1 and 4: 12 heads 44 and 83 us, 24 heads 65 and 86, 48 heads 122 and 97); R = 2 is
// between them or behind everywhere.  d = 128: R = 2 above one workgroup of R = 1 per CU (3000 tokens, R = 1 and 2: 1 head 51 and
// 77 us, 12 heads 184 and 158, 96 heads 1301 and 1125), with gates R = 1 throughout: R = 2 has no registers left for a second
// wave per SIMD (48 heads 1007 and 1030 us, 192 heads of 1000 tokens 1504 and 1664).
bool absorb_blk(const AbsorbArgs& a, int d, hipStream_t s) {
    const bool gated = a.log_g != nullptr;
    if (d == 64) {
        if (a.heads * AbsorbBlk<64, 1>::G <= 512) return gated ? launch_absorb_blk<64, 1, true>(a, s) : launch_absorb_blk<64, 1, false>(a, s);
        return gated ? launch_absorb_blk<64, 4, true>(a, s) : launch_absorb_blk<64, 4, false>(a, s);
    }
    if (gated) return launch_absorb_blk<128, 1, true>(a, s);
    return a.heads * AbsorbBlk<128, 1>::G <= 256 ? launch_absorb_blk<128, 1, false>(a, s) : launch_absorb_blk<128, 2, false>(a, s);
}

template <bool GATED>
bool launch_absorb_32(const AbsorbArgs& a, hipStream_t s) {
    LaunchScope ls("decode_absorb", s);
    hipLaunchKernelGGL((k_decode_absorb_32<GATED>), dim3(ABSORB_UNITS / 8, a.heads), dim3(512), 0, s, a.K, a.V, a.log_g, a.S, a.gam, a.D, a.T);
    return launch_ok();
}
bool absorb_mfma_applies(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.p == 2 && pr.d == pr.v && (pr.d == 32 || pr.d == 64 || pr.d == 128);
}
bool absorb_mfma(const pa_problem& pr, const DecodeLayout& L, const void* K, const void* V, const float* log_g, char* st,
                 hipStream_t s) {
    const AbsorbArgs a{(const bf16_t*)K, (const bf16_t*)V, log_g, (float*)(st + L.off_s), (float*)(st + L.off_gam), L.D, pr.T, pr.B * pr.H};
    if (pr.d != 32) return absorb_blk(a, pr.d, s);
    return log_g != nullptr ? launch_absorb_32<true>(a, s) : launch_absorb_32<false>(a, s);
}

// grid B*H: sums the blocks' partial read-outs, divides, stores
template <typename T>
__global__ __launch_bounds__(256) void k_decode_finish(const float* __restrict__ part, int nblk, T* __restrict__ o,
                                                       float* __restrict__ z, int v, int normalize) {
    __shared__ float zs;
    const int bh = blockIdx.x, tid = threadIdx.x;
    // (the parts of 16 blocks at a time on their way: one by one, 17 blocks were 17 latencies, 6.3 us; 2.5 now)
    float acc = 0.f;
    if (tid <= v) {
        const float* src = part + (size_t)bh * nblk * (v + 1) + tid;
        for (int b0 = 0; b0 < nblk; b0 += 16) {
            float x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = src[(size_t)min(b0 + i, nblk - 1) * (v + 1)];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (b0 + i < nblk) acc += x[i];
        }
    }
    if (tid == v) zs = acc;
    __syncthreads();
    const float zz = zs;
    if (tid < v) {
        const float inv = normalize ? (zz != 0.f ? 1.f / zz : 0.f) : 1.f;
        io<T>::st(o + (size_t)bh * v + tid, acc * inv);
    }
    if (tid == v && z != nullptr) z[bh] = zz;
}

pa_status decode_supported(const pa_problem& pr) {
    if (pr.p < 1 || pr.p > 4 || pr.d > DMAX || pr.v > DMAX) return PA_ERR_UNSUPPORTED;
    if ((size_t)pr.B * pr.H > 65535u) return PA_ERR_UNSUPPORTED;
    return PA_OK;
}

template <typename T, int P>
bool launch_step(const pa_problem& pr, const DecodeLayout& L, const void* q, const void* k, const void* v, const float* log_g,
                 char* st, void* o, float* z, hipStream_t s) {
    const int BH = pr.B * pr.H;
    {
        LaunchScope ls("decode_step", s);
#define PA_VEC(VV)                                                                                                          \
    if (pr.v == VV)                                                                                                         \
        hipLaunchKernelGGL((k_decode_step_vec<T, P, VV>), dim3(L.nblk, BH), dim3(256), 0, s, (const T*)q, (const T*)k,      \
                           (const T*)v, log_g, (float*)(st + L.off_s), (float*)(st + L.off_gam),                            \
                           (const uchar4*)(st + L.off_idx), (const float*)(st + L.off_mult), (float*)(st + L.off_part), L.D, \
                           pr.d, pr.scale);                                                                                 \
    else
        PA_VEC(16) PA_VEC(32) PA_VEC(64) PA_VEC(128)
#undef PA_VEC
        hipLaunchKernelGGL((k_decode_step<T, P>), dim3(L.nblk, BH), dim3(256), 0, s, (const T*)q, (const T*)k, (const T*)v, log_g,
                           (float*)(st + L.off_s), (float*)(st + L.off_gam), (const uchar4*)(st + L.off_idx),
                           (const float*)(st + L.off_mult), (float*)(st + L.off_part), L.D, pr.d, pr.v, pr.scale);
        if (!launch_ok()) return false;
    }
    LaunchScope ls("decode_finish", s);
    hipLaunchKernelGGL((k_decode_finish<T>), dim3(BH), dim3(256), 0, s, (const float*)(st + L.off_part), L.nblk, (T*)o, z, pr.v,
                       pr.normalize);
    return launch_ok();
}

template <typename T>
bool launch_step_p(const pa_problem& pr, const DecodeLayout& L, const void* q, const void* k, const void* v, const float* log_g,
                   char* st, void* o, float* z, hipStream_t s) {
    switch (pr.p) {
        case 1: return launch_step<T, 1>(pr, L, q, k, v, log_g, st, o, z, s);
        case 2: return launch_step<T, 2>(pr, L, q, k, v, log_g, st, o, z, s);
        case 3: return launch_step<T, 3>(pr, L, q, k, v, log_g, st, o, z, s);
        default: return launch_step<T, 4>(pr, L, q, k, v, log_g, st, o, z, s);
    }
}

template <typename T, int P>
bool launch_absorb_kx(const pa_problem& pr, const DecodeLayout& L, const void* K, const void* V, const float* log_g, char* st,
                      hipStream_t s) {
    const int nq = ((pr.v + 3) / 4 + 3) / 4;      // column quads per thread
    const dim3 grid((unsigned)((L.D + 63) / 64), pr.B * pr.H);
    LaunchScope ls("decode_absorb", s);
#define PA_GO(NQ, G)                                                                                                    \
    hipLaunchKernelGGL((k_decode_absorb<T, P, NQ, G>), grid, dim3(256), 0, s, (const T*)K, (const T*)V, log_g,           \
                       (float*)(st + L.off_s), (float*)(st + L.off_gam), (const uchar4*)(st + L.off_idx),                \
                       (const float*)(st + L.off_mult), L.D, pr.T, pr.d, pr.v)
    if (log_g != nullptr) {
        if (nq <= 1) PA_GO(1, true);
        else if (nq <= 2) PA_GO(2, true);
        else if (nq <= 4) PA_GO(4, true);
        else PA_GO(8, true);
    } else {
        if (nq <= 1) PA_GO(1, false);
        else if (nq <= 2) PA_GO(2, false);
        else if (nq <= 4) PA_GO(4, false);
        else PA_GO(8, false);
    }
#undef PA_GO
    return launch_ok();
}

template <typename T>
bool launch_absorb_p(const pa_problem& pr, const DecodeLayout& L, const void* K, const void* V, const float* log_g, char* st,
                     hipStream_t s) {
    switch (pr.p) {
        case 1: return launch_absorb_kx<T, 1>(pr, L, K, V, log_g, st, s);
        case 2: return launch_absorb_kx<T, 2>(pr, L, K, V, log_g, st, s);
        case 3: return launch_absorb_kx<T, 3>(pr, L, K, V, log_g, st, s);
        default: return launch_absorb_kx<T, 4>(pr, L, K, V, log_g, st, s);
    }
}

}  // namespace

size_t decode_absorb_workspace_bytes(const pa_problem& pr) {
    return decode_supported(pr) == PA_OK ? mfma_absorb_workspace_bytes(pr) : 0;
}

// With a workspace, and where the matrix-core scan applies, the prompt goes through that (the sums are then rounded to bf16
// once, like the chunk states of the forward pass).  The exact matrix-core kernel runs every other bf16, p = 2 prompt.  At
// d = 64 the scan is the faster one for long prompts of few heads (12 heads of 32768 tokens: 148 us against 376; 12 of 3072:
// 34 against 41) and the exact kernel for short ones and many heads (48 of 512: 29 against 38; 48 of 3072: 95 against 98), but which
// of the two rounds its sums is the caller's choice, made with the workspace, so the line does not follow the time.  The rest takes the float32 kernel on the
// vector ALUs.
pa_status decode_absorb(const pa_problem& pr, const void* K, const void* V, const float* log_g, void* state, void* ws,
                        size_t ws_bytes, hipStream_t s) {
    pa_status st = decode_supported(pr);
    if (st != PA_OK) return st;
    const DecodeLayout L = make_decode_layout(pr);
    if (ws != nullptr && mfma_absorb_supported(pr) && ws_bytes >= mfma_absorb_workspace_bytes(pr))
        return mfma_absorb(pr, K, V, log_g, (char*)ws, s, (float*)((char*)state + L.off_s), (float*)((char*)state + L.off_gam),
                           (int)L.D);
    if (absorb_mfma_applies(pr)) return absorb_mfma(pr, L, K, V, log_g, (char*)state, s) ? PA_OK : PA_ERR_HIP;
    const bool ok = pr.dtype == PA_DTYPE_F32 ? launch_absorb_p<float>(pr, L, K, V, log_g, (char*)state, s)
                                             : launch_absorb_p<bf16_t>(pr, L, K, V, log_g, (char*)state, s);
    return ok ? PA_OK : PA_ERR_HIP;
}

size_t decode_state_bytes(const pa_problem& pr) { return decode_supported(pr) == PA_OK ? make_decode_layout(pr).total : 0; }

pa_status decode_init(const pa_problem& pr, void* state, hipStream_t s) {
    pa_status st = decode_supported(pr);
    if (st != PA_OK) return st;
    const DecodeLayout L = make_decode_layout(pr);
    {
        // a kernel, not a memset: the call may be recorded into a graph
        LaunchScope ls("decode_zero", s);
        const size_t n4 = L.off_idx / sizeof(float4);     // S and gamma, both padded to 256 bytes
        hipLaunchKernelGGL(k_decode_zero, dim3(1024), dim3(256), 0, s, (float4*)state, n4);
        if (!launch_ok()) return PA_ERR_HIP;
    }
    char* base = (char*)state;
    return build_monomial_table(s, pr.d, pr.p, L.D, base + L.off_idx, (float*)(base + L.off_mult)) ? PA_OK : PA_ERR_HIP;
}

pa_status decode_step(const pa_problem& pr, const void* q, const void* k, const void* v, const float* log_g, void* state, void* o,
                      float* z, hipStream_t s) {
    pa_status st = decode_supported(pr);
    if (st != PA_OK) return st;
    const DecodeLayout L = make_decode_layout(pr);
    const bool ok = pr.dtype == PA_DTYPE_F32 ? launch_step_p<float>(pr, L, q, k, v, log_g, (char*)state, o, z, s)
                                             : launch_step_p<bf16_t>(pr, L, q, k, v, log_g, (char*)state, o, z, s);
    return ok ? PA_OK : PA_ERR_HIP;
}

}  // namespace pa
