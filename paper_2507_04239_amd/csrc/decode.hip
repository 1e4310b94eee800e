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
template <int HD, bool GATED>
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
        accz[r] = g0[r];
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
        if (lane == 0) g0[r] = accz[r];
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
// has decayed across the whole prompt, at the end.
//
// A state row is a pair i <= j.  A wave owns the rows of 16 consecutive j (operand row = j) for 2 consecutive i: k_j for 8
// tokens per lane is formed once per 32 tokens and multiplied by two broadcast k_i.  Eight such waves share the staged tokens
// (four waves of 4 i each take 169 us at the size below: too few waves to cover the LDS and MFMA latency).  Tokens are staged feature-major, so
// that every operand is one 16-byte LDS read.  Blocks on the diagonal also form the pairs j < i and drop them (23 % more
// products at d = 64).  The parts of an infinite product, and of any product beside an infinite value, are not the product's
// (inf - inf, 0 inf): a wave that ends with anything but finite sums forms its rows token by token instead (absorb_rows), at
// the vector kernel's speed.  The vector ALU (4 operations per product and lane) and the matrix pipe are loaded
// about equally, each less than half of the time; the rest is the chain barrier, LDS read, product, MFMA of a tile.
// MI355X, B4 H12 T3000 d64: 2160 us on the vector ALUs (k_decode_absorb, one thread per row and 4 columns) -> 156 us.
constexpr int AXT = 64;         // tokens per tile
constexpr int AXP = AXT + 8;    // pitch of a feature's tokens: 16 rows read 16 bytes each from distinct banks
template <int HD>
struct AbsorbTile {
    bf16_t k[HD][AXP], v[HD][AXP];
    float w[AXT];               // decay of each token to the end of the tile
};
// the units of a head: (j block, i pair) with the pair not beyond the block's last row
template <int HD>
constexpr int absorb_units() {
    return (HD / 16) * (HD / 16 + 1) * 4;
}
template <int HD, bool GATED>
__global__ __launch_bounds__(512, HD == 128 ? 2 : HD == 32 ? (GATED ? 5 : 6) : 4) void k_decode_absorb_mfma(const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
                                                               const float* __restrict__ log_g, float* __restrict__ S,
                                                               float* __restrict__ gam, long long D, int Tlen) {
    using namespace mfma;
    constexpr int NV = HD / 16, NP = GATED ? 3 : 2, NI = 2;
    constexpr int NPC = (HD + 63) / 64;     // pieces of 8 features per thread and operand (d = 32: of the first four waves)
    extern __shared__ __attribute__((aligned(16))) unsigned char absorb_smem[];
    AbsorbTile<HD>* tiles = reinterpret_cast<AbsorbTile<HD>*>(absorb_smem);      // [2]
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

    // thread: token `lane` of the tile, features 8 (NPC w + c) .. + 7.  Tokens past the end are zeros (log-gate 0).
    Frag kr[NPC], vr[NPC];
    float lg = 0.f, decay = 1.f;
    auto load = [&](int t0) {
        const int t = t0 + lane;
        const size_t off = (size_t)min(t, Tlen - 1) * HD + 8 * NPC * w;
        if (GATED) lg = t < Tlen ? log_g[bh * Tlen + t] : 0.f;
        if (HD == 32 && w >= 4) return;
#pragma unroll
        for (int c = 0; c < NPC; ++c) {
            kr[c].u = *(const uint4*)(Kh + off + 8 * c);
            vr[c].u = *(const uint4*)(Vh + off + 8 * c);
            if (t >= Tlen) kr[c].u = vr[c].u = make_uint4(0, 0, 0, 0);
        }
    };
    float tile_decay = 1.f;     // across the tile that `store` was last called for
    auto store = [&](AbsorbTile<HD>& dst) {
        if (HD != 32 || w < 4)
#pragma unroll
        for (int c = 0; c < NPC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int f = 8 * (NPC * w + c) + e;
                dst.k[f][lane] = (bf16_t)(((e & 1) ? kr[c].q[e / 2] >> 16 : kr[c].q[e / 2]) & 0xffffu);
                dst.v[f][lane] = (bf16_t)(((e & 1) ? vr[c].q[e / 2] >> 16 : vr[c].q[e / 2]) & 0xffffu);
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
        const AbsorbTile<HD>& tl = tiles[buf];
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

template <int HD, bool GATED>
bool absorb_mfma_t(const pa_problem& pr, const DecodeLayout& L, const void* K, const void* V, const float* log_g, char* st,
                   hipStream_t s) {
    static_assert(absorb_units<HD>() % 8 == 0, "whole workgroups");
    constexpr size_t smem = 2 * sizeof(AbsorbTile<HD>);
    auto kern = k_decode_absorb_mfma<HD, GATED>;
    if (smem > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) {
            note_hip_error(e, "hipFuncSetAttribute(max dynamic LDS)");
            return false;
        }
    }
    LaunchScope ls("decode_absorb", s);
    hipLaunchKernelGGL(kern, dim3(absorb_units<HD>() / 8, pr.B * pr.H), dim3(512), smem, s, (const bf16_t*)K, (const bf16_t*)V, log_g,
                       (float*)(st + L.off_s), (float*)(st + L.off_gam), L.D, pr.T);
    return launch_ok();
}
bool absorb_mfma_applies(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.p == 2 && pr.d == pr.v && (pr.d == 32 || pr.d == 64 || pr.d == 128);
}
bool absorb_mfma(const pa_problem& pr, const DecodeLayout& L, const void* K, const void* V, const float* log_g, char* st,
                 hipStream_t s) {
#define PA_GO(DD)                                                                  \
    if (pr.d == DD)                                                                \
        return log_g != nullptr ? absorb_mfma_t<DD, true>(pr, L, K, V, log_g, st, s) \
                                : absorb_mfma_t<DD, false>(pr, L, K, V, log_g, st, s);
    PA_GO(32) PA_GO(64) PA_GO(128)
#undef PA_GO
    return false;
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
// d = 64 the scan is the faster one for long prompts of few heads (12 heads of 65536 tokens: 579 us against 1896; 12 of 2048:
// 45 against 70) and the exact kernel for short ones (48 heads of 512: 39 against 77), but which of the two rounds its sums is
// the caller's choice, made with the workspace, so the line does not follow the time.  The rest takes the float32 kernel on the
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
