// bf16 MFMA kernels for the attention form of power attention (arXiv 2507.04239, Sec. 2 Eq. 5 with
// the kernel of Sec. 4 Eq. 7): the whole sequence is one chunk, no state is built,
//     O_i = sum_{j <= i} a_ij v_j / Z_i,   a_ij = (scale q_i . k_j)^p,   Z_i = sum_{j <= i} a_ij,
// for degrees p in {2, 3, 4}, head sizes d = v in {32, 64, 128} and any sequence length.  The paper switches to this form where
// it is the cheaper one (Sec. 4.1.2, the throughput comparison); here it is also what runs the degrees and
// head sizes the chunked MFMA family (p = 2, d = 64) does not cover.
//
// Backward pass (the paper gives none; derived from the definition): with ghat_i = dO_i / Z_i and
// gz_i = -ghat_i . O_i (normalised; ghat = dO, gz = 0 otherwise),
//     e_ij = ghat_i . v_j + gz_i                       dL / d a_ij
//     t_ij = e_ij p scale (scale q_i . k_j)^(p-1)      dL / d (q_i . k_j)
//     dQ_i = sum_{j <= i} t_ij k_j,   dK_j = sum_{i >= j} t_ij q_i,   dV_j = sum_{i >= j} a_ij ghat_i.
//
// All three kernels have one shape: a workgroup of 4 waves owns a block of rows (queries for the
// forward pass and dQ, keys for dK / dV), each wave OWN of them with its operands and accumulators
// in registers, and walks over the other side's rows in tiles of 64 that are staged row-major in
// LDS (double-buffered, one barrier per tile).  Operands that are needed transposed (V^T, K^T, Q^T,
// ghat^T as the MFMA's A operand) come from the same row-major tile through the transposing LDS
// read, so no transposed copy exists anywhere.
//
// MFMA: 32x32x16 throughout (layouts in mfma_common.hpp).  The first contraction's accumulators (16 registers: rows
// 8 k + 4 h + r of the streamed side) are two B operands of the second one, whose 16 k-slots are then the streamed rows
// 16 j + 4 h + r and 16 j + 8 + 4 h + r.  Against 16x16x32 the operands read per flop halve and a wave that has the SIMD
// to itself still issues at the full rate (31 cycles per 16x16x32 MFMA otherwise).
//
// The vector ALU's share, per pair of tokens, is what bounds d = 32 and matters everywhere, so the scale stays out of it.
// scale = fold * rest, fold a power of two and 1 <= |rest| < 2.  The operand of the scores that a wave holds for the whole
// walk (Q; K for dK / dV) is multiplied by fold as it is loaded, exactly, so that the kernels' c is q . k at the magnitude of
// the score s = rest c; they form c^p and e c^(p-1), and the factors rest^p (p fold rest^p for dQ and dK) are applied to the
// accumulators once, at the end.  Powers and sums then overflow or vanish where those of s do, within rest^p < 16; with all of
// scale^p left to the end they would where those of q . k or scale^p itself do.  (Per pair at p = 2: forward 1 multiply and
// half a conversion instead of 2.5 instructions, dQ 1.5 instead of 3.5.)
//
// Forward + backward, before and after the 32x32 form, the scale's removal and the order of the workgroups:
// p = 4, d = 32, B2 H8 T16384: 2.43 -> 1.40 ms; p = 3, d = 64, B1 H4 T16384: 1.25 -> 0.89 ms; p = 2, d = 64, B16 H12
// T1000: 0.260 -> 0.175 ms.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mfma_common.hpp"

namespace pa {
namespace mfma {
namespace {

constexpr int AT = 64;   // rows per streamed tile

template <int HD>
struct AttnTile {
    bf16_t r[AT][HD + 8];   // pitch (HD + 8) / 2 dwords = 4 (mod 8): the 16 rows of a fragment read hit distinct banks
};

template <int P>
__device__ __forceinline__ float ipow(float x) {
    float r = 1.f;
#pragma unroll
    for (int i = 0; i < P; ++i) r *= x;
    return r;
}
template <>
__device__ __forceinline__ float ipow<4>(float x) {
    const float x2 = x * x;
    return x2 * x2;
}

// z + the sum of 8 bf16 values (exact products with one, float32 sums)
__device__ __forceinline__ float sum_bf16x8(const Frag& f, float z) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const bf16x2 one = {(__bf16)1.f, (__bf16)1.f};
#pragma unroll
    for (int i = 0; i < 8; i += 2) z = __builtin_amdgcn_fdot2_f32_bf16((bf16x2){f.v[i], f.v[i + 1]}, one, z, false);
    return z;
}

// Staging of a 64-row tile of a row-major [.][HD] array: HD / 32 pieces of 16 bytes per thread,
// piece id = tid + 256 q is row id / (HD / 8), features 8 (id % (HD / 8)) .. + 7.  The pieces wait
// in registers while the tile before them is being used (plain arrays and unrolled loops in the
// kernels: wrapped in a struct they end up in scratch memory).
// T need not be a multiple of the tile: rows past the end are read as row T - 1 (keys and queries
// there are masked out by causality, or never stored) or, with ZERO, as zeros (ghat, whose rows
// past the end must not contribute to dK, dV).
template <int HD, bool ZERO>
__device__ __forceinline__ uint4 piece_load(const bf16_t* __restrict__ head_base, int row0, int id, int T) {
    const int row = row0 + id / (HD / 8);
    const uint4 u = *(const uint4*)(head_base + (size_t)min(row, T - 1) * HD + 8 * (id % (HD / 8)));
    return ZERO && row >= T ? make_uint4(0, 0, 0, 0) : u;
}
template <int HD>
__device__ __forceinline__ void piece_store(AttnTile<HD>& dst, int id, uint4 u) {
    *(uint4*)&dst.r[id / (HD / 8)][8 * (id % (HD / 8))] = u;
}
#define PA_TILE_LOAD(REGS, BASE, ROW0, ZERO)        \
    _Pragma("unroll") for (int q_ = 0; q_ < HD / 32; ++q_) REGS[q_] = piece_load<HD, ZERO>(BASE, ROW0, tid + 256 * q_, T);
#define PA_TILE_STORE(DST, REGS)                    \
    _Pragma("unroll") for (int q_ = 0; q_ < HD / 32; ++q_) piece_store<HD>(DST, tid + 256 * q_, REGS[q_]);

// row 32 blk + r32, features 16 ks + 8 h .. + 7: A operand (rows x features) or B operand
// (features x rows) of a contraction over the features
template <int HD>
__device__ __forceinline__ bf16x8 row_frag(const AttnTile<HD>& t, int blk, int ks, int lane) {
    Frag f;
    f.u = *(const uint4*)&t.r[32 * blk + (lane & 31)][16 * ks + 8 * (lane >> 5)];
    return f.v;
}
template <int HD>
__device__ __forceinline__ bf16x8 row_frag_global(const bf16_t* __restrict__ X, size_t row, int ks, int h) {
    Frag f;
    f.u = *(const uint4*)(X + row * HD + 16 * ks + 8 * h);
    return f.v;
}

// scale as fold * rest (see above)
struct ScaleParts {
    float fold, rest;
};
ScaleParts split_scale(float scale) {
    if (!std::isfinite(scale)) return {1.f, scale};
    int e = 0;
    (void)std::frexp(scale, &e);
    e = std::max(e - 1, -126);      // (a subnormal scale: |rest| < 1)
    return {std::ldexp(1.f, e), std::ldexp(scale, -e)};
}
// a held operand times `fold`: exact, but for results that are subnormal or too large for bf16
template <int N>
__device__ __forceinline__ void fold_in(bf16x8 (&f)[N], float fold) {
    if (fold == 1.f) return;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) f[i][e] = (__bf16)(fold * (float)f[i][e]);
}

// A operand of a contraction over the tile's rows: column 32 cb + r32, k-slots = rows 16 j + 4 h .. + 3 and 8 further.
// The transposing read hands lane n of a 16-lane group column n of the 4 x 16 block whose row i the lanes 4 i .. 4 i + 3
// point at (4 columns each).
template <int HD>
__device__ __forceinline__ bf16x8 col_frag(const AttnTile<HD>& t, int j, int cb, int lane) {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const int r16 = lane & 15, h = lane >> 5, odd = (lane >> 4) & 1;
    const bf16_t* p = &t.r[16 * j + 4 * h + (r16 >> 2)][32 * cb + 16 * odd + 4 * (r16 & 3)];
    union {
        bf16x8 v;
        bf16x4 h[2];
    } f;
    f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
    f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 8 * (HD + 8)));
    return f.v;
}
__device__ __forceinline__ f32x16 splat16(float x) {
    f32x16 v;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = x;
    return v;
}
// four values per accumulator quad k: rows 8 k + 4 h + r of a per-row float array
__device__ __forceinline__ void row_values(float (&o)[16], const float* base, int h) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 q = *(const float4*)(base + 8 * k + 4 * h);
        o[4 * k] = q.x; o[4 * k + 1] = q.y; o[4 * k + 2] = q.z; o[4 * k + 3] = q.w;
    }
}
// one 32-row block of an output row's columns: dst[8 k + 4 h + r] = f acc[4 k + r] (bf16); two lanes 32 apart exchange
// halves so that each stores whole 16-byte runs
__device__ __forceinline__ void store_block(bf16_t* dst, const f32x16& acc, float f, int h, bool in) {
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        union {
            bf16x4 v;
            uint2 u;
        } x, y;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x.v[r] = (__bf16)(f * acc[4 * k + r]);
            y.v[r] = (__bf16)(f * acc[4 * k + 4 + r]);
        }
        const auto d0 = __builtin_amdgcn_permlane32_swap(x.u.x, y.u.x, false, false);
        const auto d1 = __builtin_amdgcn_permlane32_swap(x.u.y, y.u.y, false, false);
        if (in) *(u32x4*)(dst + 8 * (k + h)) = (u32x4){d0[0], d1[0], d0[1], d1[1]};
    }
}
// acc += the same block of `nslab` float32 parts
__device__ __forceinline__ void add_parts(f32x16& acc, const float* part, size_t slab_stride, int nslab, int h) {
    for (int sl = 0; sl < nslab; ++sl)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 pv = *(const float4*)(part + sl * slab_stride + 8 * k + 4 * h);
            acc[4 * k] += pv.x; acc[4 * k + 1] += pv.y; acc[4 * k + 2] += pv.z; acc[4 * k + 3] += pv.w;
        }
}

// Gating (Sec. 2 "Gating"): the pair (i, j) carries exp(b_i - b_j), b the running sum of the log-gates.
// For a tile whose every pair is below the diagonal the factor is split at a reference m inside the
// gap between the two sides, exp(b_i - m) exp(m - b_j), both <= 1: one of them is staged with the tile
// (GateTile::f, per streamed row), the other is formed once per tile for the rows a lane owns.  Tiles
// on the diagonal use the difference itself (GateTile::b), where a split could overflow.  Sums are relative to blocks of
// GATE_BLOCK tokens, which a tile and a wave's rows never straddle: the reference takes in what lies between the two blocks,
// a difference in float64.
static_assert(GATE_BLOCK % AT == 0, "a tile lies in one block, and so do the 32 or 64 rows of a wave");
struct alignas(16) GateTile {
    float b[AT], f[AT];
    float m;        // the reference, from the start of the workgroup's first block
};
// streamed rows row0 .. row0 + 63 of one head, by the first wave; own: blk of the workgroup's first row; KEYS: f = exp(m - b), m the b
// of the last row, else f = exp(b - m), m that of the first.  (Vector loads and a lane's value: scalar loads make the tile's LDS reads
// wait for them, 2 % of the kernel.)
template <bool KEYS>
__device__ __forceinline__ void gate_tile_load(float& b, float& f, float& m, const float* __restrict__ bl_head,
                                               const double* __restrict__ blk_head, double own, int row0, int tid, int T) {
    if (tid < AT) {
        const int row = min(row0 + tid, T - 1);
        b = bl_head[row];
        const float ref = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), KEYS ? AT - 1 : 0));
        f = __expf(KEYS ? ref - b : b - ref);
        m = ref + (float)(blk_head[row / GATE_BLOCK] - own);
    }
}
__device__ __forceinline__ void gate_tile_store(GateTile& t, float b, float f, float m, int tid) {
    if (tid < AT) {
        t.b[tid] = b;
        t.f[tid] = f;
        if (tid == 0) t.m = m;
    }
}

// Workgroups are numbered so that the ones with the longest walk start first: grid (heads of a group, blocks, groups), so the
// longest blocks of every head of a group come before the next ones.  (With the blocks of one head after the other, the last
// heads' long walks started when most of the chip was done: at 16 heads of 16384 tokens the CUs were busy 62 % of the time, and
// the p = 4 kernels took 468 / 685 / 926 us instead of 330 / 445 / 587.)  More blocks than y is given go on in z (the device
// states 65536 as the most of either).
struct Order {
    int group, parts;       // heads per group; slices of y that a group's blocks take
};
struct Place {
    int head, rank;         // rank counts the blocks from the longest walk down
};
__device__ __forceinline__ Place place(Order o) {
    int z = (int)blockIdx.z, part = 0;
    if (o.parts > 1) {
        const int g = __builtin_amdgcn_readfirstlane(z / o.parts);
        part = z - g * o.parts;
        z = g;
    }
    return {z * o.group + (int)blockIdx.x, part * (int)gridDim.y + (int)blockIdx.y};
}
dim3 block_grid(int heads, int blocks, Order& o) {
    const int y = std::min(blocks, 32768);
    o.parts = (blocks + y - 1) / y;
    return dim3((unsigned)o.group, (unsigned)y, (unsigned)((heads + o.group - 1) / o.group * o.parts));
}

// ---- forward ----------------------------------------------------------------------------------------
// acc[vb][ib] = O^T: value columns 32 vb + .., query 32 ib + r32 of the wave's OWN queries.
// WPE: waves per SIMD the register budget is set for.
// CHUNKED (the in-chunk part of the chunked form, App. E.1, for any degree and head size): a query sees the
// keys of its own chunk of `cs` tokens only (cs a multiple of the 64-key tile), and the part that comes
// through the state has been left by other kernels: part[slab][bh][t][v] (float32, `nslab` slabs, summed
// here) joins the numerator and zpart[bh][t] the denominator before the division.
struct ChunkedIn {
    int cs = 0, nslab = 0, nslab2 = 0;
    const float* part = nullptr;     // forward: numerator; dQ kernel: dQ; dK / dV kernel: dK
    const float* part2 = nullptr;    // dK / dV kernel: dV (nslab2 slabs)
    const float* zpart = nullptr;    // forward: denominator
    const float* dot = nullptr;      // gated, dQ and dK / dV kernels: the states' part of q . dq and k . dk
};
template <int P, int HD, int OWN, int WPE, bool GATED, bool CHUNKED = false>
__global__ __launch_bounds__(256, WPE) void k_attn_fwd(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                                       const bf16_t* __restrict__ V, bf16_t* __restrict__ O,
                                                       float* __restrict__ Z, int BH, Order order, int T, ScaleParts scale, int normalize,
                                                       GateSums sums, ChunkedIn ck) {
    constexpr int NI = OWN / 32, NK = HD / 16, NV = HD / 32, WG = 4 * OWN;
    extern __shared__ __attribute__((aligned(16))) unsigned char attn_smem[];
    AttnTile<HD>* kt = reinterpret_cast<AttnTile<HD>*>(attn_smem);      // [2]
    AttnTile<HD>* vt = kt + 2;                                          // [2]
    GateTile* gtile = reinterpret_cast<GateTile*>(vt + 2);              // [2]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r32 = lane & 31, h = lane >> 5;
    const int nblk = (T + WG - 1) / WG;
    const Place at = place(order);
    const int i0 = (nblk - 1 - at.rank) * WG;
    if (i0 < 0 || at.head >= BH) return;
    const int q0 = i0 + OWN * w;                    // the wave's first query
    const bool active = q0 < T;
    const size_t head = (size_t)at.head * T;
    const bf16_t* Kh = K + head * HD;
    const bf16_t* Vh = V + head * HD;

    bf16x8 qf[NI][NK];
    f32x16 acc[NV][NI];
    float zsum[NI];     // the sum of the rounded weights over this lane's k-slots
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
        zsum[ib] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks)
            qf[ib][ks] = row_frag_global<HD>(Q, head + min(q0 + 32 * ib + r32, T - 1), ks, h);
        fold_in(qf[ib], scale.fold);
#pragma unroll
        for (int vb = 0; vb < NV; ++vb) acc[vb][ib] = splat16(0.f);
    }
    const float* bl_head = GATED ? sums.bl + head : nullptr;
    const double* blk_head = GATED ? sums.blk + (size_t)at.head * ((T + GATE_BLOCK - 1) / GATE_BLOCK) : nullptr;
    const double own_blk = GATED ? blk_head[i0 / GATE_BLOCK] : 0.;
    float d_blk = 0.f;       // from there to the wave's block
    if (GATED && WG > GATE_BLOCK) d_blk = (float)(blk_head[min(q0, T - 1) / GATE_BLOCK] - own_blk);
    float bq[NI];
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) bq[ib] = GATED ? bl_head[min(q0 + 32 * ib + r32, T - 1)] : 0.f;

    // one 64-key tile; DIAG: some pair of the tile lies above the diagonal and has to be masked
    auto tile = [&](auto diag_c, int buf, int key0) {
        constexpr bool DIAG = decltype(diag_c)::value;
        float fq[NI];
        if (GATED && !DIAG) {
            const float m = gtile[buf].m - d_blk;          // the tile's last key, from the queries' block
#pragma unroll
            for (int ib = 0; ib < NI; ++ib) fq[ib] = __expf(bq[ib] - m);
        }
        f32x16 c[2][NI];        // S^T: key 32 kb + 8 k + 4 h + r, query 32 ib + r32
        auto scores = [&](int kb) {
#pragma unroll
            for (int ib = 0; ib < NI; ++ib) c[kb][ib] = splat16(0.f);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                const bf16x8 kf = row_frag<HD>(kt[buf], kb, ks, lane);
#pragma unroll
                for (int ib = 0; ib < NI; ++ib) c[kb][ib] = mfma32(kf, qf[ib][ks], c[kb][ib]);
            }
        };
        scores(0);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            if (kb == 0) scores(1);      // in flight under the weights of the first half
            Frag pf[NI][2];
            float gk[16];
            if (GATED) row_values(gk, DIAG ? &gtile[buf].b[32 * kb] : &gtile[buf].f[32 * kb], h);
#pragma unroll
            for (int ib = 0; ib < NI; ++ib)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float a = ipow<P>(c[kb][ib][i]);
                    if (GATED) a *= DIAG ? __expf(bq[ib] - gk[i]) : fq[ib] * gk[i];
                    if (DIAG && key0 + 32 * kb + 8 * (i >> 2) + 4 * h + (i & 3) > q0 + 32 * ib + r32) a = 0.f;
                    pf[ib][i >> 3].v[i & 7] = (__bf16)a;
                }
            // the denominator sums the rounded weights, the ones the numerator uses: the output is
            // then an exact convex combination of the values
#pragma unroll
            for (int ib = 0; ib < NI; ++ib)
#pragma unroll
                for (int j = 0; j < 2; ++j) zsum[ib] = sum_bf16x8(pf[ib][j], zsum[ib]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int vb = 0; vb < NV; ++vb) {
                    const bf16x8 vf = col_frag<HD>(vt[buf], 2 * kb + j, vb, lane);
#pragma unroll
                    for (int ib = 0; ib < NI; ++ib) acc[vb][ib] = mfma32(vf, pf[ib][j].v, acc[vb][ib]);
                }
        }
    };

    const int ntile = (min(i0 + WG, T) + AT - 1) / AT;   // key tiles 0 .. ntile - 1 reach the block's last query
    // chunked: the walk starts at the chunk of the block's first query, and a wave skips the tiles before its own chunk
    const int t_lo = CHUNKED ? (i0 / ck.cs) * ck.cs / AT : 0;
    const int k_lo = CHUNKED ? (q0 / ck.cs) * ck.cs : 0;
    uint4 kr[HD / 32], vr[HD / 32];
    float gb = 0.f, gf = 0.f, gm = 0.f;
    PA_TILE_LOAD(kr, Kh, t_lo * AT, false)
    PA_TILE_LOAD(vr, Vh, t_lo * AT, false)
    if (GATED) gate_tile_load<true>(gb, gf, gm, bl_head, blk_head, own_blk, t_lo * AT, tid, T);
    PA_TILE_STORE(kt[0], kr)
    PA_TILE_STORE(vt[0], vr)
    if (GATED) gate_tile_store(gtile[0], gb, gf, gm, tid);
    __syncthreads();
    for (int t = t_lo; t < ntile; ++t) {
        const int buf = (t - t_lo) & 1, key0 = t * AT;
        if (t + 1 < ntile) {
            PA_TILE_LOAD(kr, Kh, key0 + AT, false)
            PA_TILE_LOAD(vr, Vh, key0 + AT, false)
            if (GATED) gate_tile_load<true>(gb, gf, gm, bl_head, blk_head, own_blk, key0 + AT, tid, T);
        }
        if (active && key0 <= q0 + OWN - 1 && key0 >= k_lo) {
            if (key0 + AT - 1 > q0) tile(std::true_type{}, buf, key0);
            else tile(std::false_type{}, buf, key0);
        }
        if (t + 1 < ntile) {
            PA_TILE_STORE(kt[buf ^ 1], kr)
            PA_TILE_STORE(vt[buf ^ 1], vr)
            if (GATED) gate_tile_store(gtile[buf ^ 1], gb, gf, gm, tid);
        }
        __syncthreads();
    }

    if (!active) return;
    const float sp = ipow<P>(scale.rest);
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
        const bool in = q0 + 32 * ib + r32 < T;     // (a sequence need not be a multiple of the block)
        const size_t row = head + min(q0 + 32 * ib + r32, T - 1);
        float z = sp * xor32_sum(zsum[ib]), f = sp;
        if (CHUNKED) {
            z += ck.zpart[row];
#pragma unroll
            for (int vb = 0; vb < NV; ++vb) {
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[vb][ib][i] *= sp;
                add_parts(acc[vb][ib], ck.part + row * HD + 32 * vb, (size_t)BH * T * HD, ck.nslab, h);
            }
            f = 1.f;
        }
        if (normalize) f = z != 0.f ? f / z : 0.f;
#pragma unroll
        for (int vb = 0; vb < NV; ++vb) store_block(O + row * HD + 32 * vb, acc[vb][ib], f, h, in);
        if (Z != nullptr && h == 0 && in) Z[row] = z;
    }
}

// ---- backward: preparation -------------------------------------------------------------------------
// ghat = dO / Z (bf16) and gz = -(ghat . O) (float32); un-normalised: ghat = dO, gz = 0.  Rows with
// Z == 0 give zeros.  HD / 4 lanes per row.  gz is formed from the rounded ghat, so that
// ghat . v_j + gz = ghat . (v_j - O_i) keeps its exact cancellations.
template <int HD>
__global__ __launch_bounds__(256) void k_attn_prep(const bf16_t* __restrict__ dO, const bf16_t* __restrict__ O,
                                                   const float* __restrict__ Z, bf16_t* __restrict__ Gh,
                                                   float* __restrict__ gz, long long rows, int normalize) {
    constexpr int LPR = HD / 4;
    const long long row = (long long)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    const int c4 = threadIdx.x % LPR;
    if (row >= rows) return;
    const uint2 graw = *(const uint2*)(dO + row * HD + 4 * c4);
    const float gv[4] = {bf_lo(graw.x), bf_hi(graw.x), bf_lo(graw.y), bf_hi(graw.y)};
    float inv = 1.f;
    if (normalize) {
        const float z = Z[row];
        inv = z != 0.f ? 1.f / z : 0.f;
    }
    bf16x4 o;
    float gr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[i] = (__bf16)(gv[i] * inv);
        gr[i] = (float)o[i];
    }
    *(bf16x4*)(Gh + row * HD + 4 * c4) = o;
    float delta = 0.f;
    if (normalize) {
        const uint2 oraw = *(const uint2*)(O + row * HD + 4 * c4);
        delta = gr[0] * bf_lo(oraw.x) + gr[1] * bf_hi(oraw.x) + gr[2] * bf_lo(oraw.y) + gr[3] * bf_hi(oraw.y);
#pragma unroll
        for (int off = 1; off < LPR; off <<= 1) delta += __shfl_xor(delta, off);
    }
    if (c4 == 0) gz[row] = -delta;
}

// ---- backward: dQ -----------------------------------------------------------------------------------
// acc[fb][ib] = dQ^T: features 32 fb + .., query 32 ib + r32.
template <int P, int HD, int OWN, bool GATED, bool CHUNKED>
__device__ __forceinline__ void dq_block(Place at, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                                 const bf16_t* __restrict__ V, const bf16_t* __restrict__ Gh,
                                                 const float* __restrict__ gz, bf16_t* __restrict__ dQ, int BH, int T,
                                                 ScaleParts scale, GateSums sums, float* __restrict__ qdq,
                                                 ChunkedIn ck) {
    constexpr int NI = OWN / 32, NK = HD / 16, NF = HD / 32, WG = 4 * OWN;
    extern __shared__ __attribute__((aligned(16))) unsigned char attn_smem[];
    AttnTile<HD>* kt = reinterpret_cast<AttnTile<HD>*>(attn_smem);      // [2]
    AttnTile<HD>* vt = kt + 2;                                          // [2]
    GateTile* gtile = reinterpret_cast<GateTile*>(vt + 2);              // [2]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r32 = lane & 31, h = lane >> 5;
    const int nblk = (T + WG - 1) / WG;
    const int i0 = (nblk - 1 - at.rank) * WG;
    const int q0 = i0 + OWN * w;
    const bool active = q0 < T;
    const size_t head = (size_t)at.head * T;
    const bf16_t* Kh = K + head * HD;
    const bf16_t* Vh = V + head * HD;

    bf16x8 qf[NI][NK], gf[NI][NK];
    f32x16 acc[NF][NI];
    float gzq[NI];
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
        const size_t row = head + min(q0 + 32 * ib + r32, T - 1);
        gzq[ib] = gz[row];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            qf[ib][ks] = row_frag_global<HD>(Q, row, ks, h);
            gf[ib][ks] = row_frag_global<HD>(Gh, row, ks, h);
        }
        fold_in(qf[ib], scale.fold);
#pragma unroll
        for (int fb = 0; fb < NF; ++fb) acc[fb][ib] = splat16(0.f);
    }

    const float* bl_head = GATED ? sums.bl + head : nullptr;
    const double* blk_head = GATED ? sums.blk + (size_t)at.head * ((T + GATE_BLOCK - 1) / GATE_BLOCK) : nullptr;
    // gated: rsum = sum_j e_ij c_ij^p = q_i . dq_i / (p rest^p), the row's share of the gate gradient, summed
    // here from the unrounded terms (the dot product of the stored dq with q carries bf16 noise that a
    // sum over a block of tokens amplifies)
    const double own_blk = GATED ? blk_head[i0 / GATE_BLOCK] : 0.;
    float d_blk = 0.f;       // from there to the wave's block
    if (GATED && WG > GATE_BLOCK) d_blk = (float)(blk_head[min(q0, T - 1) / GATE_BLOCK] - own_blk);
    float bq[NI], rsum[NI];
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
        bq[ib] = GATED ? bl_head[min(q0 + 32 * ib + r32, T - 1)] : 0.f;
        rsum[ib] = 0.f;
    }

    auto tile = [&](auto diag_c, int buf, int key0) {
        constexpr bool DIAG = decltype(diag_c)::value;
        float fq[NI];
        if (GATED && !DIAG) {
            const float m = gtile[buf].m - d_blk;          // the tile's last key, from the queries' block
#pragma unroll
            for (int ib = 0; ib < NI; ++ib) fq[ib] = __expf(bq[ib] - m);
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            f32x16 c[NI], e[NI];        // S^T and E^T = V ghat^T + gz: key 32 kb + 8 k + 4 h + r, query 32 ib + r32
#pragma unroll
            for (int ib = 0; ib < NI; ++ib) {
                c[ib] = splat16(0.f);
                e[ib] = splat16(gzq[ib]);
            }
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                const bf16x8 kf = row_frag<HD>(kt[buf], kb, ks, lane), vf = row_frag<HD>(vt[buf], kb, ks, lane);
#pragma unroll
                for (int ib = 0; ib < NI; ++ib) {
                    c[ib] = mfma32(kf, qf[ib][ks], c[ib]);
                    e[ib] = mfma32(vf, gf[ib][ks], e[ib]);
                }
                if (ks & 1) __builtin_amdgcn_sched_barrier(0);   // (holds the register count under 256; gated, d = 128: 5 spills)
            }
            Frag tf[NI][2];
            float gk[16];
            if (GATED) row_values(gk, DIAG ? &gtile[buf].b[32 * kb] : &gtile[buf].f[32 * kb], h);
#pragma unroll
            for (int ib = 0; ib < NI; ++ib)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float tv = e[ib][i] * ipow<P - 1>(c[ib][i]);
                    if (GATED) tv *= DIAG ? __expf(bq[ib] - gk[i]) : fq[ib] * gk[i];
                    if (DIAG && key0 + 32 * kb + 8 * (i >> 2) + 4 * h + (i & 3) > q0 + 32 * ib + r32) tv = 0.f;
                    if (GATED) rsum[ib] += tv * c[ib][i];
                    tf[ib][i >> 3].v[i & 7] = (__bf16)tv;
                }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int fb = 0; fb < NF; ++fb) {
                    const bf16x8 kc = col_frag<HD>(kt[buf], 2 * kb + j, fb, lane);   // K^T
#pragma unroll
                    for (int ib = 0; ib < NI; ++ib) acc[fb][ib] = mfma32(kc, tf[ib][j].v, acc[fb][ib]);
                }
        }
    };

    const int ntile = (min(i0 + WG, T) + AT - 1) / AT;
    const int t_lo = CHUNKED ? (i0 / ck.cs) * ck.cs / AT : 0;     // chunked: keys of the query's own chunk only
    const int k_lo = CHUNKED ? (q0 / ck.cs) * ck.cs : 0;
    uint4 kr[HD / 32], vr[HD / 32];
    float gb = 0.f, gf2 = 0.f, gm = 0.f;
    PA_TILE_LOAD(kr, Kh, t_lo * AT, false)
    PA_TILE_LOAD(vr, Vh, t_lo * AT, false)
    if (GATED) gate_tile_load<true>(gb, gf2, gm, bl_head, blk_head, own_blk, t_lo * AT, tid, T);
    PA_TILE_STORE(kt[0], kr)
    PA_TILE_STORE(vt[0], vr)
    if (GATED) gate_tile_store(gtile[0], gb, gf2, gm, tid);
    __syncthreads();
    for (int t = t_lo; t < ntile; ++t) {
        const int buf = (t - t_lo) & 1, key0 = t * AT;
        if (t + 1 < ntile) {
            PA_TILE_LOAD(kr, Kh, key0 + AT, false)
            PA_TILE_LOAD(vr, Vh, key0 + AT, false)
            if (GATED) gate_tile_load<true>(gb, gf2, gm, bl_head, blk_head, own_blk, key0 + AT, tid, T);
        }
        if (active && key0 <= q0 + OWN - 1 && key0 >= k_lo) {
            if (key0 + AT - 1 > q0) tile(std::true_type{}, buf, key0);
            else tile(std::false_type{}, buf, key0);
        }
        if (t + 1 < ntile) {
            PA_TILE_STORE(kt[buf ^ 1], kr)
            PA_TILE_STORE(vt[buf ^ 1], vr)
            if (GATED) gate_tile_store(gtile[buf ^ 1], gb, gf2, gm, tid);
        }
        __syncthreads();
    }

    if (!active) return;
    const float psp = (float)P * ipow<P>(scale.rest), dsp = psp * scale.fold;
#pragma unroll
    for (int ib = 0; ib < NI; ++ib) {
        const bool in = q0 + 32 * ib + r32 < T;
        const size_t row = head + min(q0 + 32 * ib + r32, T - 1);
#pragma unroll
        for (int fb = 0; fb < NF; ++fb) {
            if (CHUNKED) {   // what came through the state (and the normaliser), per slab
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[fb][ib][i] *= dsp;
                add_parts(acc[fb][ib], ck.part + row * HD + 32 * fb, (size_t)BH * T * HD, ck.nslab, h);
            }
            store_block(dQ + row * HD + 32 * fb, acc[fb][ib], CHUNKED ? 1.f : dsp, h, in);
        }
        if (GATED) {
            const float dot = psp * xor32_sum(rsum[ib]) + (CHUNKED ? ck.dot[row] : 0.f);
            if (in && h == 0) qdq[row] = dot;
        }
    }
}

// ---- backward: dK, dV ---------------------------------------------------------------------------------
// dk[fb][kb] = dK^T: features 32 fb + .., key 32 kb + r32 of the wave's OWN keys; dv likewise.
// S and E are formed queries x keys here, so that their accumulators are the B operand (k-slots =
// queries) of the two contractions over the queries.
template <int P, int HD, int OWN, bool GATED, bool CHUNKED>
__device__ __forceinline__ void dkdv_block(Place at, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                                   const bf16_t* __restrict__ V, const bf16_t* __restrict__ Gh,
                                                   const float* __restrict__ gz, bf16_t* __restrict__ dK,
                                                   bf16_t* __restrict__ dV, int BH, int T, ScaleParts scale,
                                                   GateSums sums, float* __restrict__ kdk,
                                                   float* __restrict__ wsum, ChunkedIn ck) {
    constexpr int NJ = OWN / 32, NK = HD / 16, NF = HD / 32, WG = 4 * OWN;
    extern __shared__ __attribute__((aligned(16))) unsigned char attn_smem[];
    AttnTile<HD>* qt = reinterpret_cast<AttnTile<HD>*>(attn_smem);      // [2]
    AttnTile<HD>* gt = qt + 2;                                          // [2]
    float(*gzt)[AT] = reinterpret_cast<float(*)[AT]>(gt + 2);           // [2][AT]
    GateTile* gtile = reinterpret_cast<GateTile*>(gzt + 2);             // [2]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r32 = lane & 31, h = lane >> 5;
    const int j0 = at.rank * WG;
    const int k0 = j0 + OWN * w;                    // the wave's first key
    const bool active = k0 < T;
    const size_t head = (size_t)at.head * T;
    const bf16_t* Qh = Q + head * HD;
    const bf16_t* Gh_h = Gh + head * HD;
    const float* gzh = gz + head;
    const float sp = ipow<P>(scale.rest), psp = (float)P * sp, dsp = psp * scale.fold;

    bf16x8 kf[NJ][NK], vf[NJ][NK];
    f32x16 dk[NF][NJ], dv[NF][NJ];
#pragma unroll
    for (int kb = 0; kb < NJ; ++kb) {
        const size_t row = head + min(k0 + 32 * kb + r32, T - 1);
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            kf[kb][ks] = row_frag_global<HD>(K, row, ks, h);
            vf[kb][ks] = row_frag_global<HD>(V, row, ks, h);
        }
        fold_in(kf[kb], scale.fold);
#pragma unroll
        for (int fb = 0; fb < NF; ++fb) {
            dk[fb][kb] = splat16(0.f);
            dv[fb][kb] = splat16(0.f);
        }
    }

    const float* bl_head = GATED ? sums.bl + head : nullptr;
    const double* blk_head = GATED ? sums.blk + (size_t)at.head * ((T + GATE_BLOCK - 1) / GATE_BLOCK) : nullptr;
    // gated: csum = sum_i e_ij a_ij = k_j . dk_j / (p rest^p), the key's share of the gate gradient, from the
    // unrounded weights
    const double own_blk = GATED ? blk_head[j0 / GATE_BLOCK] : 0.;
    float d_blk = 0.f;       // from there to the wave's block
    if (GATED && WG > GATE_BLOCK) d_blk = (float)(blk_head[min(k0, T - 1) / GATE_BLOCK] - own_blk);
    float bk[NJ], csum[NJ];
#pragma unroll
    for (int kb = 0; kb < NJ; ++kb) {
        bk[kb] = GATED ? bl_head[min(k0 + 32 * kb + r32, T - 1)] : 0.f;
        csum[kb] = 0.f;
    }

    float wprev = 0.f;   // the wave's total of csum at the end of the last complete block of queries
    auto tile = [&](auto diag_c, int buf, int q0) {
        constexpr bool DIAG = decltype(diag_c)::value;
        float fk[NJ];
        if (GATED && !DIAG) {
            const float m = gtile[buf].m - d_blk;          // the tile's first query, from the keys' block
#pragma unroll
            for (int kb = 0; kb < NJ; ++kb) fk[kb] = __expf(m - bk[kb]);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            float g0[16];
            row_values(g0, &gzt[buf][32 * qb], h);
            f32x16 c[NJ], e[NJ];        // S and E = ghat V^T + gz: query 32 qb + 8 k + 4 h + r, key 32 kb + r32
#pragma unroll
            for (int kb = 0; kb < NJ; ++kb) {
                c[kb] = splat16(0.f);
#pragma unroll
                for (int i = 0; i < 16; ++i) e[kb][i] = g0[i];
            }
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                const bf16x8 qa = row_frag<HD>(qt[buf], qb, ks, lane), ga = row_frag<HD>(gt[buf], qb, ks, lane);
#pragma unroll
                for (int kb = 0; kb < NJ; ++kb) {
                    c[kb] = mfma32(qa, kf[kb][ks], c[kb]);
                    e[kb] = mfma32(ga, vf[kb][ks], e[kb]);
                }
            }
            Frag tf[NJ][2], pf[NJ][2];
            float gq[16];
            if (GATED) row_values(gq, DIAG ? &gtile[buf].b[32 * qb] : &gtile[buf].f[32 * qb], h);
#pragma unroll
            for (int kb = 0; kb < NJ; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float pw = ipow<P - 1>(c[kb][i]);
                    if (GATED) pw *= DIAG ? __expf(gq[i] - bk[kb]) : gq[i] * fk[kb];
                    if (DIAG && q0 + 32 * qb + 8 * (i >> 2) + 4 * h + (i & 3) < k0 + 32 * kb + r32) pw = 0.f;
                    // (p = 4 without gates or mask: the square's square is one multiply less deep than c^3 c)
                    const float a = P == 4 && !GATED && !DIAG ? ipow<P>(c[kb][i]) : pw * c[kb][i];
                    if (GATED) csum[kb] += e[kb][i] * a;
                    pf[kb][i >> 3].v[i & 7] = (__bf16)a;
                    tf[kb][i >> 3].v[i & 7] = (__bf16)(e[kb][i] * pw);
                }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int fb = 0; fb < NF; ++fb) {
                    const bf16x8 qc = col_frag<HD>(qt[buf], 2 * qb + j, fb, lane);   // Q^T
                    const bf16x8 gc = col_frag<HD>(gt[buf], 2 * qb + j, fb, lane);   // ghat^T
#pragma unroll
                    for (int kb = 0; kb < NJ; ++kb) {
                        dk[fb][kb] = mfma32(qc, tf[kb][j].v, dk[fb][kb]);
                        dv[fb][kb] = mfma32(gc, pf[kb][j].v, dv[fb][kb]);
                    }
                }
        }
    };

    // query tiles t_first .. ntile - 1 reach the block's first key; chunked: up to the end of the chunk of the block's
    // last key, and a wave stops at the end of its own keys' chunk
    const int t_first = j0 / AT;
    const int ntile = ((CHUNKED ? min(((j0 + WG - 1) / ck.cs + 1) * ck.cs, T) : T) + AT - 1) / AT;
    const int q_hi = CHUNKED ? (k0 / ck.cs + 1) * ck.cs : T + AT;
    uint4 qr[HD / 32], gr[HD / 32];
    float gzr = 0.f, gb = 0.f, gf2 = 0.f, gm = 0.f;
    PA_TILE_LOAD(qr, Qh, t_first * AT, false)
    PA_TILE_LOAD(gr, Gh_h, t_first * AT, true)
    if (tid < AT) gzr = t_first * AT + tid < T ? gzh[t_first * AT + tid] : 0.f;
    if (GATED) gate_tile_load<false>(gb, gf2, gm, bl_head, blk_head, own_blk, t_first * AT, tid, T);
    PA_TILE_STORE(qt[0], qr)
    PA_TILE_STORE(gt[0], gr)
    if (tid < AT) gzt[0][tid] = gzr;
    if (GATED) gate_tile_store(gtile[0], gb, gf2, gm, tid);
    __syncthreads();
    for (int t = t_first; t < ntile; ++t) {
        const int buf = (t - t_first) & 1, q0 = t * AT;
        if (t + 1 < ntile) {
            PA_TILE_LOAD(qr, Qh, q0 + AT, false)
            PA_TILE_LOAD(gr, Gh_h, q0 + AT, true)
            if (tid < AT) gzr = q0 + AT + tid < T ? gzh[q0 + AT + tid] : 0.f;
            if (GATED) gate_tile_load<false>(gb, gf2, gm, bl_head, blk_head, own_blk, q0 + AT, tid, T);
        }
        if (active && q0 + AT - 1 >= k0 && q0 < q_hi) {
            if (q0 < k0 + OWN - 1) tile(std::true_type{}, buf, q0);   // some pair of this tile lies above the diagonal
            else tile(std::false_type{}, buf, q0);
        }
        if (GATED && !CHUNKED && active && (q0 + AT) % WG == 0) {
            // a block of queries is complete: the wave's sum goes to wsum[head][key block][query block][wave]
            // (the key block's own query block is not a boundary sum: its pairs are summed per token)
            // = what the block added to the wave's running column sums
            const int jblk = j0 / WG, iblk = q0 / WG, nblk = T / WG;
            float v = 0.f;
#pragma unroll
            for (int kb = 0; kb < NJ; ++kb) v += csum[kb];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (iblk > jblk && lane == 0) wsum[(((size_t)at.head * nblk + jblk) * nblk + iblk) * 4 + w] = sp * (v - wprev);
            wprev = v;
        }
        if (t + 1 < ntile) {
            PA_TILE_STORE(qt[buf ^ 1], qr)
            PA_TILE_STORE(gt[buf ^ 1], gr)
            if (tid < AT) gzt[buf ^ 1][tid] = gzr;
            if (GATED) gate_tile_store(gtile[buf ^ 1], gb, gf2, gm, tid);
        }
        __syncthreads();
    }

    if (!active) return;
#pragma unroll
    for (int kb = 0; kb < NJ; ++kb) {
        const bool in = k0 + 32 * kb + r32 < T;
        const size_t row = head + min(k0 + 32 * kb + r32, T - 1);
        const size_t slab_stride = (size_t)BH * T * HD;
#pragma unroll
        for (int fb = 0; fb < NF; ++fb) {
            if (CHUNKED) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    dk[fb][kb][i] *= dsp;
                    dv[fb][kb][i] *= sp;
                }
                add_parts(dk[fb][kb], ck.part + row * HD + 32 * fb, slab_stride, ck.nslab, h);
                add_parts(dv[fb][kb], ck.part2 + row * HD + 32 * fb, slab_stride, ck.nslab2, h);
            }
            store_block(dK + row * HD + 32 * fb, dk[fb][kb], CHUNKED ? 1.f : dsp, h, in);
            store_block(dV + row * HD + 32 * fb, dv[fb][kb], CHUNKED ? 1.f : sp, h, in);
        }
        if (GATED) {
            const float dot = psp * xor32_sum(csum[kb]) + (CHUNKED ? ck.dot[row] : 0.f);
            if (in && h == 0) kdk[row] = dot;
        }
    }
}

// One launch for both halves of the backward pass, or for one of them; `rank` counts the blocks from the longest walk down.
// Both: blocks of either kind alternate, so that the tail of one is filled by the other.  A walk is a serial chain (a lone wave
// takes 4 times the MFMA time for a tile), and with few workgroups the longest one sets a kernel's time.  Backward pass, dK / dV
// and then dQ -> one launch: p = 3, d = 64, 2 heads of 16384 tokens 577 -> 370 us, 4 heads 681 -> 599; p = 2, 12 heads of 4096
// 166 -> 115, 24 heads 210 -> 200; p = 4, d = 32, 4 heads of 16384 604 -> 396.
enum class Bwd { dkdv, dq, both };
template <int P, int HD, int OWN, int WPE, bool GATED, bool CHUNKED, Bwd WHAT>
__global__ __launch_bounds__(256, WPE) void k_attn_bwd(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                                       const bf16_t* __restrict__ V, const bf16_t* __restrict__ Gh,
                                                       const float* __restrict__ gz, bf16_t* __restrict__ dQ,
                                                       bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, int BH, Order order,
                                                       int T, ScaleParts scale, GateSums sums, float* __restrict__ qdq,
                                                       float* __restrict__ kdk, float* __restrict__ wsum, ChunkedIn ckq,
                                                       ChunkedIn ckk) {
    Place at = place(order);
    const bool dq = WHAT == Bwd::dq || (WHAT == Bwd::both && (at.rank & 1));
    if (WHAT == Bwd::both) at.rank >>= 1;
    if (at.rank >= (T + 4 * OWN - 1) / (4 * OWN) || at.head >= BH) return;
    if (dq)
        dq_block<P, HD, OWN, GATED, CHUNKED>(at, Q, K, V, Gh, gz, dQ, BH, T, scale, sums, qdq, ckq);
    else
        dkdv_block<P, HD, OWN, GATED, CHUNKED>(at, Q, K, V, Gh, gz, dK, dV, BH, T, scale, sums, kdk, wsum, ckk);
}

template <int HD>
constexpr size_t attn_smem_bytes() {
    return 4 * sizeof(AttnTile<HD>) + 2 * AT * sizeof(float) + 2 * sizeof(GateTile);
}
// LDS beyond the default per-kernel limit has to be requested once per kernel
template <typename F>
bool allow_smem(F* fn, size_t bytes) {
    if (bytes <= 64 * 1024) return true;
    hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) note_hip_error(e, "hipFuncSetAttribute(max dynamic LDS)");
    return e == hipSuccess;
}

// Gate gradient, the part that crosses block boundaries: xb[head][m] = sum of e_ij a_ij over the pairs
// with key block <= m < query block, from wsum[head][key block][query block][wave].
// First along the query blocks: wsum[J][m][0] <- sum over I > m (one thread per key block J) ...
__global__ __launch_bounds__(64) void k_attn_gate_rows(float* __restrict__ wsum, int nblk) {
    const int jb = blockIdx.x * 64 + threadIdx.x, bh = blockIdx.y;
    if (jb >= nblk) return;
    float* rowp = wsum + ((size_t)bh * nblk + jb) * nblk * 4;
    float run = 0.f;
    for (int i = nblk - 1; i >= jb; --i) {
        const float here = i > jb ? rowp[4 * i] + rowp[4 * i + 1] + rowp[4 * i + 2] + rowp[4 * i + 3] : 0.f;
        rowp[4 * i] = run;
        run += here;
    }
}
// ... then down the key blocks: xb[m] = sum over J <= m (one thread per boundary m)
__global__ __launch_bounds__(64) void k_attn_gate_cols(const float* __restrict__ wsum, float* __restrict__ xb, int nblk) {
    const int m = blockIdx.x * 64 + threadIdx.x, bh = blockIdx.y;
    if (m >= nblk) return;
    float acc = 0.f;
    for (int jb = 0; jb <= m; ++jb) acc += wsum[(((size_t)bh * nblk + jb) * nblk + m) * 4];
    xb[(size_t)bh * nblk + m] = acc;
}

// Rows of the block one wave owns and the waves per SIMD the kernel is compiled for, measured on MI355X.  At d = 64 the
// 32-row waves read twice the LDS bytes per flop, but two to three of them share a SIMD without spilling (4 heads of 16384
// tokens, p = 3: forward 241 us against 277 with 64 rows; dQ 322 against 375 with 64 rows and one wave per SIMD, 877 with 64
// rows and spills; dK / dV 437 against 504 with 64 keys and one wave).  The forward pass takes 64 rows all the same where the grid is
// large (fwd_wide).  At d = 32 the operands are half the size and 64 rows fit two waves (16 heads of 16384 tokens, p = 4:
// 330 / 445 / 587 us against 336 / 463 / 620 with 32).  Only dK / dV at d = 128 (192 registers of operands and accumulators)
// runs alone.
template <int HD>
struct Shape {
    static constexpr int FWD_OWN = HD == 32 ? 64 : 32, FWD_WPE = 2;
    static constexpr int DQ_OWN = HD == 32 ? 64 : 32, DQ_WPE = 2;
    static constexpr int DKDV_OWN = HD == 32 ? 64 : 32, DKDV_WPE = HD == 128 ? 1 : 2;
};

// Heads whose blocks are taken together.  All of them, as long as their K and V (Q and dO / Z) fit half of the 256 MB memory-side
// cache; beyond, every walk comes from HBM (B8 H16 T32768, d = 128, forward / dK, dV / dQ in ms: 43.8 / 80.2 / 52.3 with all heads
// together, 34.9 / 74.6 / 44.4 with 8, 40.0 / 82.1 / 49.5 with one; 192 heads of 8192, d = 64: 1.84 / 3.45 / 2.20, 1.67 / 3.08 / 2.12,
// 2.18 / 3.94 / 2.56, and 1.58 / 2.95 / 2.04 with 32).  Eight is the least: a head then has an XCD and its L2 to itself.  Groups are of
// one size, for a small last one would leave the chip idle behind it (40 heads of 32768, d = 64: 5.43 ms forward in eights, 7.87
// as 32 + 8), and a power of two where it can be (the heads that meet on an XCD are then the fewest).  In-chunk walks that read
// no block but their own share nothing: there the blocks of a head stay together and read memory in order (12 heads of 65536, d = 64,
// chunk 128: dK / dV 410 us, 429 with the heads together).
template <int HD, bool CHUNKED, int WG>
int head_group(int BH, int T, const ChunkedIn& ck) {
    if (CHUNKED && ck.cs <= WG) return 1;
    const int fit = std::max(8, (int)((128 << 20) / (4LL * T * HD)));
    if (BH <= fit) return BH;
    int g = 8;
    while (2 * g <= fit) g *= 2;
    for (; g >= 4; g /= 2)
        if (BH % g == 0) return g;
    const int groups = (BH + fit - 1) / fit;
    return (BH + groups - 1) / groups;
}

// d = 64, whole sequences: 64 query rows per wave in place of 32 read half the LDS bytes per flop, and are the faster ones once
// their blocks of 256 rows, half as many, still fill the chip (32 and 64 rows, us, p = 2): 8 heads of 16384 (512 blocks) 285 / 307, 96 of
// 2048 (768) 60.3 / 61.7, 24 of 8192 (768) 209 / 198, 256 of 1024 (1024) 47.3 / 47.6, 128 of 2048 (1024) 76.9 / 74.9, 64 of 4096 (1024)
// 142 / 135, 64 of 8192 531 / 469, 16 of 131072 33.0 / 28.9 ms.
bool fwd_wide(int BH, int T) { return T >= 2048 && (long long)BH * ((T + 255) / 256) >= 1024; }
template <int P, int HD, bool GATED, bool CHUNKED, int OWN>
bool fwd_own(hipStream_t s, const bf16_t* Q, const bf16_t* K, const bf16_t* V, bf16_t* O, float* Z, int BH, int T, float scale,
             int normalize, GateSums sums, ChunkedIn ck, const char* label) {
    constexpr int WG = 4 * OWN;
    auto kern = k_attn_fwd<P, HD, OWN, Shape<HD>::FWD_WPE, GATED, CHUNKED>;
    if (!allow_smem(kern, attn_smem_bytes<HD>())) return false;
    LaunchScope ls(label, s);
    Order order{head_group<HD, CHUNKED, WG>(BH, T, ck)};
    const dim3 grid = block_grid(BH, (T + WG - 1) / WG, order);
    hipLaunchKernelGGL(kern, grid, dim3(256), attn_smem_bytes<HD>(), s, Q, K, V, O, Z, BH, order, T,
                       split_scale(scale), normalize, sums, ck);
    return launch_ok();
}
template <int P, int HD, bool GATED, bool CHUNKED = false>
bool fwd_t(hipStream_t s, const bf16_t* Q, const bf16_t* K, const bf16_t* V, bf16_t* O, float* Z, int BH, int T, float scale,
           int normalize, GateSums sums, ChunkedIn ck = ChunkedIn(), const char* label = "attn_fwd") {
    if constexpr (HD == 64 && !CHUNKED)
        if (fwd_wide(BH, T)) return fwd_own<P, HD, GATED, CHUNKED, 64>(s, Q, K, V, O, Z, BH, T, scale, normalize, sums, ck, label);
    return fwd_own<P, HD, GATED, CHUNKED, Shape<HD>::FWD_OWN>(s, Q, K, V, O, Z, BH, T, scale, normalize, sums, ck, label);
}

template <int P, int HD, bool GATED, bool CHUNKED = false>
bool bwd_t(hipStream_t s, const bf16_t* Q, const bf16_t* K, const bf16_t* V, const bf16_t* O, const float* Z, const bf16_t* dO,
           bf16_t* Gh, float* gz, bf16_t* dQ, bf16_t* dK, bf16_t* dV, int BH, int T, float scale, int normalize,
           const AttnGate& gate, ChunkedIn ckq = ChunkedIn(), ChunkedIn ckk = ChunkedIn()) {
    const long long rows = (long long)BH * T;
    if (!CHUNKED) {
        constexpr int RPB = 256 / (HD / 4);
        LaunchScope ls("attn_bwd_prep", s);
        hipLaunchKernelGGL((k_attn_prep<HD>), dim3((unsigned)((rows + RPB - 1) / RPB)), dim3(256), 0, s, dO, O, Z, Gh, gz, rows,
                           normalize);
        if (!launch_ok()) return false;
    }
    constexpr int WG = 4 * Shape<HD>::DKDV_OWN;
    static_assert(Shape<HD>::DQ_OWN == Shape<HD>::DKDV_OWN, "the blocks of dQ and dK / dV alternate in one grid");
    const int nblk = (T + WG - 1) / WG;
    auto launch = [&](auto what, const char* name, int wgs) {
        constexpr Bwd W = decltype(what)::value;
        constexpr int WPE = W == Bwd::dq ? Shape<HD>::DQ_WPE : Shape<HD>::DKDV_WPE;
        auto kern = k_attn_bwd<P, HD, Shape<HD>::DKDV_OWN, WPE, GATED, CHUNKED, W>;
        if (!allow_smem(kern, attn_smem_bytes<HD>())) return false;
        LaunchScope ls(name, s);
        Order order{head_group<HD, CHUNKED, WG>(BH, T, ckq)};
        const dim3 grid = block_grid(BH, wgs, order);
        hipLaunchKernelGGL(kern, grid, dim3(256), attn_smem_bytes<HD>(), s, Q, K, V, Gh, gz, dQ, dK, dV, BH, order, T,
                           split_scale(scale), gate.sums, gate.qdq, gate.kdk, gate.wsum, ckq, ckk);
        return launch_ok();
    };
    // One launch holds every wave to the registers of the larger half (d = 64: two waves of dQ per SIMD instead of three), which
    // costs what the filled tail saves from 3 to 4 workgroups of each kind per CU on (d = 64, 24 heads of 4096 tokens, 768 of each
    // kind: 210 us in two, 201 in one; T1000, 1536: 124 either way; 96 heads of 4096, 3072: 782 and 801; d = 32, 1024: 1065 and
    // 1071).  Gated: 12 heads of 4096 (384 of each kind) 240 and 165, 24 heads (768) 271 and 253.  In-chunk, whole backward passes
    // of the tiled kernels, d = 32: 24 heads of 1024 tokens, chunk 128, 114 and 106; 1 of 16384, chunk 4096, 538 and 487; 12 of
    // 16384, chunk 256, 727 and 720; no shape slower in one.  At d = 128 dQ would lose half of its waves.
    bool both = false;
    if constexpr (HD < 128) {
        both = (long long)BH * nblk <= 768;
        if (both && !launch(std::integral_constant<Bwd, Bwd::both>{}, CHUNKED ? "chunk_bwd" : "attn_bwd", 2 * nblk)) return false;
    }
    if (!both && !launch(std::integral_constant<Bwd, Bwd::dkdv>{}, CHUNKED ? "chunk_bwd_dkdv" : "attn_bwd_dkdv", nblk)) return false;
    if (GATED && !CHUNKED) {
        const int ngate = T / WG;
        LaunchScope ls2("attn_gate_boundary", s);
        hipLaunchKernelGGL(k_attn_gate_rows, dim3((ngate + 63) / 64, BH), dim3(64), 0, s, gate.wsum, ngate);
        hipLaunchKernelGGL(k_attn_gate_cols, dim3((ngate + 63) / 64, BH), dim3(64), 0, s, gate.wsum, gate.xb, ngate);
        if (!launch_ok()) return false;
    }
    if (!both && !launch(std::integral_constant<Bwd, Bwd::dq>{}, CHUNKED ? "chunk_bwd_dq" : "attn_bwd_dq", nblk)) return false;
    return true;
}

}  // namespace

int attn_gate_block(int d) { return 4 * (d == 128 ? Shape<128>::DKDV_OWN : d == 64 ? Shape<64>::DKDV_OWN : Shape<32>::DKDV_OWN); }

bool attn_shape_ok(int p, int d) { return (p == 2 || p == 3 || p == 4) && (d == 32 || d == 64 || d == 128); }

bool launch_attn_fwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, bf16_t* O, float* Z, int BH,
                     int T, float scale, int normalize, GateSums sums) {
#define PA_CASE(PP, DD)                                                                                      \
    if (p == PP && d == DD)                                                                                  \
        return sums.bl != nullptr ? fwd_t<PP, DD, true>(s, Q, K, V, O, Z, BH, T, scale, normalize, sums)            \
                             : fwd_t<PP, DD, false>(s, Q, K, V, O, Z, BH, T, scale, normalize, sums);
    PA_CASE(2, 32) PA_CASE(2, 64) PA_CASE(2, 128)
    PA_CASE(3, 32) PA_CASE(3, 64) PA_CASE(3, 128)
    PA_CASE(4, 32) PA_CASE(4, 64) PA_CASE(4, 128)
#undef PA_CASE
    return false;
}

bool launch_chunk_fwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, bf16_t* O, float* Z, int BH,
                      int T, int cs, float scale, int normalize, const float* part, int nslab, const float* zpart, const char* label,
                      GateSums sums) {
    ChunkedIn ck;
    ck.cs = cs;
    ck.nslab = nslab;
    ck.part = part;
    ck.zpart = zpart;
    if (cs % AT != 0) return false;
    if (sums.bl != nullptr) return p == 2 && d == 64 && fwd_t<2, 64, true, true>(s, Q, K, V, O, Z, BH, T, scale, normalize, sums, ck, label);
#define PA_CASE(PP, DD) \
    if (p == PP && d == DD) return fwd_t<PP, DD, false, true>(s, Q, K, V, O, Z, BH, T, scale, normalize, GateSums(), ck, label);
    PA_CASE(2, 32) PA_CASE(2, 64) PA_CASE(2, 128)
    PA_CASE(3, 32) PA_CASE(3, 64)
    PA_CASE(4, 32)
#undef PA_CASE
    return false;
}

bool launch_attn_prep(hipStream_t s, int d, const bf16_t* dO, const bf16_t* O, const float* Z, bf16_t* Gh, float* gz, long long rows,
                      int normalize) {
    LaunchScope ls("attn_bwd_prep", s);
    if (d == 32)
        hipLaunchKernelGGL((k_attn_prep<32>), dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, s, dO, O, Z, Gh, gz, rows, normalize);
    else if (d == 64)
        hipLaunchKernelGGL((k_attn_prep<64>), dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, s, dO, O, Z, Gh, gz, rows, normalize);
    else if (d == 128)
        hipLaunchKernelGGL((k_attn_prep<128>), dim3((unsigned)((rows + 7) / 8)), dim3(256), 0, s, dO, O, Z, Gh, gz, rows, normalize);
    else
        return false;
    return launch_ok();
}

bool launch_chunk_bwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, const bf16_t* Gh,
                      const float* gz, bf16_t* dQ, bf16_t* dK, bf16_t* dV, int BH, int T, int cs, float scale, const float* part_dq,
                      int nslab_dq, const float* part_dk, int nslab_dk, const float* part_dv, int nslab_dv, const AttnGate& gate,
                      const float* dotq, const float* dotk) {
    ChunkedIn ckq, ckk;
    ckq.cs = ckk.cs = cs;
    ckq.part = part_dq;
    ckq.nslab = nslab_dq;
    ckk.part = part_dk;
    ckk.nslab = nslab_dk;
    ckk.part2 = part_dv;
    ckk.nslab2 = nslab_dv;
    ckq.dot = dotq;
    ckk.dot = dotk;
    if (cs % AT != 0) return false;
    if (gate.sums.bl != nullptr)
        return p == 2 && d == 64 &&
               bwd_t<2, 64, true, true>(s, Q, K, V, nullptr, nullptr, nullptr, const_cast<bf16_t*>(Gh), const_cast<float*>(gz), dQ, dK, dV, BH, T,
                                        scale, 1, gate, ckq, ckk);
#define PA_CASE(PP, DD)     \
    if (p == PP && d == DD) \
        return bwd_t<PP, DD, false, true>(s, Q, K, V, nullptr, nullptr, nullptr, const_cast<bf16_t*>(Gh), const_cast<float*>(gz), dQ, dK, dV, BH, T, scale, 1, AttnGate(), ckq, ckk);
    PA_CASE(2, 32) PA_CASE(2, 64) PA_CASE(2, 128)
    PA_CASE(3, 32) PA_CASE(3, 64)
    PA_CASE(4, 32)
#undef PA_CASE
    return false;
}

bool launch_attn_bwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, const bf16_t* O,
                     const float* Z, const bf16_t* dO, bf16_t* Gh, float* gz, bf16_t* dQ, bf16_t* dK, bf16_t* dV, int BH, int T,
                     float scale, int normalize, const AttnGate& gate) {
#define PA_CASE(PP, DD)                                                                                                          \
    if (p == PP && d == DD)                                                                                                      \
        return gate.sums.bl != nullptr ? bwd_t<PP, DD, true>(s, Q, K, V, O, Z, dO, Gh, gz, dQ, dK, dV, BH, T, scale, normalize, gate) \
                                  : bwd_t<PP, DD, false>(s, Q, K, V, O, Z, dO, Gh, gz, dQ, dK, dV, BH, T, scale, normalize, gate);
    PA_CASE(2, 32) PA_CASE(2, 64) PA_CASE(2, 128)
    PA_CASE(3, 32) PA_CASE(3, 64) PA_CASE(3, 128)
    PA_CASE(4, 32) PA_CASE(4, 64) PA_CASE(4, 128)
#undef PA_CASE
    return false;
}

}  // namespace mfma
}  // namespace pa
