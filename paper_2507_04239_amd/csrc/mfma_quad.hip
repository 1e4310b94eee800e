// Chunk-state kernels for degree p = 2 at d = v in {64, 128}, bf16 (arXiv 2507.04239, Sec. 2 "Chunked form", App. E.2 - E.4,
// embedding of Sec. 4.1.1 with d_tile = 8): the state scan, its read-out and the gradient of the embedding.  The pairs inside
// a chunk are the attention-form kernels' job (launch_chunk_fwd / launch_chunk_bwd), which add what these kernels leave.
//
// All three are contractions of phi (D = 36 or 136 tiles of 64 rows) with the head size, D HD multiply-adds per token each, on
// v_mfma_f32_32x32x16_bf16 (layouts in mfma_common.hpp), and in all three the vector ALU has as much to do with phi as the
// matrix cores have with the product.  So phi lives in registers in operand order, formed once per (row, token) with 1.5
// instructions (a multiply and half a conversion), every wave holds enough columns for one formation (64 or 128), and two
// waves share a SIMD so that one's multiplies run under the other's MFMAs.
//
// The chunk states are bf16, [BH][chunk][tile][a 8][v HD][b 8], tiles by columns: (ti, tj), ti <= tj, is number
// tj (tj + 1) / 2 + ti.  Off-diagonal tiles carry their multiplicity 2.  The normaliser is kept as the HD x HD matrix
// Gamma = sum k k^T (forward) or Omega = sum gz q q^T (backward).  Forward slot n - 1 is the sum over the chunks before n,
// backward slot n the sum over the chunks after n.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mfma_common.hpp"

namespace pa {
namespace mfma {
namespace {

template <int HD>
struct QD {
    static constexpr int NB = HD / 8, NTILE = NB * (NB + 1) / 2, TILE = 8 * HD * 8;
    static constexpr size_t STATE = (size_t)NTILE * TILE, GAM = (size_t)HD * HD;
};

__device__ __forceinline__ void unpack8(float (&x)[8], const uint4& u) {
    x[0] = bf_lo(u.x); x[1] = bf_hi(u.x); x[2] = bf_lo(u.y); x[3] = bf_hi(u.y);
    x[4] = bf_lo(u.z); x[5] = bf_hi(u.z); x[6] = bf_lo(u.w); x[7] = bf_hi(u.w);
}
__device__ __forceinline__ void unpack4(float (&x)[4], const uint2& u) {
    x[0] = bf_lo(u.x); x[1] = bf_hi(u.x); x[2] = bf_lo(u.y); x[3] = bf_hi(u.y);
}
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    union {
        __attribute__((ext_vector_type(2))) __bf16 v;
        uint32_t u;
    } o;
    o.v[0] = (__bf16)a;
    o.v[1] = (__bf16)b;
    return o.u;
}
// ---- state scan ----------------------------------------------------------------------------------------
// Update-state and the cumulative sum over chunks:
//   forward   S_n = sum_{j < n cs}      phi(k_j) v_j^T           (X = K, Y = V)
//   REV       R_n = sum_{i >= (n+1) cs} phi(q_i) ghat_i^T        (X = Q, Y = ghat)
// A wave owns 2 R values a, 16 values b (two adjacent tile columns) and all HD columns: 128 accumulators.  A 32-row MFMA block is
// 2 a x 16 b, so the factor x[a] is the same along each 16-lane row: a lane holds x[a] of one token and the multiply takes the
// token it needs by DPP (row_newbcast).  Four waves share the token rows, staged row-major in LDS, and take operands that run
// along tokens through the transposing read, so no transposed copy of anything exists.  Blocks on the diagonal compute the tile
// below it too (2560 rows for 2304 at d = 64, 9216 for 8704) and do not store it.  The last workgroup of a head has the normaliser.
//
// The sequence is cut into segments.  TOT: a workgroup adds up one segment's own total (float32, to memory).  Then either
// k_quad_prefix sums the totals of segments of one chunk (d = 64), or every segment starts from the sum of the totals before it
// and is walked once more, leaving a state per chunk (d = 128, where one head's workgroups are many and its float32 totals large).
template <int HD>
struct ScanCfg {
    static constexpr int R = HD == 64 ? 4 : 2, AU = 2 * R, NC = HD / 32;
    static constexpr int NG = HD == 64 ? 5 : 36;      // workgroups of 4 units (AU a x 16 b); + 1 for the normaliser
    static constexpr int XF = HD == 64 ? 64 : 32;     // features of X a workgroup stages: all, or its 16 a and 16 b
    static constexpr int XP = XF + 16, YP = HD + 16;  // pitches: 8 rows x 32 bytes of a transposing read on distinct banks
    static constexpr int ST = 64;                     // tokens per stage
    static constexpr int TOTF = 4 * R * NC * 16 * 64; // floats of a workgroup's total
};
template <int HD>
struct ScanSmem {
    bf16_t x[2][ScanCfg<HD>::ST][ScanCfg<HD>::XP];
    bf16_t y[2][ScanCfg<HD>::ST][ScanCfg<HD>::YP];
    float w[2][ScanCfg<HD>::ST];
};

struct ScanArgs {
    const bf16_t *X, *Y;
    const float* gz;         // REV: per token, the weight of the normaliser
    const float* tw;         // GATED: per token, the decay that goes with it (to the end, REV: from the start, of its chunk)
    const float* lam;        // GATED: [BH][nchunk] decay across a chunk
    bf16_t *st, *gam;
    float* tot;              // [BH][nseg][NG + 1][TOTF]
    int T, cs, nchunk, nseg, seg_chunks, heads;
    int tot_segs;            // TOT: segments whose total is formed (all, or all but the walk's last)
    float fold, out_scale;   // X is multiplied by fold (a power of two) on the way in, the state by out_scale on the way out
};

// where a wave's accumulators stand: unit (4 g + w) -> 16 b from 16 J, AU a from a0
template <int HD>
__device__ __forceinline__ void scan_unit(int u, int& J, int& a0) {
    constexpr int PER = 16 / ScanCfg<HD>::AU;     // units per (16 a, 16 b)
    J = 0;
    while (u >= PER * (J + 1)) {
        u -= PER * (J + 1);
        ++J;
    }
    a0 = ScanCfg<HD>::AU * u;
}
// a lane's accumulators c[0 .. 3] times fx and c[4 .. 7] times fy, as bf16: lanes 32 apart exchange halves, so that a lane of half
// 0 holds 8 consecutive rows of the first kind and its partner those of the second
__device__ __forceinline__ u32x4 pack_runs(const float* c, float fx, float fy) {
    const uint32_t x0 = pack2(fx * c[0], fx * c[1]), x1 = pack2(fx * c[2], fx * c[3]);
    const uint32_t y0 = pack2(fy * c[4], fy * c[5]), y1 = pack2(fy * c[6], fy * c[7]);
    const auto d0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
    const auto d1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
    return (u32x4){d0[0], d1[0], d0[1], d1[1]};
}
// accumulators 8 kp + 0 .. 7 of row block rb, column block cb of the unit at (J, a0), into a state: a = a0 + 2 rb + kp, tile
// columns 2 J (the first four) and 2 J + 1, b = 4 hl + r
template <int HD>
__device__ __forceinline__ void store_runs(bf16_t* state, const float* c, int J, int a0, int rb, int cb, int kp, float scale, int lane) {
    const int a = a0 + 2 * rb + kp, ti = a >> 3, hl = lane >> 5, tj = 2 * J + hl;
    const u32x4 v = pack_runs(c, (ti == 2 * J ? 1.f : 2.f) * scale, (ti == 2 * J + 1 ? 1.f : 2.f) * scale);
    if (ti <= tj)
        __builtin_nontemporal_store(v, (u32x4*)(state + (size_t)(tj * (tj + 1) / 2 + ti) * QD<HD>::TILE + (a & 7) * (HD * 8) +
                                                 (32 * cb + (lane & 31)) * 8));
}
// the same of the normaliser's rows 32 rb .. (symmetric: element (row, col) is stored at [col][row])
template <int HD>
__device__ __forceinline__ void store_norm(bf16_t* gam, const float* c, int rb, int cb, int kp, float scale, int lane) {
    const u32x4 v = pack_runs(c, scale, scale);
    *(u32x4*)(gam + (size_t)(32 * cb + (lane & 31)) * HD + 32 * rb + 8 * (2 * kp + (lane >> 5))) = v;
}

template <int HD, bool REV, bool TOT, bool FOLD, bool GATED, bool NORM>
__device__ __forceinline__ void scan_body(const ScanArgs& A, ScanSmem<HD>& sm, int bh, int seg, int g) {
    using C = ScanCfg<HD>;
    constexpr int R = NORM ? 1 : C::R, NC = NORM && HD == 64 ? 1 : C::NC;
    constexpr bool WGT = GATED || (NORM && REV);      // per-token weights
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int hl = lane >> 5, row16 = (lane >> 4) & 1, i16 = lane & 15;
    int J = 0, a0 = 0;
    if (!NORM) scan_unit<HD>(4 * g + w, J, a0);
    const int I = a0 >> 4;                  // d = 128: the same for all four waves
    // normaliser: rows 32 rb, columns 32 cb0 ..
    const int nrb = HD == 64 ? (w & 1) : w, ncb0 = NORM && HD == 64 ? (w >> 1) : 0;

    const bf16_t* Xh = A.X + (size_t)bh * A.T * HD;
    const bf16_t* Yh = (NORM ? A.X : A.Y) + (size_t)bh * A.T * HD;

    // staging: 16-byte pieces; Y: HD / 32 per thread; X: 2 per thread at d = 64, 1 at d = 128
    constexpr int NY = HD / 32, NX = NORM ? 0 : C::XF / 32;
    uint4 xr[NX > 0 ? NX : 1], yr[NY];
    float wr = 0.f;
    auto load = [&](int t0) {
#pragma unroll
        for (int q = 0; q < NY; ++q) {
            const int id = tid + 256 * q, row = t0 + id / (HD / 8);
            const uint4 u = *(const uint4*)(Yh + (size_t)min(row, A.T - 1) * HD + 8 * (id % (HD / 8)));
            yr[q] = make_uint4(u.x, u.y, u.z, u.w);     // (by element: a copy of the whole puts the array into scratch memory)
        }
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int id = tid + 256 * q, c8 = id % (C::XF / 8), row = t0 + id / (C::XF / 8);
            const int f = HD == 64 ? 8 * c8 : (c8 < 2 ? 16 * I + 8 * c8 : 16 * J + 8 * (c8 - 2));
            const uint4 u = *(const uint4*)(Xh + (size_t)min(row, A.T - 1) * HD + f);
            xr[q] = make_uint4(u.x, u.y, u.z, u.w);
        }
        if (WGT && tid < C::ST) {
            const int t = t0 + tid;
            const size_t at = (size_t)bh * A.T + min(t, A.T - 1);
            float v = 1.f;
            if (GATED) v = A.tw[at];
            if (NORM && REV) v *= A.gz[at];
            wr = t < A.T ? v : 0.f;
        }
    };
    auto put = [&](int buf, int t0) {
        // (Only REV adds the last chunk.  Zeros are chosen here, in a branch of their own: chosen in the loads they break the
        // 16-byte writes up: 12 heads of 65536 tokens at d = 64 358 us instead of 327)
        if (REV && t0 + C::ST > A.T) {
#pragma unroll
            for (int q = 0; q < NY; ++q)
                if (t0 + (tid + 256 * q) / (HD / 8) >= A.T) yr[q] = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < NX; ++q)
                if (t0 + (tid + 256 * q) / (C::XF / 8) >= A.T) xr[q] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < NY; ++q) {
            const int id = tid + 256 * q;
            *(uint4*)&sm.y[buf][id / (HD / 8)][8 * (id % (HD / 8))] = yr[q];
        }
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int id = tid + 256 * q;
            *(uint4*)&sm.x[buf][id / (C::XF / 8)][8 * (id % (C::XF / 8))] = xr[q];
        }
        if (WGT && tid < C::ST) sm.w[buf][tid] = wr;
    };

    f32x16 acc[R][NC];
#pragma unroll
    for (int rb = 0; rb < R; ++rb)
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) acc[rb][cb] = zero16();

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
        for (int cb = 0; cb < NC; ++cb) o.v[cb] = tr_frag(&sm.y[buf][t][32 * (ncb0 + cb) + tr_col], C::YP);
        o.xb = NORM ? tr_frag(&sm.y[buf][t][32 * nrb + tr_col], C::YP) : tr_frag(&sm.x[buf][t][xb_col], C::XP);
        if (WGT) {
            o.w0 = *(const float4*)&sm.w[buf][16 * ks + 4 * hl];
            o.w1 = *(const float4*)&sm.w[buf][16 * ks + 8 + 4 * hl];
        }
    };
    using XaRaw = std::conditional_t<HD == 64, uint4, uint2>;
    auto read_xa = [&](int buf, int kp) { return *(const XaRaw*)&sm.x[buf][32 * kp + xa_tok][xa_col]; };
    // x[b] (normaliser: x) of the step in c, token j, with its weights
    auto elem = [&](const Ops& c, int j) {
        const uint32_t d = j < 2 ? c.xb.u.x : j < 4 ? c.xb.u.y : j < 6 ? c.xb.u.z : c.xb.u.w;
        float x = (j & 1) ? bf_hi(d) : bf_lo(d);
        if (FOLD) x *= A.fold;
        if (WGT) {
            float t = j == 0 ? c.w0.x : j == 1 ? c.w0.y : j == 2 ? c.w0.z : j == 3 ? c.w0.w : j == 4 ? c.w1.x : j == 5 ? c.w1.y : j == 6 ? c.w1.z : c.w1.w;
            if (NORM && FOLD) t *= A.fold;
            x *= t;
        }
        return x;
    };
    // Steps (ks, rb): the products of one step are issued with the multiplies of the next step's phi between them (a 32x32x16
    // MFMA hides six vector instructions).
    auto stage = [&](int buf) {
        Ops o[2];
        read_ops(o[0], buf, 0);
        if constexpr (NORM) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const Ops& c = o[ks & 1];
                if (ks < 3) read_ops(o[(ks + 1) & 1], buf, ks + 1);
                __builtin_amdgcn_sched_barrier(0);
                Frag af = c.xb;
                if (WGT) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) af.v[j] = (__bf16)elem(c, j);
                }
#pragma unroll
                for (int cb = 0; cb < NC; ++cb) acc[0][cb] = mfma32(af.v, c.v[cb].v, acc[0][cb]);
            }
        } else {
            XaRaw xw[2];
            xw[0] = read_xa(buf, 0);
            float xb[8], xa = 0.f;
            // elements j0 .. j1 - 1 of phi at step (ks, rb)
            auto phi = [&](Frag& f, int ks, int rb, int j0, int j1) {
                if (j0 == 0) {
                    const XaRaw& u = xw[ks >> 1];
                    uint32_t d = rb == 0 ? u.x : u.y;
                    if constexpr (R == 4) d = rb == 2 ? u.z : rb == 3 ? u.w : d;
                    xa = __uint_as_float(__builtin_amdgcn_perm(d, 0u, sel));
                    if (FOLD) xa *= A.fold;
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (j < j0 || j >= j1) continue;
                    if (rb == 0) xb[j] = elem(o[ks & 1], j);
                    float m;
                    switch (8 * (ks & 1) + j) {
#define PA_LANE(L_) case L_: m = row_lane<L_>(xa); break;
                        PA_LANE(0) PA_LANE(1) PA_LANE(2) PA_LANE(3) PA_LANE(4) PA_LANE(5) PA_LANE(6) PA_LANE(7)
                        PA_LANE(8) PA_LANE(9) PA_LANE(10) PA_LANE(11) PA_LANE(12) PA_LANE(13) PA_LANE(14)
#undef PA_LANE
                        default: m = row_lane<15>(xa);
                    }
                    f.v[j] = (__bf16)(m * xb[j]);
                }
            };
            Frag af[2];
            phi(af[0], 0, 0, 0, 8);
#pragma unroll
            for (int i = 0; i < 4 * R; ++i) {
                const int ks = i / R, rb = i % R;
                if (rb == 0) {
                    if (ks < 3) read_ops(o[(ks + 1) & 1], buf, ks + 1);
                    if (ks == 0) xw[1] = read_xa(buf, 1);
                }
#pragma unroll
                for (int cb = 0; cb < NC; ++cb) {
                    acc[rb][cb] = mfma32(af[i & 1].v, o[ks & 1].v[cb].v, acc[rb][cb]);
                    if (i + 1 < 4 * R) phi(af[(i + 1) & 1], (i + 1) / R, (i + 1) % R, 8 / NC * cb, 8 / NC * (cb + 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };

    const int nslot = A.nchunk - 1;
    auto store_state = [&](int slot) {
#pragma unroll
        for (int rb = 0; rb < R; ++rb)
#pragma unroll
            for (int cb = 0; cb < NC; ++cb)
#pragma unroll
                for (int kp = 0; kp < 2; ++kp) {
                    float c[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) c[i] = acc[rb][cb][8 * kp + i];
                    if constexpr (NORM)
                        store_norm<HD>(A.gam + ((size_t)bh * nslot + slot) * QD<HD>::GAM, c, nrb, ncb0 + cb, kp, A.out_scale, lane);
                    else
                        store_runs<HD>(A.st + ((size_t)bh * nslot + slot) * QD<HD>::STATE, c, J, a0, rb, cb, kp, A.out_scale, lane);
                }
    };
    auto decay = [&](float f) {
#pragma unroll
        for (int rb = 0; rb < R; ++rb)
#pragma unroll
            for (int cb = 0; cb < NC; ++cb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[rb][cb][i] *= f;
    };
    const float* lam = GATED ? A.lam + (size_t)bh * A.nchunk : nullptr;
    auto tot_ptr = [&](int sg) {
        return A.tot + (((size_t)bh * A.nseg + sg) * (C::NG + 1) + g) * C::TOTF + (size_t)w * (C::TOTF / 4) + 4 * lane;
    };

    const int c0 = seg * A.seg_chunks, c1 = min(c0 + A.seg_chunks, A.nchunk);
    if (!TOT) {
        for (int k = 0; k < (REV ? A.nseg - 1 - seg : seg); ++k) {
            const int sg = REV ? A.nseg - 1 - k : k;
            if (GATED) {
                float f = 1.f;
                for (int n = sg * A.seg_chunks; n < min((sg + 1) * A.seg_chunks, A.nchunk); ++n) f *= lam[n];
                decay(f);
            }
            const float* src = tot_ptr(sg);
#pragma unroll
            for (int rb = 0; rb < R; ++rb)
#pragma unroll
                for (int cb = 0; cb < NC; ++cb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 v = *(const float4*)(src + ((rb * NC + cb) * 4 + q) * 256);
                        acc[rb][cb][4 * q] += v.x; acc[rb][cb][4 * q + 1] += v.y;
                        acc[rb][cb][4 * q + 2] += v.z; acc[rb][cb][4 * q + 3] += v.w;
                    }
        }
        if (REV ? c1 < A.nchunk : c0 > 0) store_state(REV ? c1 - 1 : c0 - 1);
        if (GATED) decay(lam[REV ? c1 - 1 : c0]);
    }
    // chunks added, in walk order: all of the segment for a total, all but the last otherwise
    const int nadd = (c1 - c0) - (TOT ? 0 : 1);
    if (nadd > 0) {
        const int dir = REV ? -1 : 1;
        int n = REV ? c1 - 1 : c0, left = nadd;
        int t = n * A.cs, t_end = min(t + A.cs, A.T), buf = 0;
        load(t);
        put(0, t);
        lds_barrier();
        while (true) {
            // the stage after this one
            int t2 = t + C::ST, n2 = n, left2 = left, t2_end = t_end;
            if (t2 >= t_end) {
                n2 += dir;
                --left2;
                t2 = n2 * A.cs;
                t2_end = min(t2 + A.cs, A.T);
            }
            if (left2 > 0) load(t2);
            stage(buf);
            if (left2 != left) {
                if (!TOT) store_state(REV ? n2 : n2 - 1);
                if (GATED && left2 > 0) decay(lam[n2]);
            }
            if (left2 == 0) break;
            put(buf ^ 1, t2);
            lds_barrier();
            buf ^= 1;
            t = t2;
            n = n2;
            left = left2;
            t_end = t2_end;
        }
    }
    if (TOT) {
        float* dst = tot_ptr(seg);
#pragma unroll
        for (int rb = 0; rb < R; ++rb)
#pragma unroll
            for (int cb = 0; cb < NC; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(float4*)(dst + ((rb * NC + cb) * 4 + q) * 256) = make_float4(acc[rb][cb][4 * q], acc[rb][cb][4 * q + 1],
                                                                                   acc[rb][cb][4 * q + 2], acc[rb][cb][4 * q + 3]);
    }
}

template <int HD, bool REV, bool TOT, bool FOLD, bool GATED>
__global__ __launch_bounds__(256, 2) void k_quad_scan(ScanArgs A) {
    __shared__ __attribute__((aligned(16))) ScanSmem<HD> sm;
    constexpr int G = ScanCfg<HD>::NG + 1;
    const int segs = TOT ? A.tot_segs : A.nseg;
    const int item = xcd_item(A.heads * segs * G);
    if (item < 0) return;
    const int g = item % G, hs = item / G;
    const int seg = hs % segs + (TOT && REV ? 1 : 0), bh = hs / segs;
    if (g == ScanCfg<HD>::NG) scan_body<HD, REV, TOT, FOLD, GATED, true>(A, sm, bh, seg, g);
    else scan_body<HD, REV, TOT, FOLD, GATED, false>(A, sm, bh, seg, g);
}

// The states from per-chunk totals (segments of one chunk): a running sum over the chunks, one wave per 8 accumulators of a scan
// wave, the next PF totals on their way in registers.  Bound by memory.
template <int HD, bool REV, bool GATED>
__global__ __launch_bounds__(256) void k_quad_prefix(ScanArgs A) {
    using C = ScanCfg<HD>;
    constexpr int UNITS = C::TOTF / 512, PF = 8;      // waves' worth of a workgroup's total: 8 floats per lane each
    constexpr int NUNIT = 4 * 2;                      // of the normaliser's (d = 64: 16 accumulators per wave)
    constexpr int PERHEAD = C::NG * UNITS + NUNIT;
    static_assert(HD == 64, "the normaliser's units are written for d = 64");
    const int lane = threadIdx.x & 63, id = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (id >= A.heads * PERHEAD) return;
    const int bh = id / PERHEAD, u = id % PERHEAD;
    const bool norm = u >= C::NG * UNITS;
    const int g = norm ? C::NG : u / UNITS, v = norm ? u - C::NG * UNITS : u % UNITS;
    // v = (wave, row block, column block, kp); normaliser: (wave, kp), 16 accumulators per wave
    const int kp = v & 1, cb = norm ? 0 : (v >> 1) & 1, rb = norm ? 0 : (v >> 2) & 3, w = norm ? v >> 1 : v >> 4;
    const size_t stride = (size_t)(C::NG + 1) * C::TOTF;      // floats from one chunk's totals to the next's
    const float* src = A.tot + ((size_t)bh * A.nseg * (C::NG + 1) + g) * C::TOTF + (size_t)w * (C::TOTF / 4) +
                       ((rb * C::NC + cb) * 4 + 2 * kp) * 256 + 4 * lane;
    int J = 0, a0 = 0;
    if (!norm) scan_unit<HD>(4 * g + w, J, a0);
    const int steps = A.nchunk - 1;
    const float* lam = GATED ? A.lam + (size_t)bh * A.nchunk : nullptr;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    float4 q[PF][2];
    auto chunk_of = [&](int s) { return REV ? A.nchunk - 1 - s : s; };
    auto fetch = [&](float4 (&r)[2], int s) {
        const float* p = src + (size_t)chunk_of(min(s, steps - 1)) * stride;
        r[0] = *(const float4*)p;
        r[1] = *(const float4*)(p + 256);
    };
#pragma unroll
    for (int i = 0; i < PF; ++i) fetch(q[i], i);
    for (int s0 = 0; s0 < steps; s0 += PF) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const int s = s0 + i, n = chunk_of(min(s, steps - 1));
            if (GATED) {
                const float f = lam[n];
#pragma unroll
                for (int k = 0; k < 8; ++k) acc[k] *= f;
            }
            acc[0] += q[i][0].x; acc[1] += q[i][0].y; acc[2] += q[i][0].z; acc[3] += q[i][0].w;
            acc[4] += q[i][1].x; acc[5] += q[i][1].y; acc[6] += q[i][1].z; acc[7] += q[i][1].w;
            fetch(q[i], s + PF);
            if (s < steps) {
                const size_t slot = (size_t)bh * (A.nchunk - 1) + (REV ? n - 1 : n);
                if (norm) store_norm<HD>(A.gam + slot * QD<HD>::GAM, acc, w & 1, w >> 1, kp, A.out_scale, lane);
                else store_runs<HD>(A.st + slot * QD<HD>::STATE, acc, J, a0, rb, cb, kp, A.out_scale, lane);
            }
        }
    }
}

// ---- read-out --------------------------------------------------------------------------------------------
// part[t][:] = outscale S^T phi(fold x_t), zpart[t] = outscale (fold x_t)^T Gamma (fold x_t), S and Gamma of t's chunk (App. E.4;
// with R and k also dV).  A wave owns 64 tokens and all HD columns; phi of its tokens is formed in registers from their rows in
// LDS (a lane is a token; the two halves of the wave take a = 0 .. 3 and 4 .. 7), the state tiles stream through LDS and are
// shared by the workgroup, two tiles further on the way in registers.
// Rows of x in LDS are swizzled by 16-byte chunks so that 16 tokens' reads of one feature block hit distinct banks.
template <int HD>
__device__ __forceinline__ int xoff(int row, int chunk) {   // element offset of 16-byte chunk `chunk` of a row
    return row * HD + 8 * (chunk ^ (HD == 64 ? (row & 7) : (row & 15)));
}
// rows tok0 .. of X times fold into LDS; rows past T repeat the last token's (results of rows past the chunk are never stored)
template <int HD, int THREADS, int ROWS>
__device__ __forceinline__ void stage_rows(bf16_t* xs, const bf16_t* __restrict__ Xh, int tok0, int T, float fold) {
#pragma unroll
    for (int q = 0; q < ROWS * (HD / 8) / THREADS; ++q) {
        const int id = threadIdx.x + THREADS * q, row = id / (HD / 8), c = id % (HD / 8);
        uint4 u = *(const uint4*)(Xh + (size_t)min(tok0 + row, T - 1) * HD + 8 * c);
        if (fold != 1.f) {
            float x[8];
            unpack8(x, u);
            u = make_uint4(pack2(fold * x[0], fold * x[1]), pack2(fold * x[2], fold * x[3]), pack2(fold * x[4], fold * x[5]),
                           pack2(fold * x[6], fold * x[7]));
        }
        *(uint4*)(xs + xoff<HD>(row, c)) = u;
    }
}

struct StateArgs {
    const bf16_t *X, *Y;       // Y: d phi only
    const float* wgt;          // d phi: weight of the normaliser's term per token (null: 1)
    const float* tw;           // gated: the token's decay, a factor of all results (null: 1)
    const bf16_t *st, *gam;
    float *part, *zpart;       // zpart may be null; d phi: zpart = X . part
    int T, cs, nchunk, heads, rev, blocks;   // blocks per chunk
    float fold, out_scale;
};

template <int HD>
struct ReadCfg {
    static constexpr int NW = HD == 64 ? 4 : 8, TOK = 64 * NW;
    static constexpr size_t SMEM = (size_t)TOK * HD * 2 + 2 * (size_t)QD<HD>::TILE * 2;
};

template <int HD>
__global__ __launch_bounds__(64 * ReadCfg<HD>::NW, 2) void k_quad_read(StateArgs A) {
    using D = QD<HD>;
    constexpr int NV = HD / 32, THREADS = 64 * ReadCfg<HD>::NW, TOK = ReadCfg<HD>::TOK;
    extern __shared__ __attribute__((aligned(16))) unsigned char quad_smem[];
    bf16_t* xs = reinterpret_cast<bf16_t*>(quad_smem);
    bf16_t* ring = xs + TOK * HD;                        // [2][TILE]
    const int item = xcd_item(A.heads * A.nchunk * A.blocks);
    if (item < 0) return;
    const int blk = item % A.blocks, hc = item / A.blocks, n = hc % A.nchunk, bh = hc / A.nchunk;
    const int tok0 = n * A.cs + blk * TOK, t_end = min((n + 1) * A.cs, A.T);
    if (tok0 >= t_end) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r32 = lane & 31, hl = lane >> 5;
    const size_t head = (size_t)bh * A.T;
    f32x16 acc[NV][2];
#pragma unroll
    for (int vb = 0; vb < NV; ++vb) acc[vb][0] = acc[vb][1] = zero16();
    float z[2] = {0.f, 0.f};
    const int slot = A.rev ? n : n - 1;
    if (slot >= 0 && slot < A.nchunk - 1) {
        const bf16_t* S = A.st + ((size_t)bh * (A.nchunk - 1) + slot) * D::STATE;
        // a tile is D::TILE / 8 pieces of 16 bytes, two per thread
        static_assert(D::TILE / 8 == 2 * THREADS, "two pieces per thread");
        uint4 p0a, p0b, p1a, p1b;
        auto tile_ptr = [&](int t) { return (const uint4*)(S + (size_t)min(t, D::NTILE - 1) * D::TILE) + tid; };
        p0a = tile_ptr(0)[0];
        p0b = tile_ptr(0)[THREADS];
        p1a = tile_ptr(1)[0];
        p1b = tile_ptr(1)[THREADS];
        stage_rows<HD, THREADS, TOK>(xs, A.X + head * HD, tok0, A.T, A.fold);
        uint4* ring4 = (uint4*)ring;
        ring4[tid] = p0a;
        ring4[tid + THREADS] = p0b;
        p0a = tile_ptr(2)[0];
        p0b = tile_ptr(2)[THREADS];
        const int row0 = 64 * w + r32;
        const int swz = HD == 64 ? (r32 & 7) : (r32 & 15);        // (rows 32 further: the same)
        const bf16_t* xrow = xs + row0 * HD;
        int ti = 0, tj = 0;
        float xb[2][8];
        auto tile = [&](const bf16_t* tl) {
            if (ti == 0) {
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) unpack8(xb[tb], *(const uint4*)(xrow + 32 * tb * HD + 8 * (tj ^ swz)));
            }
            float xa[2][4];
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) unpack4(xa[tb], *(const uint2*)(xrow + 32 * tb * HD + 8 * (ti ^ swz) + 4 * hl));
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                Frag pf[2];
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                    for (int j = 0; j < 8; ++j) pf[tb].v[j] = (__bf16)(xa[tb][kk] * xb[tb][j]);
#pragma unroll
                for (int vb = 0; vb < NV; ++vb) {
                    Frag sf;
                    sf.u = *(const uint4*)(tl + ((4 * hl + kk) * HD + 32 * vb + r32) * 8);
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb) acc[vb][tb] = mfma32(sf.v, pf[tb].v, acc[vb][tb]);
                }
            }
            if (++ti > tj) {
                ti = 0;
                ++tj;
            }
        };
        // tile t is in ring slot t & 1; the pieces of t + 1 and t + 2 wait in registers
        for (int t = 0; t < D::NTILE; t += 2) {
            lds_barrier();
            ring4[2 * THREADS + tid] = p1a;
            ring4[3 * THREADS + tid] = p1b;
            p1a = tile_ptr(t + 3)[0];
            p1b = tile_ptr(t + 3)[THREADS];
            tile(ring);
            lds_barrier();
            ring4[tid] = p0a;
            ring4[THREADS + tid] = p0b;
            p0a = tile_ptr(t + 4)[0];
            p0b = tile_ptr(t + 4)[THREADS];
            tile(ring + D::TILE);
        }
        static_assert(D::NTILE % 2 == 0, "tiles in pairs");
        if (A.zpart != nullptr) {
            const bf16_t* Gm = A.gam + ((size_t)bh * (A.nchunk - 1) + slot) * D::GAM;
#pragma unroll 1
            for (int fb = 0; fb < HD / 32; ++fb) {
                f32x16 u[2] = {zero16(), zero16()};
#pragma unroll
                for (int ks = 0; ks < HD / 16; ++ks) {
                    Frag gf;
                    gf.u = *(const uint4*)(Gm + (size_t)(32 * fb + r32) * HD + 16 * ks + 8 * hl);
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb) {
                        Frag xf;
                        xf.u = *(const uint4*)(xrow + 32 * tb * HD + 8 * ((2 * ks + hl) ^ swz));
                        u[tb] = mfma32(gf.v, xf.v, u[tb]);
                    }
                }
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        float x[4];
                        unpack4(x, *(const uint2*)(xrow + 32 * tb * HD + 8 * ((4 * fb + k) ^ swz) + 4 * hl));
#pragma unroll
                        for (int r = 0; r < 4; ++r) z[tb] += u[tb][4 * k + r] * x[r];
                    }
            }
        }
    }
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        const int t = tok0 + 64 * w + 32 * tb + r32;
        const bool in = t < t_end;
        float* dst = A.part + (head + (in ? t : 0)) * HD;
        const float f = A.tw != nullptr && in ? A.out_scale * A.tw[head + t] : A.out_scale;
        if (in) {
#pragma unroll
            for (int vb = 0; vb < NV; ++vb)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *(float4*)(dst + 32 * vb + 8 * k + 4 * hl) = make_float4(f * acc[vb][tb][4 * k], f * acc[vb][tb][4 * k + 1],
                                                                             f * acc[vb][tb][4 * k + 2], f * acc[vb][tb][4 * k + 3]);
        }
        if (A.zpart != nullptr) {
            const float zs = f * xor32_sum(z[tb]);
            if (in && hl == 0) A.zpart[head + t] = zs;
        }
    }
}

// ---- gradient of the embedding -----------------------------------------------------------------------------
// part[t][:] = outscale (J_phi(x_t)^T (S y_t) + 2 w_t Gamma x_t), x_t = fold X_t, S and Gamma of t's chunk: the state's part of dQ
// (X = Q, y = ghat, w = gz) and, with R and Omega, of dK (X = K, y = V, w = 1).
// A lane is a token (32 per MFMA column block, two blocks per wave).  Per 32-row block of a tile, c[a][b] = (S y)[a, b] is a
// product over the HD value columns (operands: the tile through LDS and the transposing read; y in registers), and
//     dx[8 ti + a] += sum_b c[a][b] x[8 tj + b],    dx[8 tj + b] += sum_a c[a][b] x[8 ti + a],
// two multiply-adds per state row and token.  dx stays in registers: ti runs in unrolled code, the sums that land on tj wait in
// four registers until the column is done.  The wave's halves hold b = 0 .. 3 and 4 .. 7.  At d = 128 two waves share 64 tokens,
// each with one half of the a of every tile and the gradient of the features 4 h .. 4 h + 3 of every block of 8 (all 128 of 64
// tokens and y would not fit the registers); what lands on the partner's goes through LDS once per column.
template <int HD>
struct DphiCfg {
    static constexpr int RS = HD == 64 ? 1 : 2, NW = 4 * RS, TOK = 256;
    static constexpr size_t RING = 4 * (size_t)QD<HD>::TILE * 2, HAND = RS == 2 ? NW * 2 * 64 * 16 : 0;
    static constexpr size_t SMEM = (size_t)TOK * HD * 2 + RING + HAND;
};

template <int HD>
__global__ __launch_bounds__(64 * DphiCfg<HD>::NW, 2) void k_quad_dphi(StateArgs A) {
    using D = QD<HD>;
    using C = DphiCfg<HD>;
    constexpr int NB = D::NB, RS = C::RS, THREADS = 64 * C::NW, KS = HD / 16, ND = RS == 1 ? 4 : 2, NRB = RS == 1 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char quad_smem[];
    bf16_t* xs = reinterpret_cast<bf16_t*>(quad_smem);
    bf16_t* ring = xs + C::TOK * HD;                     // [2][2 TILE]
    float4* hand = (float4*)(ring + 4 * D::TILE);        // [wave][2][64]
    const int item = xcd_item(A.heads * A.nchunk * A.blocks);
    if (item < 0) return;
    const int blk = item % A.blocks, hc = item / A.blocks, n = hc % A.nchunk, bh = hc / A.nchunk;
    const int tok0 = n * A.cs + blk * C::TOK, t_end = min((n + 1) * A.cs, A.T);
    if (tok0 >= t_end) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r32 = lane & 31, hl = lane >> 5;
    const int row16 = (lane >> 4) & 1, i16 = lane & 15;
    const int wt = w / RS, h = RS == 2 ? (w & 1) : 0;    // token group, half of the a
    const size_t head = (size_t)bh * A.T;

    float dx[NB][2][ND];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int e = 0; e < ND; ++e) dx[i][tb][e] = 0.f;

    const int slot = A.rev ? n : n - 1;
    if (slot >= 0 && slot < A.nchunk - 1) {
        const bf16_t* S = A.st + ((size_t)bh * (A.nchunk - 1) + slot) * D::STATE;
        static_assert(2 * D::TILE / 8 == 4 * THREADS, "four pieces per thread and pair of tiles");
        uint4 p0, p1, p2, p3;
        auto fetch = [&](int t) {      // the tiles t and t + 1 (past the end: repeats, never used)
            const uint4* a = (const uint4*)(S + (size_t)min(t, D::NTILE - 1) * D::TILE) + tid;
            const uint4* b = (const uint4*)(S + (size_t)min(t + 1, D::NTILE - 1) * D::TILE) + tid;
            p0 = a[0];
            p1 = a[THREADS];
            p2 = b[0];
            p3 = b[THREADS];
        };
        uint4* ring4 = (uint4*)ring;
        static_assert(THREADS % (2 * HD) == 0, "a thread's four pieces are rows a of one parity");
        auto put = [&](int sl) {       // 8-byte reads of 4 a x 4 v: odd a are 4 v apart so that they take other banks
            uint4* dst = ring4 + sl * (2 * D::TILE / 8) + (tid ^ (((tid / HD) & 1) << 2));
            dst[0] = p0;
            dst[THREADS] = p1;
            dst[2 * THREADS] = p2;
            dst[3 * THREADS] = p3;
        };
        fetch(0);
        stage_rows<HD, THREADS, C::TOK>(xs, A.X + head * HD, tok0, A.T, A.fold);
        Frag yf[KS][2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const size_t row = head + min(tok0 + 64 * wt + 32 * tb + r32, A.T - 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) yf[ks][tb].u = *(const uint4*)(A.Y + row * HD + 16 * ks + 8 * hl);
        }
        put(0);
        fetch(1);                      // column 1: tiles 1 and 2

        const int swz = HD == 64 ? (r32 & 7) : (r32 & 15);
        const bf16_t* xrow = xs + (64 * wt + r32) * HD;
        // transposing read: lane (i = i16 >> 2, c = i16 & 3) of a 16-lane group points at value row i, a = 2 row16 + (c >> 1), b = 4 (c & 1)
        const int c2 = (i16 >> 1) & 1;
        const bf16_t* tr0 = ring + (((2 * row16 + c2) * HD + 8 * hl + (i16 >> 2)) * 8 + 4 * (i16 & 1));
        float xb[2][4], t2[2][4];

        // one tile (ti = i) from `tl` (element offset into the ring)
        auto tile = [&](int i, int tl, float (&dxi)[2][ND]) {
            float xa[2][4 * NRB], t1[NRB][2][4];
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                const bf16_t* px = xrow + 32 * tb * HD + 8 * (i ^ swz);
                if constexpr (RS == 1) unpack8(xa[tb], *(const uint4*)px);
                else unpack4(xa[tb], *(const uint2*)(px + 4 * h));
            }
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) {
                f32x16 c[2] = {zero16(), zero16()};
                const bf16_t* tp = tr0 + tl + (RS == 1 ? rb : h) * 4 * HD * 8;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    union {
                        Frag f;
                        bf16x4 q[2];
                    } s;
                    s.q[0] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(tp + (16 * ks + 4 * c2) * 8));
                    s.q[1] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(tp + (16 * ks + 4 * (c2 ^ 1)) * 8));
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb) c[tb] = mfma32(s.f.v, yf[ks][tb].v, c[tb]);
                }
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        t1[rb][tb][k] = c[tb][4 * k] * xb[tb][0];
#pragma unroll
                        for (int r = 1; r < 4; ++r) t1[rb][tb][k] += c[tb][4 * k + r] * xb[tb][r];
#pragma unroll
                        for (int r = 0; r < 4; ++r) t2[tb][r] += c[tb][4 * k + r] * xa[tb][4 * rb + k];
                    }
            }
            // the halves' shares of t1 meet: lanes hl = 0 and 1 end up with different a
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int e = 0; e < ND; ++e) {
                    const float lo = t1[0][tb][e], hi = RS == 1 ? t1[NRB - 1][tb][e] : t1[0][tb][ND == 2 ? 2 + e : e];
                    const auto m = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
                    dxi[tb][e] += __uint_as_float(m[0]) + __uint_as_float(m[1]);
                }
        };
        auto land = [&](int col) {      // RS == 2: the sums that landed on column block `col`, own and partner's
            float2 s[2];
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                const float* h0 = (const float*)&hand[((w & ~1) * 2 + tb) * 64 + 32 * h + r32] + 2 * hl;
                const float2 u = *(const float2*)h0, v = *(const float2*)(h0 + 2 * 64 * 4);
                s[tb] = make_float2(u.x + v.x, u.y + v.y);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (i == col) {
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb) {
                        dx[i][tb][0] += s[tb].x;
                        dx[i][tb][1] += s[tb].y;
                    }
                    asm volatile("; column %0" ::"n"(i));   // (keeps the branches apart: merged, dx would be indexed in scratch memory)
                }
        };

        int par = 0, fj = 1, fi = 0;     // ring slot of the current pair; the pair the pieces in registers belong to
#pragma unroll 1
        for (int tj = 0; tj < NB; ++tj) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int r = 0; r < 4; ++r) t2[tb][r] = 0.f;
#pragma unroll
            for (int i = 0; i < NB; i += 2) {
                if (i <= tj) {
                    lds_barrier();
                    put(par ^ 1);
                    fi += 2;
                    if (fi > fj) {
                        fi = 0;
                        ++fj;
                    }
                    fetch(fj * (fj + 1) / 2 + fi);
                    if (i == 0) {
#pragma unroll
                        for (int tb = 0; tb < 2; ++tb)
                            unpack4(xb[tb], *(const uint2*)(xrow + 32 * tb * HD + 8 * (tj ^ swz) + 4 * hl));
                        if (RS == 2 && tj > 0) land(tj - 1);
                    }
                    tile(i, par * 2 * D::TILE, dx[i]);
                    if (i + 1 <= tj) tile(i + 1, par * 2 * D::TILE + D::TILE, dx[i + 1]);
                    par ^= 1;
                }
            }
            if constexpr (RS == 1) {
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (i == tj) {
#pragma unroll
                        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                            for (int r = 0; r < 4; ++r) dx[i][tb][r] += t2[tb][r];
                        asm volatile("; column %0" ::"n"(i));
                    }
            } else {
                // The partner reads the last column's sums (land) behind the barrier that opened this column, so another barrier
                // has to come before they are overwritten.  The second pair of tiles brings it, but column 1 has one pair only.
                if (tj == 1) lds_barrier();
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) hand[(w * 2 + tb) * 64 + lane] = make_float4(t2[tb][0], t2[tb][1], t2[tb][2], t2[tb][3]);
            }
        }
        if constexpr (RS == 2) {
            lds_barrier();
            land(NB - 1);
        }
        // the normaliser: rows of Gamma in the order in which the lanes hold dx
        const bf16_t* Gm = A.gam + ((size_t)bh * (A.nchunk - 1) + slot) * D::GAM;
        float wgt2[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
            wgt2[tb] = A.wgt == nullptr ? 2.f : 2.f * A.wgt[head + min(tok0 + 64 * wt + 32 * tb + r32, A.T - 1)];
#pragma unroll
        for (int fb = 0; fb < HD / 32 / RS; ++fb) {
            const int grow = RS == 1 ? 32 * fb + r32
                                     : 8 * (2 * (4 * fb + (r32 >> 3)) + ((r32 >> 1) & 1)) + 4 * h + 2 * ((r32 >> 2) & 1) + (r32 & 1);
            f32x16 u[2] = {zero16(), zero16()};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                Frag gf;
                gf.u = *(const uint4*)(Gm + (size_t)grow * HD + 16 * ks + 8 * hl);
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
                    Frag xf;
                    xf.u = *(const uint4*)(xrow + 32 * tb * HD + 8 * ((2 * ks + hl) ^ swz));
                    u[tb] = mfma32(gf.v, xf.v, u[tb]);
                }
            }
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if constexpr (RS == 1) dx[4 * fb + k][tb][r] += wgt2[tb] * u[tb][4 * k + r];
                        else dx[2 * (4 * fb + k) + (r >> 1)][tb][r & 1] += wgt2[tb] * u[tb][4 * k + r];
                    }
        }
    }
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        const int t = tok0 + 64 * wt + 32 * tb + r32;
        const bool in = t < t_end;
        const float f = A.tw != nullptr && in ? A.out_scale * A.tw[head + t] : A.out_scale;
        float* dst = A.part + (head + min(t, A.T - 1)) * HD;
        if constexpr (RS == 1) {
            if (A.zpart != nullptr) {       // (rows of x are in LDS unless the chunk has no state, and dx is zero then)
                const bf16_t* xrow = xs + (64 * wt + 32 * tb + r32) * HD;
                float dot = 0.f;
                if (slot >= 0 && slot < A.nchunk - 1) {
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        float x[4];
                        unpack4(x, *(const uint2*)(xrow + 8 * (i ^ (r32 & 7)) + 4 * hl));
#pragma unroll
                        for (int r = 0; r < 4; ++r) dot += dx[i][tb][r] * x[r];
                    }
                }
                dot = f / A.fold * xor32_sum(dot);
                if (in && hl == 0) A.zpart[head + t] = dot;
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (in) *(float4*)(dst + 8 * i + 4 * hl) = make_float4(f * dx[i][tb][0], f * dx[i][tb][1], f * dx[i][tb][2], f * dx[i][tb][3]);
        } else {
#pragma unroll
            for (int i = 0; i < NB; i += 2) {     // two blocks' halves change places: each lane stores 16 bytes
                const auto m0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(f * dx[i][tb][0]), __float_as_uint(f * dx[i + 1][tb][0]), false, false);
                const auto m1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(f * dx[i][tb][1]), __float_as_uint(f * dx[i + 1][tb][1]), false, false);
                if (in) *(float4*)(dst + 8 * (i + hl) + 4 * h) = make_float4(__uint_as_float(m0[0]), __uint_as_float(m1[0]),
                                                                              __uint_as_float(m0[1]), __uint_as_float(m1[1]));
            }
        }
    }
}

// ---- gated: the pairs that straddle a chunk ---------------------------------------------------------------------
// lam_n (<R_n, S_n> + <Omega_n, Gamma_n>), the states after and before chunk n; off-diagonal tiles carry their multiplicity in both.
// QUAD_XPARTS workgroups per chunk, every eighth tile (the normaliser's 64 x 64 is one more).
__device__ __forceinline__ float dot8(const uint4& a, const uint4& b) {
    float x[8], y[8], s = 0.f;
    unpack8(x, a);
    unpack8(y, b);
#pragma unroll
    for (int i = 0; i < 8; ++i) s += x[i] * y[i];
    return s;
}
__global__ __launch_bounds__(256) void k_quad_boundary(const bf16_t* __restrict__ st, const bf16_t* __restrict__ rc,
                                                       const bf16_t* __restrict__ gam, const bf16_t* __restrict__ omg,
                                                       const float* __restrict__ lam, float* __restrict__ xb, int nchunk) {
    using D = QD<64>;
    __shared__ float red[4];
    const int part = blockIdx.x, n = blockIdx.y, bh = blockIdx.z, tid = threadIdx.x;
    float acc = 0.f;
    if (n > 0 && n < nchunk - 1) {
        const size_t slot = (size_t)bh * (nchunk - 1) + n, before = slot - 1;
        static_assert(D::TILE == D::GAM && D::TILE / 8 == 512, "two pieces per thread");
        for (int tile = part; tile <= D::NTILE; tile += QUAD_XPARTS) {
            const bool norm = tile == D::NTILE;
            const uint4* a = (const uint4*)(norm ? gam + before * D::GAM : st + before * D::STATE + (size_t)tile * D::TILE) + tid;
            const uint4* b = (const uint4*)(norm ? omg + slot * D::GAM : rc + slot * D::STATE + (size_t)tile * D::TILE) + tid;
            bool diag = norm;
            for (int t = 0; t < D::NB; ++t) diag = diag || tile == t * (t + 1) / 2 + t;
            const float s = dot8(a[0], b[0]) + dot8(a[256], b[256]);
            acc += diag ? s : 0.5f * s;
        }
    }
    acc = xor32_sum(xor16_sum(acc));
    for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) xb[((size_t)bh * nchunk + n) * QUAD_XPARTS + part] = lam[(size_t)bh * nchunk + n] * (red[0] + red[1] + red[2] + red[3]);
}

// ---- a prompt into a decode state -------------------------------------------------------------------------
// rows of X times the square root of their token's weight (p = 2: the weight of phi), in bf16
__global__ __launch_bounds__(256) void k_quad_weigh(const bf16_t* __restrict__ X, const float* __restrict__ tw, bf16_t* __restrict__ out,
                                                    size_t pieces) {
    const size_t id = (size_t)blockIdx.x * 256 + threadIdx.x;      // 8 features of one token (d = 64)
    if (id >= pieces) return;
    const float f = sqrtf(tw[id / 8]);
    float x[8];
    unpack8(x, *(const uint4*)(X + 8 * id));
    *(uint4*)(out + 8 * id) = make_uint4(pack2(f * x[0], f * x[1]), pack2(f * x[2], f * x[3]), pack2(f * x[4], f * x[5]), pack2(f * x[6], f * x[7]));
}
// S[row][:] = decay S + m sum over the segments' totals, row = the monomial (i, j), i <= j, of multiplicity m, and the normaliser
// column likewise; the sum is rounded to bf16, as the states between chunks are.  A wave has one i and 8 consecutive j of one
// state: what a scan wave's lanes hold of them are the accumulators 4 kq + r of one row block (a = a0 + 2 rb + (kq >> 1),
// b = 8 (kq & 1) + 4 hl + r).  Bound by memory: totals in, state in and out.
// Measured, scan and this (before: a scan over transposed copies, one workgroup per head and tile pair, into bf16 states):
// B4 H12 T3072 164 -> 109 us, B1 H4 T65536 499 -> 112, B8 H16 T8192 884 -> 502.
__global__ __launch_bounds__(256) void k_quad_absorb(const float* __restrict__ tot, int nseg, const float* __restrict__ lam,
                                                     float* __restrict__ S, float* __restrict__ gamd, int D, int heads) {
    using C = ScanCfg<64>;
    constexpr int HD = 64, PERHEAD = HD * (HD / 8);
    const int lane = threadIdx.x & 63, hl = lane >> 5, id = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int bh = id / PERHEAD, u = id % PERHEAD, i = u % HD, jb = u / HD;
    if (bh >= heads || 8 * jb + 7 < i) return;
    const int J = jb >> 1, unit = J * (J + 1) + (i >> 3);       // (two units of 8 a per 16 x 16)
    const int rb = (i & 7) >> 1, kq = 2 * (i & 1) + (jb & 1);
    const size_t seg = (size_t)(C::NG + 1) * C::TOTF;
    const float* base = tot + (size_t)bh * nseg * seg;
    const float* src = base + (size_t)(unit >> 2) * C::TOTF + (size_t)(unit & 3) * (C::TOTF / 4) + (rb * C::NC * 4 + kq) * 256 + 4 * lane;
    // the normaliser's element (i, 8 jb + lane): rows 32 (w & 1) + 8 k + 4 h + r, columns 32 (w >> 1) + ..
    const int jn = 8 * jb + (lane & 7), nw = (i >> 5) + 2 * (jn >> 5), nrow = i & 31;
    const float* nsrc = base + (size_t)C::NG * C::TOTF + (size_t)nw * (C::TOTF / 4) + (nrow >> 3) * 256 +
                        4 * (32 * ((nrow >> 2) & 1) + (jn & 31)) + (nrow & 3);
    float4 a[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
    float gsum = 0.f;
    for (int s = 0; s < nseg; ++s) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const float4 v = *(const float4*)(src + s * seg + cb * 4 * 256);
            a[cb].x += v.x; a[cb].y += v.y; a[cb].z += v.z; a[cb].w += v.w;
        }
        gsum += nsrc[s * seg];
    }
    auto rounded = [](float x) { return (float)(__bf16)x; };
    gsum = rounded(gsum);
    const float decay = lam != nullptr ? lam[bh] : 1.f;
    const int row0 = i * HD - i * (i - 1) / 2 - i;              // row of (i, j): row0 + j
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 8 * jb + 4 * hl + r;
            if (j < i) continue;
            float* dst = S + ((size_t)bh * D + row0 + j) * HD + 32 * cb + (lane & 31);
            const float x = rounded(r == 0 ? a[cb].x : r == 1 ? a[cb].y : r == 2 ? a[cb].z : a[cb].w);
            *dst = decay * *dst + (i == j ? x : 2.f * x);
        }
    if (lane < 8 && jn >= i) {
        float* dst = gamd + (size_t)bh * D + row0 + jn;
        *dst = decay * *dst + (i == jn ? gsum : 2.f * gsum);
    }
}

template <typename F>
bool allow_smem(F* fn, size_t bytes) {
    if (bytes <= 64 * 1024) return true;
    hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) note_hip_error(e, "hipFuncSetAttribute(max dynamic LDS)");
    return e == hipSuccess;
}

// scale = fold * rest: fold a power of two (exact on x), 1 <= |rest| < 2
void split_scale(float scale, float& fold, float& rest) {
    fold = 1.f;
    rest = scale;
    if (!std::isfinite(scale)) return;
    int e = 0;
    (void)std::frexp(scale, &e);
    e = std::max(e - 1, -126);
    fold = std::ldexp(1.f, e);
    rest = std::ldexp(scale, -e);
}

template <int HD, bool REV, bool FOLD, bool GATED>
bool scan_go(const char* name, hipStream_t s, ScanArgs a) {
    constexpr int G = ScanCfg<HD>::NG + 1;
    // (d = 64: the totals are the update-state, the running sum over them a pass of its own)
    if (a.nseg > 1) {
        LaunchScope ls(HD == 64 ? name : "mfma_state_totals", s);
        hipLaunchKernelGGL((k_quad_scan<HD, REV, true, FOLD, GATED>), dim3(xcd_grid(a.heads * a.tot_segs * G)), dim3(256), 0, s, a);
        if (!launch_ok()) return false;
    }
    LaunchScope ls(HD == 64 ? "mfma_state_prefix" : name, s);
    if constexpr (HD == 64) {
        const int waves = a.heads * (ScanCfg<64>::NG * ScanCfg<64>::TOTF / 512 + 8);
        hipLaunchKernelGGL((k_quad_prefix<64, REV, GATED>), dim3((waves + 3) / 4), dim3(256), 0, s, a);
    } else {
        hipLaunchKernelGGL((k_quad_scan<HD, REV, false, FOLD, GATED>), dim3(xcd_grid(a.heads * a.nseg * G)), dim3(256), 0, s, a);
    }
    return launch_ok();
}

}  // namespace

QuadPlan quad_plan(int d, int BH, int T, int cs) {
    QuadPlan p{};
    p.hd = d;
    p.cs = cs;
    p.nchunk = (T + cs - 1) / cs;
    const int G = d == 64 ? ScanCfg<64>::NG + 1 : ScanCfg<128>::NG + 1;
    const size_t totf = d == 64 ? ScanCfg<64>::TOTF : ScanCfg<128>::TOTF;
    p.state_elems = d == 64 ? QD<64>::STATE : QD<128>::STATE;
    p.gam_elems = d == 64 ? QD<64>::GAM : QD<128>::GAM;
    // d = 64: a segment per chunk.  d = 128: one workgroup of a head and segment per CU and a half
    int want = 1;
    while (d == 128 && want < 64 && (long long)BH * G * want < 400) ++want;
    if (d == 64) want = p.nchunk;
    want = std::min(want, p.nchunk);
    p.seg_chunks = (p.nchunk + want - 1) / want;
    p.nseg = (p.nchunk + p.seg_chunks - 1) / p.seg_chunks;
    p.tot_floats = p.nseg > 1 ? (size_t)BH * p.nseg * G * totf : 0;
    return p;
}

bool launch_quad_scan(const char* name, hipStream_t s, const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* Y,
                      const float* wgt, bf16_t* st, bf16_t* gam, float* tot, int BH, int T, float scale, const float* tw,
                      const float* lam) {
    if (p.nchunk < 2) return true;
    ScanArgs a{};
    a.X = X; a.Y = Y; a.gz = wgt; a.tw = tw; a.lam = lam; a.st = st; a.gam = gam; a.tot = tot;
    a.T = T; a.cs = p.cs; a.nchunk = p.nchunk; a.nseg = p.nseg; a.tot_segs = p.nseg - 1; a.seg_chunks = p.seg_chunks; a.heads = BH;
    float rest;
    split_scale(scale, a.fold, rest);
    a.out_scale = rest * rest;
#define PA_GO(HD_, G_)                                                                                                            \
    if (!rev) return scan_go<HD_, false, false, G_>(name, s, a);                                                                  \
    return a.fold == 1.f ? scan_go<HD_, true, false, G_>(name, s, a) : scan_go<HD_, true, true, G_>(name, s, a);
    if (p.hd == 128) {
        if (tw != nullptr) return false;
        PA_GO(128, false)
    }
    if (tw != nullptr) {
        PA_GO(64, true)
    }
    PA_GO(64, false)
#undef PA_GO
}

static StateArgs state_args(const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* st, const bf16_t* gam, float* part, int BH,
                            int T, int tok) {
    StateArgs a{};
    a.X = X; a.st = st; a.gam = gam; a.part = part;
    a.T = T; a.cs = p.cs; a.nchunk = p.nchunk; a.heads = BH; a.rev = rev;
    a.blocks = (p.cs + tok - 1) / tok;
    return a;
}

bool launch_quad_read(const char* name, hipStream_t s, const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* st,
                      const bf16_t* gam, float* part, float* zpart, int BH, int T, float scale, const float* tw) {
    float rest;
#define PA_GO(HD_)                                                                                                          \
    if (p.hd == HD_) {                                                                                                      \
        using C = ReadCfg<HD_>;                                                                                             \
        StateArgs a = state_args(p, rev, X, st, gam, part, BH, T, C::TOK);                                                  \
        a.zpart = zpart;                                                                                                    \
        a.tw = tw;                                                                                                          \
        split_scale(scale, a.fold, rest);                                                                                   \
        a.out_scale = rest * rest;                                                                                          \
        if (!allow_smem(k_quad_read<HD_>, C::SMEM)) return false;                                                           \
        LaunchScope ls(name, s);                                                                                            \
        hipLaunchKernelGGL(k_quad_read<HD_>, dim3(xcd_grid(BH * a.nchunk * a.blocks)), dim3(64 * C::NW), C::SMEM, s, a);     \
        return launch_ok();                                                                                                 \
    }
    PA_GO(64) PA_GO(128)
#undef PA_GO
    return false;
}

bool launch_quad_dphi(const char* name, hipStream_t s, const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* Y,
                      const float* wgt, const bf16_t* st, const bf16_t* gam, float* part, int BH, int T, float scale, const float* tw,
                      float* dot) {
    float rest;
    if (dot != nullptr && p.hd != 64) return false;
#define PA_GO(HD_)                                                                                                          \
    if (p.hd == HD_) {                                                                                                      \
        using C = DphiCfg<HD_>;                                                                                             \
        StateArgs a = state_args(p, rev, X, st, gam, part, BH, T, C::TOK);                                                  \
        a.Y = Y;                                                                                                            \
        a.wgt = wgt;                                                                                                        \
        a.tw = tw;                                                                                                          \
        a.zpart = dot;                                                                                                      \
        split_scale(scale, a.fold, rest);                                                                                   \
        a.out_scale = scale * rest;                                                                                         \
        if (!allow_smem(k_quad_dphi<HD_>, C::SMEM)) return false;                                                           \
        LaunchScope ls(name, s);                                                                                            \
        hipLaunchKernelGGL(k_quad_dphi<HD_>, dim3(xcd_grid(BH * a.nchunk * a.blocks)), dim3(64 * C::NW), C::SMEM, s, a);     \
        return launch_ok();                                                                                                 \
    }
    PA_GO(64) PA_GO(128)
#undef PA_GO
    return false;
}

bool launch_quad_boundary(hipStream_t s, const QuadPlan& p, const bf16_t* st, const bf16_t* rc, const bf16_t* gam, const bf16_t* omg,
                          const float* lam, float* xb, int BH) {
    LaunchScope ls("mfma_gate_boundary", s);
    hipLaunchKernelGGL(k_quad_boundary, dim3(QUAD_XPARTS, p.nchunk, BH), dim3(256), 0, s, st, rc, gam, omg, lam, xb, p.nchunk);
    return launch_ok();
}

// segments of the prompt, each a workgroup's own: about two workgroups per CU, of at least four stages
QuadAbsorbPlan quad_absorb_plan(int BH, int T) {
    QuadAbsorbPlan p{};
    const int want = std::max(1, 512 / (BH * (ScanCfg<64>::NG + 1)));
    p.cs = std::max(256, ((T + want - 1) / want + 63) / 64 * 64);
    p.nseg = (T + p.cs - 1) / p.cs;
    p.tot_floats = (size_t)BH * p.nseg * (ScanCfg<64>::NG + 1) * ScanCfg<64>::TOTF;
    return p;
}
bool launch_quad_absorb(hipStream_t s, const QuadAbsorbPlan& p, const bf16_t* K, const bf16_t* V, const float* tw, const float* lam,
                        bf16_t* wK, float* tot, float* S, float* gamd, int D, int BH, int T) {
    if (tw != nullptr) {
        const size_t pieces = (size_t)BH * T * 8;
        LaunchScope ls("decode_absorb_weigh", s);
        hipLaunchKernelGGL(k_quad_weigh, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, K, tw, wK, pieces);
        if (!launch_ok()) return false;
        K = wK;
    }
    ScanArgs a{};
    a.X = K; a.Y = V; a.tot = tot;
    a.T = T; a.cs = p.cs; a.nchunk = a.nseg = a.tot_segs = p.nseg; a.seg_chunks = 1; a.heads = BH;
    a.fold = a.out_scale = 1.f;
    {
        LaunchScope ls("decode_absorb_scan", s);
        hipLaunchKernelGGL((k_quad_scan<64, false, true, false, false>), dim3(xcd_grid(BH * p.nseg * (ScanCfg<64>::NG + 1))), dim3(256), 0, s,
                           a);
        if (!launch_ok()) return false;
    }
    LaunchScope ls("decode_absorb_convert", s);
    hipLaunchKernelGGL(k_quad_absorb, dim3((unsigned)(BH * 64 * 8 / 4)), dim3(256), 0, s, (const float*)tot, p.nseg, lam, S, gamd, D, BH);
    return launch_ok();
}

}  // namespace mfma
}  // namespace pa
