// Shared definitions of the bf16 MFMA kernel family for degree p = 2 (gfx950, wave64).
//
// Chunked form of arXiv 2507.04239 (Sec. 2 "Chunked form", App. E) with the tiled
// symmetric-power embedding of Sec. 4.1.1 at d_tile = 8:  the expanded row (ti, tj, a, b),
// ti <= tj, of phi(x) is x[8 ti + a] * x[8 tj + b]; tiles off the diagonal carry the
// multiplicity 2, which is applied once, to the state (instead of sqrt(2) on both sides).
// Expanded operands are built in registers in MFMA operand order and never stored.
//
// MFMAs used: v_mfma_f32_32x32x16_bf16 (mfma32 below) and v_mfma_f32_16x16x32_bf16.  Operand layout of the latter (lane l,
// r16 = l % 16, g = l / 16):
//   A: row r16,   k-slots 8g..8g+7        B: column r16, k-slots 8g..8g+7
//   C: column r16, rows 4g..4g+3 (4 floats)
// Only the pairing of A and B k-slots matters, so k-slots are assigned to whatever order
// the data is already in (no shuffles between the two MFMAs of the attention form).
//
// A 64-row state tile (bf16) is stored as [a][v][b]: the 8 expanded rows b of one (a, v) are
// contiguous, which is the MFMA operand of a contraction over rows (the read-out).  The
// contraction over v (d phi in the backward pass) reads the same copy: it stages the tile in LDS
// and lets the transposing LDS read (ds_read_b64_tr_b16) gather 8 value columns per lane.
#pragma once

#include "common.hpp"

namespace pa {
namespace mfma {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int DH = 64;                         // head size (d = v)
constexpr int QBLK = 128;                      // token rows the chunk length is a multiple of
constexpr int TBLK = 64;                       // tokens per block of the feature-major copies

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 32x32x16 (lane l, r32 = l % 32, h = l / 32): A row r32, k-slots 8h..8h+7;  B column r32, k-slots 8h..8h+7;
// C column r32, register 4 k + r: row 8 k + 4 h + r
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

union Frag {
    bf16x8 v;
    uint4 u;
    u32x4 q;
    uint2 h[2];
};

template <int L>
__device__ __forceinline__ float row_lane(float x) {   // the value of lane L of this lane's 16-lane row
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + L, 0xf, 0xf, false));
}
__device__ __forceinline__ f32x16 zero16() {
    f32x16 v;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = 0.f;
    return v;
}
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
// 8 k-slots (rows base + 0 .. 3 of the lanes' 16-lane group, and 8 rows further), one column per lane
__device__ __forceinline__ Frag tr_frag(const bf16_t* p, int pitch) {
    union {
        Frag f;
        bf16x4 h[2];
    } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 8 * pitch));
    return u.f;
}

// Work items in contiguous runs per XCD (workgroups are dealt to the 8 XCDs round-robin by their linear id), so that the items
// that read the same memory sit side by side on one L2
__device__ __forceinline__ int xcd_item(int total, int block) {
    const int xcd = block & 7, q = block >> 3;
    const int base = total / 8, extra = total % 8;
    if (q >= base + (xcd < extra ? 1 : 0)) return -1;
    return xcd * base + min(xcd, extra) + q;
}
__device__ __forceinline__ int xcd_item(int total) { return xcd_item(total, (int)blockIdx.x); }
__host__ __device__ inline unsigned xcd_grid(int total) { return 8u * (unsigned)((total + 7) / 8); }

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also fences global memory,
// i.e. waits for every outstanding global load, which would drain a register prefetch ring.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Cross-lane sums without the LDS pipe: v_permlane16_swap / v_permlane32_swap exchange 16-lane rows (resp.
// 32-lane halves) between two registers.
__device__ __forceinline__ float xor16_sum(float x) {   // x + (value in lane ^ 16), in every lane
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ void halves(float x, float& lo, float& hi) {   // lane (l & 31) of each half, in every lane
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    lo = __uint_as_float(q[0]);
    hi = __uint_as_float(q[1]);
}
__device__ __forceinline__ float xor32_sum(float x) {
    float lo, hi;
    halves(x, lo, hi);
    return lo + hi;
}

// ---- launchers (each defined next to its kernels) ------------------------------------------

// ---- resident-state kernels (chunk states kept in registers; see mfma_resident.hip) ----------------
struct ResidentPlan {
    int nhp, nslab;            // half-pairs per wave; workgroups (slabs of state rows) per head
    int nseg, seg_chunks;      // segments the sequence is cut into, chunks per segment
    size_t acc_floats;         // accumulator floats per wave
    size_t tot_bytes, part_bytes, gram_bytes;   // per-segment totals; per-slab partial read-outs; per-chunk Gram matrices
};
ResidentPlan resident_plan(int HD, int BH, int T, int cs);
// One pass over the sequence with the state in registers.  readout = false: every segment but the last
// adds up its own total into `tot`.  readout = true: each segment starts from the totals before it and
// writes, per slab, part[slab][bh][t][:] = (state entering t's chunk)^T phi(Qr_t) * snap_scale.
// rev: the state holds the chunks after the current one (state gradient).
// mode 2 (d phi): part[slab][bh][t][:] = J_phi(Qr_t)^T (state . Gr_t) * snap_scale, Gr the token-major rows the state's
// value columns are contracted with
bool launch_res_walk(const char* name, hipStream_t s, int HD, bool rev, int mode, const bf16_t* Xt, const bf16_t* Yt,
                     const bf16_t* Qr, const bf16_t* Gr, float* tot, float* part, int BH, int T, int cs, const ResidentPlan& pl,
                     float snap_scale);
// out[bh][n] (bf16, HD x HD) = out_scale * sum over the chunks before (rev: after) n of sum_t w_t x_t x_t^T;
// gram: float32 scratch [BH][T / cs][HD][HD]; wgt may be null (w = 1)
bool launch_gram(hipStream_t s, int HD, const bf16_t* Xt, const float* wgt, float* gram, bf16_t* out, int BH, int T, int cs,
                 bool rev, float out_scale);

// feature-major copy in blocks of 64 tokens for any head size the resident kernels take
bool launch_transpose_hd(hipStream_t s, int HD, const bf16_t* in, bf16_t* out, int BH, int T);
// normaliser terms per token from the HD x HD states gam[bh][T / cs]: vec[bh][t][:] = cvec * wgt_t * G x_t (float32),
// sca[bh][t] = csca * x_t^T G x_t; vec, sca and wgt may each be null
bool launch_gram_apply(hipStream_t s, int HD, const bf16_t* X, const bf16_t* gam, const float* wgt, float* vec, float* sca,
                       int BH, int T, int cs, float cvec, float csca);

// a prompt of T tokens (a multiple of 64; d = 64) into decode states S [BH][D][64], gamd [BH][D]: scratch of tot_floats.
// Gates: tw [BH][T], the decay from a token to the prompt's end, lam [BH] across the prompt, wK [BH][T][64] scratch
struct QuadAbsorbPlan {
    int cs, nseg;
    size_t tot_floats;
};
QuadAbsorbPlan quad_absorb_plan(int BH, int T);
bool launch_quad_absorb(hipStream_t s, const QuadAbsorbPlan& p, const bf16_t* K, const bf16_t* V, const float* tw, const float* lam,
                        bf16_t* wK, float* tot, float* S, float* gamd, int D, int BH, int T);

// ---- chunked form for any degree and tile width (state kept in memory; see mfma_tiled.hip) -------------
// One tile of the tiled symmetric-power embedding: its p block indices (non-decreasing) and its multiplicity
struct TileDesc {
    unsigned char t[4];
    float mult;
};
struct TiledPlan {
    int p, dt, hd, vp;            // degree, tile width, head size, value columns of a state row (hd + 16)
    int ntile, rows_per_tile;     // tiles of the embedding, dt^p rows each
    int nunit_real, nunit;        // 64-row units that hold state, and the count the layout is padded to (a multiple of 4)
    int nentry;                   // entries of the tile table (padding entries have multiplicity 0)
    size_t state_elems;           // bf16 elements of one (head, chunk) state
};
bool tiled_shape_ok(int p, int d, int dt);
int tiled_default_dt(int p);
TiledPlan tiled_plan(int p, int d, int dt);
bool launch_tiled_table(hipStream_t s, const TiledPlan& pl, TileDesc* tab);
// Yp[row] = [Y[row] (hd values), col[row] (1 when col is null), 15 zeros], bf16
bool launch_tiled_pack(hipStream_t s, int hd, const bf16_t* Y, const float* col, bf16_t* Yp, long long rows);
// st[bh][c] = multiplicity x sum over the chunks before c (rev: after c) of phi(xscale X_t) Yp_t^T
bool launch_tiled_scan(const char* name, hipStream_t s, const TiledPlan& pl, bool rev, const bf16_t* X, const bf16_t* Yp,
                       const TileDesc* tab, bf16_t* st, int BH, int T, int cs, float xscale);
// part[bh][t][:] = (state of t's chunk)^T phi(xscale X_t), columns 0 .. hd - 1; zpart[bh][t] (may be null) = column hd
bool launch_tiled_readout(const char* name, hipStream_t s, const TiledPlan& pl, const bf16_t* X, const TileDesc* tab, const bf16_t* st,
                          float* part, float* zpart, int BH, int T, int cs, float xscale);
// part[bh][t][:] = outscale J_phi(xscale X_t)^T (state of t's chunk . Yp_t)
bool launch_tiled_dphi(const char* name, hipStream_t s, const TiledPlan& pl, const bf16_t* X, const bf16_t* Yp, const TileDesc* tab,
                       const bf16_t* st, float* part, int BH, int T, int cs, float xscale, float outscale);

// ---- chunked form, p = 2, d = v in {64, 128}: states formed and used with phi in registers (see mfma_quad.hip) ---------
struct QuadPlan {
    int hd, cs, nchunk;           // chunks of cs tokens, the last one shorter where cs does not divide T
    int nseg, seg_chunks;         // segments the scan is cut into
    size_t state_elems, gam_elems;   // bf16 elements of one state and of one normaliser, nchunk - 1 of each per head
    size_t tot_floats;            // scratch of the scan
};
QuadPlan quad_plan(int d, int BH, int T, int cs);
// Gates (d = 64; null without): tw [BH][T], the decay that goes with a token (GateBuf::kfac, rev: qfac; the other one where a
// state is used), lam [BH][nchunk].
// st, gam: the states before (rev: after) each chunk.  rev: wgt = gz, X enters multiplied by scale.
bool launch_quad_scan(const char* name, hipStream_t s, const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* Y, const float* wgt,
                      bf16_t* st, bf16_t* gam, float* tot, int BH, int T, float scale, const float* tw, const float* lam);
// part[bh][t][:] = (state of t's chunk)^T phi(scale X_t), zpart[bh][t] (may be null) = the same of the normaliser; zeros where
// the chunk has no state
bool launch_quad_read(const char* name, hipStream_t s, const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* st,
                      const bf16_t* gam, float* part, float* zpart, int BH, int T, float scale, const float* tw);
// part[bh][t][:] = d/dX_t of phi(scale X_t) . (state of t's chunk . Y_t) and of wgt_t times the normaliser's part (wgt null: 1); dot[bh][t] (may be null) = X_t . part
bool launch_quad_dphi(const char* name, hipStream_t s, const QuadPlan& p, bool rev, const bf16_t* X, const bf16_t* Y, const float* wgt,
                      const bf16_t* st, const bf16_t* gam, float* part, int BH, int T, float scale, const float* tw, float* dot);
// d = 64: xb[bh][n][QUAD_XPARTS] = terms of the sum over the pairs that straddle the whole of chunk n, from the states
constexpr int QUAD_XPARTS = 8;
bool launch_quad_boundary(hipStream_t s, const QuadPlan& p, const bf16_t* st, const bf16_t* rc, const bf16_t* gam, const bf16_t* omg,
                          const float* lam, float* xb, int BH);

// running sums of the log-gates as the attention kernels read them (see GateBuf; null: no gates)
struct GateSums {
    const float* bl = nullptr;
    const double* blk = nullptr;
};
// attention form (chunk == T): p in {2, 3, 4}, d = v in {32, 64, 128}, any T.
// Gh [BH][T][d] bf16 and gz [BH][T] float32 are scratch of the backward pass.
bool attn_shape_ok(int p, int d);
// bl (null when not gated): [BH][T] running sums of the log-gates from the start of the sequence
bool launch_attn_fwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, bf16_t* O, float* Z, int BH,
                     int T, float scale, int normalize, GateSums sums = GateSums());
// The in-chunk part of the chunked form on the attention-form kernels (keys of the query's own chunk of cs
// tokens), plus what came through the state: part[slab][BH][T][d] (float32, nslab slabs) joins the numerator,
// zpart[BH][T] the denominator
bool launch_chunk_fwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, bf16_t* O, float* Z, int BH,
                      int T, int cs, float scale, int normalize, const float* part, int nslab, const float* zpart,
                      const char* label = "chunk_fwd", GateSums sums = GateSums());
// ghat = dO / Z (bf16) and gz = -(ghat . O) (float32) per token, d in {32, 64, 128}
bool launch_attn_prep(hipStream_t s, int d, const bf16_t* dO, const bf16_t* O, const float* Z, bf16_t* Gh, float* gz, long long rows,
                      int normalize);
// Gated backward pass (sums non-null; T a multiple of attn_gate_block(d)): also leaves what the gradient of
// the log-gates needs: qdq [BH][T] = q_i . dq_i, kdk [BH][T] = k_j . dk_j (from float32 accumulators) and
// xb [BH][T / block] = the sum of e_ij a_ij over the pairs j <= end of block m < i.
// wsum: scratch, BH * (T / block)^2 * 4 floats.
struct AttnGate {
    GateSums sums;
    float *qdq = nullptr, *kdk = nullptr, *xb = nullptr, *wsum = nullptr;
};
int attn_gate_block(int d);
// backward of launch_chunk_fwd: the in-chunk gradients plus the per-slab parts that came through the states (float32
// [slab][BH][T][d]; the slab counts include the normaliser's slab where there is one).  Gated (p = 2, d = 64): gate.sums
// from the start of the chunk, gate.qdq and gate.kdk, to which the states' parts dotq and dotk [BH][T] are added.
bool launch_chunk_bwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, const bf16_t* Gh,
                      const float* gz, bf16_t* dQ, bf16_t* dK, bf16_t* dV, int BH, int T, int cs, float scale, const float* part_dq,
                      int nslab_dq, const float* part_dk, int nslab_dk, const float* part_dv, int nslab_dv,
                      const AttnGate& gate = AttnGate(), const float* dotq = nullptr, const float* dotk = nullptr);
bool launch_attn_bwd(hipStream_t s, int p, int d, const bf16_t* Q, const bf16_t* K, const bf16_t* V, const bf16_t* O,
                     const float* Z, const bf16_t* dO, bf16_t* Gh, float* gz, bf16_t* dQ, bf16_t* dK, bf16_t* dV, int BH, int T,
                     float scale, int normalize, const AttnGate& gate = AttnGate());

}  // namespace mfma
}  // namespace pa
