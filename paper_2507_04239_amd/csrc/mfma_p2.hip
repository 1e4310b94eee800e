// Host side of the bf16 MFMA kernel families: support check, workspace layout and the launch
// sequences of the forward and backward passes: chunk states for p = 2 (mfma_quad.hip, mfma_resident.hip) and for any degree
// (mfma_tiled.hip), and the attention form (no state) for p in {2, 3, 4}, d = v in {32, 64, 128}.
#include <algorithm>

#include "mfma_common.hpp"

namespace pa {
namespace {

using namespace mfma;

// resident-state kernels: workspace of the forward pass (the backward part is appended)
struct ResLayout {
    ResidentPlan pl;
    size_t off_kt, off_vt, off_gam, off_gram, off_tot, off_part, off_zpart;
    size_t off_qt, off_ght, off_gh, off_gz, off_omg, off_totr, off_pdq, off_pdk;   // backward only
    size_t total;
};
ResLayout make_res_layout(const pa_problem& pr, bool backward) {
    ResLayout L{};
    const int BH = pr.B * pr.H;
    L.pl = resident_plan(pr.d, BH, pr.T, pr.chunk);
    const size_t tok = (size_t)BH * pr.T * pr.d * 2;
    const size_t gm = (size_t)BH * (pr.T / pr.chunk) * pr.d * pr.d * 2;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    L.off_kt = take(tok);
    L.off_vt = take(tok);
    L.off_gam = take(gm);
    L.off_gram = take(L.pl.gram_bytes);
    L.off_tot = take(L.pl.tot_bytes);
    L.off_part = take(L.pl.part_bytes);
    L.off_zpart = take((size_t)BH * pr.T * sizeof(float));
    if (backward || pr.keep_state) {
        const size_t slab = (size_t)BH * pr.T * pr.d * sizeof(float);
        L.off_qt = take(tok);
        L.off_ght = take(tok);
        L.off_gh = take(tok);
        L.off_gz = take((size_t)BH * pr.T * sizeof(float));
        L.off_omg = take(gm);
        L.off_totr = take(L.pl.tot_bytes);
        L.off_pdq = take((L.pl.nslab + 1) * slab);     // the last slab is the normaliser's share
        L.off_pdk = take((L.pl.nslab + 1) * slab);
    }
    L.total = off;
    return L;
}
bool resident_ok(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.p == 2 && (pr.d == 64 || pr.d == 128) && pr.v == pr.d && pr.chunk > 0 &&
           pr.chunk % QBLK == 0 && pr.T % pr.chunk == 0 && !pr.gated && (size_t)pr.B * pr.H <= 65535u;
}
// gated: the boundary sums of the gate gradient are kept per block of keys of the dK / dV kernel
bool attn_ok(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.d == pr.v && attn_shape_ok(pr.p, pr.d) && pr.chunk == pr.T &&
           (!pr.gated || pr.T % attn_gate_block(pr.d) == 0) && (size_t)pr.B * pr.H <= 65535u;
}
// One chunk: the attention-form kernels.
bool use_quad(const pa_problem& pr);
bool quad_states(const pa_problem& pr, bool backward);
bool use_attn(const pa_problem& pr, bool backward) {
    if (use_quad(pr)) return !quad_states(pr, backward);
    return attn_ok(pr) && pr.impl != PA_IMPL_RESIDENT && pr.impl != PA_IMPL_TILED;
}
bool use_tiled(const pa_problem& pr);
// The resident-state kernels run when asked for by name, and wherever they are the only matrix-core kernels
// for the chunked form
bool use_resident(const pa_problem& pr) {
    if (pr.impl == PA_IMPL_TILED || !resident_ok(pr)) return false;
    return pr.impl == PA_IMPL_RESIDENT || (!use_quad(pr) && !attn_ok(pr) && !use_tiled(pr));
}

// tiled kernels (any degree and tile width, chunk states in memory): workspace of the forward pass, the backward
// part appended
struct TiledLayout {
    TiledPlan pl;
    size_t off_tab, off_vp, off_sc, off_part, off_zpart;
    size_t off_gh, off_gz, off_gp, off_rc, off_pdq, off_pdk;   // backward only
    size_t total;
};
int tiled_dt(const pa_problem& pr) { return pr.d_tile > 0 ? pr.d_tile : tiled_default_dt(pr.p); }
TiledLayout make_tiled_layout(const pa_problem& pr, bool backward) {
    TiledLayout L{};
    const size_t BH = (size_t)pr.B * pr.H;
    L.pl = tiled_plan(pr.p, pr.d, tiled_dt(pr));
    const size_t rows = BH * pr.T;
    const size_t st = BH * (pr.T / pr.chunk) * L.pl.state_elems * 2;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    L.off_tab = take((size_t)L.pl.nentry * sizeof(TileDesc));
    L.off_vp = take(rows * L.pl.vp * 2);
    L.off_sc = take(st);
    L.off_part = take(rows * pr.d * sizeof(float));
    L.off_zpart = take(rows * sizeof(float));
    if (backward || pr.keep_state) {
        L.off_gh = take(rows * pr.d * 2);
        L.off_gz = take(rows * sizeof(float));
        L.off_gp = take(rows * L.pl.vp * 2);
        L.off_rc = take(st);
        L.off_pdq = take(rows * pr.d * sizeof(float));
        L.off_pdk = take(rows * pr.d * sizeof(float));
    }
    L.total = off;
    return L;
}
bool tiled_ok(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.d == pr.v && pr.chunk > 0 && pr.chunk % QBLK == 0 && pr.T % pr.chunk == 0 &&
           pr.chunk < pr.T && !pr.gated && tiled_shape_ok(pr.p, pr.d, tiled_dt(pr)) && (size_t)pr.B * pr.H <= 65535u;
}

// attention form, backward: ghat (bf16) and gz (float32) per token
struct AttnLayout {
    size_t off_gh, off_gz, off_wsum, total;
};
AttnLayout make_attn_layout(const pa_problem& pr, bool backward) {
    AttnLayout L{};
    if (!backward) return L;
    const size_t rows = (size_t)pr.B * pr.H * pr.T;
    L.off_gh = 0;
    L.off_gz = align_up(rows * pr.d * 2, 256);
    L.off_wsum = L.off_gz + align_up(rows * sizeof(float), 256);
    L.total = L.off_wsum;
    if (pr.gated) {
        const size_t nblk = (size_t)(pr.T / attn_gate_block(pr.d));
        L.total += align_up((size_t)pr.B * pr.H * nblk * nblk * 4 * sizeof(float), 256);
    }
    return L;
}

// Chunk-state kernels with phi in registers (mfma_quad.hip): what AUTO and MFMA run for the chunked form of p = 2 at d = 64 and
// (un-gated) 128, whatever multiple of 128 tokens the chunk is.  The states they keep are quad_chunk tokens apart: the result does
// not depend on that beyond rounding, and states are rounded less often the fewer they are.
bool quad_ok(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.p == 2 && (pr.d == 64 || pr.d == 128) && pr.v == pr.d && pr.chunk > 0 &&
           pr.chunk % QBLK == 0 && pr.chunk < pr.T && (!pr.gated || pr.d == 64) && pr.d_tile == 0 && (size_t)pr.B * pr.H <= 65535u;
}
bool use_quad(const pa_problem& pr) { return (pr.impl == PA_IMPL_AUTO || pr.impl == PA_IMPL_MFMA) && quad_ok(pr); }
// Tokens per state.  A state's traffic falls with the distance, the pairs in between grow with it; the step is flat around the
// best (ms, forward + backward): 12 heads of 65536, d = 64: 512 3.23, 768 3.00, 1024 3.05, 1280 2.97, 1536 3.03, 2048 3.24;
// 32 heads of 32768, d = 128: 512 17.6, 768 18.4, 1024 17.4, 1536 18.0, 2048 18.0.  (Multiples of 256 at d = 64 and of 512 at
// d = 128 fill the workgroups of the per-chunk kernels.)
// Where the states of both passes take more than 256 MB a longer chunk is taken as asked for: fewer states is how a caller trades
// time for memory (backward, 32 heads of 32768, d = 128: 6.4 GB of workspace at 1024 tokens, 4.1 at 2048, 2.9 at 4096; 12 of 65536,
// d = 64: 1459 MB at 1280, 822 at 4096, and 2319 us, 2993).  Below there is nothing to save (1 head of 16384, d = 64, forward: 79 us,
// 253 at a chunk of 8192).
int quad_chunk(const pa_problem& pr) {
    const int own = pr.d == 64 ? 1280 : 1024;
    if (pr.chunk <= own) return own;
    const QuadPlan pl = quad_plan(pr.d, pr.B * pr.H, pr.T, own);
    const size_t states = (size_t)pr.B * pr.H * (pl.nchunk - 1) * (pl.state_elems + pl.gam_elems) * 2;
    return 2 * states > (256u << 20) ? pr.chunk : own;
}
// Shorter sequences run as one chunk, without a state.  The whole pass grows with the square of the length once the chip is full
// and with the length while it is not (few heads: one walk is the time); a pass with states has a constant part for few heads and
// steps where a kernel's workgroups begin another round of the CUs.  So the line lies elsewhere for few heads.  Measured at 1 .. 20
// heads, 24, 32, 40, 48, 64, 96 (heads x tokens: us whole, with states):
//   d = 64 forward    1 x 7168 75, 76;       4 x 8192 86, 80;       12 x 8192 126, 132;     48 x 8192 387, 413;     12 x 9216 150, 138
//   d = 64 backward   1 x 7168 131, 139;     8 x 7168 213, 215;     12 x 6144 214, 238;     12 x 7168 286, 259;     48 x 7168 1057, 979
//   gated forward     1 x 5120 103, 96;      12 x 5120 109, 109;    16 x 5632 126, 136;     24 x 6144 160, 200
//   gated backward    1 x 5120 169, 166;     12 x 5632 247, 263;    12 x 6144 284, 271;     16 x 5632 326, 292;     48 x 5120 709, 721;
//                     48 x 6144 999, 919
//   d = 128 forward   1 x 18432 342, 328;    2 x 20480 414, 428;    4 x 24576 671, 685;     8 x 24576 1263, 1430;   12 x 18432 1086, 1073;
//                     16 x 18432 1396, 1686; 16 x 20480 1739, 1818; 32 x 18432 2892, 2919
//   d = 128 backward  1 x 8192 494, 492;     3 x 10240 623, 619;    4 x 16384 1112, 1097;   8 x 16384 1999, 1989;   16 x 14336 2985, 2993;
//                     32 x 14336 6252, 6081
// With more than 6 heads a forward pass of 8192 tokens is up to 6 % faster whole, and runs with states all the same, as one with
// gates between 5633 and 7168 does at 20 heads and more: the states may be kept for the backward pass, which gains more by them
// (48 x 8192, d = 64, both passes: 413 + 956 us kept, 387 + 1138 whole and rebuilt), and results do not depend on keep_state.
int quad_whole_upto(const pa_problem& pr, bool backward) {
    const int heads = pr.B * pr.H;
    if (pr.gated) return backward ? (heads >= 9 && heads <= 14 ? 5632 : 5248) : heads <= 11 ? 5120 : 5632;
    if (pr.d == 64) return backward ? (heads <= 10 ? 7296 : 6400) : (heads <= 6 ? 7424 : 8191);
    if (backward) return heads <= 2 ? 8192 : heads == 3 ? 9984 : heads <= 10 ? 16384 : 14336;
    return heads == 1 ? 17408 : heads <= 3 ? 20480 : heads <= 10 ? 24576 : heads >= 13 && heads <= 16 ? 20480 : 18432;
}
bool quad_states(const pa_problem& pr, bool backward) { return use_quad(pr) && pr.T > quad_whole_upto(pr, backward); }
// the forward pass leaves its states for the backward pass
bool quad_kept(const pa_problem& pr) { return pr.keep_state != 0 && quad_states(pr, false); }
struct QuadLayout {
    QuadPlan pl;
    size_t off_st, off_gam, off_part, off_zpart, off_tot;
    size_t off_gh, off_gz, off_rc, off_omg, off_pdq, off_pdk;   // backward only
    size_t off_tot2;                                            // scratch of the other scan, where both run side by side
    size_t off_dotq, off_dotk;                                  // ... gated: the states' part of q . dq and k . dk
    size_t total;
};
QuadLayout make_quad_layout(const pa_problem& pr, bool backward) {
    QuadLayout L{};
    const size_t BH = (size_t)pr.B * pr.H, rows = BH * pr.T;
    L.pl = quad_plan(pr.d, (int)BH, pr.T, quad_chunk(pr));
    const size_t nslot = BH * (L.pl.nchunk - 1);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    // A scan's totals are dead before the first kernel behind it on its stream writes a part: they share the parts' space, once
    // they are more than the 32 MB of all L2 caches.  (Below, lines of the totals are still in other XCDs' caches when the parts
    // are written over them, and what is saved is little: shared and apart, forward, d = 64: 4 heads of 8192 tokens, 22 MB of totals,
    // 81.7 and 79.6 us, 1 of 32768, 20 MB, 85.9 and 84.1; 4 of 16384, 41 MB, 101.7 and 101.4; 4 of 65536, 164 MB, 288 and 294.)
    const size_t tot = L.pl.tot_floats * sizeof(float), slab = rows * pr.d * sizeof(float);
    const bool share = tot > (32u << 20);
    L.off_st = take(nslot * L.pl.state_elems * 2);
    L.off_gam = take(nslot * L.pl.gam_elems * 2);
    L.off_zpart = take(rows * sizeof(float));
    L.off_tot = share ? off : take(tot);
    L.off_part = off;                    // forward: the read-out; backward: dV and then dK, behind the scan of R
    const size_t over = share ? tot : 0;
    if (!backward && !pr.keep_state) {
        take(std::max(slab, over));
    } else {
        take(std::max(2 * align_up(slab, 256), over));
        L.off_pdk = L.off_part + align_up(slab, 256);
        L.off_gh = take(rows * pr.d * 2);
        L.off_gz = take(rows * sizeof(float));
        L.off_rc = take(nslot * L.pl.state_elems * 2);
        L.off_omg = take(nslot * L.pl.gam_elems * 2);
        L.off_tot2 = share || quad_kept(pr) ? off : take(tot);
        L.off_pdq = off;                 // dQ, behind the scan of S unless the forward pass has left that
        take(quad_kept(pr) ? slab : std::max(slab, over));
        if (pr.gated) {
            L.off_dotq = take(rows * sizeof(float));
            L.off_dotk = take(rows * sizeof(float));
        }
    }
    L.total = off;
    return L;
}

// The tiled kernels run when asked for by name or for a tile width, and wherever no other matrix-core kernel takes the
// chunked form of the problem (degrees 3 and 4, d = 32)
bool use_tiled(const pa_problem& pr) {
    if (!tiled_ok(pr)) return false;
    if (pr.impl == PA_IMPL_TILED) return true;
    if (pr.impl == PA_IMPL_RESIDENT) return false;
    return pr.d_tile > 0 || (!use_quad(pr) && !attn_ok(pr));
}

}  // namespace

int mfma_state_spacing(const pa_problem& pr, bool backward) {
    if (use_quad(pr)) return quad_states(pr, backward) ? quad_chunk(pr) : pr.T;
    return use_attn(pr, backward) ? pr.T : pr.chunk;
}
int mfma_gate_chunk(const pa_problem& pr, bool backward) { return use_attn(pr, backward) ? pr.T : quad_chunk(pr); }
size_t mfma_gate_slots(const pa_problem& pr) {
    if (!use_quad(pr) || !quad_states(pr, true)) return 0;
    const int cs = quad_chunk(pr);
    return (size_t)((pr.T + cs - 1) / cs) * QUAD_XPARTS;
}
int mfma_gate_fin_chunk(const pa_problem& pr, const char* ws, int& xparts, const float*& dotk) {
    const bool attn = use_attn(pr, true);
    xparts = attn ? 1 : QUAD_XPARTS;
    dotk = attn ? nullptr : (const float*)(ws + make_quad_layout(pr, true).off_dotk);
    return attn ? attn_gate_block(pr.d) : quad_chunk(pr);
}

// (whole, a gated sequence has to be a multiple of the attention form's key block, as all lines of quad_whole_upto are)
int mfma_whole_rows(const pa_problem& pr, bool backward) {
    if (!use_quad(pr)) return pr.chunk;
    return pr.gated && !quad_states(pr, backward) ? attn_gate_block(pr.d) : 1;
}

pa_status mfma_supported(const pa_problem& pr, bool backward) {
    if (use_quad(pr)) return PA_OK;
    if (pr.impl == PA_IMPL_RESIDENT) return resident_ok(pr) ? PA_OK : PA_ERR_UNSUPPORTED;
    if (pr.impl == PA_IMPL_TILED || pr.d_tile > 0) return tiled_ok(pr) ? PA_OK : PA_ERR_UNSUPPORTED;
    return attn_ok(pr) || resident_ok(pr) || tiled_ok(pr) ? PA_OK : PA_ERR_UNSUPPORTED;
}

long long mfma_state_rows(const pa_problem& pr) {
    if (use_quad(pr)) return (long long)(pr.d / 8) * (pr.d / 8 + 1) / 2 * 64;
    if (use_tiled(pr)) {
        const TiledPlan pl = tiled_plan(pr.p, pr.d, tiled_dt(pr));
        return (long long)pl.ntile * pl.rows_per_tile;
    }
    if (use_resident(pr)) return (long long)(pr.d / 8) * (pr.d / 8 + 1) / 2 * 64;
    return 0;      // attention form
}

size_t mfma_workspace_bytes(const pa_problem& pr, bool backward) {
    if (use_quad(pr)) return quad_states(pr, backward) ? make_quad_layout(pr, backward).total : make_attn_layout(pr, backward).total;
    if (use_tiled(pr)) return make_tiled_layout(pr, backward).total;
    if (use_resident(pr)) return make_res_layout(pr, backward).total;
    return make_attn_layout(pr, backward).total;
}

// Scratch of a fixed size.  The totals of the scan and the spacing are the kernels' own affair: what counts is whether the states as
// far apart as they were asked for fit, beside one float32 value per element of O.  Such a problem runs as the attention form, which
// needs no scratch, where the kernels' own spacing does not fit (1 head of 24576 tokens, d = 64: 252 us).
bool mfma_fit(pa_problem& pr, bool chosen, size_t bytes) {
    if (!use_quad(pr) || pr.gated) return false;
    const size_t BH = (size_t)pr.B * pr.H, nasked = (size_t)((pr.T + pr.chunk - 1) / pr.chunk);
    const QuadPlan pl = quad_plan(pr.d, (int)BH, pr.T, quad_chunk(pr));
    const size_t asked = BH * (nasked * (pl.state_elems + pl.gam_elems) * 2 + (size_t)pr.T * pr.d * sizeof(float));
    // (d = 128: a chunk chosen by the library was the whole sequence up to 24575 tokens before it was chosen for speed alone)
    const bool whole = chosen && pr.d == 128 && pr.T < 24576;
    if (asked > bytes && !whole) return false;
    pr.chunk = pr.T;
    return true;
}

#define PA_TRY(CALL) \
    if (!(CALL)) return PA_ERR_HIP;

pa_status mfma_fwd(const Ctx& c, const void* Q, const void* K, const void* V, void* O, float* Z) {
    const pa_problem& pr = c.prob;
    const int BH = pr.B * pr.H;
    if (use_attn(pr, false)) {
        PA_TRY(launch_attn_fwd(c.stream, pr.p, pr.d, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (bf16_t*)O, Z, BH, pr.T,
                               pr.scale, pr.normalize, GateSums{c.gate.bl, c.gate.blk}))
        return PA_OK;
    }
    if (use_quad(pr)) {
        // states, read-out; the in-chunk part and the division on the chunk-local attention kernel
        const QuadLayout L = make_quad_layout(pr, pr.keep_state != 0);
        bf16_t *st = (bf16_t*)(c.ws + L.off_st), *gam = (bf16_t*)(c.ws + L.off_gam);
        float *part = (float*)(c.ws + L.off_part), *zpart = (float*)(c.ws + L.off_zpart);
        PA_TRY(launch_quad_scan("mfma_state_scan", c.stream, L.pl, false, (const bf16_t*)K, (const bf16_t*)V, nullptr, st, gam,
                                (float*)(c.ws + L.off_tot), BH, pr.T, 1.0f, c.gate.kfac, c.gate.lam))
        PA_TRY(launch_quad_read("mfma_query_state", c.stream, L.pl, false, (const bf16_t*)Q, st, gam, part, zpart, BH, pr.T, pr.scale,
                                c.gate.qfac))
        PA_TRY(launch_chunk_fwd(c.stream, pr.p, pr.d, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (bf16_t*)O, Z, BH, pr.T,
                                L.pl.cs, pr.scale, pr.normalize, part, 1, zpart, "mfma_fwd_chunk", GateSums{c.gate.bl, c.gate.blk}))
        return PA_OK;
    }
    if (use_tiled(pr)) {
        // tile table, values extended by the normaliser's one, state scan, read-out; the in-chunk part and the
        // division on the chunk-local attention kernel
        const TiledLayout L = make_tiled_layout(pr, pr.keep_state != 0);
        TileDesc* tab = (TileDesc*)(c.ws + L.off_tab);
        bf16_t* Vp = (bf16_t*)(c.ws + L.off_vp);
        bf16_t* Sc = (bf16_t*)(c.ws + L.off_sc);
        float* part = (float*)(c.ws + L.off_part);
        float* zpart = (float*)(c.ws + L.off_zpart);
        PA_TRY(launch_tiled_table(c.stream, L.pl, tab))
        PA_TRY(launch_tiled_pack(c.stream, pr.d, (const bf16_t*)V, nullptr, Vp, (long long)BH * pr.T))
        PA_TRY(launch_tiled_scan("tiled_state_scan", c.stream, L.pl, false, (const bf16_t*)K, Vp, tab, Sc, BH, pr.T, pr.chunk, 1.0f))
        PA_TRY(launch_tiled_readout("tiled_query_state", c.stream, L.pl, (const bf16_t*)Q, tab, Sc, part, zpart, BH, pr.T, pr.chunk,
                                    pr.scale))
        PA_TRY(launch_chunk_fwd(c.stream, pr.p, pr.d, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (bf16_t*)O, Z, BH, pr.T,
                                pr.chunk, pr.scale, pr.normalize, part, 1, zpart))
        return PA_OK;
    }
    if (use_resident(pr)) {
        const ResLayout R = make_res_layout(pr, pr.keep_state != 0);
        bf16_t* Kt = (bf16_t*)(c.ws + R.off_kt);
        bf16_t* Vt = (bf16_t*)(c.ws + R.off_vt);
        bf16_t* Gam = (bf16_t*)(c.ws + R.off_gam);
        float* gram = (float*)(c.ws + R.off_gram);
        float* tot = (float*)(c.ws + R.off_tot);
        float* part = (float*)(c.ws + R.off_part);
        float* zpart = (float*)(c.ws + R.off_zpart);
        PA_TRY(launch_transpose_hd(c.stream, pr.d, (const bf16_t*)K, Kt, BH, pr.T))
        PA_TRY(launch_transpose_hd(c.stream, pr.d, (const bf16_t*)V, Vt, BH, pr.T))
        PA_TRY(launch_gram(c.stream, pr.d, Kt, nullptr, gram, Gam, BH, pr.T, pr.chunk, false, 1.0f))
        if (R.pl.nseg > 1)
            PA_TRY(launch_res_walk("res_state_totals", c.stream, pr.d, false, 0, Kt, Vt, nullptr, nullptr, tot, nullptr, BH, pr.T,
                                   pr.chunk, R.pl, 1.0f))
        PA_TRY(launch_res_walk("res_state_walk", c.stream, pr.d, false, 1, Kt, Vt, (const bf16_t*)Q, nullptr, tot, part, BH, pr.T,
                               pr.chunk, R.pl, pr.scale * pr.scale))
        // the normaliser's share of the denominator, then the in-chunk part on the attention-form kernel
        PA_TRY(launch_gram_apply(c.stream, pr.d, (const bf16_t*)Q, Gam, nullptr, nullptr, zpart, BH, pr.T, pr.chunk, 0.f,
                                 pr.scale * pr.scale))
        PA_TRY(launch_chunk_fwd(c.stream, pr.p, pr.d, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (bf16_t*)O, Z, BH,
                                pr.T, pr.chunk, pr.scale, pr.normalize, part, R.pl.nslab, zpart))
        return PA_OK;
    }
    return PA_ERR_UNSUPPORTED;     // (no family: not reached behind mfma_supported)
}

// The backward pass with states has two strands, dQ from S and dK, dV from R, that do not fill the chip to their ends: the first
// runs on a second stream (created once, default priority).
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr, scanned = nullptr;
    bool ok = false;
    int device = -1;
};
// One side stream per host thread (so that calls from several threads never share one), bound to the
// device of the thread's first backward call; a call on any other device simply runs both strands on the
// caller's stream.  power_attn_release_thread() destroys it.
static thread_local SideStream t_side;
static SideStream side_stream() {
    SideStream& s = t_side;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return SideStream{};
    if (s.device < 0) {
        s.device = dev;
        s.ok = hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) == hipSuccess &&
               hipEventCreateWithFlags(&s.fork, hipEventDisableTiming) == hipSuccess &&
               hipEventCreateWithFlags(&s.join, hipEventDisableTiming) == hipSuccess &&
               hipEventCreateWithFlags(&s.scanned, hipEventDisableTiming) == hipSuccess;
    }
    return s.device == dev ? s : SideStream{};
}

void mfma_release_side_stream() {
    SideStream& s = t_side;
    if (s.stream != nullptr) (void)hipStreamDestroy(s.stream);
    if (s.fork != nullptr) (void)hipEventDestroy(s.fork);
    if (s.join != nullptr) (void)hipEventDestroy(s.join);
    if (s.scanned != nullptr) (void)hipEventDestroy(s.scanned);
    s = SideStream{};
}

pa_status mfma_bwd(const Ctx& c, const void* Q, const void* K, const void* V, const void* O, const float* Z,
                   const void* dO, void* dQ, void* dK, void* dV) {
    const pa_problem& pr = c.prob;
    const int BH = pr.B * pr.H;
    if (use_attn(pr, true)) {
        const AttnLayout A = make_attn_layout(pr, true);
        AttnGate ag;
        if (pr.gated) {
            ag.sums = GateSums{c.gate.bl, c.gate.blk};
            ag.qdq = c.gate.db;
            ag.kdk = c.gate.db2;
            ag.xb = c.gate.xb;
            ag.wsum = (float*)(c.ws + A.off_wsum);
        }
        PA_TRY(launch_attn_bwd(c.stream, pr.p, pr.d, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)O, Z,
                               (const bf16_t*)dO, (bf16_t*)(c.ws + A.off_gh), (float*)(c.ws + A.off_gz), (bf16_t*)dQ, (bf16_t*)dK,
                               (bf16_t*)dV, BH, pr.T, pr.scale, pr.normalize, ag))
        return PA_OK;
    }
    if (use_quad(pr)) {
        // dQ's state part from S, the state gradient R, dV's and dK's from R; one kernel then adds the in-chunk gradients
        const QuadLayout L = make_quad_layout(pr, true);
        bf16_t *st = (bf16_t*)(c.ws + L.off_st), *gam = (bf16_t*)(c.ws + L.off_gam);
        bf16_t *rc = (bf16_t*)(c.ws + L.off_rc), *omg = (bf16_t*)(c.ws + L.off_omg), *Gh = (bf16_t*)(c.ws + L.off_gh);
        float *gz = (float*)(c.ws + L.off_gz), *tot = (float*)(c.ws + L.off_tot);
        float *pdv = (float*)(c.ws + L.off_part), *pdq = (float*)(c.ws + L.off_pdq), *pdk = (float*)(c.ws + L.off_pdk);
        const bf16_t *q = (const bf16_t*)Q, *k = (const bf16_t*)K, *v = (const bf16_t*)V;
        hipStream_t s = c.stream;
        PA_TRY(launch_attn_prep(s, pr.d, (const bf16_t*)dO, (const bf16_t*)O, Z, Gh, gz, (long long)BH * pr.T, pr.normalize))
        const GateBuf& gt = c.gate;       // (all null without gates)
        float *dotq = pr.gated ? (float*)(c.ws + L.off_dotq) : nullptr, *dotk = pr.gated ? (float*)(c.ws + L.off_dotk) : nullptr;
        // Two strands that meet at the in-chunk gradients: dQ's part from S (on the side stream), and R with dV's and dK's.  Neither
        // fills the chip to its end.
        SideStream side = side_stream();
        if (profile_enabled()) side.ok = false;   // timed kernel by kernel: no overlap
        hipStream_t s2 = side.ok ? side.stream : s;
        if (side.ok && (hipEventRecord(side.fork, s) != hipSuccess || hipStreamWaitEvent(s2, side.fork, 0) != hipSuccess)) return PA_ERR_HIP;
        PA_TRY(launch_quad_scan("mfma_state_grad_scan", s, L.pl, true, q, Gh, gz, rc, omg, tot, BH, pr.T, pr.scale, gt.qfac, gt.lam))
        if (pr.gated && side.ok && hipEventRecord(side.scanned, s) != hipSuccess) return PA_ERR_HIP;
        if (!quad_kept(pr))
            PA_TRY(launch_quad_scan("mfma_state_scan_bwd", s2, L.pl, false, k, v, nullptr, st, gam, (float*)(c.ws + L.off_tot2), BH, pr.T, 1.0f,
                                    gt.kfac, gt.lam))
        PA_TRY(launch_quad_dphi("mfma_dq_state", s2, L.pl, false, q, Gh, gz, st, gam, pdq, BH, pr.T, pr.scale, gt.qfac, dotq))
        PA_TRY(launch_quad_read("mfma_dv_state", s, L.pl, true, k, rc, omg, pdv, nullptr, BH, pr.T, 1.0f, gt.kfac))
        PA_TRY(launch_quad_dphi("mfma_dk_state", s, L.pl, true, k, v, nullptr, rc, omg, pdk, BH, pr.T, 1.0f, gt.kfac, dotk))
        if (pr.gated) {
            if (side.ok && hipStreamWaitEvent(s2, side.scanned, 0) != hipSuccess) return PA_ERR_HIP;
            PA_TRY(launch_quad_boundary(s2, L.pl, st, rc, gam, omg, gt.lam, gt.xb, BH))
        }
        if (side.ok && (hipEventRecord(side.join, s2) != hipSuccess || hipStreamWaitEvent(s, side.join, 0) != hipSuccess)) return PA_ERR_HIP;
        AttnGate ag;
        ag.sums = GateSums{gt.bl, gt.blk};
        ag.qdq = gt.db;
        ag.kdk = gt.db2;
        PA_TRY(launch_chunk_bwd(s, pr.p, pr.d, q, k, v, Gh, gz, (bf16_t*)dQ, (bf16_t*)dK, (bf16_t*)dV, BH, pr.T, L.pl.cs, pr.scale, pdq,
                                1, pdk, 1, pdv, 1, ag, dotq, dotk))
        return PA_OK;
    }
    if (use_tiled(pr)) {
        // dQ's state part from S and [ghat, gz]; the state gradient R from phi(q) [ghat, gz]^T, read out with phi(k) for
        // dV and contracted with [v, 1] for dK; one kernel then adds the in-chunk gradients
        const TiledLayout L = make_tiled_layout(pr, true);
        TileDesc* tab = (TileDesc*)(c.ws + L.off_tab);
        bf16_t* Vp = (bf16_t*)(c.ws + L.off_vp);
        bf16_t* Sc = (bf16_t*)(c.ws + L.off_sc);
        bf16_t* Gh = (bf16_t*)(c.ws + L.off_gh);
        float* gz = (float*)(c.ws + L.off_gz);
        bf16_t* Gp = (bf16_t*)(c.ws + L.off_gp);
        bf16_t* Rc = (bf16_t*)(c.ws + L.off_rc);
        float* pdv = (float*)(c.ws + L.off_part);
        float* pdq = (float*)(c.ws + L.off_pdq);
        float* pdk = (float*)(c.ws + L.off_pdk);
        const bf16_t *q = (const bf16_t*)Q, *k = (const bf16_t*)K, *v = (const bf16_t*)V;
        const long long rows = (long long)BH * pr.T;
        hipStream_t st = c.stream;
        PA_TRY(launch_attn_prep(st, pr.d, (const bf16_t*)dO, (const bf16_t*)O, Z, Gh, gz, rows, pr.normalize))
        PA_TRY(launch_tiled_pack(st, pr.d, Gh, gz, Gp, rows))
        if (!pr.keep_state) {
            PA_TRY(launch_tiled_table(st, L.pl, tab))
            PA_TRY(launch_tiled_pack(st, pr.d, v, nullptr, Vp, rows))
            PA_TRY(launch_tiled_scan("tiled_state_scan_bwd", st, L.pl, false, k, Vp, tab, Sc, BH, pr.T, pr.chunk, 1.0f))
        }
        PA_TRY(launch_tiled_dphi("tiled_dq", st, L.pl, q, Gp, tab, Sc, pdq, BH, pr.T, pr.chunk, pr.scale, pr.scale))
        PA_TRY(launch_tiled_scan("tiled_state_grad_scan", st, L.pl, true, q, Gp, tab, Rc, BH, pr.T, pr.chunk, pr.scale))
        PA_TRY(launch_tiled_readout("tiled_dv", st, L.pl, k, tab, Rc, pdv, nullptr, BH, pr.T, pr.chunk, 1.0f))
        PA_TRY(launch_tiled_dphi("tiled_dk", st, L.pl, k, Vp, tab, Rc, pdk, BH, pr.T, pr.chunk, 1.0f, 1.0f))
        PA_TRY(launch_chunk_bwd(st, pr.p, pr.d, q, k, v, Gh, gz, (bf16_t*)dQ, (bf16_t*)dK, (bf16_t*)dV, BH, pr.T, pr.chunk, pr.scale,
                                pdq, 1, pdk, 1, pdv, 1))
        return PA_OK;
    }
    if (use_resident(pr)) {
        // Every part that goes through a state is left per slab in float32 by a walk that keeps that state in
        // registers: J_phi(q)^T (S ghat) for dQ from a forward walk, R^T phi(k) for dV and J_phi(k)^T (R v) for dK
        // from two backward walks over R (the two contractions want the accumulators in different orientations);
        // the normaliser's shares come from the d x d states; one kernel then adds the in-chunk gradients.
        const ResLayout R = make_res_layout(pr, true);
        const float s2 = pr.scale * pr.scale;
        const size_t slab = (size_t)BH * pr.T * pr.d;   // floats
        bf16_t* Kt = (bf16_t*)(c.ws + R.off_kt);
        bf16_t* Vt = (bf16_t*)(c.ws + R.off_vt);
        bf16_t* Qt = (bf16_t*)(c.ws + R.off_qt);
        bf16_t* Ght = (bf16_t*)(c.ws + R.off_ght);
        bf16_t* Gh = (bf16_t*)(c.ws + R.off_gh);
        float* gz = (float*)(c.ws + R.off_gz);
        bf16_t* Gam = (bf16_t*)(c.ws + R.off_gam);
        bf16_t* Omg = (bf16_t*)(c.ws + R.off_omg);
        float* gram = (float*)(c.ws + R.off_gram);
        float* totS = (float*)(c.ws + R.off_tot);
        float* totR = (float*)(c.ws + R.off_totr);
        float* pdv = (float*)(c.ws + R.off_part);
        float* pdq = (float*)(c.ws + R.off_pdq);
        float* pdk = (float*)(c.ws + R.off_pdk);
        const bf16_t *q = (const bf16_t*)Q, *k = (const bf16_t*)K, *v = (const bf16_t*)V;
        hipStream_t st = c.stream;
        PA_TRY(launch_attn_prep(st, pr.d, (const bf16_t*)dO, (const bf16_t*)O, Z, Gh, gz, (long long)BH * pr.T, pr.normalize))
        PA_TRY(launch_transpose_hd(st, pr.d, q, Qt, BH, pr.T))
        PA_TRY(launch_transpose_hd(st, pr.d, Gh, Ght, BH, pr.T))
        if (!pr.keep_state) {
            PA_TRY(launch_transpose_hd(st, pr.d, k, Kt, BH, pr.T))
            PA_TRY(launch_transpose_hd(st, pr.d, v, Vt, BH, pr.T))
            PA_TRY(launch_gram(st, pr.d, Kt, nullptr, gram, Gam, BH, pr.T, pr.chunk, false, 1.0f))
            if (R.pl.nseg > 1)
                PA_TRY(launch_res_walk("res_state_totals", st, pr.d, false, 0, Kt, Vt, nullptr, nullptr, totS, nullptr, BH, pr.T,
                                       pr.chunk, R.pl, 1.0f))
        }
        PA_TRY(launch_gram(st, pr.d, Qt, gz, gram, Omg, BH, pr.T, pr.chunk, true, s2))
        PA_TRY(launch_gram_apply(st, pr.d, q, Gam, gz, pdq + R.pl.nslab * slab, nullptr, BH, pr.T, pr.chunk, 2.f * s2, 0.f))
        PA_TRY(launch_gram_apply(st, pr.d, k, Omg, nullptr, pdk + R.pl.nslab * slab, nullptr, BH, pr.T, pr.chunk, 2.f, 0.f))
        PA_TRY(launch_res_walk("res_dq_walk", st, pr.d, false, 2, Kt, Vt, q, Gh, totS, pdq, BH, pr.T, pr.chunk, R.pl, s2))
        if (R.pl.nseg > 1)
            PA_TRY(launch_res_walk("res_grad_totals", st, pr.d, true, 0, Qt, Ght, nullptr, nullptr, totR, nullptr, BH, pr.T,
                                   pr.chunk, R.pl, 1.0f))
        PA_TRY(launch_res_walk("res_dv_walk", st, pr.d, true, 1, Qt, Ght, k, nullptr, totR, pdv, BH, pr.T, pr.chunk, R.pl, s2))
        PA_TRY(launch_res_walk("res_dk_walk", st, pr.d, true, 2, Qt, Ght, k, v, totR, pdk, BH, pr.T, pr.chunk, R.pl, s2))
        PA_TRY(launch_chunk_bwd(st, pr.p, pr.d, q, k, v, Gh, gz, (bf16_t*)dQ, (bf16_t*)dK, (bf16_t*)dV, BH, pr.T, pr.chunk, pr.scale,
                                pdq, R.pl.nslab + 1, pdk, R.pl.nslab + 1, pdv, R.pl.nslab))
        return PA_OK;
    }
    return PA_ERR_UNSUPPORTED;
}

// ---- a prompt into a decode state, through the state scan ----------------------------------------------
// The sum the decode state needs is what the forward scan accumulates: per-segment totals (float32, of phi rounded to bf16, on
// which the state kernels' scan runs as it is), which one more kernel adds, in the decode step's basis (monomials x_i x_j, i <= j,
// multiplicity on the state), to the decode state.  Gates: keys scaled by the square root of their decay to the prompt's end,
// the old state by the decay across the whole prompt.
namespace {

struct AbsorbLayout {
    QuadAbsorbPlan pl;
    size_t off_wk, off_gate, total;
};
AbsorbLayout make_absorb_layout(const pa_problem& pr) {
    AbsorbLayout L{};
    L.pl = quad_absorb_plan(pr.B * pr.H, pr.T);
    L.off_wk = align_up(L.pl.tot_floats * sizeof(float), 256);
    L.off_gate = align_up(L.off_wk + (pr.gated ? (size_t)pr.B * pr.H * pr.T * DH * sizeof(bf16_t) : 0), 256);      // (weighted keys)
    pa_problem gp = pr;
    gp.chunk = pr.T;
    L.total = L.off_gate + gate_workspace_bytes(gp, false);
    return L;
}

}  // namespace

bool mfma_absorb_supported(const pa_problem& pr) {
    return pr.dtype == PA_DTYPE_BF16 && pr.p == 2 && pr.d == DH && pr.v == DH && pr.T % QBLK == 0 &&
           (size_t)pr.B * pr.H <= 65535u;
}
size_t mfma_absorb_workspace_bytes(const pa_problem& pr) { return mfma_absorb_supported(pr) ? make_absorb_layout(pr).total : 0; }

pa_status mfma_absorb(const pa_problem& pr, const void* K, const void* V, const float* log_g, char* ws, hipStream_t s, float* S,
                      float* gamd, int D) {
    const AbsorbLayout L = make_absorb_layout(pr);
    const float *kfac = nullptr, *lam = nullptr;
    if (log_g != nullptr) {
        pa_problem gp = pr;
        gp.chunk = pr.T;
        gp.gated = 1;
        Ctx c{gp, s, ws, L.total, gate_buffers(gp, false, ws + L.off_gate)};
        pa_status st = gate_prepare(c, log_g, pr.T, true);
        if (st != PA_OK) return st;
        kfac = c.gate.kfac;
        lam = c.gate.lam;
    }
    PA_TRY(launch_quad_absorb(s, L.pl, (const bf16_t*)K, (const bf16_t*)V, kfac, lam, (bf16_t*)(ws + L.off_wk), (float*)ws, S, gamd, D, pr.B * pr.H, pr.T))
    return PA_OK;
}

}  // namespace pa
