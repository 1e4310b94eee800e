"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header declares,
validates arguments and sizes workspaces without touching a GPU."""
import ctypes
import os
import re

import pytest

from paper_2507_04239_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.library_path()):
        import __graft_entry__ as g
        g.build()
    return binding.load_library()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "power_attn.h")).read()
    declared = set(re.findall(r"\b(power_attn_\w+)\s*\(", header))
    assert declared == set(binding.EXPORTED_SYMBOLS)
    for sym in declared:
        assert getattr(lib, sym) is not None


def test_status_strings(lib):
    assert lib.power_attn_status_string(0) == b"ok"
    assert b"workspace" in lib.power_attn_status_string(3)


def test_validation_and_sizes(lib):
    ok = binding.make_problem(1, 1, 256, 16, 16, 2, 32, dtype="f32")
    assert lib.power_attn_supported(ctypes.byref(ok), 1) == 0
    assert binding.power_attn_state_rows(ok) == 136
    assert binding.power_attn_workspace_bytes(ok, True) > binding.power_attn_workspace_bytes(ok, False) > 0
    # a ragged last chunk is a valid request, but only the chunked matrix-core kernels take it
    ragged = binding.make_problem(1, 1, 256, 16, 16, 2, 48)
    assert lib.power_attn_supported(ctypes.byref(ragged), 0) == 2
    assert binding.power_attn_workspace_bytes(ragged, False) == 0
    # padded inside the workspace by the tiled kernels (d = 32); the kernels of d = 64 take any length
    for d, padded in ((32, True), (64, False)):
        for T in (300, 9000):
            ragged_mfma = binding.make_problem(1, 2, T, d, d, 2, 128)
            assert lib.power_attn_supported(ctypes.byref(ragged_mfma), 1) == 0
            whole = binding.make_problem(1, 2, (T + 127) // 128 * 128, d, d, 2, 128)
            for backward in (False, True):
                a, b = (binding.power_attn_workspace_bytes(pr, backward) for pr in (ragged_mfma, whole))
                assert a > b > 0 if padded else a <= b, (d, T, backward)
    assert binding.power_attn_workspace_bytes(ragged_mfma, True) > 0
    odd_p = binding.make_problem(1, 1, 256, 16, 16, 3, 32, normalize=True)
    assert lib.power_attn_supported(ctypes.byref(odd_p), 0) == 1
    odd_p_unnorm = binding.make_problem(1, 1, 256, 16, 16, 3, 32, normalize=False)
    assert lib.power_attn_supported(ctypes.byref(odd_p_unnorm), 1) == 0
    big_p = binding.make_problem(1, 1, 256, 16, 16, 8, 32)
    assert lib.power_attn_supported(ctypes.byref(big_p), 0) == 2
    # null pointers are rejected before anything is launched (no GPU needed to see that)
    assert lib.power_attn_fwd(ctypes.byref(ok), None, None, None, None, None, None, 0, None) == 1
    assert lib.power_attn_fwd(None, None, None, None, None, None, None, 0, None) == 1
    # a real-looking call with no workspace is refused with the workspace status
    fake = ctypes.c_void_p(256)
    assert lib.power_attn_fwd(ctypes.byref(ok), fake, fake, fake, fake, None, None, 0, None) == 3


@pytest.mark.parametrize("chunk", [0, 1, 7])
@pytest.mark.parametrize("d,p", [(16, 1), (32, 2), (64, 2), (128, 4)])
def test_float32_attention_form_asks_for_no_states(lib, d, p, chunk):
    """Its scratch is one float per token (backward), at any chunk; the sizes beside it keep the chunked kernels' states."""
    bytes_of = binding.power_attn_workspace_bytes
    T = 7 * 429
    pr = binding.make_problem(2, 3, T, d, d, p, chunk, normalize=p % 2 == 0, dtype="f32")
    assert 0 < bytes_of(pr, False) <= 256 and 4 * 6 * T <= bytes_of(pr, True) < 4 * 6 * T + 256
    for other in (dict(impl="generic"), dict(gated=True)):
        pr = binding.make_problem(2, 3, T, d, d, p, chunk, normalize=p % 2 == 0, dtype="f32", **other)
        assert bytes_of(pr, False) >= 4 * 6 * T * d


def test_scratch_of_the_state_scans_shares_the_space_of_what_follows(lib):
    """12 heads of 65536 tokens, d = 64: 51 states of 295 KB and float32 totals of 786 KB a head; the totals are dead when the parts
    [T][64] in float32 are written.  (States and totals apart from the parts: 881 MB forward, 2063 MB backward.)"""
    heads, T = 12, 65536
    state, total, part, bf16 = (heads * n for n in (51 * (36 * 4096 + 4096) * 2, 52 * 6 * 4 * 32768, T * 64 * 4, T * 64 * 2))
    small = 3 * heads * T * 4 + 16 * 256
    pr = binding.make_problem(1, heads, T, 64, 64, 2, 128)
    assert total > part and 2 * part < total
    assert binding.power_attn_workspace_bytes(pr, False) <= state + total + small
    assert binding.power_attn_workspace_bytes(pr, True) <= 2 * (state + total) + bf16 + small
    kept = binding.make_problem(1, heads, T, 64, 64, 2, 128, keep_state=True)
    assert binding.power_attn_workspace_bytes(kept, True) <= 2 * state + total + part + bf16 + small


@pytest.mark.parametrize("d,heads,T,gated", [(64, 12, 65536, False), (64, 24, 32768, True), (128, 32, 32768, False)])
def test_a_longer_chunk_takes_less_workspace(lib, d, heads, T, gated):
    """The chunk is how a caller trades time for memory: beyond the spacing the kernels choose, each doubling drops half of the states.
    Few states are kept as the kernels choose, whatever is asked for."""
    small = [binding.power_attn_workspace_bytes(binding.make_problem(1, 1, 20480, d, d, 2, c, gated=gated), True) for c in (128, 1024, 2048, 8192)]
    assert max(small) - min(small) <= 256        # (sums of the gates per chunk)
    for backward in (False, True):
        need = [binding.power_attn_workspace_bytes(binding.make_problem(1, heads, T, d, d, 2, c, gated=gated), backward)
                for c in (128, 1024, 2048, 4096, 8192)]
        state = (d // 8 * (d // 8 + 1) // 2 * 64 * d + d * d) * 2 * heads * (2 if backward else 1)
        assert need[0] == need[1]
        for n, (a, b) in enumerate(zip(need[1:], need[2:])):
            assert a - b >= (T // (2048 << n) // 2 - 1) * state, (backward, need)


@pytest.mark.parametrize("d,gated", [(64, False), (64, True), (128, False)])
def test_kept_states_fit_what_the_backward_pass_asks_for(lib, d, gated):
    """keep_state: both passes take the backward pass's size, also where only the forward pass forms states."""
    lines = {64: (5120, 5632, 6400, 7168, 7296, 7424, 8191), 128: (8192, 9984, 14336, 16384, 17408, 18432, 20480, 24576)}[d]
    for heads in (1, 2, 3, 6, 8, 9, 11, 12, 14, 16, 48):
        for T in sorted({t + k for t in lines for k in (-128, 0, 1, 100, 128)}):
            for chunk in (128, 1024, 2048):
                pr = binding.make_problem(1, heads, T, d, d, 2, chunk, keep_state=True, gated=gated)
                need = [binding.power_attn_workspace_bytes(pr, b) for b in (False, True)]
                assert need[0] <= need[1], (heads, T, chunk, need)


def test_state_rows_match_the_embedding_dimension(lib):
    import math
    for d, p in [(16, 2), (32, 4), (12, 3)]:
        pr = binding.make_problem(1, 1, 64, d, d, p, 32, normalize=(p % 2 == 0), impl="generic")
        assert binding.power_attn_state_rows(pr) == math.comb(d + p - 1, p)


def test_automatic_chunk_choice():
    """chunk = 0 lets the library choose (host logic only): the attention form (one chunk) for short
    sequences, the chunked form beyond; an explicit chunk is returned unchanged."""
    from paper_2507_04239_amd import binding
    mk = binding.make_problem
    rc = binding.power_attn_resolved_chunk
    assert rc(mk(1, 12, 65536, 64, 64, 2, 128)) == 128
    assert rc(mk(1, 12, 65536, 64, 64, 2, 0)) == 256          # bf16, p = 2, d = 64: measured best chunk
    assert rc(mk(1, 12, 65536 + 128, 64, 64, 2, 0)) == 128    # 256 does not divide T
    assert rc(mk(1, 12, 65536 + 5, 64, 64, 2, 0)) == 256      # ragged: chunked all the same
    assert rc(mk(1, 12, 3000, 64, 64, 2, 0)) == 3000          # short and ragged: attention form, any length
    assert rc(mk(4, 12, 4096, 64, 64, 2, 0)) == 4096          # short: attention form
    assert rc(mk(4, 12, 8192, 64, 64, 2, 0)) == 256
    assert rc(mk(4, 12, 4096, 64, 64, 2, 0, gated=True)) == 256
    assert rc(mk(4, 12, 2048, 64, 64, 2, 0, gated=True)) == 2048
    assert rc(mk(4, 12, 512, 64, 64, 2, 0)) == 512
    # d = 128, p = 2: chunked from 18k tokens on (not gated: the chunked kernels take no gates there)
    assert rc(mk(8, 16, 32768, 128, 128, 2, 0)) == 256
    assert rc(mk(8, 16, 16384, 128, 128, 2, 0)) == 16384
    assert rc(mk(8, 16, 32768, 128, 128, 2, 0, gated=True)) == 32768
    assert rc(mk(8, 16, 32768, 128, 128, 4, 0)) == 32768
    # d = 32, p = 2: the tiled chunked kernels beyond 4096 tokens
    assert rc(mk(4, 8, 8192, 32, 32, 2, 0)) == 256
    assert rc(mk(4, 8, 4096, 32, 32, 2, 0)) == 4096
    assert rc(mk(4, 8, 8192, 32, 32, 2, 0, gated=True)) == 8192     # (they take no gates)
    # p = 3, d = 64: chunked matrix-core kernels exist (tiled), the attention form is the faster one at these lengths
    assert rc(mk(1, 4, 16384, 64, 64, 3, 0, normalize=False)) == 16384
    # p = 4, d = 32: the state is 52360 x 33 per head, the attention form stays cheaper far beyond 16k tokens
    assert rc(mk(2, 8, 16384, 32, 32, 4, 0, dtype="bf16")) == 16384
    # float32, small head: state 136 x 17; chunked from a few hundred tokens on
    assert rc(mk(1, 1, 64, 16, 16, 2, 0, dtype="f32")) == 64
    assert rc(mk(1, 1, 4096, 16, 16, 2, 0, dtype="f32")) == 64   # generic kernels: measured best chunk
    assert rc(mk(1, 1, 96, 16, 16, 2, 0, dtype="f32", impl="generic")) == 96
    assert rc(mk(1, 1, 4000, 16, 16, 2, 0, dtype="f32")) == 32   # largest power of two <= 64 dividing T
    assert binding.power_attn_workspace_bytes(mk(1, 12, 65536, 64, 64, 2, 0), False) == \
        binding.power_attn_workspace_bytes(mk(1, 12, 65536, 64, 64, 2, 256), False)
    assert rc(mk(1, 1, 100, 16, 16, 2, 7)) == 7                  # an explicit chunk is returned as it is ...
    assert not binding.power_attn_supported(mk(1, 1, 100, 16, 16, 2, 7), False)   # ... supported or not
    assert rc(mk(1, 1, 100, 16, 16, 2, -1)) == 0                 # invalid


def test_tiled_kernels_host_logic():
    """Which problems the tiled matrix-core kernels (degree and tile width as parameters) take, the state rows
    of their embedding C(d / d_tile + p - 1, p) d_tile^p (Sec. 4.1.1), and when the automatic choice runs them."""
    import math
    from paper_2507_04239_amd import binding
    mk, ok, rows = binding.make_problem, binding.power_attn_supported, binding.power_attn_state_rows

    def tspow_rows(d, p, dt):
        return math.comb(d // dt + p - 1, p) * dt ** p

    for (p, dt, d) in [(2, 4, 32), (2, 8, 32), (2, 16, 32), (3, 4, 32), (4, 2, 32), (4, 4, 32),
                       (2, 4, 64), (2, 8, 64), (2, 16, 64), (3, 4, 64)]:
        pr = mk(1, 2, 1024, d, d, p, 128, normalize=(p % 2 == 0), impl="tiled", d_tile=dt)
        assert ok(pr, True) and ok(pr, False), (p, dt, d)
        assert rows(pr) == tspow_rows(d, p, dt), (p, dt, d)
    # the default widths: 8, 4, 2 for p = 2, 3, 4
    assert rows(mk(1, 2, 1024, 32, 32, 2, 128, impl="tiled")) == tspow_rows(32, 2, 8)
    assert rows(mk(1, 2, 1024, 32, 32, 3, 128, normalize=False, impl="tiled")) == tspow_rows(32, 3, 4) == 7680
    assert rows(mk(1, 2, 1024, 32, 32, 4, 128, impl="tiled")) == tspow_rows(32, 4, 2) == 62016
    # config 4 as stated with no family named: the tiled kernels, not the vector-ALU family (52360 rows there)
    assert rows(mk(2, 8, 16384, 32, 32, 4, 128)) == 62016
    assert rows(mk(2, 8, 16384, 32, 32, 4, 128, d_tile=4)) == 84480
    assert rows(mk(2, 8, 16384, 32, 32, 4, 128, impl="generic")) == 52360
    # a tile width is a request for these kernels: p = 2, d = 64 otherwise runs the d_tile = 8 family of its own
    assert rows(mk(1, 12, 65536, 64, 64, 2, 128)) == 2304
    assert rows(mk(1, 12, 65536, 64, 64, 2, 128, d_tile=4)) == tspow_rows(64, 2, 4) == 2176
    assert rows(mk(1, 12, 65536, 64, 64, 2, 128, d_tile=16)) == 2560
    # not taken: widths that are not built, one chunk, chunks that are not a multiple of 128, gates, float32, d = 128 beyond p = 2 with width 8
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 128, d_tile=8), True)
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 128, d_tile=3), True)
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 1024, impl="tiled"), True)
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 64, impl="tiled"), True)
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 128, impl="tiled", gated=True), True)
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 128, impl="tiled", dtype="f32"), True)
    assert ok(mk(1, 2, 1024, 128, 128, 2, 128, impl="tiled"), True)
    assert rows(mk(1, 2, 1024, 128, 128, 2, 128, impl="tiled")) == tspow_rows(128, 2, 8) == 8704
    assert not ok(mk(1, 2, 1024, 128, 128, 2, 128, d_tile=4), True)
    assert not ok(mk(1, 2, 1024, 128, 128, 3, 128, impl="tiled", normalize=False), True)
    assert ok(mk(1, 2, 1024, 32, 32, 4, 128, gated=True), True)           # automatic: the vector-ALU family takes it
    assert rows(mk(1, 2, 1024, 32, 32, 4, 128, gated=True)) == 52360
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 128, d_tile=-1), True)        # invalid


def test_support_matrix_host_logic():
    """Which problems the matrix-core kernels take (host logic only, nothing is launched)."""
    from paper_2507_04239_amd import binding
    mk, ok, rows = binding.make_problem, binding.power_attn_supported, binding.power_attn_state_rows
    # chunked form: p = 2, d = 64, chunk a multiple of 128
    assert ok(mk(1, 2, 1024, 64, 64, 2, 128, impl="mfma"), True)
    assert rows(mk(1, 2, 1024, 64, 64, 2, 128, impl="mfma")) == 36 * 64            # tiled embedding, d_tile = 8
    assert not ok(mk(1, 2, 1024, 64, 64, 2, 64, impl="mfma"), True)
    # d = 128 chunked (136 tiles of 64 rows); the resident-state kernels when asked for by name
    assert ok(mk(1, 2, 1024, 128, 128, 2, 256, impl="mfma"), True)
    assert rows(mk(1, 2, 1024, 128, 128, 2, 256, impl="mfma")) == 136 * 64
    assert ok(mk(1, 2, 1024, 64, 64, 2, 128, impl="resident"), True)
    assert ok(mk(1, 2, 1024, 128, 128, 2, 256, impl="resident"), True)
    assert not ok(mk(1, 2, 1024, 64, 64, 2, 64, impl="resident"), True)            # chunk a multiple of 128
    assert not ok(mk(1, 2, 1024, 32, 32, 4, 128, impl="resident"), True)           # p = 2 only
    assert not ok(mk(1, 2, 1024, 64, 64, 2, 128, impl="resident", gated=True), True)
    assert ok(mk(1, 2, 1024, 128, 128, 2, 256, impl="auto"), True)                 # ... the generic family runs it
    assert rows(mk(1, 2, 1024, 128, 128, 2, 256)) == 8704                          # auto: the tiled embedding (Sec. 4.1.1)
    assert rows(mk(1, 2, 1024, 128, 128, 2, 256, impl="generic")) == 8256          # C(129, 2), Lemma 4.2
    # attention form: one chunk, degrees 2-4, head sizes 32 / 64 / 128, any length
    for p, d in ((2, 32), (3, 64), (4, 128), (4, 32)):
        assert ok(mk(1, 1, 1000, d, d, p, 1000, normalize=(p % 2 == 0), impl="mfma"), True), (p, d)
        assert rows(mk(1, 1, 1000, d, d, p, 1000, normalize=(p % 2 == 0), impl="mfma")) == 0
    assert not ok(mk(1, 1, 1024, 48, 48, 2, 1024, impl="mfma"), True)
    assert not ok(mk(1, 1, 1024, 64, 32, 2, 1024, impl="mfma"), True)              # d != v
    # with gates the sequence has to be a multiple of the dK / dV kernel's key block
    assert ok(mk(1, 1, 1024, 128, 128, 2, 1024, impl="mfma", gated=True), True)
    assert not ok(mk(1, 1, 1000, 128, 128, 2, 1000, impl="mfma", gated=True), True)
    assert ok(mk(1, 1, 1000, 128, 128, 2, 1000, impl="auto", gated=True), True)    # generic
    assert not ok(mk(1, 1, 128, 32, 32, 4, 128, impl="mfma", gated=True), True)    # d = 32: blocks of 256 keys
    assert ok(mk(1, 1, 256, 32, 32, 4, 256, impl="mfma", gated=True), True)
    # f32 never runs on the MFMA kernels
    assert not ok(mk(1, 1, 256, 64, 64, 2, 128, dtype="f32", impl="mfma"), True)


def test_decode_state_size_host_logic():
    from paper_2507_04239_amd import binding
    import math
    for (B, H, d, p) in ((1, 12, 64, 2), (2, 3, 32, 4), (1, 1, 128, 2)):
        prob = binding.make_problem(B, H, 1, d, d, p, 1)
        D = math.comb(d + p - 1, p)
        need = binding.power_attn_decode_state_bytes(prob)
        assert need >= B * H * D * (d + 1) * 4          # the float32 state itself
        assert need <= B * H * D * (d + 1) * 4 + D * 8 + B * H * ((D + 127) // 128) * (d + 1) * 4 + 5 * 256
    assert binding.power_attn_decode_state_bytes(binding.make_problem(1, 1, 1, 200, 200, 2, 1)) == 0   # head size above 128
    assert binding.power_attn_decode_state_bytes(binding.make_problem(1, 1, 1, 16, 16, 5, 1, normalize=False)) == 0


def test_state_spacing(lib):
    """What a pass forms: T where it has no states, else what the kernels choose, or a longer chunk that is taken as asked for."""
    mk, spacing = binding.make_problem, binding.power_attn_state_spacing
    assert [spacing(mk(1, 12, 65536, 64, 64, 2, 128), b) for b in (False, True)] == [1280, 1280]
    assert [spacing(mk(1, 32, 32768, 128, 128, 2, 256), b) for b in (False, True)] == [1024, 1024]
    assert [spacing(mk(1, 12, 65536, 64, 64, 2, 4096), b) for b in (False, True)] == [4096, 4096]
    assert [spacing(mk(1, 12, 7000, 64, 64, 2, 128), b) for b in (False, True)] == [7000, 1280]
    assert [spacing(mk(1, 12, 5001, 64, 64, 2, 128, gated=True), b) for b in (False, True)] == [5001, 5001]       # (padded)
    assert spacing(mk(2, 8, 16384, 32, 32, 4, 128), False) == 128 and spacing(mk(2, 8, 16384, 32, 32, 4, 0), False) == 16384
    assert spacing(mk(1, 2, 4096, 64, 64, 2, 256, impl="resident"), True) == 256
    assert spacing(mk(1, 1, 256, 16, 16, 2, 32, dtype="f32"), False) == 256
    assert spacing(mk(1, 1, 256, 16, 16, 2, 32, dtype="f32", impl="generic"), False) == 32
    assert spacing(mk(1, 1, 256, 16, 16, 2, 48), False) == 0 and spacing(mk(1, 1, 256, 16, 16, 3, 32), False) == 0


def test_plans_are_kept_by_value(lib):
    """What is looked up once per set of fields: integers of any kind are taken by their value at the call, floats are refused."""
    import numpy as np
    import torch
    Q = torch.empty(1, 1, 1024, 32, dtype=torch.bfloat16)

    def degree(p, chunk=1024, d_tile=0):
        ref, status, _ = binding._plan_of(0, Q, Q, p, chunk, False, 1.0, "auto", False, False, d_tile)
        assert status == 0
        return ref.contents.p, ref.contents.chunk, ref.contents.d_tile

    for kind in (int, np.int64, np.array, torch.tensor):
        assert degree(kind(2), kind(128), kind(8)) == (2, 128, 8), kind
    p, chunk = torch.tensor(2), np.array(128)
    assert degree(p, chunk) == (2, 128, 0)
    p.fill_(3)
    chunk[...] = 256
    assert degree(p, chunk) == (3, 256, 0)
    for bad in (dict(p=2.0), dict(p=2, chunk=128.0)):
        with pytest.raises(TypeError):
            degree(**bad)


def test_prompt_scratch_holds_weighted_keys_only_with_gates(lib):
    """Un-gated, the scratch of the hand-over is the float32 totals of its segments and nothing per token."""
    size = binding.power_attn_decode_absorb_workspace_bytes
    for heads, T in ((12, 65536), (1, 128), (200, 512)):
        plain, gated = (size(binding.make_problem(1, heads, T, 64, 64, 2, 1, gated=g)) for g in (False, True))
        assert plain % (heads * 6 * 4 * 32768) == 0 and plain > 0
        assert gated >= plain + heads * T * 64 * 2


STATIC_LONG = [
    # B, H, T, d, chunk: more than the static scratch as the kernels would space their states, less as asked for
    (1, 1, 24576, 64, 1024), (1, 1, 22528, 64, 1024), (1, 3, 9000, 64, 1024), (1, 1, 20480, 128, 0), (3, 11, 18500, 128, 0),
]


def test_static_scratch_takes_the_states_that_fit_as_asked_for(lib):
    """Without a GPU a call that is taken ends at the scratch array's address (4: HIP error), a refused one before (3)."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch")
    fake = ctypes.c_void_p(256)

    def status(*a, **k):
        return lib.power_attn_fwd_static(ctypes.byref(binding.make_problem(*a, **k)), fake, fake, fake, fake, fake, None)

    for B, H, T, d, c in STATIC_LONG:
        pr = binding.make_problem(B, H, T, d, d, 2, c)
        assert binding.power_attn_workspace_bytes(pr, False) > lib.power_attn_static_scratch_bytes()
        assert status(B, H, T, d, d, 2, c) == 4, (B, H, T, d, c)
    for T in (16384, 57344):
        for c in (512, 1024, 2048, 4096, 8192, 28672):
            if c < T and T * 256 + T // c * 303104 <= 16 << 20:
                assert status(1, 1, T, 64, 64, 2, c) == 4, (T, c)
    # refused as ever: too many states, or too many tokens
    for a in ((1, 12, 65536, 64, 64, 2, 128), (1, 1, 65536, 64, 64, 2, 32768), (1, 1, 24576, 64, 64, 2, 128), (1, 1, 24576, 128, 128, 2, 0),
              (1, 1, 20480, 128, 128, 2, 2048)):
        assert status(*a) == 3, a
