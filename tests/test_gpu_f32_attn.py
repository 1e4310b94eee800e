"""GPU parity of the float32 attention-form kernels (what an "auto" float32 call of up to a few thousand tokens runs,
whatever its chunk) against the float64 oracle, and their agreement with the chunked float32 kernels."""
import numpy as np
import pytest

from oracle import power_attn_oracle as orc
from paper_2507_04239_amd import binding, inputs

from gpu_util import assert_close, rel_l2, run_fwd_bwd, to_dev, to_np

pytestmark = pytest.mark.gpu

CASES = [
    # p, d, B, H, T, chunk, normalize, scale
    (2, 16, 1, 1, 256, 32, True, 1.0),
    # a single token (un-normalised: with the division its dQ and dK are 0 in exact arithmetic, and no error is relative to 0)
    (2, 16, 1, 1, 1, 1, False, 1.0),
    (2, 32, 1, 2, 15, 15, True, 1.0),         # one partial tile
    (2, 32, 1, 1, 17, 17, True, 1.3),         # a tile and a row
    (2, 64, 2, 1, 65, 13, True, 0.7),         # the fifth tile goes back to the first wave
    (4, 32, 1, 1, 100, 50, True, 1.0),
    (4, 64, 1, 2, 96, 96, True, 1.0),
    (1, 32, 1, 1, 77, 7, False, 1.0),         # degree 1: weights of either sign
    (3, 64, 1, 1, 130, 65, False, -1.1),
    (2, 128, 1, 1, 200, 40, True, 1.0),
    (4, 128, 1, 1, 33, 33, False, 0.5),
    (2, 16, 4, 128, 33, 33, True, 1.0),       # 32 rows per workgroup (512 workgroups and more)
    (2, 64, 4, 64, 47, 47, True, 1.0),
    (2, 128, 4, 128, 20, 20, True, 1.0),
]


def _bound(T, d):
    # sums of at most T + d products in float32: independent roundings grow with the root of their number; 8 of cancellation
    return 8 * (T + d) ** 0.5 * 2.0 ** -24


def _kernels(f):
    binding.profile_begin()
    out = f()
    return out, {n for n in binding.profile_end() if "table" not in n}


def _check_heads(got, Q, K, V, G, p, normalize, chunk=None):
    """The first and the last head against the oracle."""
    B, H, T, d = Q.shape
    for b, h in {(0, 0), (B - 1, H - 1)}:
        sl = (slice(b, b + 1), slice(h, h + 1))
        O, Z = orc.fwd_bhtd(Q[sl], K[sl], V[sl], p, chunk, normalize, 1.0)
        dQ, dK, dV = orc.bwd_bhtd(Q[sl], K[sl], V[sl], G[sl], p, chunk, normalize, 1.0)
        want = dict(O=O, Z=Z, dQ=dQ, dK=dK, dV=dV)
        assert_close({n: x[sl] for n, x in got.items()}, want, "f32", f"head {b} {h}")
        for n, w in want.items():
            assert rel_l2(got[n][sl], w) <= _bound(T, d), n


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c))
def test_float32_attention_form(case):
    p, d, B, H, T, chunk, normalize, scale = case
    print("case", case, flush=True)
    Q, K, V, G = inputs.make_qkvg(B, H, T, d, seed=9100 + CASES.index(case), dtype="f32")
    if T > 60:
        Q[0, 0, 3] = 0        # Z = 0: no output, no gradient
    got = run_fwd_bwd(Q, K, V, G, p, chunk, "f32", normalize, scale)
    ref = run_fwd_bwd(Q, K, V, G, p, chunk, "f32", normalize, scale, impl="generic")
    O, Z = orc.fwd_bhtd(Q, K, V, p, None, normalize, scale)
    dQ, dK, dV = orc.bwd_bhtd(Q, K, V, G, p, None, normalize, scale)
    want = dict(O=O, Z=Z, dQ=dQ, dK=dK, dV=dV)
    assert_close(got, want, "f32", f"float32 attention form {case}")
    for n, w in want.items():
        e_new, e_old = rel_l2(got[n], w), rel_l2(ref[n], w)
        print(f"{n}: {e_new:.2e} (chunked kernels {e_old:.2e})", flush=True)
        assert e_new <= max(2 * e_old, _bound(T, d))


# 32 rows per workgroup (512 workgroups and more), with several 64-row steps of the four waves, lengths on either side of a
# step and of a block; (d = 128: forward pass only, the backward pass keeps 16)
@pytest.mark.parametrize("p,d,B,H,T", [
    (2, 16, 2, 64, 129), (4, 16, 3, 60, 95), (2, 32, 2, 90, 65), (3, 32, 2, 64, 161), (1, 32, 1, 60, 300), (2, 64, 2, 52, 150),
    (4, 64, 1, 64, 257), (3, 64, 1, 128, 127), (2, 128, 1, 64, 259), (1, 128, 2, 43, 191),
])
def test_wide_blocks_over_several_steps(p, d, B, H, T):
    print("case", p, d, B, H, T, flush=True)
    assert B * H * ((T + 31) // 32) >= 512
    normalize = p % 2 == 0
    Q, K, V, G = inputs.make_qkvg(B, H, T, d, seed=9210 + T, dtype="f32")
    got, names = _kernels(lambda: run_fwd_bwd(Q, K, V, G, p, T, "f32", normalize))
    assert names == {"f32_attn_fwd", "f32_attn_dq", "f32_attn_dkdv"}
    _check_heads(got, Q, K, V, G, p, normalize)


# either side of T = 4096 with B H T > 262144, of B H T = 262144 beyond it, and of T = 16384
@pytest.mark.parametrize("H,T,attention", [(65, 4096, True), (63, 4097, True), (64, 4097, False), (16, 16384, True), (1, 16385, False)])
def test_lines_of_the_dispatch(H, T, attention):
    p, d = 2, 16
    print("case", H, T, flush=True)
    Q, K, V, G = inputs.make_qkvg(1, H, T, d, seed=9220 + T % 100, dtype="f32")
    got, names = _kernels(lambda: run_fwd_bwd(Q, K, V, G, p, 0, "f32"))
    assert all(n.startswith("f32_attn_") == attention for n in names) and names, names
    _check_heads(got, Q, K, V, G, p, True, 256)


def test_static_scratch_takes_a_length_without_small_divisors():
    """No chunk but 1 and T divides a prime T: what used to mean a state per token needs no scratch here."""
    import torch
    from paper_2507_04239_amd.binding import power_attn_fwd_static
    B, H, T, d = 1, 8, 1009, 64
    print("case", T, flush=True)
    Q, K, V, _ = inputs.make_qkvg(B, H, T, d, seed=9250, dtype="f32", with_grad=False)
    tq, tk, tv = (to_dev(x, "f32") for x in (Q, K, V))
    O, Z = torch.full_like(tv, float("nan")), torch.full((B, H, T), float("nan"), device="cuda:0")
    power_attn_fwd_static(tq, tk, tv, O, Z, 2, 0)
    want_O, want_Z = orc.fwd_bhtd(Q, K, V, 2, None, True, 1.0)
    assert_close(dict(O=to_np(O), Z=to_np(Z)), dict(O=want_O, Z=want_Z), "f32", "static scratch")


def test_float32_attention_form_repeats_bit_for_bit():
    Q, K, V, G = inputs.make_qkvg(1, 3, 150, 32, seed=9200, dtype="f32")
    a = run_fwd_bwd(Q, K, V, G, 2, 50, "f32")
    b = run_fwd_bwd(Q, K, V, G, 2, 50, "f32")
    for n in a:
        assert np.array_equal(a[n], b[n]), n
