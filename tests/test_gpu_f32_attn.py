"""GPU parity of the float32 attention-form kernels (what an "auto" float32 call of up to a few thousand tokens runs,
whatever its chunk) against the float64 oracle, and their agreement with the chunked float32 kernels."""
import numpy as np
import pytest

from oracle import power_attn_oracle as orc
from paper_2507_04239_amd import inputs

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
        # sums of at most T products in float32: T 2^-24 relative to the sum of magnitudes, 8 of cancellation
        assert e_new <= max(2 * e_old, 8 * (T + d) * 2.0 ** -24)


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
