"""The attention-form kernels at scales far from one: what has to stay in range is scale q.k and its powers, not those of q.k
or of the scale."""
import numpy as np
import pytest

from oracle import power_attn_oracle as orc
from paper_2507_04239_amd import inputs

from gpu_util import assert_close, run_fwd_bwd

pytestmark = pytest.mark.gpu

SHAPES = [
    # p, d, T, normalize, gated
    (4, 32, 320, True, False),
    (4, 64, 200, True, False),
    (4, 128, 256, True, True),
    (4, 32, 512, False, True),
    (3, 64, 200, False, False),
    (2, 128, 130, True, False),
    (2, 64, 256, True, True),
]


@pytest.mark.parametrize("shift", [-40, 40])
@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "-".join(str(x) for x in c))
def test_power_of_two_scale_against_operands_that_undo_it(case, shift):
    """scale = 2^shift with Q 2^-shift is the problem at scale 1 exactly: every output is the same to the bit, dQ times
    2^shift.  ((q.k)^4 is up to 2^160 larger than (scale q.k)^4 here, and scale^4 = 2^-160 is no float32.)"""
    p, d, T, normalize, gated = case
    print("case", case, shift, flush=True)
    Q, K, V, G = inputs.make_qkvg(1, 2, T, d, seed=9600 + T + d, dtype="bf16")
    lg = inputs.make_log_gates(1, 2, T, 9601 + T, 0.02) if gated else None
    one = run_fwd_bwd(Q, K, V, G, p, T, "bf16", normalize, 1.0, impl="mfma", log_g=lg)
    far = run_fwd_bwd(Q * 2.0 ** -shift, K, V, G, p, T, "bf16", normalize, 2.0 ** shift, impl="mfma", log_g=lg)
    far["dQ"] = far["dQ"] * np.float32(2.0 ** -shift)
    for n, want in one.items():
        assert np.isfinite(far[n]).all(), n
        assert np.array_equal(far[n], want), n


@pytest.mark.parametrize("p,d,scale", [(4, 64, 1.7e-12), (4, 32, -2.9e11), (3, 128, -0.6e-12), (2, 64, 3.3e-20)])
def test_far_scale_against_the_oracle(p, d, scale):
    print("case", p, d, scale, flush=True)
    T, normalize = 200, p % 2 == 0
    Q, K, V, G = inputs.make_qkvg(1, 1, T, d, seed=9700 + d, dtype="bf16")
    Q = np.ldexp(Q, -int(np.floor(np.log2(abs(scale)))))       # scores as large as at an ordinary scale; still bf16 numbers
    got = run_fwd_bwd(Q, K, V, G, p, T, "bf16", normalize, scale, impl="mfma")
    s = float(np.float32(scale))
    O, Z = orc.fwd_bhtd(Q, K, V, p, None, normalize, s)
    dQ, dK, dV = orc.bwd_bhtd(Q, K, V, G, p, None, normalize, s)
    assert_close(got, dict(O=O, Z=Z, dQ=dQ, dK=dK, dV=dV), "bf16", f"scale {scale}")


def test_chunked_in_chunk_kernels_at_a_far_scale():
    """The in-chunk part and the part through the state (tiled kernels, p = 2) carry the same scale."""
    p, d, T, chunk, shift = 2, 128, 512, 128, -40
    print("case chunked", flush=True)
    Q, K, V, G = inputs.make_qkvg(1, 2, T, d, seed=9800, dtype="bf16")
    one = run_fwd_bwd(Q, K, V, G, p, chunk, "bf16", True, 1.0, impl="tiled")
    far = run_fwd_bwd(Q * 2.0 ** -shift, K, V, G, p, chunk, "bf16", True, 2.0 ** shift, impl="tiled")
    far["dQ"] = far["dQ"] * np.float32(2.0 ** -shift)
    assert_close(far, one, "bf16", "chunked, scale 2^-40", 0.1)
