"""The attention-form backward pass runs both of its halves in one launch while the grid is small and in two beyond (d = 32,
64): both against the oracle on either side of the line, through a sequence with a block that is not full."""
import pytest

from oracle import power_attn_oracle as orc
from paper_2507_04239_amd import inputs

from gpu_util import assert_close, run_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,d,H,T", [
    (2, 64, 384, 129),      # 768 blocks of 128 rows of each kind: the last in one launch
    (2, 64, 385, 129),      # the first in two
    (2, 32, 768, 33),      # blocks of 256 rows
    (2, 32, 769, 33),
])
def test_backward_on_either_side_of_the_one_launch_line(p, d, H, T):
    print("case", p, d, H, T, flush=True)
    Q, K, V, G = inputs.make_qkvg(1, H, T, d, seed=9500 + H, dtype="bf16")
    got = run_fwd_bwd(Q, K, V, G, p, T, "bf16", impl="mfma")
    for h in (0, H - 1):
        sl = (slice(None), slice(h, h + 1))
        O, Z = orc.fwd_bhtd(Q[sl], K[sl], V[sl], p, None, True, 1.0)
        dQ, dK, dV = orc.bwd_bhtd(Q[sl], K[sl], V[sl], G[sl], p, None, True, 1.0)
        assert_close({n: x[sl] for n, x in got.items()}, dict(O=O, Z=Z, dQ=dQ, dK=dK, dV=dV), "bf16", f"head {h}")
