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


def test_more_row_blocks_than_one_grid_dimension_takes():
    """8.4 M tokens of one head are 65664 blocks of 128 rows.  Keys (and upstream gradients) are zero but in the first and the
    last chunk, so those two chunks come out as they do when they are the whole sequence."""
    import torch
    from paper_2507_04239_amd import power_attn_bwd, power_attn_fwd
    p, d, chunk, n = 2, 128, 4096, 2052
    T = chunk * n
    print("case", T, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(9550)
    Q, K, V, G = (torch.randn((1, 1, T, d), device=dev, generator=gen, dtype=torch.bfloat16) * s for s in (d ** -.5, d ** -.5, 1., 1.))
    for x in (K, G):
        x[:, :, chunk:-chunk] = 0
    ends = lambda x: torch.cat([x[:, :, :chunk], x[:, :, -chunk:]], 2).contiguous()

    def step(q, k, v, g):
        O, Z = power_attn_fwd(q, k, v, p, chunk, impl="tiled")
        dQ, dK, dV = power_attn_bwd(q, k, v, O, Z, g, p, chunk, impl="tiled")
        return dict(O=O, Z=Z, dQ=dQ, dK=dK, dV=dV)

    got = step(Q, K, V, G)
    want = step(*(ends(x) for x in (Q, K, V, G)))
    for x in (got["dQ"], got["dK"], got["dV"]):
        assert not x[:, :, chunk:-chunk].any()
    to_np = lambda x: x.float().cpu().numpy()
    assert_close({m: to_np(ends(x)) for m, x in got.items()}, {m: to_np(x) for m, x in want.items()}, "bf16", f"T = {T}", 0.1)
