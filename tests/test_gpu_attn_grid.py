"""The attention-form backward pass runs both of its halves in one launch while the grid is small and in two beyond (d = 32,
64): both against the oracle on either side of the line, through a sequence with a block that is not full."""
import pytest

from oracle import power_attn_oracle as orc
from paper_2507_04239_amd import binding, inputs

from gpu_util import assert_close, run_fwd_bwd, to_dev, to_np

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


def _run(case, kernels, Q, K, V, G, p, chunk, impl, normalize=True, log_g=None):
    print("case", case, flush=True)
    binding.profile_begin()
    got = run_fwd_bwd(Q, K, V, G, p, chunk, "bf16", normalize, impl=impl, log_g=log_g)
    names = set(binding.profile_end())
    assert kernels <= names and not ({"attn_bwd", "attn_bwd_dq", "chunk_bwd", "chunk_bwd_dq"} - kernels) & names, names
    for h in (0, Q.shape[1] - 1):
        sl = (slice(None), slice(h, h + 1))
        lg = None if log_g is None else log_g[sl]
        O, Z = orc.fwd_bhtd(Q[sl], K[sl], V[sl], p, None, normalize, 1.0, log_g=lg)
        grads = orc.bwd_bhtd(Q[sl], K[sl], V[sl], G[sl], p, None, normalize, 1.0, log_g=lg)
        assert_close({n: x[sl] for n, x in got.items()}, dict(zip(("O", "Z", "dQ", "dK", "dV", "dlog_g"), (O, Z, *grads))), "bf16", f"head {h}")


@pytest.mark.parametrize("p,d,H,T,one", [(2, 64, 384, 256, True), (2, 64, 385, 256, False), (4, 32, 384, 512, True), (4, 32, 385, 512, False)])
def test_gated_backward_on_either_side_of_the_one_launch_line(p, d, H, T, one):
    """2 blocks of 128 (256) rows a head: the sums across the block boundary come from the dK / dV half of either launch."""
    Q, K, V, G = inputs.make_qkvg(1, H, T, d, seed=9510 + H, dtype="bf16")
    lg = inputs.make_log_gates(1, H, T, 9511, 0.02)
    _run((p, d, H, T), {"attn_bwd"} if one else {"attn_bwd_dkdv", "attn_bwd_dq"}, Q, K, V, G, p, T, "mfma", log_g=lg)


@pytest.mark.parametrize("p,d,H,T,one", [(2, 32, 768, 256, True), (2, 32, 769, 256, False), (3, 64, 12, 256, True), (2, 32, 384, 384, True),
                                         (2, 32, 385, 384, False), (2, 128, 3, 384, False)])
def test_in_chunk_backward_on_either_side_of_the_one_launch_line(p, d, H, T, one):
    """The in-chunk kernels of the tiled family, chunks of 128 (d = 32: half a block of rows, the last block not full at T = 384)."""
    Q, K, V, G = inputs.make_qkvg(1, H, T, d, seed=9520 + H, dtype="bf16")
    _run((p, d, H, T), {"chunk_bwd"} if one else {"chunk_bwd_dkdv", "chunk_bwd_dq"}, Q, K, V, G, p, 128, "tiled", p % 2 == 0)


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


@pytest.mark.parametrize("d,H,T,p", [(128, 9, 32768, 2), (128, 16, 32768, 2), (64, 12, 65536, 2)])
def test_heads_in_groups(d, H, T, p):
    """Heads whose keys and values outgrow the memory-side cache are taken in groups: 5 + 4 (the last one short), 8 + 8, 4 + 4 + 4.
    Every head against the chunked kernels."""
    import torch
    from paper_2507_04239_amd import power_attn_bwd, power_attn_fwd
    print("case", d, H, T, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(9560 + H)
    Q, K, V, G = (torch.randn((1, H, T, d), device=dev, generator=gen, dtype=torch.bfloat16) * s for s in (d ** -.5, d ** -.5, 1., 1.))

    def step(chunk):
        O, Z = power_attn_fwd(Q, K, V, p, chunk, impl="mfma")
        return dict(zip(("O", "Z", "dQ", "dK", "dV"), (O, Z, *power_attn_bwd(Q, K, V, O, Z, G, p, chunk, impl="mfma"))))

    got, want = step(T), step(256)
    for n, w in want.items():
        e = (got[n].float() - w.float()).flatten(2).norm(dim=2) / w.float().flatten(2).norm(dim=2)
        print(n, e.max().item(), flush=True)
        assert e.max() <= 1e-2, n       # two bf16 evaluations, each within about 4e-3 of the definition


@pytest.mark.parametrize("p,H,T,gated", [(2, 127, 2048, False), (2, 128, 2047, False), (2, 128, 2048, False), (3, 114, 2100, False),
                                         (4, 103, 2305, False), (2, 128, 2048, True), (4, 114, 2176, True)])
def test_forward_on_either_side_of_the_wide_wave_line(p, H, T, gated):
    """d = 64: 64 rows per wave from 1024 blocks of 256 rows and 2048 tokens on, through blocks that are not full."""
    import torch
    from paper_2507_04239_amd import power_attn_fwd
    d = 64
    print("case", p, H, T, gated, flush=True)
    Q, K, V, _ = inputs.make_qkvg(1, H, T, d, seed=9570 + H, dtype="bf16", with_grad=False)
    lg = inputs.make_log_gates(1, H, T, 9571, 0.02) if gated else None
    tq, tk, tv = (to_dev(x, "bf16") for x in (Q, K, V))
    O, Z = power_attn_fwd(tq, tk, tv, p, T, p % 2 == 0, impl="mfma", log_g=None if lg is None else torch.from_numpy(lg).to("cuda:0"))
    for h in (0, H - 1):
        sl = (slice(None), slice(h, h + 1))
        wO, wZ = orc.fwd_bhtd(Q[sl], K[sl], V[sl], p, None, p % 2 == 0, 1.0, log_g=None if lg is None else lg[sl])
        assert_close(dict(O=to_np(O[sl]), Z=to_np(Z[sl])), dict(O=wO, Z=wZ), "bf16", f"head {h}")
