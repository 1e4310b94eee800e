"""The exact matrix-core hand-over of a prompt into a decode state (bf16 tokens, p = 2) at the edges of its 64-token tiles,
for each head size it has, on top of a state that already holds tokens, against the sum written out in float64."""
import numpy as np
import pytest

from paper_2507_04239_amd import binding, inputs

from gpu_util import rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T", [1, 31, 64, 65, 128, 200])
def test_exact_hand_over(T, d, gated):
    import torch
    B, H, past, p = 1, 3, 70, 2
    print("case", T, d, gated, flush=True)
    n = past + T
    _, K, V, _ = inputs.make_qkvg(B, H, n, d, seed=9300 + T + d, dtype="bf16", with_grad=False)
    lg = inputs.make_log_gates(B, H, n, 9400 + T, 0.05) if gated else None
    if gated:
        lg[0, 1, n // 2] = -np.inf          # a gate of zero forgets everything before it
    tk, tv = to_dev(K, "bf16"), to_dev(V, "bf16")
    tl = None if lg is None else torch.from_numpy(np.ascontiguousarray(lg)).to("cuda:0")
    state = binding.power_attn_decode_init(binding.make_problem(B, H, 1, d, d, p, 1, True, 1.0, "bf16", "auto", False, gated))
    for lo, hi in ((0, past), (past, n)):
        prob = binding.make_problem(B, H, hi - lo, d, d, p, 1, True, 1.0, "bf16", "auto", False, gated)
        binding.power_attn_decode_absorb(prob, tk[:, :, lo:hi].contiguous(), tv[:, :, lo:hi].contiguous(), state,
                                         None if tl is None else tl[:, :, lo:hi].contiguous(), fast=False)
    torch.cuda.synchronize()
    i, j = np.triu_indices(d)
    D = len(i)
    n_s = B * H * D * d
    off_gam = ((n_s * 4 + 255) // 256 * 256) // 4
    words = state.view(torch.float32)
    S = to_np(words[:n_s]).reshape(B, H, D, d)
    gam = to_np(words[off_gam: off_gam + B * H * D]).reshape(B, H, D)
    mult = np.where(i == j, 1.0, 2.0)
    for h in range(H):
        k, v = K[0, h].astype(np.float64), V[0, h].astype(np.float64)
        w = np.ones(n)
        if gated:
            for t in range(n - 2, -1, -1):
                w[t] = w[t + 1] * np.exp(np.float64(lg[0, h, t + 1]))
        phi = k[:, i] * k[:, j] * mult * w[:, None]
        # float32 sums of exact products (gated: products rounded three times): n 2^-24 relative to the sum of magnitudes
        for got, want, mag in ((S[0, h], phi.T @ v, np.abs(phi).T @ np.abs(v)), (gam[0, h], phi.sum(0), np.abs(phi).sum(0))):
            assert rel_l2(got, want) <= 2e-6
            assert np.all(np.abs(got - want) <= (n + 8) * 2.0 ** -24 * mag + 1e-30)


def _recurrence(K, V, lg, S, gam):
    """The state after the tokens K, V [T, d], in float32 and in order."""
    i, j = np.triu_indices(K.shape[1])
    mult = np.where(i == j, 1.0, 2.0).astype(np.float32)
    with np.errstate(all="ignore"):
        for t in range(K.shape[0]):
            g = np.float32(1.0 if lg is None else np.exp(np.float32(lg[t])))
            coef = mult * (K[t, i] * K[t, j])
            S = g * S + coef[:, None] * V[t][None, :]
            gam = g * gam + coef
    return S, gam


NOT_FINITE = ["infinite product", "infinite value", "infinite key", "not a number", "overflowing sum", "infinite state"]
NOT_FINITE_GATED = ["infinite state, vanishing gates", "infinite state, a gate of zero", "growing gates"]


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("what,gated", [(w, g) for w in NOT_FINITE for g in (False, True)] + [(w, True) for w in NOT_FINITE_GATED])
def test_hand_over_of_numbers_that_are_not_finite(what, d, gated):
    """Infinities in the tokens, products that overflow and states that already hold infinities leave what the recurrence
    leaves in float32: infinities of the same sign and NaN in the same places, and finite sums everywhere else."""
    import torch
    B, H, T, p = 1, 2, 100, 2
    print("case", what, d, gated, flush=True)
    _, K, V, _ = inputs.make_qkvg(B, H, T, d, seed=9350 + d, dtype="bf16", with_grad=False)
    lg = inputs.make_log_gates(B, H, T, 9450, 0.05) if gated else None
    K, V = K.copy(), V.copy()
    K[0, 1, 20] = np.sign(K[0, 1, 20])      # products with an empty lower half
    if what == "infinite product":
        K[0, 1, 70, 3], K[0, 1, 70, d - 2] = 2.0 ** 66, -2.0 ** 67
    elif what == "infinite value":
        V[0, 1, 20, 5] = np.inf
        V[0, 1, 90, 6] = -np.inf
    elif what == "infinite key":
        K[0, 1, 33, 17] = -np.inf
    elif what == "not a number":
        K[0, 1, 40, 9] = np.nan
    elif what == "overflowing sum":
        K[0, 1, 50:60, 4] = 2.0 ** 63
        V[0, 1, 50:60, 1] = 1.0
    if what == "infinite state, vanishing gates":
        lg[:] = -2.0            # their product is no float32
    elif what == "infinite state, a gate of zero":
        lg[0, 1, 50] = -np.inf
    elif what == "growing gates":
        lg[0, 1] = 1.5          # (log-gates are <= 0 in use)
    tk, tv = to_dev(K, "bf16"), to_dev(V, "bf16")
    tl = None if lg is None else torch.from_numpy(np.ascontiguousarray(lg)).to("cuda:0")
    n_s = B * H * (d * (d + 1) // 2) * d
    D = d * (d + 1) // 2
    off_gam = ((n_s * 4 + 255) // 256 * 256) // 4
    one = binding.make_problem(B, H, 1, d, d, p, 1, True, 1.0, "bf16", "auto", False, gated)
    state = binding.power_attn_decode_init(one)
    words = state.view(torch.float32)
    if "infinite state" in what:
        words[(D + 3) * d + 1] = np.inf
        words[off_gam + D + 7] = -np.inf
    S0 = to_np(words[:n_s]).reshape(H, D, d)
    gam0 = to_np(words[off_gam: off_gam + H * D]).reshape(H, D)
    prob = binding.make_problem(B, H, T, d, d, p, 1, True, 1.0, "bf16", "auto", False, gated)
    binding.power_attn_decode_absorb(prob, tk, tv, state, tl, fast=False)
    torch.cuda.synchronize()
    S = to_np(words[:n_s]).reshape(H, D, d)
    gam = to_np(words[off_gam: off_gam + H * D]).reshape(H, D)
    bad = 0
    for h in range(H):
        want_S, want_g = _recurrence(K[0, h], V[0, h], None if lg is None else lg[0, h], S0[h], gam0[h])
        with np.errstate(all="ignore"):
            mag_S, mag_g = _recurrence(np.abs(K[0, h]), np.abs(V[0, h]), None if lg is None else lg[0, h], np.abs(S0[h]), np.abs(gam0[h]))
        for got, want, mag in ((S[h], want_S, mag_S), (gam[h], want_g, mag_g)):
            assert np.array_equal(np.isnan(got), np.isnan(want))
            inf = np.isinf(want)
            assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
            fin = np.isfinite(want)
            bad += int((~fin).sum())
            # two float32 sums of T terms, each product rounded up to three times
            assert np.all(np.abs(got[fin].astype(np.float64) - want[fin]) <= 2 * (T + 8) * 2.0 ** -24 * mag[fin].astype(np.float64) + 1e-30)
    assert bad > 0


@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
@pytest.mark.parametrize("d,heads", [(64, 25), (64, 26), (128, 3), (128, 4)])      # the last with small blocks, the first with large ones
@pytest.mark.parametrize("T", [1, 64, 129, 193])
def test_exact_hand_over_of_many_heads(T, d, heads, gated):
    """Small and large blocks around the stages of 64 tokens, of which three are under way at once; one head in the middle holds an
    infinite value and keys whose products are no float32 of either sign."""
    import torch
    print("case", T, d, heads, gated, flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(T + d + heads)
    K, V = (torch.randn(1, heads, T, d, device="cuda:0", generator=gen).bfloat16() for _ in range(2))
    lg = -0.05 * torch.rand(1, heads, T, device="cuda:0", generator=gen) if gated else None
    odd = heads // 2
    V[0, odd, T // 2, 5] = float("inf")
    K[0, odd, T - 1, 3], K[0, odd, T - 1, 40] = 2.0 ** 66, 2.0 ** 67
    K[0, odd, T // 3, 3], K[0, odd, T // 3, 40] = -2.0 ** 66, 2.0 ** 67
    one = binding.make_problem(1, heads, 1, d, d, 2, 1, dtype="bf16", gated=gated)
    state = binding.power_attn_decode_init(one)
    prob = binding.make_problem(1, heads, T, d, d, 2, 1, dtype="bf16", gated=gated)
    words = binding.power_attn_decode_absorb(prob, K, V, state, lg, fast=False).view(torch.float32)
    D = d * (d + 1) // 2
    n, off = heads * D * d, (heads * D * d * 4 + 255) // 256 * 64
    S, gam = words[:n].view(heads, D, d), words[off:off + heads * D].view(heads, D)
    i, j = torch.triu_indices(d, d, device="cuda:0")
    for h in sorted({0, heads - 1, odd}):
        if h == odd:
            want_S, want_g = _recurrence(*(to_np(a[0, h].float()) for a in (K, V)), None if lg is None else to_np(lg[0, h]),
                                         np.zeros((D, d), np.float32), np.zeros(D, np.float32))
            for got, want in ((to_np(S[h]), want_S), (to_np(gam[h]), want_g)):
                assert not np.isfinite(want).all()
                assert np.array_equal(np.isnan(got), np.isnan(want))
                inf = np.isinf(want)
                assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
            continue
        k, v = K[0, h].double(), V[0, h].double()
        phi = k[:, i] * k[:, j] * torch.where(i == j, 1.0, 2.0)
        if gated:
            b = torch.cumsum(lg[0, h].double(), 0)
            phi = phi * torch.exp(b[-1:] - b)[:, None]
        pt = phi.t().contiguous()
        tol = (T + 8) * 2.0 ** -24          # as above
        assert bool(((S[h].double() - pt @ v).abs() <= tol * (pt.abs() @ v.abs()) + 1e-30).all())
        assert bool(((gam[h].double() - pt.sum(1)).abs() <= tol * pt.abs().sum(1) + 1e-30).all())
