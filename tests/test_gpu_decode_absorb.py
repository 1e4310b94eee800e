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
