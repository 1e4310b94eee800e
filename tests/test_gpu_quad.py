"""Chunk-state kernels of p = 2 at d = 64 and 128: lengths around their tiles (64-token stages, blocks of 256 and 512 tokens,
states 1280 or 1024 tokens apart, a last chunk of any length), few and many heads (the state scan in segments or in one walk),
kept and rebuilt states, scales with and without a power of two, gates, against the definition in float64 on the GPU."""
import numpy as np
import pytest

from gpu_util import assert_close, run_fwd_bwd

pytestmark = pytest.mark.gpu


def reference(Q, K, V, G, scale, normalize, log_g=None, block=2048):
    """One head in float64, rows of queries in blocks: O, Z, dQ, dK, dV (and dlog_g) as the header defines them (p = 2)."""
    import torch
    q, k, v, g = (torch.from_numpy(a).to("cuda:0", torch.float64) for a in (Q, K, V, G))
    T = q.shape[0]
    b_sum = None if log_g is None else torch.cumsum(torch.from_numpy(log_g).to("cuda:0", torch.float64), 0)
    db = q.new_zeros(T)
    O, Z, dQ, dK, dV = torch.zeros_like(v), q.new_zeros(T), torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for a in range(0, T, block):
        b = min(a + block, T)
        kt, vt = k[:b].t().contiguous(), v[:b].t().contiguous()
        s = scale * (q[a:b] @ kt)
        s.masked_fill_(torch.arange(b, device=q.device)[None, :] > torch.arange(a, b, device=q.device)[:, None], 0.0)
        w = s * s
        if b_sum is not None:
            f = torch.exp((b_sum[a:b, None] - b_sum[None, :b]).clamp_(max=0.0))
            w *= f
        Z[a:b] = w.sum(1)
        den = torch.where(Z[a:b, None] == 0, float("inf"), Z[a:b, None]) if normalize else 1.0      # (a row without weight gives 0)
        O[a:b] = (w @ v[:b]) / den
        gh = g[a:b] / den
        e = gh @ vt
        if normalize:
            e -= (gh * O[a:b]).sum(1, keepdim=True)
        t = 2.0 * scale * e * s
        if b_sum is not None:
            t *= f
            ea = e * w
            db[a:b] += ea.sum(1)
            db[:b] -= ea.sum(0)
        dQ[a:b] = t @ k[:b]
        dK[:b] += t.t().contiguous() @ q[a:b]
        dV[:b] += w.t().contiguous() @ gh
    out = {n: x.cpu().numpy() for n, x in zip(("O", "Z", "dQ", "dK", "dV"), (O, Z, dQ, dK, dV))}
    if b_sum is not None:
        out["dlog_g"] = torch.flip(torch.cumsum(torch.flip(db, [0]), 0), [0]).cpu().numpy()
    return out


CASES = [
    # heads, T, d, chunk asked for, scale, normalize, keep (, mean log-gate)
    (1, 7169, 64, 128, 1.0, True, True),       # whole
    (1, 7297, 64, 128, 1.0, True, False),      # the shortest backward pass with states at 1 .. 10 heads
    (12, 6401, 64, 128, 1.0, True, True),      # ... and at more; the forward pass has none to keep
    (1, 7425, 64, 128, 1.0, False, False),     # the shortest forward pass at 1 .. 6 heads
    (7, 8192, 64, 128, 1.0, True, True),       # ... and at more
    (2, 8192, 64, 128, 0.3, True, True),
    (1, 8959, 64, 256, 1.0, True, False),      # 7 x 1280 - 1, 7 x 1280, one token of an eighth chunk
    (3, 8960, 64, 128, 1.0, True, False),
    (1, 8961, 64, 128, 2.0, True, True),
    (13, 9300, 64, 128, 1.0, False, False),
    (1, 8193, 128, 128, 1.0, True, True),      # d = 128: states 1024 apart; the shortest backward pass at 1 and 2 heads
    (3, 9985, 128, 128, 1.0, True, False),     # ... at 3
    (1, 14337, 128, 128, 1.0, True, True),
    (11, 14337, 128, 128, 1.0, True, False),   # ... at more than 10
    (1, 18433, 128, 256, 0.7, True, True),
    (4, 20000, 128, 256, 1.0, True, False),    # whole forward at 4 .. 10 heads, states backward
    (2, 19456, 128, 128, 1.0, True, False),    # 19 x 1024
    (14, 18500, 128, 256, 1.0, False, True),   # one walk per head: no segments
    (1, 5120, 64, 128, 1.0, True, True, 0.02),     # gated: the longest sequence that runs whole
    (2, 5121, 64, 128, 1.0, True, False, 0.02),    # ... and the shortest with states, one token in the last chunk; the backward pass padded
    (2, 5121, 64, 128, 1.0, True, True, 0.02),     # ... kept states that the backward pass does not use, in the workspace it asks for
    (1, 5249, 64, 384, 1.0, True, True, 0.02),     # ... and the shortest backward pass
    (15, 5504, 64, 1024, 1.0, True, True, 0.02),   # whole forward at many heads (no multiple of the chunk), states backward
    (15, 5400, 64, 4096, 1.0, True, False, 0.02),  # ... padded to whole blocks, not to whole chunks
    (1, 5632, 64, 128, 1.0, True, True, 0.02),
    (2, 5633, 64, 128, 1.0, True, True, 0.02),     # 513 tokens in the last chunk
    (1, 6400, 64, 256, 0.3, True, False, 0.1),     # 5 x 1280
    (13, 6401, 64, 384, 1.0, False, False, 0.005),
    (48, 13000, 64, 1408, 1.0, True, True),    # over 256 MB of states: chunks beyond the spacing of the kernels are taken as they are
    (30, 22000, 64, 8192, 0.6, True, False),
    (5, 18500, 128, 2176, 1.0, True, True),
    (48, 13000, 64, 1920, 1.0, True, False, 0.02),
    (2, 7000, 64, 1920, 1.0, True, False, 0.02),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c))
def test_long_sequences(case):
    heads, T, d, chunk, scale, normalize, keep = case[:7]
    what = f"heads={heads} T={T} d={d} chunk={chunk} scale={scale} norm={normalize} keep={keep} gates={case[7:]}"
    print(what, flush=True)
    rng = np.random.default_rng(7 * T + d)

    def bf16(a):
        import torch
        return torch.from_numpy(a.astype(np.float32)).bfloat16().float().numpy()

    Q, K, V, G = (bf16(rng.standard_normal((1, heads, T, d), dtype=np.float32) * s) for s in (d ** -0.5, d ** -0.5, 1.0, 1.0))
    lg = None if len(case) == 7 else -case[7] * rng.standard_exponential((1, heads, T), dtype=np.float32)
    got = run_fwd_bwd(Q, K, V, G, 2, chunk, "bf16", normalize=normalize, scale=scale, keep_state=keep, log_g=lg)
    for h in sorted({0, heads - 1}):
        want = reference(Q[0, h], K[0, h], V[0, h], G[0, h], scale, normalize, None if lg is None else lg[0, h])
        assert_close({n: a[0, h] for n, a in got.items()}, want, "bf16", f"{what} head {h}")


@pytest.mark.parametrize("d,T", [(64, 9000), (128, 18500)])
def test_runs_are_bit_identical_and_chunks_agree(d, T):
    """Fixed order of sums, no float atomics; and the chunk asked for does not change which kernels run."""
    rng = np.random.default_rng(d)
    Q, K, V, G = (rng.standard_normal((1, 2, T, d), dtype=np.float32) * s for s in (d ** -0.5, d ** -0.5, 1.0, 1.0))
    a = run_fwd_bwd(Q, K, V, G, 2, 128, "bf16")
    b = run_fwd_bwd(Q, K, V, G, 2, 128, "bf16", keep_state=True)
    c = run_fwd_bwd(Q, K, V, G, 2, 384, "bf16")
    for n in a:
        assert np.array_equal(a[n], b[n]), n
        assert np.array_equal(a[n], c[n]), n


def device_inputs(seed, heads, T, d, gated):
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    x = [(torch.randn(1, heads, T, d, device="cuda:0", generator=gen) * s).bfloat16() for s in (d ** -0.5, d ** -0.5, 1.0, 1.0)]
    return x + [-0.02 * torch.rand(1, heads, T, device="cuda:0", generator=gen) if gated else None]


def step(x, ws, keep):
    from paper_2507_04239_amd import power_attn_bwd, power_attn_fwd
    q, k, v, g, lg = x
    O, Z = power_attn_fwd(q, k, v, 2, 128, workspace=ws, keep_state=keep, log_g=lg)
    return (O, Z, *power_attn_bwd(q, k, v, O, Z, g, 2, 128, workspace=ws, keep_state=keep, log_g=lg))


def scratch(x, keep):
    import torch
    from paper_2507_04239_amd import binding
    B, H, T, d = x[0].shape
    prob = binding.make_problem(B, H, T, d, d, 2, 128, keep_state=keep, gated=x[4] is not None)
    assert binding.power_attn_state_spacing(prob, False) < T and binding.power_attn_state_spacing(prob, True) < T
    need = max(binding.power_attn_workspace_bytes(prob, b) for b in (False, True))
    return torch.full((need,), 255, dtype=torch.uint8, device="cuda:0")        # (NaN in float32 and bf16: nothing unwritten is read)


def alone(x, keep):
    import torch
    out = step(x, scratch(x, keep), keep)
    torch.cuda.synchronize()
    return out


SHARED = [(64, 9000, False, True), (64, 9000, False, False), (64, 7000, True, True), (64, 7000, True, False), (128, 18560, False, True),
          (128, 18560, False, False)]


@pytest.mark.parametrize("d,T,gated,keep", SHARED)
def test_steps_queued_on_one_workspace(d, T, gated, keep):
    """Steps on different inputs, one after the other on one workspace without waiting: the next forward pass overwrites states that the
    backward pass before it, on two streams, still reads, and totals overwrite parts, unless all is ordered.  Bits as alone."""
    import torch
    print(f"d={d} T={T} gated={gated} keep={keep}", flush=True)
    xs = [device_inputs(seed, 1, T, d, gated) for seed in (1, 2, 3)]
    want = [alone(x, keep) for x in xs]
    ws = scratch(xs[0], keep)
    got = [step(x, ws, keep) for x in xs]
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert all(torch.equal(s, t) and bool(torch.isfinite(s.float()).all()) for s, t in zip(a, b))


def test_two_threads_with_states():
    """Two host threads, each with a stream, a side stream of the library's and a workspace of its own, at the same time: bits as alone."""
    import threading
    import torch
    from paper_2507_04239_amd import binding
    print("two threads", flush=True)
    shapes = [(64, 9000, False), (64, 7000, True)]
    xs = [device_inputs(10 + i, 2, T, d, g) for i, (d, T, g) in enumerate(shapes)]
    want = [alone(x, False) for x in xs]
    got, errors = [None, None], []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                ws = scratch(xs[i], False)
                for _ in range(4):
                    got[i] = step(xs[i], ws, False)
                stream.synchronize()
            binding.load_library().power_attn_release_thread()
        except Exception as e:   # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for a, b in zip(got, want):
        assert all(torch.equal(s, t) for s, t in zip(a, b))


@pytest.mark.parametrize("d,T", [(64, 9000), (128, 18560)])
def test_replayed_step_with_states(d, T):
    """A captured step, replayed with the program's own work between: bits as alone each time."""
    import torch
    print(f"d={d} T={T}", flush=True)
    a, b = device_inputs(21, 1, T, d, False), device_inputs(22, 1, T, d, False)
    want = [alone(x, False) for x in (a, b)]
    x = [None if t is None else t.clone() for t in a]
    ws = scratch(x, False)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        step(x, ws, False)           # (the library's side stream exists before the capture)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        out = step(x, ws, False)
    for n in (0, 1, 1, 0):
        for s, t in zip(x[:4], (a, b)[n][:4]):
            s.copy_(t)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(s, t) for s, t in zip(out, want[n])), n
        ws.fill_(255)
        step((b, a)[n], ws, False)   # eager work on the same workspace
        torch.cuda.synchronize()


def test_zero_rows_with_states():
    """Queries that are all zero have Z = 0: O = 0 and no gradient flows through the row, in chunks with a state before them too."""
    print("zero rows", flush=True)
    T = 9000
    Q, K, V, G = (t[0].float().cpu().numpy() for t in device_inputs(31, 1, T, 64, False)[:4])
    for t in (5, 1279, 1280, 8960, 8999):
        Q[0, t] = 0
    K[0, 1300] = V[0, 2600] = 0
    got = run_fwd_bwd(Q[None], K[None], V[None], G[None], 2, 128, "bf16")
    assert_close({n: a[0, 0] for n, a in got.items()}, reference(Q[0], K[0], V[0], G[0], 1.0, True), "bf16", "zero rows")
    for t in (5, 1279, 1280, 8960, 8999):
        assert not got["O"][0, 0, t].any() and not got["dQ"][0, 0, t].any() and got["Z"][0, 0, t] == 0


@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
@pytest.mark.parametrize("heads,T", [(1, 128), (3, 640), (90, 384), (2, 4224)])     # one segment, a short last one, long ones, many
def test_prompt_totals(heads, T, gated):
    """The decode state after a prompt, through the state scan: phi and the sum are rounded to bf16 (2^-8 each), with gates the two
    scaled keys of a product as well; the sums are float32."""
    import torch
    from paper_2507_04239_amd import binding
    print(f"heads={heads} T={T} gated={gated}", flush=True)
    torch.manual_seed(T + heads)
    K, V = (torch.randn(1, heads, T, 64, device="cuda:0").bfloat16() for _ in range(2))
    lg = -0.02 * torch.rand(1, heads, T, device="cuda:0") if gated else None
    prob = binding.make_problem(1, heads, T, 64, 64, 2, 1, dtype="bf16", gated=gated)
    assert binding.power_attn_decode_absorb_workspace_bytes(prob) > 0
    state = binding.power_attn_decode_init(binding.make_problem(1, heads, 1, 64, 64, 2, 1, dtype="bf16", gated=gated))
    flat = binding.power_attn_decode_absorb(prob, K, V, state, lg, fast=True).view(torch.float32)
    n, off = heads * 2080 * 64, (heads * 2080 * 64 * 4 + 255) // 256 * 64
    S, gam = flat[:n].view(heads, 2080, 64), flat[off:off + heads * 2080].view(heads, 2080)
    i, j = torch.triu_indices(64, 64, device="cuda:0")
    for h in sorted({0, heads - 1}):
        k, v = K[0, h].double(), V[0, h].double()
        phi = k[:, i] * k[:, j] * torch.where(i == j, 1.0, 2.0)
        if gated:
            b = torch.cumsum(lg[0, h].double(), 0)
            phi = phi * torch.exp(b[-1:] - b)[:, None]
        pt = phi.t().contiguous()
        tol = (4.1 if gated else 2.05) * 2.0 ** -8 + (T + 8) * 2.0 ** -24        # (and second-order terms)
        assert bool(((S[h].double() - pt @ v).abs() <= tol * (pt.abs() @ v.abs())).all())
        assert bool(((gam[h].double() - pt.sum(1)).abs() <= tol * pt.abs().sum(1)).all())
