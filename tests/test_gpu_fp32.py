"""fp32 tensors: the forms of the kernels that the smaller parity cases do not reach (a workgroup's waves take the key tiles of
one group of rows in one, two, four or eight ways, chosen by the number of groups and the length of the
run of rows; test_fp32_forms_of_the_gpu_tests has which), at lengths around their tiles, against the fp64 oracle on single heads."""
import pytest

import synth_inputs
from ha_testutil import assert_close, assert_lse_close, have_gpu, run_oracle, to_device, to_host
from oracle import hyperattn_oracle as orc

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("H,n,d,b,m,causal,n_min", [
    (16, 4096, 64, 128, 40, 0, 4096),     # one way: 128-row tiles
    (16, 4096, 128, 128, 33, 0, 4096),
    (8, 4096, 64, 64, 64, 1, 1024),       # two ways: 64-row tiles, blocks of 64
    (6, 4032, 128, 63, 7, 0, 4096),       # four, one row of the second 32-row tile idle
    (6, 4032, 64, 63, 7, 0, 4096),        # two, one row idle
    (3, 1056, 64, 33, 31, 0, 4096),       # four: 32-row tiles, one row in the second
    (1, 264, 128, 33, 0, 1, 132)])
def test_forward_fp32_forms(H, n, d, b, m, causal, n_min):
    import paper_2310_05869_amd as ha
    print(f"fp32 forms H={H} n={n} d={d} b={b} m={m} causal={causal}", flush=True)
    cfg = dict(B=1, H=H, n=n, d=d, dtype="fp32", law="iid", b=b, m=m, r=7, causal=causal, n_min=n_min, seed=1)
    Q, K, V = synth_inputs.make_qkv(cfg)
    out, lse = ha.hyperattn_forward(*(to_device(x, "fp32") for x in (Q, K, V)), b, m, 7, causal=bool(causal), n_min=n_min, seed=1)
    for hd in sorted({0, H - 1}):
        ref_o, ref_l = run_oracle(*(x[:, hd:hd + 1] for x in (Q, K, V)), cfg)
        assert_close(to_host(out)[:, hd:hd + 1], ref_o, "fp32", f"out, head {hd}")
        assert_lse_close(to_host(lse)[:, hd:hd + 1], ref_l, "fp32", f"lse, head {hd}")


@pytest.mark.parametrize("H,n,d,causal", [(16, 4097, 64, True), (16, 4127, 128, False), (8, 4160, 64, False),
                                          (1, 31, 64, True), (2, 33, 128, True), (1, 1, 64, False)])
def test_exact_attention_fp32_forms(H, n, d, causal):
    import paper_2310_05869_amd as ha
    print(f"fp32 exact forms H={H} n={n} d={d} causal={causal}", flush=True)
    Q, K, V = synth_inputs.iid_qkv(1, H, n, d, "fp32")
    out, lse = ha.exact_attn_forward(*(to_device(x, "fp32") for x in (Q, K, V)), causal=causal)
    hd = H - 1
    ref_o, ref_l = orc.exact_attention(*(x[0, hd] for x in (Q, K, V)), causal=causal)
    assert_close(to_host(out)[0, hd], ref_o, "fp32", "out")
    assert_lse_close(to_host(lse)[0, hd], ref_l, "fp32", "lse")


@pytest.mark.parametrize("H,n,d,b,m,causal,n_min", [
    (32, 4096, 64, 128, 100, 0, 4096),    # one way in every pass, samples included
    (32, 4096, 128, 128, 128, 1, 2048),
    (30, 896, 128, 128, 64, 0, 4096),     # one way, delta formed and samples' sums added in the pass
    (5, 2112, 64, 33, 65, 0, 4096),       # four ways, one row in the second 32-row tile
    (1, 264, 128, 33, 5, 1, 132)])
def test_backward_fp32_forms(H, n, d, b, m, causal, n_min):
    """Criterion |got - ref| <= 2^-14 bound (fp32 sums of up to 2^10 terms; bound: the oracle on absolute values)."""
    import torch

    import paper_2310_05869_amd as ha
    print(f"fp32 backward forms H={H} n={n} d={d} b={b} m={m} causal={causal}", flush=True)
    cfg = dict(B=1, H=H, n=n, d=d, dtype="fp32", law="iid", b=b, m=m, r=7, causal=causal, n_min=n_min, seed=1)
    Q, K, V = synth_inputs.make_qkv(cfg)
    G = synth_inputs.iid_qkv(1, H, n, d, "fp32", seed=5)[0]
    tq, tk, tv, tg = (to_device(x, "fp32") for x in (Q, K, V, G))
    kw = dict(causal=bool(causal), n_min=n_min, seed=1)
    ws = ha.alloc_workspace(ha.make_shape(1, H, n, d, ha.HA_FP32), ha.make_params(b, m, 7, causal, n_min, 1))
    out, lse = ha.hyperattn_forward(tq, tk, tv, b, m, 7, workspace=ws, **kw)
    got = ha.hyperattn_backward(tq, tk, tv, out, lse, tg, b, m, 7, fwd_workspace=ws, **kw)
    again = ha.hyperattn_backward(tq, tk, tv, out, lse, tg, b, m, 7, fwd_workspace=ws, **kw)
    assert all(torch.equal(x, y) for x, y in zip(got, again))
    hd = H - 1
    one = [x[:, hd:hd + 1] for x in (Q, K, V, G)]
    ref = orc.hyperattn_backward(*one, b=b, m=m, r=7, **kw)
    bound = orc.hyperattn_backward(*one, b=b, m=m, r=7, absolute=True, **kw)
    for name, x, y, lim in zip(("dQ", "dK", "dV"), got, ref, bound):
        err = abs(to_host(x)[:, hd:hd + 1] - y)
        assert (err <= 2.0 ** -14 * lim + 2.0 ** -100).all(), (name, err.max())


@pytest.mark.parametrize("H,n,d,causal", [(32, 2079, 64, True), (32, 2079, 128, True), (16, 4100, 128, False)])
def test_exact_backward_fp32_forms(H, n, d, causal):
    import torch

    import paper_2310_05869_amd as ha
    print(f"fp32 exact backward forms H={H} n={n} d={d} causal={causal}", flush=True)
    Q, K, V = synth_inputs.iid_qkv(1, H, n, d, "fp32")
    G = synth_inputs.iid_qkv(1, H, n, d, "fp32", seed=5)[0]
    tq, tk, tv, tg = (to_device(x, "fp32") for x in (Q, K, V, G))
    out, lse = ha.exact_attn_forward(tq, tk, tv, causal=causal)
    got = ha.exact_attn_backward(tq, tk, tv, out, lse, tg, causal=causal)
    torch.cuda.synchronize()
    hd = H - 1
    one = [x[:, hd:hd + 1] for x in (Q, K, V, G)]
    okw = dict(b=1, m=0, r=1, causal=True, n_min=n) if causal else dict(b=n, m=0, r=1, causal=False)
    ref = orc.hyperattn_backward(*one, **okw)
    bound = orc.hyperattn_backward(*one, absolute=True, **okw)
    for name, x, y, lim in zip(("dQ", "dK", "dV"), got, ref, bound):
        err = abs(to_host(x)[:, hd:hd + 1] - y)
        # sums of up to 4100 terms, 2^-24 each
        assert (err <= 2.0 ** -12 * lim + 2.0 ** -100).all(), (name, err.max())


# passes that share launches: one to four levels, blocks and base blocks that no tile of 32 divides, no samples, more samples
# than a slab, several draws of a key; and a problem whose passes stay apart (one wave per group of rows)
@pytest.mark.parametrize("B,H,n,n_min,d,b,m", [(1, 2, 1024, 512, 64, 64, 64), (1, 1, 1600, 100, 64, 50, 33), (2, 1, 1040, 130, 128, 65, 0),
                                               (1, 3, 512, 256, 128, 32, 200), (1, 16, 4096, 2048, 64, 128, 128)])
def test_backward_fp32_shared_launches(B, H, n, n_min, d, b, m):
    import torch

    import paper_2310_05869_amd as ha
    print(f"fp32 shared launches B={B} H={H} n={n} n_min={n_min} d={d} b={b} m={m}", flush=True)
    Q, K, V = synth_inputs.iid_qkv(B, H, n, d, "fp32")
    G = synth_inputs.iid_qkv(B, H, n, d, "fp32", seed=5)[0]
    tq, tk, tv, tg = (to_device(x, "fp32") for x in (Q, K, V, G))
    ws = ha.alloc_workspace(ha.make_shape(B, H, n, d, ha.HA_FP32), ha.make_params(b, m, 7, True, n_min, 2))
    kw = dict(causal=True, n_min=n_min, seed=2)
    out, lse = ha.hyperattn_forward(tq, tk, tv, b, m, 7, workspace=ws, **kw)
    got = [torch.full_like(tq, float("nan")) for _ in range(3)]  # every row is written before it is added to
    ha.hyperattn_backward(tq, tk, tv, out, lse, tg, b, m, 7, fwd_workspace=ws, grads=tuple(got), **kw)
    again = ha.hyperattn_backward(tq, tk, tv, out, lse, tg, b, m, 7, fwd_workspace=ws, **kw)
    torch.cuda.synchronize()
    for x, y in zip(got, again):
        assert torch.equal(x, y)
    for bi, hd in sorted({(0, 0), (B - 1, H - 1)}):
        one = [x[bi:bi + 1, hd:hd + 1] for x in (Q, K, V, G)]
        okw = dict(b=b, m=m, r=7, causal=True, n_min=n_min, seed=2)
        ref = orc.hyperattn_backward(*one, **okw)
        bound = orc.hyperattn_backward(*one, absolute=True, **okw)
        for name, x, y, lim in zip(("dQ", "dK", "dV"), got, ref, bound):
            err = abs(to_host(x)[bi:bi + 1, hd:hd + 1] - y)
            # sums of up to some thousand terms, 2^-24 each
            assert (err <= 2.0 ** -12 * lim + 2.0 ** -100).all(), (name, err.max())


# eight ways: ragged last tiles, a way without a tile, more workgroups than CUs (11 x 33)
@pytest.mark.parametrize("H,n,d,causal", [(1, 2079, 64, True), (1, 2100, 64, False), (1, 513, 128, True), (2, 700, 128, False),
                                          (11, 1025, 128, True)])
def test_exact_fp32_eight_waves(H, n, d, causal):
    test_exact_attention_fp32_forms(H, n, d, causal)
    test_exact_backward_fp32_forms(H, n, d, causal)


def _frobenius(got, ref):
    return float(((got - ref) ** 2).sum() ** 0.5 / (ref ** 2).sum() ** 0.5)


@pytest.mark.parametrize("d,n,b,m,causal,n_min", [(64, 2048, 128, 128, 0, 4096), (128, 2048, 256, 256, 0, 4096)])
def test_log_row_sums_fp32_rounding(d, n, b, m, causal, n_min):
    """Log row sums near ln 2048 + 1/2 = 8.1: one rounding of the result is 2^-20 / sqrt(12) = 2.8e-7 at the root mean square,
    3.4e-8 of the value; sums and scores add to it.  Bound 4.2e-8, below what a logarithm of the result's own size adds (1.4e-7
    and the function's own error: 5e-8 in all)."""
    import paper_2310_05869_amd as ha
    print(f"fp32 log row sums d={d} n={n}", flush=True)
    cfg = dict(B=1, H=2, n=n, d=d, dtype="fp32", law="iid", b=b, m=m, r=7, causal=causal, n_min=n_min, seed=3)
    Q, K, V = synth_inputs.make_qkv(cfg, seed=9)
    _, lse = ha.hyperattn_forward(*(to_device(x, "fp32") for x in (Q, K, V)), b, m, 7, causal=bool(causal), n_min=n_min, seed=3)
    err = _frobenius(to_host(lse), run_oracle(Q, K, V, cfg)[1])
    print(f"  {err:.2e}", flush=True)
    assert err <= 4.2e-8


def test_query_gradients_fp32_rounding():
    """dQ of a causal problem against 64 bits, relative Frobenius.  dS = P (dP - delta): a chain of k fp32 products is off by
    about sqrt(k) times a rounding; bound 4.4e-7 between the two forms measured, dP as two chains of 64 (4.0e-7) and
    as one of 128 (4.8e-7)."""
    import paper_2310_05869_amd as ha
    d, n, b, m, n_min = 128, 1024, 128, 64, 256
    print("fp32 dQ rounding", flush=True)
    cfg = dict(B=1, H=2, n=n, d=d, dtype="fp32", law="iid", b=b, m=m, r=7, causal=1, n_min=n_min, seed=3)
    Q, K, V = synth_inputs.make_qkv(cfg, seed=9)
    G = synth_inputs.iid_qkv(1, 2, n, d, "fp32", seed=5)[0]
    t = [to_device(x, "fp32") for x in (Q, K, V, G)]
    kw = dict(causal=True, n_min=n_min, seed=3)
    ws = ha.alloc_workspace(ha.make_shape(1, 2, n, d, ha.HA_FP32), ha.make_params(b, m, 7, 1, n_min, 3))
    out, lse = ha.hyperattn_forward(*t[:3], b, m, 7, workspace=ws, **kw)
    dQ = ha.hyperattn_backward(*t[:3], out, lse, t[3], b, m, 7, fwd_workspace=ws, **kw)[0]
    err = _frobenius(to_host(dQ), orc.hyperattn_backward(Q, K, V, G, b=b, m=m, r=7, **kw)[0])
    print(f"  {err:.2e}", flush=True)
    assert err <= 4.4e-7


@pytest.mark.parametrize("d", [64, 128])
def test_stages_past_four_gib(d):
    """Block and sampled stage of one fp32 head whose tensors pass 4 GiB, the reach of a 32-bit byte offset: blocks at the
    start, beyond 2 GiB and at the end against fp64 attention, 2^-14 of the values' magnitude (sums of 64 terms)."""
    import torch

    import paper_2310_05869_amd as ha
    n = (1 << 30) // d + 128  # a multiple of 64
    print(f"fp32 stages n={n} d={d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    rows = torch.randn((n + 192, d), generator=gen, device="cuda") * d ** -0.25
    q, k, v = (rows[at:at + n].view(1, n, d) for at in (0, 64, 192))
    samples = torch.tensor([0, 1, n // 2, n // 2 + 1, n - 2, n - 1, n // 3, 5], dtype=torch.int32, device="cuda")
    for stage in ("block", "sampled"):
        if stage == "block":
            out, lse = ha.ha_block_attn(q, k, v, 64)
        else:
            out, lse = ha.ha_sampled_attn(q, k, v, samples, torch.arange(n, dtype=torch.int32, device="cuda").view(1, n), 64)
        for at in (0, n // 2 // 64 * 64 + 64, n // 64 * 64 - 128, n - 64):
            mine = slice(at, at + 64)
            keys = torch.arange(at, at + 64, device="cuda") if stage == "block" else samples[samples // 64 != at // 64].long()
            s = q[0, mine].double() @ k[0, keys].double().T.contiguous()
            if stage == "sampled":
                s = s + torch.log(torch.tensor(n / samples.numel(), dtype=torch.float64))
            ref = s.softmax(-1) @ v[0, keys].double()
            bound = s.softmax(-1) @ v[0, keys].double().abs()
            assert ((out[0, mine] - ref).abs() <= 2.0 ** -14 * bound).all(), (stage, at)
            assert torch.allclose(lse[0, mine].double(), s.logsumexp(-1), atol=2e-5), (stage, at)
        del out, lse


def test_more_workgroups_than_one_launch_holds():
    """2^24 + 64 blocks of one row: a launch of 256 threads each would count past 32 bits.  A softmax over one key is 1, so
    every row's result is its value row, bit for bit."""
    import torch

    import paper_2310_05869_amd as ha
    groups, n, d = 4, (1 << 22) + 16, 64
    print(f"fp32 block stage, {groups * n} workgroups", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    v = torch.randn((groups, n, d), generator=gen, device="cuda")
    q = 0.1 * v
    out, lse = ha.ha_block_attn(q, q, v, 1)
    assert torch.equal(out, v)
    assert torch.allclose(lse, (q.double() ** 2).sum(-1).float(), atol=1e-5, rtol=1e-5)
