"""GPU parity of the Algorithm 2 / Lemma 2 options (hyperattn_forward_alg2) against the
oracle's dense evaluation: the rows of T bit-exact; the rows drawn by squared value norm
(Lemma 2, inverse of the cumulative law in fp64 on both sides) equal except where the
oracle's uniform lies within 1e-9 of a boundary of that law (counted, and replayed in the
oracle like a projection too close to zero); log tau and log d~ within fp32 accuracy, outputs
within the forward's tolerance (bf16: 2e-3 + half an ulp; fp32: 1e-5 + 1e-5 |ref|).  Where
fewer than 16 sampled rows carry a row's whole value product (Lemma 2 with a small m) the
rounding of the weights to bf16 as matrix-core operands does not average out and an element
may also use 2^-8 sum_j w_j |v_j| (the oracle run on |V| with the draws of V); the share of
the elements that need it is printed and must stay below 0.5 %."""
import numpy as np
import pytest

import synth_inputs
from oracle import hyperattn_oracle as orc
from ha_testutil import LSE_TOL, assert_close, have_gpu, out_tolerance, to_device, to_host

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def ha():
    import paper_2310_05869_amd as mod
    mod.lib()
    return mod


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


CASES = [  # dtype, d, n, b, m, r, cap_scale, kappa, vnorm
    ("bf16", 64, 512, 64, 48, 5, 0.0, 0.0, False),      # no caps: the Section 4 estimator
    ("bf16", 64, 512, 64, 48, 5, 8.0, 1.2, False),      # both caps bind on part of the rows (12 % / 65 %)
    ("bf16", 128, 768, 96, 100, 6, 1e-4, 2.0, False),   # cap below every entry
    ("bf16", 128, 768, 96, 100, 6, 4.0, 1.1, True),     # Lemma 2's value product, caps binding (27 % / 86 %)
    ("fp32", 64, 384, 32, 20, 4, 25.0, 1.5, True),
    ("fp32", 64, 384, 32, 20, 4, 0.0, 0.0, True),
    ("bf16", 64, 600, 200, 7, 7, 10.0, 0.0, True),      # block not a multiple of the row tile, cap without lower cap
    ("bf16", 128, 2048, 256, 256, 7, 8.0, 1.2, False),  # the benchmark's b and m: two query tiles per block, four key tiles per segment
    ("bf16", 128, 2048, 256, 256, 7, 4.0, 1.1, True),
    ("bf16", 64, 1536, 512, 300, 6, 6.0, 1.3, True),    # four query tiles per block, five ragged sample tiles
    ("bf16", 64, 1000, 8, 130, 3, 5.0, 1.5, False),     # tiny blocks, tau rows over ragged key tiles
]


@pytest.mark.parametrize("dtype,d,n,b,m,r,cap_scale,kappa,vnorm", CASES)
def test_alg2_options_match_the_oracle(ha, torch, dtype, d, n, b, m, r, cap_scale, kappa, vnorm):
    print(f"alg2 {dtype} d={d} n={n} b={b} m={m} r={r} cap={cap_scale} kappa={kappa} vnorm={vnorm}", flush=True)
    cfg = dict(B=1, H=2, n=n, d=d, dtype=dtype, law="iid")
    Q, K, V = synth_inputs.make_qkv(cfg, seed=11 + n)
    rng = np.random.default_rng(n)
    V = V * rng.uniform(0.2, 2.0, size=(1, 2, n, 1)).astype(np.float32)       # unequal value-row norms
    V = synth_inputs.round_to_bf16(V) if dtype == "bf16" else V.astype(np.float32)
    seed = 5
    tq, tk, tv = (to_device(x, dtype) for x in (Q, K, V))
    out, lse, ws = ha.hyperattn_forward_alg2(tq, tk, tv, b, m, r, seed=seed, cap_scale=cap_scale, kappa=kappa,
                                             vnorm_sampling=vnorm)
    torch.cuda.synchronize()
    shape = ha.make_shape(1, 2, n, d, ha.HA_BF16 if dtype == "bf16" else ha.HA_FP32)
    params = ha.make_params(b, m, r, False, 4096, seed)
    views = ha.alg2_workspace_views(ws, shape, params)
    replay = {}
    if vnorm:
        for bh in range(2):
            w = (V[0, bh].astype(np.float64) ** 2).sum(axis=1)
            np.testing.assert_allclose(views["vnorm_w"][bh].cpu().numpy(), w, rtol=1e-13)
            marg = []
            idx, logw = orc.vnorm_samples(V[0, bh], seed, bh, m, margin=marg)
            got = views["vnorm_samples"][bh, 0].cpu().numpy()
            for r_ in np.nonzero(got != idx)[0]:
                assert marg[r_] < 1e-9 and abs(int(got[r_]) - int(idx[r_])) == 1, (bh, r_, got[r_], idx[r_], marg[r_])
                replay.setdefault(bh, {})[int(r_)] = int(got[r_])
            idx, logw = orc.vnorm_samples(V[0, bh], seed, bh, m, replay=replay.get(bh))
            np.testing.assert_allclose(views["vnorm_logw"][bh, 0].cpu().numpy(), logw, rtol=1e-6, atol=1e-6)
        print(f"  Lemma 2 draws within rounding of a boundary (replayed): {sum(len(v) for v in replay.values())}", flush=True)
    ref_out, ref_lse, ref_tau = orc.hyperattn_forward_alg2(Q, K, V, b=b, m=m, r=r, seed=seed, cap_scale=cap_scale,
                                                           kappa=kappa, vnorm_sampling=vnorm, vnorm_replay=replay)
    if cap_scale > 0 or kappa > 0:   # the options must actually act in this instance, or the case tests nothing
        plain = orc.hyperattn_forward_alg2(Q, K, V, b=b, m=m, r=r, seed=seed)[1]
        changed = np.abs(plain - ref_lse) > 1e-9
        print(f"  caps change log d~ on {changed.mean():.0%} of the rows", flush=True)
        assert changed.any()
    np.testing.assert_array_equal(views["tau_rows"][0].cpu().numpy(), orc.tau_rows(seed, n, m))
    np.testing.assert_allclose(views["log_tau"][:, 0].cpu().numpy(), ref_tau, rtol=2e-5, atol=2e-5)
    np.testing.assert_allclose(to_host(lse), ref_lse, rtol=3e-5, atol=3e-5)
    absv = None
    if dtype == "bf16" and 0 < m < 16:   # squared row norms, hence the draws, are those of V
        absv = orc.hyperattn_forward_alg2(Q, K, np.abs(V), b=b, m=m, r=r, seed=seed, cap_scale=cap_scale, kappa=kappa,
                                          vnorm_sampling=vnorm, vnorm_from=V, vnorm_replay=replay)[0]
    assert_close(to_host(out), ref_out, dtype, "out", absv, 0.005)


CAUSAL_CASES = [  # dtype, d, n, n_min, b, m, r, cap_scale, kappa, vnorm
    ("bf16", 128, 2048, 256, 128, 64, 6, 6.0, 1.3, False),     # three levels, 1 + 2 + 4 nodes
    ("bf16", 128, 2048, 256, 128, 64, 6, 5.0, 1.2, True),
    ("bf16", 64, 1024, 128, 32, 40, 5, 8.0, 1.5, True),        # nodes of 512, 256, 128 rows; ragged sample tiles
    ("fp32", 64, 512, 64, 32, 20, 4, 10.0, 1.5, True),
    ("fp32", 64, 512, 64, 32, 20, 4, 0.0, 0.0, False),         # no caps: the Section 4 causal forward
    ("bf16", 64, 4096, 1024, 256, 256, 7, 8.0, 1.2, False),    # the benchmark's b and m, two levels
]


@pytest.mark.parametrize("dtype,d,n,n_min,b,m,r,cap_scale,kappa,vnorm", CAUSAL_CASES)
def test_alg2_options_on_causal_problems(ha, torch, dtype, d, n, n_min, b, m, r, cap_scale, kappa, vnorm):
    """Algorithm 4 with Algorithm 2 as printed at every off-diagonal node: every node's rows of T bit-exact,
    log tau of every node, Lemma 2's draws per node (replayed where a uniform sits within rounding of a
    boundary), then log D~ and the outputs."""
    print(f"alg2 causal {dtype} d={d} n={n} n_min={n_min} b={b} m={m} r={r} cap={cap_scale} kappa={kappa} vnorm={vnorm}", flush=True)
    H = 2
    cfg = dict(B=1, H=H, n=n, d=d, dtype=dtype, law="iid")
    Q, K, V = synth_inputs.make_qkv(cfg, seed=23 + n)
    rng = np.random.default_rng(n + 1)
    V = V * rng.uniform(0.1, 1.0, size=(1, H, n, 1)).astype(np.float32)          # unequal value-row norms
    V = synth_inputs.round_to_bf16(V) if dtype == "bf16" else V.astype(np.float32)
    seed = 8
    tq, tk, tv = (to_device(x, dtype) for x in (Q, K, V))
    out, lse, ws = ha.hyperattn_forward_alg2(tq, tk, tv, b, m, r, seed=seed, cap_scale=cap_scale, kappa=kappa,
                                             vnorm_sampling=vnorm, causal=True, n_min=n_min)
    torch.cuda.synchronize()
    shape = ha.make_shape(1, H, n, d, ha.HA_BF16 if dtype == "bf16" else ha.HA_FP32)
    params = ha.make_params(b, m, r, True, n_min, seed)
    views = ha.alg2_workspace_views(ws, shape, params)
    levels = int(np.log2(n // n_min))
    replay = {}
    for level in range(levels):
        s_rows = n >> (level + 1)
        for node in range(1 << level):
            heap = (1 << level) - 1 + node
            np.testing.assert_array_equal(views["tau_rows"][heap].cpu().numpy(), orc.tau_rows(seed, s_rows, m, heap))
            if vnorm:
                for bh in range(H):
                    k0 = 2 * node * s_rows
                    marg = []
                    idx, _ = orc.vnorm_samples(V[0, bh, k0:k0 + s_rows], seed, bh, m, margin=marg, heap=heap, n_heads=H)
                    got = views["vnorm_samples"][bh, heap].cpu().numpy()
                    for r_ in np.nonzero(got != idx)[0]:
                        assert marg[r_] < 1e-9 and abs(int(got[r_]) - int(idx[r_])) == 1, (bh, heap, r_, marg[r_])
                        replay.setdefault((bh, heap), {})[int(r_)] = int(got[r_])
                    _, logw = orc.vnorm_samples(V[0, bh, k0:k0 + s_rows], seed, bh, m, replay=replay.get((bh, heap)),
                                                heap=heap, n_heads=H)
                    np.testing.assert_allclose(views["vnorm_logw"][bh, heap].cpu().numpy(), logw, rtol=1e-6, atol=1e-6)
    okw = dict(b=b, m=m, r=r, seed=seed, cap_scale=cap_scale, kappa=kappa, vnorm_sampling=vnorm, causal=True,
               n_min=n_min, vnorm_replay=replay)
    ref_out, ref_lse, ref_tau = orc.hyperattn_forward_alg2(Q, K, V, **okw)
    if cap_scale > 0 or kappa > 0:
        plain = orc.hyperattn_forward_alg2(Q, K, V, b=b, m=m, r=r, seed=seed, causal=True, n_min=n_min)[1]
        changed = np.abs(plain - ref_lse) > 1e-9
        print(f"  caps change log D~ on {changed.mean():.0%} of the rows; replayed draws {sum(len(v) for v in replay.values())}",
              flush=True)
        assert changed.any()
    np.testing.assert_allclose(views["log_tau"].cpu().numpy(), ref_tau, rtol=3e-5, atol=3e-5)
    np.testing.assert_allclose(to_host(lse), ref_lse, rtol=3e-5, atol=5e-5)
    absv = None
    if dtype == "bf16" and 0 < m < 16:
        absv = orc.hyperattn_forward_alg2(Q, K, np.abs(V), vnorm_from=V, **okw)[0]
    assert_close(to_host(out), ref_out, dtype, "out", absv, 0.005)


def test_alg2_rejects_bad_arguments(ha, torch):
    print("alg2 errors", flush=True)
    shape = ha.make_shape(1, 1, 256, 64, ha.HA_BF16)
    with pytest.raises(ha.HyperAttnError):          # causal: n / n_min must be a power of two
        ha.ha_alg2_workspace_layout(shape, ha.make_params(64, 16, 7, True, 96, 0))
    q = torch.zeros((1, 1, 256, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ha.HyperAttnError):
        ha.hyperattn_forward_alg2(q, q, q, 64, 16, 7, workspace=torch.zeros(256, dtype=torch.uint8, device="cuda"))
    # a causal problem at or below n_min is plain exact causal attention
    out, lse, _ = ha.hyperattn_forward_alg2(q, q, q, 64, 16, 7, causal=True, n_min=256, cap_scale=2.0, kappa=1.5)
    ref, _ = ha.exact_attn_forward(q, q, q, causal=True)
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("dtype,d,n,b,m,r,cap_scale,kappa,vnorm", [
    ("bf16", 64, 300, 100, 130, 4, 6.0, 1.3, False),    # a block's last tile padded after a full one
    ("bf16", 128, 256, 256, 40, 5, 0.0, 0.0, False),    # one block: no sample is kept, every row of T sums nothing
    ("bf16", 64, 48, 16, 33, 3, 5.0, 1.2, False),       # one key tile, seven of eight ranges empty
    ("bf16", 128, 2080, 65, 300, 6, 6.0, 1.4, False),   # ranges of four and five tiles, the last ragged; blocks across tiles
    ("bf16", 64, 2080, 65, 257, 6, 0.0, 1.4, False)])   # lower cap alone, three row tiles, the last of one row
def test_alg2_caps_in_the_node_kernel(ha, torch, dtype, d, n, b, m, r, cap_scale, kappa, vnorm):
    """The forward kernel's cap mode and the sorted walk of the rows of T at the edges of their tiles: criteria as above."""
    test_alg2_options_match_the_oracle(ha, torch, dtype, d, n, b, m, r, cap_scale, kappa, vnorm)


@pytest.mark.parametrize("vnorm", [False, True])
@pytest.mark.parametrize("d,H,n,b,m,r,cap_scale,kappa", [
    (64, 2, 300, 100, 130, 4, 6.0, 1.3),     # four ways; padded tail of a block, samples from its next tile on
    (128, 2, 256, 256, 40, 5, 0.0, 0.0),     # one block: no sample is kept, every row of T sums nothing
    (64, 2, 48, 16, 33, 3, 5.0, 1.2),        # ways without a tile of the block; seven of eight key ranges empty
    (128, 2, 2080, 65, 300, 6, 6.0, 1.4),    # ragged ranges, blocks across tiles
    (64, 2, 650, 65, 0, 4, 0.0, 0.0),        # no samples at all
    (128, 40, 896, 64, 77, 5, 6.0, 1.3),     # four ways, blocks of two row tiles
    (64, 80, 896, 128, 31, 5, 6.0, 1.3),     # one way
    (128, 80, 700, 100, 0, 5, 0.0, 0.0),     # four, no samples
    (64, 80, 700, 100, 65, 5, 0.0, 1.4),     # one; lower cap alone
    (64, 24, 704, 64, 96, 5, 6.0, 1.3),      # two ways: 5 tiles of keys, the second way's turn at the samples without one
    (64, 24, 704, 64, 40, 5, 6.0, 1.3),      # 4 tiles
    (64, 24, 704, 64, 20, 5, 0.0, 1.4),      # 3: the second way comes to the samples behind its loop
    (128, 35, 896, 128, 70, 5, 6.0, 1.3),    # one way
    (128, 70, 700, 100, 31, 5, 0.0, 1.4)])   # one, blocks that its rows do not fill
def test_alg2_fp32_caps_in_the_node_kernel(ha, torch, d, H, n, b, m, r, cap_scale, kappa, vnorm):
    """The fp32 forward kernel's cap and value modes and the sums of the rows of T at the edges of their tiles and for each number of
    ways (test_fp32_forms_of_the_gpu_tests); two heads (all share the draws, but the first two Lemma 2's of such a call) against the oracle:
    criteria as above."""
    print(f"alg2 fp32 d={d} H={H} n={n} b={b} m={m} r={r} cap={cap_scale} kappa={kappa} vnorm={vnorm}", flush=True)
    Q, K, V = (x.astype(np.float32) for x in synth_inputs.make_qkv(dict(B=1, H=H, n=n, d=d, dtype="fp32", law="iid"), seed=n))
    out, lse, ws = ha.hyperattn_forward_alg2(*(to_device(x, "fp32") for x in (Q, K, V)), b, m, r, seed=5, cap_scale=cap_scale,
                                             kappa=kappa, vnorm_sampling=vnorm)
    torch.cuda.synchronize()
    views = ha.alg2_workspace_views(ws, ha.make_shape(1, H, n, d, ha.HA_FP32), ha.make_params(b, m, r, False, 4096, 5))
    ends = [0, 1 if vnorm else H - 1]
    ref_out, ref_lse, ref_tau = orc.hyperattn_forward_alg2(Q[:, ends], K[:, ends], V[:, ends], b=b, m=m, r=r, seed=5,
                                                           cap_scale=cap_scale, kappa=kappa, vnorm_sampling=vnorm)
    np.testing.assert_allclose(views["log_tau"][ends, 0].cpu().numpy(), ref_tau, rtol=2e-5, atol=2e-5)
    np.testing.assert_allclose(to_host(lse)[:, ends], ref_lse, rtol=3e-5, atol=3e-5)
    assert_close(to_host(out)[:, ends], ref_out, "fp32", "out")


def test_alg2_more_workgroups_than_one_launch_holds(ha, torch):
    """All levels' nodes together are 20 M workgroups of 256 threads, each level's own 4 M: more than a launch counts.  Heads
    are independent and share the draws, so halves of the heads give the same bits."""
    H, n, n_min = 8, 1 << 20, 1 << 15
    print(f"alg2 {H * (n // 2) * 5} workgroups", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    q, k, v = ((torch.randn((1, H, n, 64), generator=gen, device="cuda") / 8 ** 0.5).to(torch.bfloat16) for _ in range(3))
    kw = dict(causal=True, n_min=n_min, seed=2)
    out, lse, _ = ha.hyperattn_forward_alg2(q, k, v, 1, 0, 7, **kw)
    for half in (slice(0, H // 2), slice(H // 2, H)):
        o, l, _ = ha.hyperattn_forward_alg2(*(x[:, half].contiguous() for x in (q, k, v)), 1, 0, 7, **kw)
        assert torch.equal(out[:, half], o) and torch.equal(lse[:, half], l)


def test_alg2_more_heads_than_one_launch_holds(ha, torch):
    """2^20 heads, the most that a call takes: 2^23 workgroups of 512 threads sum the rows of T.  Halves of the heads give
    the same bits."""
    H, n = 1 << 20, 16
    print(f"alg2 {H} heads", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    q, k, v = ((torch.randn((1, H, n, 64), generator=gen, device="cuda") / 8 ** 0.5).to(torch.bfloat16) for _ in range(3))
    kw = dict(seed=2, cap_scale=4.0, kappa=1.2)
    out, lse, _ = ha.hyperattn_forward_alg2(q, k, v, 8, 4, 3, **kw)
    for half in (slice(0, H // 2), slice(H // 2, H)):
        o, l, _ = ha.hyperattn_forward_alg2(*(x[:, half].contiguous() for x in (q, k, v)), 8, 4, 3, **kw)
        assert torch.equal(out[:, half], o) and torch.equal(lse[:, half], l)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("cap_scale,kappa", [(8.0, 0.0), (0.0, 0.0), (8.0, 1.3)])
@pytest.mark.parametrize("vnorm", [False, True])
@pytest.mark.parametrize("d,H,n,b,m,r,n_min", [
    (64, 1, 2048, 64, 64, 7, 0),
    (128, 1, 2048, 128, 128, 7, 0),
    (64, 1, 4096, 256, 256, 7, 0),
    (128, 40, 896, 64, 77, 5, 0),
    (64, 80, 896, 128, 31, 5, 0),      # fp32: one way
    (64, 24, 704, 64, 96, 5, 0),       # fp32: two
    (128, 35, 896, 128, 70, 5, 0),     # fp32: one
    (64, 1, 2048, 64, 64, 7, 512),     # causal, two levels
    (128, 1, 2048, 64, 64, 7, 256),
    (64, 1, 1024, 2, 5, 5, 2)])        # nine levels, folded one by one
def test_alg2_scores_far_apart(ha, torch, d, H, n, b, m, r, n_min, vnorm, cap_scale, kappa, dtype):
    """Clustered inputs, whose sampled or drawn keys can exceed all of a row's block by hundreds: the masked sum, the capped sum of
    the samples and the output's weights have scales of their own.  log d~ of every row within the rounding of the scores: a score is
    a sum of d products, its error at most (d + 2) 2^-24 sum_c |q_c k_c| <= e (the row's largest), and log d~ moves by no more than twice that
    (through the cap and by itself) plus LSE_TOL of its own value.  Outputs where the row's weights fit fp32 (sum_j w_j |v_j| <
    1e30), within the weights' relative error exp(4 e) - 1 (score and log d~), 2^-8 for bf16 operands (2^-9 each for the weights
    and, causal, for the partial rows)."""
    print(f"alg2 clustered {dtype} d={d} H={H} n={n} b={b} m={m} r={r} n_min={n_min} cap={cap_scale} kappa={kappa} vnorm={vnorm}", flush=True)
    causal = n_min > 0
    Q, K, V = synth_inputs.make_qkv(dict(B=1, H=H, n=n, d=d, dtype=dtype, law="mixture"), seed=n + d)
    kw = dict(seed=5, cap_scale=cap_scale, kappa=kappa, vnorm_sampling=vnorm, causal=causal, n_min=n_min or 4096)
    out, lse, ws = ha.hyperattn_forward_alg2(*(to_device(x, dtype) for x in (Q, K, V)), b, m, r, **kw)
    torch.cuda.synchronize()
    views = ha.alg2_workspace_views(ws, ha.make_shape(1, H, n, d, ha.HA_BF16 if dtype == "bf16" else ha.HA_FP32),
                                    ha.make_params(b, m, r, causal, n_min or 4096, 5))
    ends = sorted({0, 1 if vnorm else H - 1} & set(range(H)))
    replay = {}
    if vnorm:
        for bh in ends:
            for heap in range(views["vnorm_samples"].shape[1]):
                level = (heap + 1).bit_length() - 1
                s = n >> (level + 1) if causal else n
                k0 = 2 * (heap + 1 - (1 << level)) * s
                marg = []
                idx, _ = orc.vnorm_samples(V[0, bh, k0:k0 + s], 5, bh, m, margin=marg, heap=heap, n_heads=H)
                got = views["vnorm_samples"][bh, heap].cpu().numpy()
                for j in np.nonzero(got != idx)[0]:
                    assert marg[j] < 1e-9 and abs(int(got[j]) - int(idx[j])) == 1, (bh, heap, j, marg[j])
                    replay.setdefault((bh, heap), {})[int(j)] = int(got[j])
    Qe, Ke, Ve = (x[:, ends] for x in (Q, K, V))
    okw = dict(b=b, m=m, r=r, vnorm_replay=replay, **kw)
    with np.errstate(over="ignore", invalid="ignore"):
        ref_out, ref_lse, _ = orc.hyperattn_forward_alg2(Qe, Ke, Ve, **okw)
        absv = orc.hyperattn_forward_alg2(Qe, Ke, np.abs(Ve), vnorm_from=Ve, **okw)[0]
    heavy = np.nan_to_num(absv, nan=np.inf).max(axis=-1)
    far = heavy > 1e45     # a weight beyond e^104 of the row's sum
    print(f"  rows whose weights exceed their sum by more than e^104: {int(far.sum())}", flush=True)
    if not causal and kappa == 0 and cap_scale > 0 and n >= 2048:
        assert far.any()
    e = (d + 2) * 2.0 ** -24 * (np.abs(Qe) @ np.abs(Ke).swapaxes(-1, -2)).max(axis=-1)
    got = to_host(lse)[:, ends]
    err = np.abs(got - ref_lse) - (2 * e + LSE_TOL[dtype] * np.maximum(1.0, np.abs(ref_lse)))
    assert np.isfinite(got).all() and (err <= 0).all(), (f"log d~: {int((~np.isfinite(got)).sum())} rows not finite, "
                                                         f"{int((err > 0).sum())} of {err.size} out of tolerance")
    fits = heavy < 1e30
    o = to_host(out)[:, ends][fits]
    tol = (np.expm1(4 * e[fits])[:, None] + (2.0 ** -8 if dtype == "bf16" else 0.0)) * absv[fits] + out_tolerance(ref_out[fits], dtype)
    bad = ~(np.abs(o - ref_out[fits]) <= tol)
    assert not bad.any(), f"out: {int(bad.any(axis=-1).sum())} of {len(bad)} rows out of tolerance, {int((~np.isfinite(o)).any(axis=-1).sum())} not finite"


@pytest.mark.parametrize("d,n,b,m", [(128, 35072, 256, 256),   # lists of more than four chunks per range, blocks of whole tiles
                                     (64, 35000, 100, 130),    # ranges of 68 and 69 tiles, blocks that cut tiles
                                     (128, 35200, 1600, 33), (64, 1088, 64, 40)])
@pytest.mark.parametrize("spread", [0.0, 1.5])
def test_alg2_row_sums_over_long_ranges(ha, torch, d, n, b, m, spread):
    """tau against 64-bit sums over the keys outside of the row's sorted block.  spread > 0: keys of very different lengths, so that the
    exponentials' reference moves many times (scores to 40, each a sum whose rounding is within 2e-5 of that)."""
    print(f"alg2 tau d={d} n={n} b={b} m={m} spread={spread}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + d)
    q, k, v = (torch.randn((1, 2, n, d), generator=gen, device="cuda") * d ** -0.25 for _ in range(3))
    k = k * torch.exp(spread * torch.randn((1, 2, n, 1), generator=gen, device="cuda")).clamp(max=12.0)
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    _, _, ws = ha.hyperattn_forward_alg2(q, k, v, b, m, 7, seed=3, cap_scale=4.0, kappa=1.2)
    views = ha.alg2_workspace_views(ws, ha.make_shape(1, 2, n, d, ha.HA_BF16), ha.make_params(b, m, 7, False, 4096, 3))
    base = ha.workspace_views(ws, ha.make_shape(1, 2, n, d, ha.HA_BF16), ha.make_params(b, m, 7, False, 4096, 3))
    rows = views["tau_rows"].reshape(-1)[:m].long()
    for h in range(2):
        blk_q, blk_k = torch.empty(n, dtype=torch.long, device="cuda"), torch.empty(n, dtype=torch.long, device="cuda")
        at = torch.arange(n, device="cuda") // b
        blk_q[base["perm_q"].reshape(2, n)[h].long()] = at
        blk_k[base["perm_k"].reshape(2, n)[h].long()] = at
        s = torch.matmul(q[0, h, rows].double(), k[0, h].double().t().contiguous())
        s = s.masked_fill(blk_q[rows][:, None] == blk_k[None, :], float("-inf"))
        want = torch.logsumexp(s, -1).max().item()
        got = views["log_tau"].reshape(2, -1)[h, 0].item()
        assert abs(got - want) <= 2e-5 * (1.0 + abs(want)), (h, got, want)
