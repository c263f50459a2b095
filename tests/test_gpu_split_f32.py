"""fp32 attention on operands split in three bf16 parts: every form of the kernels at lengths that no tile divides, against
64-bit attention; infinities; powers of two, which change no bit of a product."""
import pytest

from ha_testutil import have_gpu
from test_gpu_backward import _run_case

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


def _inputs(torch, H, n, d, seed, count=4):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [torch.randn((1, H, n, d), generator=gen, device="cuda") * d ** -0.25 for _ in range(count)]


def _reference(torch, q, k, v, g, causal):
    """Output, log row sums and gradients of one head in 64 bits."""
    q, k, v = (x.double().detach().requires_grad_(True) for x in (q, k, v))
    s = torch.matmul(q, k.transpose(-1, -2).contiguous())
    if causal:
        s = s.masked_fill(torch.ones(s.shape[-2:], dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    lse = torch.logsumexp(s, -1)
    out = torch.matmul(torch.exp(s - lse[..., None]), v)
    out.backward(g.double())
    return out.detach(), lse.detach(), q.grad, k.grad, v.grad


@pytest.mark.parametrize("d,H,n,causal", [
    (64, 13, 4013, False),   # one way; a last tile of 13 keys, a last workgroup of 45 rows
    (64, 70, 2007, True),
    (64, 9, 3700, False),    # two ways, the second without a last tile
    (64, 33, 2031, True),
    (64, 20, 1001, True),    # four ways
    (64, 3, 1003, True),     # eight
    (64, 1, 33, False),
    (128, 8, 4013, False),   # one way
    (128, 66, 2007, True),
    (128, 9, 3001, True),    # four
    (128, 2, 777, False),    # eight (backward: four)
])
def test_exact_forms(ha, torch, d, H, n, causal):
    """Outputs within the fp32 criterion 1e-5 + 1e-5 |ref|; gradients: 2-norm of the error at most 1e-6 of the gradient's (sums of up to n
    terms in fp32, 2^-24 each with random signs, measured 3e-7 to 7e-7)."""
    print(f"split fp32 d={d} H={H} n={n} causal={causal}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, n + d)
    out, lse = ha.exact_attn_forward(q, k, v, causal=causal)
    grads = ha.exact_attn_backward(q, k, v, out, lse, g, causal=causal)
    for h in {0, H - 1}:
        ref = _reference(torch, *(x[:, h:h + 1] for x in (q, k, v, g)), causal)
        assert ((out[:, h:h + 1].double() - ref[0]).abs() <= 1e-5 + 1e-5 * ref[0].abs()).all()
        assert ((lse[:, h:h + 1].double() - ref[1]).abs() <= 2e-5).all()
        for got, want in zip(grads, ref[2:]):
            assert (got[:, h:h + 1].double() - want).norm() <= 1e-6 * want.norm()


@pytest.mark.parametrize("d,H,n", [(64, 13, 4000), (64, 2, 700), (128, 8, 4096), (128, 2, 700)])
def test_infinite_values(ha, torch, d, H, n):
    """A value row of +inf makes the outputs of every row that sees it +inf, as a sum of products in fp32 does; a key whose score is -inf has
    no weight."""
    print(f"split fp32 inf d={d} H={H} n={n}", flush=True)
    q, k, v = _inputs(torch, H, n, d, d, 3)
    v[:, :, 5, 3] = float("inf")
    out, _ = ha.exact_attn_forward(q, k, v)
    assert torch.isposinf(out[..., 3]).all()
    assert torch.isfinite(out[..., :3]).all() and torch.isfinite(out[..., 4:]).all()
    v[:, :, 5, 3] = 0.0
    q[..., 7] = q[..., 7].abs() + 0.1
    k[:, :, 9, 7] = float("-inf")
    out, lse = ha.exact_attn_forward(q, k, v)
    others = [i for i in range(n) if i != 9]
    s = torch.matmul(q[:, :1].double(), k[:, :1, others].double().transpose(-1, -2).contiguous())
    want = torch.matmul(torch.softmax(s, -1), v[:, :1, others].double())
    assert ((out[:, :1].double() - want).abs() <= 1e-5 + 1e-5 * want.abs()).all()
    assert torch.isfinite(lse).all()


@pytest.mark.parametrize("d,H,n,causal", [(64, 13, 4000, False), (64, 2, 700, True), (128, 8, 4096, False), (128, 2, 700, True)])
def test_powers_of_two_change_no_bit(ha, torch, d, H, n, causal):
    print(f"split fp32 scales d={d} H={H} n={n}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, 2 * n)
    a, b = 2.0 ** 30, 2.0 ** -50
    out, lse = ha.exact_attn_forward(q, k, v, causal=causal)
    out2, lse2 = ha.exact_attn_forward(q * a, k / a, v * b, causal=causal)
    assert torch.equal(lse, lse2) and torch.equal(out * b, out2)
    grads = ha.exact_attn_backward(q, k, v, out, lse, g, causal=causal)
    grads2 = ha.exact_attn_backward(q * a, k / a, v * b, out2, lse2, g, causal=causal)
    for x, y, scale in zip(grads, grads2, (b / a, b * a, 1.0)):
        assert torch.equal(x * scale, y)


@pytest.mark.parametrize("d,n,b,m,causal,n_min", [(128, 256, 32, 4096, 0, 4096), (64, 256, 32, 4096, 0, 4096), (128, 256, 32, 4096, 1, 64),
                                                  (128, 8192, 4096, 4096, 0, 4096), (64, 8192, 4096, 4096, 1, 4096)])
def test_most_sampled_keys(ha, torch, d, n, b, m, causal, n_min):
    """The longest lists that a pass keeps in LDS beside its tiles (the oracle's bounds, as in the backward's other tests)."""
    print(f"split fp32 lists d={d} n={n} b={b} m={m} causal={causal}", flush=True)
    cfg = dict(B=1, H=1, n=n, d=d, dtype="fp32", law="iid", b=b, m=m, r=7, causal=causal, n_min=n_min, seed=3)
    _run_case(ha, torch, cfg)


@pytest.mark.parametrize("d,H,n", [(64, 13, 2000), (64, 2, 700), (128, 2, 700)])
def test_values_of_2_to_the_minus_100(ha, torch, d, H, n):
    """Their lowest parts are still normal numbers: the 2-norm bounds of test_exact_forms."""
    print(f"split fp32 small values d={d} H={H} n={n}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, d + n)
    v = v * 2.0 ** -100
    out, lse = ha.exact_attn_forward(q, k, v)
    dq = ha.exact_attn_backward(q, k, v, out, lse, g)[0]
    ref = _reference(torch, *(x[:, :1] for x in (q, k, v, g)), False)
    assert (out[:, :1].double() - ref[0]).norm() <= 1e-6 * ref[0].norm()
    assert (dq[:, :1].double() - ref[2]).norm() <= 1e-6 * ref[2].norm()


@pytest.mark.parametrize("exponent", [-101, -110, -118, -124])
@pytest.mark.parametrize("d,H,n", [(64, 13, 2000), (64, 2, 700), (128, 8, 4013), (128, 2, 700)])
def test_small_values(ha, torch, d, H, n, exponent):
    """Each is taken with an absolute error of up to 2^-125, and the weights of a row add up to 1."""
    print(f"split fp32 values of 2^{exponent} d={d} H={H} n={n}", flush=True)
    q, k, v = _inputs(torch, H, n, d, d + n, 3)
    v = v * 2.0 ** exponent
    out, lse = ha.exact_attn_forward(q, k, v)
    q1, k1, v1 = (x[:, :1].double() for x in (q, k, v))
    s = torch.matmul(q1, k1.transpose(-1, -2).contiguous())
    want = torch.matmul(torch.softmax(s, -1), v1)
    assert ((out[:, :1].double() - want).abs() <= 2.0 ** -125 + 1e-5 * want.abs() + 1e-6 * v1.abs().max()).all()


# Every form of the kernels: one way, two, four, eight (tests of infinities and of largest numbers).
FORMS = [(64, 13, 4000, False), (64, 9, 3700, False), (64, 20, 1001, True), (64, 2, 700, False), (128, 8, 4096, False),
         (128, 9, 2501, True), (128, 2, 700, False)]


def _far_scores(torch, q, k, partner, key):
    """Column 7 carries nothing but key 9's score: partner (both signs of its bits, no two alike) times key."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q[..., 7] = partner * (1.0 + torch.rand(q.shape[:-1], generator=gen, device="cuda"))
    k[..., 7] = 0.0
    k[:, :, 9, 7] = key


@pytest.mark.parametrize("partner,key", [(3e5, float("-inf")), (1e20, -1e20), (1e20, -3.4028234e38)])
@pytest.mark.parametrize("d,H,n,causal", FORMS)
def test_scores_that_overflow(ha, torch, d, H, n, causal, partner, key):
    """A score of -inf, as an infinite key or as products past the largest number, is a key without weight, forward and backward: all
    but the column of dQ that 0 times the key enters, as without the key."""
    print(f"split fp32 far scores d={d} H={H} n={n} causal={causal} {partner} {key}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, n + 1)
    _far_scores(torch, q, k, partner, key)
    out, lse = ha.exact_attn_forward(q, k, v, causal=causal)
    grads = ha.exact_attn_backward(q, k, v, out, lse, g, causal=causal)
    k0 = k.clone()
    k0[:, :, 9, 7] = -1e25 / partner  # a score of -1e25: no weight either
    ref = _reference(torch, *(x[:, H - 1:] for x in (q, k0, v, g)), causal)
    got = [x[:, H - 1:].double() for x in (out, lse, *grads)]
    if key == float("-inf"):
        got[2], ref[2][..., 7] = got[2].clone(), 0.0
        got[2][..., 7] = 0.0
    assert ((got[0] - ref[0]).abs() <= 1e-5 + 1e-5 * ref[0].abs()).all()
    assert ((got[1] - ref[1]).abs() <= 2e-5).all()
    for x, want in zip(got[2:], ref[2:]):  # (dQ's and dK's column 7 is partner times the others: a norm of its own)
        for cols in ([7], [c for c in range(d) if c != 7]):
            assert (x[..., cols] - want[..., cols]).norm() <= 2e-6 * want[..., cols].norm()


@pytest.mark.parametrize("value", [0x7f800000, 0x7f800001, 0x7fc00000, 0x7f7fffff])
@pytest.mark.parametrize("d,H,n,causal", FORMS)
def test_value_at_the_end_of_the_range(ha, torch, d, H, n, causal, value):
    """One value, infinite, NaN (a signalling one too) or the largest number: its column is that times its weight, the others are as without it;
    the other way round, through dO, for dV."""
    print(f"split fp32 last values d={d} H={H} n={n} causal={causal} {value:#x}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, n + 2)
    x = torch.tensor([value], dtype=torch.int32).view(torch.float32).item() if value != 0x7f800001 else None
    for t, row in ((v, 5), (g, n - 1)):
        t[..., 3] = -1e34 if value == 0x7f800000 else 0.0  # (sums that are far from the largest number, whatever is added to them)
        if x is None:
            t.view(torch.int32)[:, :, row, 3] = value
        else:
            t[:, :, row, 3] = x
    out, lse = ha.exact_attn_forward(q, k, v, causal=causal)
    v1 = v.clone()
    v1[..., 3] = 0.0
    out1, lse1 = ha.exact_attn_forward(q, k, v1, causal=causal)
    s = torch.matmul(q[:, :1].double(), k[:, :1].double().transpose(-1, -2).contiguous())
    weights = torch.exp(s - lse[:, :1, :, None].double())
    rows = slice(5, n) if causal else slice(0, n)
    assert torch.equal(lse, lse1)
    other = [c for c in range(d) if c != 3]
    assert ((out[..., other] - out1[..., other]).abs() <= 1e-5 + 1e-5 * out1[..., other].abs()).all()
    dv = ha.exact_attn_backward(q, k, v1, out1, lse1, g, causal=causal)[2]
    seen = {0x7f800000: torch.isposinf, 0x7f800001: torch.isnan, 0x7fc00000: torch.isnan}.get(value)
    if seen is not None:
        assert seen(out[:, :, rows, 3]).all() and seen(dv[..., 3]).all()
    else:
        for got, want in ((out[:, :1, rows, 3].double(), weights[:, :, rows, 5] * x), (dv[:, :1, :, 3].double(), weights[:, :, n - 1, :] * x)):
            assert ((got - want).abs() <= 2e-5 * want.abs()).all()
    assert torch.isfinite(dv[..., other]).all()


@pytest.mark.parametrize("d,H,n,b,m,causal,n_min", [(64, 16, 4096, 128, 128, False, 4096), (64, 8, 4096, 256, 256, False, 4096), (64, 2, 2048, 64, 64, True, 512),
                                                    (128, 8, 4096, 256, 256, False, 4096), (128, 2, 2048, 64, 64, True, 512)])
def test_scores_that_overflow_in_nodes(ha, torch, d, H, n, b, m, causal, n_min):
    """The same through the blocks and samples: bit for bit what scores of -1e25, which overflow nowhere, give."""
    print(f"split fp32 far scores, nodes d={d} H={H} n={n} b={b} m={m} causal={causal}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, n + 3)
    shape, params = ha.make_shape(1, H, n, d, ha.HA_FP32), ha.make_params(b, m, 7, causal, n_min, 0)
    got = []
    for key in (-1e20, -1e5):
        _far_scores(torch, q, k, 1e20, key)
        ws = ha.alloc_workspace(shape, params)
        out, lse = ha.hyperattn_forward(q, k, v, b, m, 7, causal=causal, n_min=n_min, seed=0, workspace=ws)
        got.append((out, lse, *ha.hyperattn_backward(q, k, v, out, lse, g, b, m, 7, causal=causal, n_min=n_min, seed=0, fwd_workspace=ws)))
    for x, want in zip(*got):
        assert torch.isfinite(want).all()
        assert torch.equal(x, want)


@pytest.mark.parametrize("d", [64, 128])
def test_one_product(ha, torch, d):
    """The first row of a causal head has one key, and its log row sum is their score: with one column each, a single product of two numbers.
    Its parts leave out at most 2^-24.2 of it, and it is rounded once: at most 2^-23.1; r.m.s. over all mantissas 2^-25.21 (2^-25.24 rounded
    alone, as a fused fp32 product is), here within what 8192 samples scatter."""
    print(f"split fp32 one product d={d}", flush=True)
    H, n = 8192, 32
    q, k, v = _inputs(torch, H, n, d, d + 5, 3)
    for t in (q, k):
        t.zero_()
        t[..., d - 5] = torch.rand(t.shape[:-1], generator=torch.Generator(device="cuda").manual_seed(11 if t is q else 12), device="cuda") + 1.0
    _, lse = ha.exact_attn_forward(q, k, v, causal=True)
    want = q[:, :, 0, d - 5].double() * k[:, :, 0, d - 5].double()
    err = (lse[:, :, 0].double() - want) / want
    assert err.abs().max() <= 2.0 ** -23.1
    assert err.square().mean().sqrt() <= 2.0 ** -25.1


@pytest.mark.parametrize("kind", ["one column", "sparse"])
@pytest.mark.parametrize("d,H,n,causal", FORMS)
def test_products_that_few_terms_carry(ha, torch, d, H, n, causal, kind):
    """Scores to 250 and gradients that one column carries, or two of d columns: next to no term whose rounding could average the others'.  Errors
    (2-norm; largest of a log row sum) as of products and sums in fp32, whose matrix instructions have, over eight shapes, geometric
    means, split in brackets: one column: dK 2.6e-7 (2.3e-7), dV 2.5e-7 (1.9e-7), lse 1.5e-5 (1.5e-5); sparse: dK 1.5e-5 (1.4e-5), dV
    3.1e-6 (3.4e-6), lse 1.2e-4 (8.5e-5).  Bounds: lse, scores of s each rounded to 2^-23 s and once more in the sum, 2^-22 of the largest score;
    gradients of one column, products to 2^-23 with weights to the scores' errors, where both average over n, 1e-6."""
    print(f"split fp32 few terms d={d} H={H} n={n} causal={causal} {kind}", flush=True)
    q, k, v, g = _inputs(torch, H, n, d, n + 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    if kind == "one column":
        for t, col, scale, low, width in ((q, 5, 2.0 ** -12, 6.0, 10.0), (k, 5, 2.0 ** -12, 6.0, 10.0), (v, 7, 2.0 ** -14, 1.0, 1.0), (g, 7, 2.0 ** -14, 1.0, 1.0)):
            t *= scale
            t[..., col] = torch.rand(t.shape[:-1], generator=gen, device="cuda") * width + low
    else:
        for t in (q, k, v, g):
            t *= (torch.rand(t.shape, generator=gen, device="cuda") < 2 / d) * (d / 2)
    out, lse = ha.exact_attn_forward(q, k, v, causal=causal)
    grads = ha.exact_attn_backward(q, k, v, out, lse, g, causal=causal)
    ref = _reference(torch, *(x[:, :1] for x in (q, k, v, g)), causal)
    top = torch.matmul(q[:, :1].double(), k[:, :1].double().transpose(-1, -2).contiguous()).abs().max().item()
    assert (lse[:, :1].double() - ref[1]).abs().max() <= 2.0 ** -22 * max(top, 1.0)
    if kind == "one column":
        for got, want in zip(grads[1:], ref[3:]):
            assert (got[:, :1].double() - want).norm() <= 1e-6 * want.norm()
    else:
        for got, want, bound in zip(grads, ref[2:], (6e-5, 6e-5, 2e-5)):
            assert (got[:, :1].double() - want).norm() <= bound * want.norm()


@pytest.mark.parametrize("vnorm", [False, True])
@pytest.mark.parametrize("d,H,n,b,m,ways", [(64, 2, 300, 100, 130, 4), (64, 24, 704, 64, 96, 2), (64, 24, 704, 64, 20, 2), (64, 80, 896, 128, 31, 1),
                                            (128, 2, 300, 100, 130, 4), (128, 35, 896, 128, 70, 1)])
def test_second_run_with_caps(ha, torch, d, H, n, b, m, ways, vnorm):
    """Rows with a score of +inf, whose outputs are not finite in any arithmetic, share workgroups with rows that have none: these are what
    they are when that score is 1e30.  (Their workgroups run their loops, with the barriers of the caps, twice.)"""
    print(f"split fp32 second run, caps d={d} H={H} n={n} b={b} m={m} vnorm={vnorm}", flush=True)
    shape, params = ha.make_shape(1, H, n, d, ha.HA_FP32), ha.make_params(b, m, 5, False, 4096, 5)
    assert ha.ha_fp32_ways(shape, params)[0] == ways
    q, k, v = _inputs(torch, H, n, d, n + 6, 3)
    q[..., 7] = 0.0
    q[:, :, 10:30, 7] = 1e20
    k[..., 7] = 0.0
    got = []
    for key in (1e20, 1e10):
        k[:, :, 9, 7] = key
        out, lse, _ = ha.hyperattn_forward_alg2(q, k, v, b, m, 5, seed=5, cap_scale=6.0, vnorm_sampling=vnorm)
        got.append((out, lse))
    (out, lse), (out1, lse1) = got
    assert not torch.isfinite(lse[:, :, 10:30]).all()
    assert torch.isfinite(lse1).all()
    rows = [i for i in range(n) if not 10 <= i < 30]
    assert ((out[:, :, rows] - out1[:, :, rows]).abs() <= 1e-5 + 1e-5 * out1[:, :, rows].abs()).all()
    # (when a wave's references move depends on all of its rows)
    assert ((lse[:, :, rows] - lse1[:, :, rows]).abs() <= 2e-5 * lse1[:, :, rows].abs().clamp(min=1.0)).all()
