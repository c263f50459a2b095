"""Rows that a call has no business with do not reach its results: rows behind the tensors, rows of the next head and rows
of the next diagonal block hold NaN or Inf, and what does not depend on them stays bit for bit what it is without them
(a masked weight is 0, and 0 times NaN or Inf is NaN: such rows must not be loaded at all)."""
import pytest

from ha_testutil import have_gpu

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


def _dtype(torch, name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _rows(torch, gen, H, n, d, dtype, behind, poisoned_heads=()):
    """[1, H, n, d] at the front of a buffer whose next 256 rows hold `behind`; heads of `poisoned_heads` hold it too."""
    buf = torch.full(((H * n + 256) * d,), behind, dtype=dtype, device="cuda")
    x = buf[:H * n * d].view(1, H, n, d)
    x.copy_((torch.randn((1, H, n, d), generator=gen, device="cuda") * d ** -0.25).to(dtype))
    for h in poisoned_heads:
        x[:, h] = behind
    return x


def _generator(torch, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,d,H,n", [("bf16", 64, 1, 257), ("bf16", 128, 1, 257), ("bf16", 64, 2, 321), ("bf16", 128, 2, 321),
                                         ("bf16", 64, 2, 641), ("bf16", 128, 2, 705),   # two wave groups, the second's last tile past the end
                                         ("bf16", 64, 2, 5), ("bf16", 128, 100, 300),   # one wave group
                                         ("bf16", 128, 40, 8200),                       # eight waves
                                         ("fp32", 64, 2, 33), ("fp32", 128, 2, 5), ("fp32", 64, 20, 2050)])
def test_exact_forward_reads_its_own_rows_only(ha, torch, dtype, d, H, n, causal):
    print(f"exact forward bounds {dtype} d={d} H={H} n={n} causal={causal}", flush=True)
    dt = _dtype(torch, dtype)
    results = []
    for behind in (0.0, float("nan"), float("inf")):
        gen = _generator(torch, n)
        q, k, v = (_rows(torch, gen, H, n, d, dt, behind, (H - 1,) if H > 1 else ()) for _ in range(3))
        results.append(ha.exact_attn_forward(q, k, v, causal=causal))
    own = slice(0, H - 1) if H > 1 else slice(0, 1)
    assert torch.isfinite(results[0][0]).all()
    for out, lse in results[1:]:
        assert torch.equal(out[:, own], results[0][0][:, own])
        assert torch.equal(lse[:, own], results[0][1][:, own])


@pytest.mark.parametrize("dtype,d,H,n_min", [("bf16", 64, 2, 320), ("bf16", 128, 2, 320), ("bf16", 64, 2, 704), ("bf16", 128, 2, 704), ("bf16", 64, 70, 320),
                                             ("bf16", 128, 3, 65), ("fp32", 64, 2, 320), ("fp32", 128, 2, 33)])
def test_next_diagonal_block_stays_out(ha, torch, dtype, d, H, n_min):
    """The first n_min rows of a causal call see nothing of the rows behind them."""
    print(f"next block {dtype} d={d} H={H} n_min={n_min}", flush=True)
    dt = _dtype(torch, dtype)
    results = []
    for value in (0.0, float("inf"), float("nan")):
        gen = _generator(torch, n_min)
        q, k, v = (_rows(torch, gen, H, 2 * n_min, d, dt, 0.0) for _ in range(3))
        v[:, :, n_min:] = value
        results.append(ha.hyperattn_forward(q, k, v, n_min if n_min < 64 else n_min // 5 if n_min % 5 == 0 else n_min // 11, 16, 7, causal=True, n_min=n_min, seed=1))
    assert torch.isfinite(results[0][0]).all()
    for out, lse in results[1:]:
        assert torch.equal(out[:, :, :n_min], results[0][0][:, :, :n_min])
        assert torch.equal(lse, results[0][1])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,d,H,n", [("fp32", 64, 1, 1), ("fp32", 128, 2, 5), ("fp32", 64, 2, 23), ("fp32", 128, 1, 33),
                                         ("fp32", 64, 2, 300), ("fp32", 64, 40, 2079), ("fp32", 128, 40, 2050),  # one wave per 32 rows
                                         ("bf16", 64, 1, 1), ("bf16", 128, 2, 65), ("bf16", 64, 2, 321)])
def test_exact_backward_reads_its_own_rows_only(ha, torch, dtype, d, H, n, causal):
    """NaN behind Q, K, V, dO, the output and the log row sums, and in the last of several heads: the same gradients."""
    print(f"exact backward bounds {dtype} d={d} H={H} n={n} causal={causal}", flush=True)
    dt = _dtype(torch, dtype)
    own = slice(0, H - 1) if H > 1 else slice(0, 1)
    results = []
    for behind in (0.0, float("nan")):
        gen = _generator(torch, n)
        q, k, v, g = (_rows(torch, gen, H, n, d, dt, behind, (H - 1,) if H > 1 else ()) for _ in range(4))
        out = _rows(torch, gen, H, n, d, dt, behind)
        lse = _rows(torch, gen, H, n, 1, torch.float32, behind).view(1, H, n)
        out32 = _rows(torch, gen, H, n, d, torch.float32, behind) if dtype == "bf16" else None
        ha.exact_attn_forward(q, k, v, causal=causal, out=out, lse=lse, out_f32=out32)
        results.append(ha.exact_attn_backward(q, k, v, out, lse, g, causal=causal, out_f32=out32))
    for x, y in zip(*results):
        assert torch.isfinite(x).all()
        assert torch.equal(x[:, own], y[:, own])


@pytest.mark.parametrize("d,H,n,n_min", [(64, 32, 2048, 0), (128, 32, 2048, 0), (64, 16, 2048, 0), (64, 1, 512, 0),  # one, two, four waves
                                         (64, 32, 2048, 1024), (128, 2, 1024, 256)])
@pytest.mark.parametrize("first", [64, 192])
def test_fp32_causal_rows_see_no_later_tile(ha, torch, d, H, n, n_min, first):
    """fp32, causal: rows of V from a multiple of 64 on are Inf; the rows before it do not load them."""
    print(f"fp32 later rows d={d} H={H} n={n} n_min={n_min} first={first}", flush=True)
    results = []
    for value in (0.0, float("inf")):
        gen = _generator(torch, n + H)
        q, k, v = (_rows(torch, gen, H, n, d, torch.float32, 0.0) for _ in range(3))
        v[:, :, first:] = value
        results.append(ha.hyperattn_forward(q, k, v, 64, 16, 7, causal=True, n_min=n_min, seed=1) if n_min
                       else ha.exact_attn_forward(q, k, v, causal=True))
    assert torch.isfinite(results[0][0]).all()
    assert torch.equal(results[0][0][:, :, :first], results[1][0][:, :, :first])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("b,m", [(32, 0), (32, 40), (64, 40), (128, 17)])
def test_capped_rows_see_only_their_keys(ha, torch, d, b, m):
    """Algorithm 2's caps, causal: Inf in the value of a node's first key reaches the one sorted block that holds the key
    (and sampled rows, none here), not the rows whose key lists are filled up to whole tiles."""
    print(f"caps, filled key lists d={d} b={b} m={m}", flush=True)
    n, n_min = 1024, 256
    seed = next(s for s in range(100) if m == 0 or 0 not in set(ha.ha_make_samples(s, 1, 1, 256, m)))
    gen = _generator(torch, d + b)
    q, k, v = (_rows(torch, gen, 2, n, d, torch.bfloat16, 0.0) for _ in range(3))
    v[:, :, 512] = float("inf")   # the second node of level 1: keys 512 ... 767, queries 768 ... 1023
    out, lse, _ = ha.hyperattn_forward_alg2(q, k, v, b, m, 7, seed=seed, cap_scale=6.0 if m else 0.0, kappa=1.2 if m else 0.0,
                                            causal=True, n_min=n_min)
    assert torch.isfinite(lse).all()
    assert torch.isfinite(out[:, :, :512]).all()
    hit = ~torch.isfinite(out[:, :, 768:]).all(dim=-1)
    assert (hit.sum(dim=-1) == b).all(), hit.sum(dim=-1)
