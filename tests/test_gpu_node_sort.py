"""Small calls, whose attention launch sorts its nodes by itself, against the sorting launches (which
hyperattn_forward_timed always takes): the permutations and everything computed from them are the same bits."""
import math

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


CASES = [  # dtype, d, B, H, n, b, m, r, n_min (0: unmasked)
    ("bf16", 64, 1, 2, 4096, 256, 256, 7, 0),      # 16 keys per thread, the last full size
    ("bf16", 64, 1, 2, 4160, 64, 300, 7, 0),       # 32 per thread from here on; more samples than threads
    ("bf16", 128, 1, 1, 8192, 256, 64, 8, 0),      # the longest node, all 256 buckets
    ("bf16", 128, 2, 3, 1300, 100, 77, 6, 0),      # heads at odd addresses, blocks that no tile divides
    ("bf16", 64, 1, 3, 15, 5, 4, 1, 0),            # fewer keys than a thread holds, two buckets
    ("bf16", 64, 1, 2, 513, 513, 40, 7, 0),        # one block: no sample is kept
    ("bf16", 128, 1, 2, 999, 37, 0, 7, 0),         # no samples; 4 keys per thread at odd addresses
    ("bf16", 64, 1, 3, 1505, 35, 50, 7, 0),        # 8 keys
    ("bf16", 64, 1, 3, 5005, 77, 50, 7, 0),        # 32 keys
    ("bf16", 64, 1, 2, 8192, 128, 96, 7, 1024),    # three levels
    ("bf16", 128, 1, 2, 2080, 65, 33, 5, 520),     # two levels, odd sizes
    ("bf16", 64, 1, 16, 2048, 512, 600, 7, 0),     # four tiles per block, more samples than threads
    ("bf16", 64, 1, 32, 4096, 256, 256, 7, 0),     # the most workgroups
    ("fp32", 64, 1, 1, 1024, 64, 64, 7, 0),
    ("fp32", 128, 1, 3, 777, 21, 50, 8, 0),
    ("fp32", 64, 1, 4, 4096, 64, 64, 7, 1024),
    ("fp32", 64, 2, 8, 2048, 256, 256, 7, 0),
    ("fp32", 64, 1, 16, 4096, 128, 64, 7, 0),      # one wave per group of rows
    ("fp32", 128, 1, 32, 2048, 128, 0, 7, 0),      # likewise, no samples
    ("fp32", 128, 1, 8, 8192, 128, 2000, 8, 0),    # likewise, the longest node, the most that its LDS holds
    ("fp32", 64, 1, 6, 8192, 256, 256, 7, 0),      # likewise
    ("fp32", 64, 1, 9, 4096, 64, 1000, 8, 0),      # two
    ("fp32", 128, 1, 16, 2048, 64, 64, 7, 0),      # four, the most workgroups
]

EIGHT_WAVES = [  # more than 256 tiles of 128 rows, at most 256 of 256: workgroups of eight waves
    ("bf16", 64, 1, 12, 4096, 256, 256, 7, 0),
    ("bf16", 64, 1, 12, 8192, 256, 256, 7, 4096),  # one level
    ("bf16", 128, 1, 8, 8192, 256, 100, 8, 0),     # the longest node, all buckets
    ("bf16", 64, 4, 25, 300, 150, 20, 3, 0),       # fewer keys than threads
    ("bf16", 128, 4, 5, 1500, 150, 77, 6, 0),      # 4 keys per thread at odd addresses, the last waves' past the end
    ("bf16", 64, 1, 24, 2048, 512, 600, 7, 0),     # two tiles per block, more samples than threads
    ("bf16", 128, 1, 16, 3200, 200, 100, 7, 0),    # waves that end in the second 128 rows of a tile
    ("bf16", 64, 1, 12, 3000, 300, 100, 7, 0),     # blocks whose second tile holds 44 rows
]


def tiles(rows, B, H, n, b, n_min):
    """Tiles of up to `rows` query rows in the node launch."""
    levels, covered = (int(math.log2(n // n_min)), n // 2) if n_min else (1, n)
    return levels * B * H * (covered // b) * -(-b // rows)


@pytest.mark.parametrize("law", ["iid", "equal", "steep"])
@pytest.mark.parametrize("dtype,d,B,H,n,b,m,r,n_min", CASES + EIGHT_WAVES)
def test_sort_inside_the_attention_launch(ha, torch, dtype, d, B, H, n, b, m, r, n_min, law):
    print(f"node sort {dtype} d={d} B={B} H={H} n={n} b={b} m={m} r={r} n_min={n_min} {law}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + r)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = ((torch.randn((B, H, n, d), generator=gen, device="cuda") * d ** -0.25).to(dt) for _ in range(3))
    if law == "equal":  # every key in one bucket: the order is that of the rows
        q, k = (x[:, :, :1].expand(B, H, n, d).contiguous() for x in (q, k))
    elif law == "steep":  # scores far apart: references move, by what all lanes of a wave see
        q = q * 4
    shape = ha.make_shape(B, H, n, d, ha.HA_BF16 if dtype == "bf16" else ha.HA_FP32)
    params = ha.make_params(b, m, r, n_min > 0, n_min or 4096, 3)
    assert ha.ha_call_routes(shape, params)[0]     # by the rule of the dispatch itself
    if dtype == "bf16":
        eight = tiles(128, B, H, n, b, n_min) > 256 >= tiles(256, B, H, n, b, n_min)
        assert eight == ((dtype, d, B, H, n, b, m, r, n_min) in EIGHT_WAVES)
    names = ("perm_q", "perm_k", "pos_k") + (("samp_blk",) if m else ())
    results = []
    for call in (ha.hyperattn_forward, ha.hyperattn_forward_timed):
        ws = ha.alloc_workspace(shape, params).fill_(0x5A)
        out, lse = call(q, k, v, b, m, r, causal=n_min > 0, n_min=n_min or 4096, seed=3, workspace=ws)[:2]
        torch.cuda.synchronize()
        views = ha.binding.workspace_views(ws, shape, params)
        results.append((out, lse, {name: views[name].clone() for name in names}))
    (out0, lse0, views0), (out1, lse1, views1) = results
    for name in names:
        assert torch.equal(views0[name], views1[name]), name
    assert torch.isfinite(out0.float()).all()
    assert torch.equal(out0, out1) and torch.equal(lse0, lse1)
