"""fp32 tensors on the fp32 matrix cores: the forms of the kernels that the smaller parity cases do not
reach (one, two or four waves per group of 32 queries, chosen by the number of groups and the length of the
run of rows), at lengths around their tiles, against the fp64 oracle on single heads."""
import pytest

import synth_inputs
from ha_testutil import assert_close, assert_lse_close, have_gpu, run_oracle, to_device, to_host
from oracle import hyperattn_oracle as orc

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("H,n,d,b,m,causal,n_min", [
    (16, 4096, 64, 128, 40, 0, 4096),     # one wave per group: 128-row tiles
    (16, 4096, 128, 128, 33, 0, 4096),
    (8, 4096, 64, 64, 64, 1, 1024),       # two waves per group: 64-row tiles, blocks of 64
    (6, 4032, 128, 63, 7, 0, 4096),       # two waves, one row of the tile idle
    (3, 1056, 64, 33, 31, 0, 4096),       # four waves per group: 32-row tiles, one row in the second
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
