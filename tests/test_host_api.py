"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol the header declares, rejects bad arguments before touching the
device, lays out the workspace as documented, and its random draws are
bit-identical to the oracle's independently written generator."""
import ctypes
import os
import re

import numpy as np
import pytest

from oracle import hyperattn_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ha():
    import paper_2310_05869_amd as mod
    if not os.path.exists(mod.binding.LIB_PATH):
        from paper_2310_05869_amd import build
        build.build_library()
    mod.lib()
    return mod


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "hyperattn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ha_\w+|hyperattn_\w+|exact_attn_\w+)\s*\(", text)))


def test_header_symbols_are_exported_and_bound(ha):
    declared = _declared_functions()
    assert "hyperattn_forward" in declared and "ha_lsh_hash" in declared
    handle = ctypes.CDLL(ha.binding.LIB_PATH)
    for name in declared:
        assert hasattr(handle, name), f"{name} declared in hyperattn.h but not exported"
    assert sorted(ha.exported_symbols()) == declared


def test_struct_layouts_match_header(ha):
    assert ctypes.sizeof(ha.HaShape) == 20
    assert ctypes.sizeof(ha.HaParams) == 32 and ha.HaParams.seed.offset == 24


@pytest.mark.parametrize("seed,d,r", [(0, 128, 7), (0, 64, 7), (12345, 128, 8), (2 ** 63 + 5, 64, 1)])
def test_projection_bit_identical_to_oracle(ha, seed, d, r):
    R = ha.ha_make_projection(seed, d, r)
    np.testing.assert_array_equal(R.astype(np.float64), orc.make_projection(seed, d, r))


@pytest.mark.parametrize("first", [0, 1 << 40])
def test_projection_series_agree_with_the_library_functions(ha, first):
    """R is generated from series and falls back to log / cos near a rounding boundary of bf16: 32 seeds x 1024
    entries (several boundary cases among them) hold the oracle's bits."""
    for seed in range(first, first + 32):
        np.testing.assert_array_equal(ha.ha_make_projection(seed, 128, 8).astype(np.float64), orc.make_projection(seed, 128, 8))


@pytest.mark.parametrize("seed,level,node,n_keys,m", [(0, 0, 0, 32768, 256), (0, 4, 15, 4096, 256), (7, 2, 3, 1000, 33),
                                                      (1, 0, 0, 1, 5), (3, 1, 0, 2 ** 24, 512)])
def test_samples_bit_identical_to_oracle(ha, seed, level, node, n_keys, m):
    np.testing.assert_array_equal(ha.ha_make_samples(seed, level, node, n_keys, m),
                                  orc.make_samples(seed, level, node, n_keys, m))


def test_workspace_layout(ha):
    sh = ha.make_shape(1, 32, 131072, 128, ha.HA_BF16)
    p = ha.make_params(256, 256, 7, True, 4096, 0)
    lay = ha.ha_workspace_layout(sh, p)
    assert (lay.levels, lay.total_nodes, lay.n_cov) == (5, 31, 65536)
    offs = [lay.codes_q, lay.codes_k, lay.perm_q, lay.perm_k, lay.pos_k, lay.samples, lay.proj, lay.part_o,
            lay.part_l, lay.total_bytes]
    assert all(o % 256 == 0 for o in offs) and offs == sorted(offs)
    assert lay.part_l - lay.part_o == 5 * 32 * 65536 * 128 * 2     # bf16 tensors: bf16 partial outputs
    assert ha.ha_workspace_bytes(sh, p) == lay.total_bytes
    # unmasked: one level covering all n rows, no partial buffers
    p2 = ha.make_params(256, 256, 7, False, 4096, 0)
    lay2 = ha.ha_workspace_layout(ha.make_shape(1, 32, 32768, 128, ha.HA_BF16), p2)
    assert (lay2.levels, lay2.total_nodes, lay2.n_cov) == (1, 1, 32768)
    assert lay2.part_l == lay2.part_o
    # causal with n <= n_min: exact attention only
    lay3 = ha.ha_workspace_layout(ha.make_shape(1, 2, 1024, 64, ha.HA_BF16), p)
    assert lay3.levels == 0 and lay3.total_nodes == 0


def test_backward_workspace_layout(ha):
    """The backward keeps one accumulated fp32 row per tensor row and pass (two buffers, the first one used by dQ
    and then by dK), delta, and the sampled keys' rows per query chunk: not one buffer per level."""
    sh = ha.make_shape(1, 32, 131072, 128, ha.HA_BF16)
    p = ha.make_params(256, 256, 7, True, 4096, 0)
    lay = ha.binding.HaBwdWsLayout()
    assert ha.lib().ha_backward_workspace_layout(ctypes.byref(sh), ctypes.byref(p), ctypes.byref(lay)) == 0
    rows = 32 * 131072
    assert lay.acc_a - lay.delta == rows * 4 and lay.acc_b - lay.acc_a == rows * 128 * 4
    assert lay.samp_k - lay.acc_b == rows * 128 * 4
    # per level: 32 heads x 2^l nodes x ceil(s / 2048) chunks x 256 samples, s = n >> (l + 1): 32 chunks per head and level
    samp_rows = 5 * 32 * 32 * 256
    assert lay.samp_v - lay.samp_k == samp_rows * 128 * 4 and lay.total_bytes - lay.samp_v == samp_rows * 128 * 4
    assert lay.total_bytes == ha.ha_backward_workspace_bytes(sh, p) < 6 * 2 ** 30
    # fp32 tensors have a backward pass too, with the same buffers
    assert ha.ha_backward_workspace_bytes(ha.make_shape(1, 32, 131072, 128, ha.HA_FP32), p) == lay.total_bytes
    # exact attention (the recursion that never splits): delta only
    p0 = ha.make_params(1, 0, 1, True, 131072, 0)
    assert ha.ha_backward_workspace_bytes(sh, p0) == rows * 4


def test_backward_workspace_of_an_unmasked_problem(ha):
    """Its passes write the gradients: delta and the sampled keys' rows, no accumulated rows; bounded by 2 * 1023 * 128
    sampled rows where the chunks are short."""
    lay = ha.binding.HaBwdWsLayout()
    sh, p = ha.make_shape(1, 12, 16384, 64, ha.HA_BF16), ha.make_params(256, 256, 7, False, 4096, 0)
    assert ha.lib().ha_backward_workspace_layout(ctypes.byref(sh), ctypes.byref(p), ctypes.byref(lay)) == 0
    rows = 12 * 16384
    assert lay.acc_a == lay.acc_b == lay.samp_k == rows * 4
    assert lay.samp_v - lay.samp_k == (rows // 2 + 12 * 256) * 64 * 4   # chunks of 512: 32 per head, 256 rows each, below the bound s / 2 + m
    assert ha.ha_backward_workspace_bytes(sh, ha.make_params(256, 0, 7, False, 4096, 0)) == rows * 4


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype_d", [("HA_BF16", 64), ("HA_FP32", 128)])
def test_backward_workspace_grows_with_the_problem(ha, causal, dtype_d):
    """A workspace of a problem serves every one with fewer rows, heads or samples, although short problems cut their
    queries into shorter chunks and keep more rows per sample; and it holds the rows of its own chunks."""
    dtype, d = getattr(ha, dtype_d[0]), dtype_d[1]
    b, n_min = 8, 512
    sizes = [n_min << k for k in range(1, 11)] if causal else [b * k for k in (1, 31, 32, 255, 256, 4095, 8192, 37500, 65535, 65536, 131071, 131072)]

    def layout(H, n, m):
        lay = ha.binding.HaBwdWsLayout()
        sh, p = ha.make_shape(1, H, n, d, dtype), ha.make_params(b, m, 7, causal, n_min, 0)
        assert ha.lib().ha_backward_workspace_layout(ctypes.byref(sh), ctypes.byref(p), ctypes.byref(lay)) == 0
        return lay

    def rows_needed(H, n, m):
        nodes = [(2 ** l, n >> (l + 1)) for l in range((n // n_min).bit_length() - 1)] if causal else [(1, n)]
        chunks = lambda c: H * sum(k * -(-s // min(s, c)) for k, s in nodes)
        chunk = 2048
        while chunk // 2 >= 256 and chunk // 2 >= 2 * m and chunks(chunk) * -(-m // 128) < 1024:
            chunk //= 2
        return chunks(chunk) * m

    total = {}
    for H in (1, 3, 12, 64):
        for n in sizes:
            for m in (0, 1, 127, 128, 129, 256, 700, 1024, 1025, 4096):
                lay = layout(H, n, m)
                assert lay.samp_v - lay.samp_k >= rows_needed(H, n, m) * d * 4, (H, n, m)
                assert lay.total_bytes - lay.samp_v >= rows_needed(H, n, m) * d * 4, (H, n, m)
                total[H, n, m] = lay.total_bytes
    for axis in range(3):
        values = sorted({key[axis] for key in total})
        for key, size in total.items():
            at = values.index(key[axis])
            if at > 0:
                below = tuple(values[at - 1] if x == axis else key[x] for x in range(3))
                assert total[below] <= size, (below, total[below], key, size)



def test_backward_shared_launches_hold_their_workgroups(ha):
    """A launch of 256 threads per workgroup counts its threads in 32 bits: passes share one of at most 2^23 workgroups.
    Short blocks, a workgroup each, make the levels' launches far larger than the base case's."""
    routes = lambda BH, n, d, b, m, n_min: ha.ha_call_routes(ha.make_shape(1, BH, n, d, ha.HA_FP32), ha.make_params(b, m, 7, True, n_min, 0))[1]
    assert routes(1024, 16384, 64, 1, 0, 64) == 0                # 2^20 in the base case's launch, 2^24 in a level's
    assert routes(512, 16384, 64, 1, 0, 64) == 1 << 23           # the most that a launch holds
    assert routes(4, 4096, 64, 64, 64, 1024) == 2 * 4 * 4096 // 32 + 128   # dK / dV, dQ, sampled keys: 64 query chunks, two groups of 32
    for BH in (1, 48, 1024, 1 << 16):
        for n_min, b in ((16, 1), (16, 16), (64, 1), (96, 3), (96, 32), (512, 64)):
            for levels in (1, 4, 8):
                for m in (0, 33, 256):
                    if BH * (n_min << levels) <= 1 << 30:
                        assert routes(BH, n_min << levels, 64, b, m, n_min) <= 1 << 23
    assert ha.ha_call_routes(ha.make_shape(1, 4, 4096, 64, ha.HA_BF16), ha.make_params(64, 64, 7, True, 1024, 0))[1] == 0


@pytest.mark.parametrize("dtype,d,H,n,b,m,r,n_min,sorts", [("bf16", *c) for c in [
    (64, 24, 2048, 64, 64, 7, 0, True),        # 768 workgroups: three to a CU
    (64, 8, 5760, 64, 64, 7, 0, True),         # the longest node of which three fit the LDS
    (64, 6, 5888, 64, 64, 7, 0, False),        # two: 552 workgroups have 512 places
    (64, 5, 5888, 64, 64, 7, 0, True),
    (64, 10, 6144, 256, 256, 7, 0, True),      # eight waves
    (64, 11, 6144, 256, 256, 7, 0, False),
    (64, 6, 12288, 256, 256, 7, 3072, False),  # two levels, 576 workgroups of 6144 keys
    (64, 17, 4096, 256, 1024, 7, 0, True),
    (64, 17, 4096, 256, 1024, 8, 0, False),    # more buckets: two
    (64, 32, 2048, 64, 64, 7, 0, True),        # a second round
    (64, 33, 2048, 64, 64, 7, 0, False),
    (64, 40, 2112, 96, 96, 7, 0, False),       # a second round of threads that hold half of what they could
    (64, 32, 4096, 256, 256, 7, 0, True),
    (64, 22, 3500, 100, 77, 7, 0, False),      # heads not at 16 bytes
    (64, 20, 5120, 256, 256, 7, 0, False),
    (64, 1, 8256, 64, 64, 7, 0, False),        # more keys than a workgroup's threads hold
    (128, 32, 1024, 64, 64, 7, 0, True),
    (128, 33, 1024, 64, 64, 7, 0, False),      # two to a CU
]] + [("fp32", *c) for c in [
    (64, 16, 4096, 64, 64, 7, 0, True),        # two ways: 1024 workgroups
    (64, 17, 4096, 64, 64, 7, 0, False),
    (64, 9, 4096, 64, 1000, 8, 0, True),       # 576, of which a CU holds two by their registers and by their tables
    (64, 2, 8192, 128, 2000, 7, 0, True),      # four ways, 512: three by their registers, two by the LDS
    (64, 2, 8192, 128, 2000, 8, 0, False),     # with more buckets' tables one
    (64, 8, 8192, 128, 2000, 7, 0, True),      # one way, 512: two
    (64, 8, 8192, 128, 2000, 8, 0, False),     # one
    (64, 6, 8192, 256, 256, 7, 0, True),       # one way, 384 of 8192 keys
    (64, 3, 8192, 256, 256, 7, 0, False),      # four, 768
    (128, 8, 8192, 128, 2000, 8, 0, True),     # one way, 512, of which a CU holds one in any case
    (128, 2, 8192, 128, 2000, 8, 0, False),    # four, 512: the tables cost the second
    (128, 48, 2048, 128, 128, 7, 0, True),     # one way, 768
    (128, 44, 2048, 128, 128, 7, 0, False),    # four, 2816
    (128, 16, 2048, 64, 64, 7, 0, True),       # four, 1024
    (128, 18, 2048, 64, 64, 7, 0, False),      # 1152
    (128, 61, 1000, 100, 64, 7, 0, False),     # blocks that the tiles do not divide: 2440
    (128, 2, 8192, 64, 64, 7, 0, True),        # 512 of 8192 keys
    (128, 3, 8192, 64, 64, 7, 0, False),       # 768
    (128, 4, 8192, 128, 128, 7, 0, True),      # one way, 256
    (128, 6, 4096, 256, 256, 7, 0, True),      # four, 768
    (128, 8, 4096, 32, 64, 7, 0, True),        # 1024, of blocks that 64 rows do not fill
    (128, 12, 4096, 64, 64, 7, 1024, False),   # two levels, 1536
]])
def test_forward_sorts_in_the_attention_launch(ha, dtype, d, H, n, b, m, r, n_min, sorts):
    """While its workgroups fit the chip, the sort's tables in the LDS counted."""
    shape = ha.make_shape(1, H, n, d, ha.HA_BF16 if dtype == "bf16" else ha.HA_FP32)
    assert bool(ha.ha_call_routes(shape, ha.make_params(b, m, r, n_min > 0, n_min or 4096, 0))[0]) == sorts


@pytest.mark.parametrize("d,H,n,b,m,n_min,forward,backward", [  # (n_min 0: unmasked)
    # Algorithm 2's caps and value sampling
    (64, 2, 300, 100, 130, 0, 4, 4), (64, 80, 896, 128, 31, 0, 1, 1), (64, 80, 700, 100, 65, 0, 1, 1), (64, 24, 704, 64, 96, 0, 2, 4),
    (64, 24, 704, 64, 40, 0, 2, 4), (64, 24, 704, 64, 20, 0, 2, 4), (128, 40, 896, 64, 77, 0, 4, 4), (128, 80, 700, 100, 0, 0, 4, 1),
    (128, 35, 896, 128, 70, 0, 1, 1), (128, 70, 700, 100, 31, 0, 1, 1),
    # forward, forward and backward
    (64, 16, 4096, 128, 40, 0, 1, 1), (128, 16, 4096, 128, 33, 0, 1, 1), (64, 8, 4096, 64, 64, 1024, 2, 0), (128, 6, 4032, 63, 7, 0, 4, 4),
    (64, 6, 4032, 63, 7, 0, 2, 4), (64, 3, 1056, 33, 31, 0, 4, 4), (64, 32, 4096, 128, 100, 0, 1, 1), (128, 32, 4096, 128, 128, 2048, 1, 1),
    (128, 30, 896, 128, 64, 0, 4, 1), (64, 5, 2112, 33, 65, 0, 4, 4),
    # scores that overflow
    (64, 16, 4096, 128, 128, 0, 1, 1), (64, 8, 4096, 256, 256, 0, 2, 4), (64, 2, 2048, 64, 64, 512, 4, 0), (128, 8, 4096, 256, 256, 0, 1, 1),
    (128, 2, 2048, 64, 64, 512, 4, 0)])
def test_fp32_forms_of_the_gpu_tests(ha, d, H, n, b, m, n_min, forward, backward):
    """The forms of the fp32 node kernels that tests on the GPU were given their sizes for: where a limit of the dispatch moves, they move too."""
    shape = ha.make_shape(1, H, n, d, ha.HA_FP32)
    assert ha.ha_fp32_ways(shape, ha.make_params(b, m, 5, n_min > 0, n_min or 4096, 0)) == (forward, backward)
    assert ha.ha_fp32_ways(ha.make_shape(1, H, n, d, ha.HA_BF16), ha.make_params(b, m, 5, n_min > 0, n_min or 4096, 0)) == (0, 0)


def test_forward_workgroup_counts(ha):
    """Records of the stamped forward: one per 128-query tile of every node (levels x half the rows when causal)
    and of the base case; none for fp32 tensors, which run the kernel without matrix cores."""
    p = ha.make_params(256, 256, 7, True, 4096, 0)
    assert ha.ha_forward_workgroups(ha.make_shape(1, 32, 131072, 128, ha.HA_BF16), p) == (5 * 32 * 65536 // 128, 32 * 131072 // 128)
    assert ha.ha_forward_workgroups(ha.make_shape(1, 32, 131072, 128, ha.HA_FP32), p) == (0, 0)
    pu = ha.make_params(256, 256, 7, False, 4096, 0)
    assert ha.ha_forward_workgroups(ha.make_shape(2, 4, 32768, 64, ha.HA_BF16), pu) == (8 * 32768 // 128, 0)
    assert ha.ha_forward_workgroups(ha.make_shape(1, 0, 32768, 64, ha.HA_BF16), pu) == (0, 0)
    nw, bw = ctypes.c_int64(0), ctypes.c_int64(0)
    bad = ha.make_shape(1, 1, 1000, 64, ha.HA_BF16)
    assert ha.lib().ha_forward_workgroups(ctypes.byref(bad), ctypes.byref(pu), ctypes.byref(nw), ctypes.byref(bw)) == -3
    assert ha.lib().ha_forward_workgroups(ctypes.byref(bad), ctypes.byref(pu), None, ctypes.byref(bw)) != 0


@pytest.mark.parametrize("shape,params,status", [
    ((1, 1, 1024, 96, 0), (64, 64, 7, 0, 4096, 0), -3),     # d not 64/128
    ((1, 1, 1000, 64, 0), (64, 64, 7, 0, 4096, 0), -3),     # n % b
    ((1, 1, 1024, 64, 0), (64, 64, 9, 0, 4096, 0), -3),     # r > 8
    ((1, 1, 1024, 64, 0), (64, 64, 0, 0, 4096, 0), -3),     # r < 1
    ((1, 1, 1024, 64, 0), (64, 5000, 7, 0, 4096, 0), -3),   # m too large
    ((1, 1, 1024, 64, 0), (0, 64, 7, 0, 4096, 0), -3),      # b < 1
    ((1, 1, 3072, 64, 0), (64, 64, 7, 1, 1024, 0), -3),     # n / n_min not a power of two
    ((1, 1, 2048, 64, 0), (96, 64, 7, 1, 1024, 0), -3),     # n_min % b
    ((1, 1, 2048, 64, 0), (64, 64, 7, 1, 0, 0), -3),        # n_min < 1
    ((1, 1, 1024, 64, 2), (64, 64, 7, 0, 4096, 0), -2),     # dtype
])
def test_bad_arguments_are_rejected_on_the_host(ha, shape, params, status):
    sh = ha.make_shape(*shape)
    p = ha.make_params(*params)
    lay = ha.HaWsLayout()
    assert ha.lib().ha_workspace_layout(ctypes.byref(sh), ctypes.byref(p), ctypes.byref(lay)) == status
    assert ha.ha_workspace_bytes(sh, p) == 0
    # the forward call reports the same error before any pointer is used
    assert ha.lib().hyperattn_forward(None, None, None, None, None, ctypes.byref(sh), ctypes.byref(p), None, 0,
                                      None) == status


def test_null_pointers_and_strerror(ha):
    sh = ha.make_shape(1, 1, 1024, 64, 0)
    p = ha.make_params(64, 64, 7)
    assert ha.lib().hyperattn_forward(None, None, None, None, None, ctypes.byref(sh), ctypes.byref(p), None, 0,
                                      None) == -1
    assert ha.lib().hyperattn_forward(None, None, None, None, None, None, None, None, 0, None) == -1
    assert ha.lib().exact_attn_forward(None, None, None, None, None, ctypes.byref(sh), 0, None) == -1
    assert ha.lib().ha_make_projection(0, 64, 7, None) == -1
    assert ha.lib().ha_lsh_hash(None, None, 10, 64, 0, None, 7, None) == -1
    assert ha.lib().ha_lsh_hash(None, None, 10, 65, 0, None, 7, None) == -3
    assert ha.lib().ha_seg_sort(None, None, None, 1, 2 ** 25, None) == -3
    for code in (0, -1, -2, -3, -4, -5, -6):
        assert ha.strerror(code) and ha.strerror(code) != "unknown status"
    assert ha.strerror(-99) == "unknown status"


def test_misaligned_arrays_are_rejected_on_the_host(ha):
    """Tensors must start at a 16-byte boundary, float / index arrays at a 4-byte one; the check
    runs on the host before anything is enqueued (the addresses here are never dereferenced)."""
    sh = ha.make_shape(1, 1, 1024, 64, 0)
    p = ha.make_params(64, 64, 7)
    ok = 0x7F0000000000
    fwd = ha.lib().hyperattn_forward
    assert fwd(ok + 8, ok, ok, ok, ok, ctypes.byref(sh), ctypes.byref(p), ok, 1 << 30, None) == -6
    assert fwd(ok, ok, ok + 2, ok, ok, ctypes.byref(sh), ctypes.byref(p), ok, 1 << 30, None) == -6
    assert fwd(ok, ok, ok, ok, ok + 2, ctypes.byref(sh), ctypes.byref(p), ok, 1 << 30, None) == -6
    assert ha.lib().exact_attn_forward(ok, ok + 4, ok, ok, ok, ctypes.byref(sh), 0, None) == -6
    assert ha.lib().ha_lsh_hash(ok + 4, ok, 10, 64, 0, ok, 7, None) == -6
    assert ha.lib().ha_seg_sort(ok, ok + 1, ok, 1, 16, None) == -6
    assert "aligned" in ha.strerror(-6)


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_with_and_without_torchs_private_name(ha, monkeypatch, raw):
    """The current stream's handle, also from a torch whose private shortcut is gone."""
    from types import SimpleNamespace as NS
    fake = NS(_C=NS(_cuda_getCurrentRawStream=lambda device: 100 + device) if raw else NS(),
              cuda=NS(current_device=lambda: 3, current_stream=lambda: NS(cuda_stream=103)))
    monkeypatch.setattr(ha.binding, "_torch_module", fake)
    assert ha.binding._stream(None) == 103
    assert ha.binding._stream(NS(cuda_stream=7)) == 7


def test_product_package_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2310_05869_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower(), (dirpath, f)
