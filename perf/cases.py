"""What the speed of this framework is measured on.

Every case is one pass through the public entry points of `paper_2310_05869_amd`,
as a program that uses the framework makes it: tensors resident on the GPU,
workspaces and outputs allocated once and kept, one call (forward) or two
(forward and backward) per pass.

`pass` of a case:
  fwd          hyperattn_forward
  train        hyperattn_forward with the unrounded output (bf16) + hyperattn_backward
  exact        exact_attn_forward
  exact_train  exact_attn_forward with the unrounded output (bf16) + exact_attn_backward
  alg2         hyperattn_forward_alg2 (Algorithm 2's caps; value sampling where `vnorm`)

`law` of the inputs:
  iid      Q, K, V ~ N(0, 1) / d^(1/4): the softmax scale folded into Q and K
  mixture  Q, K from 64 Gaussian clusters per head (uneven buckets, scores up to
           +-250), V ~ N(0, 1)
"""
import math

import torch

import paper_2310_05869_amd as ha


def _case(name, kind, B, H, n, d, dtype="bf16", law="iid", b=256, m=256, r=7, causal=False, n_min=4096, **more):
    return dict(name=name, **{"pass": kind}, B=B, H=H, n=n, d=d, dtype=dtype, law=law, b=b, m=m, r=r, causal=causal,
                n_min=n_min, **more)


def listed():
    return [
        # the fp32 configuration: one small head, where a call is its launches
        _case("fwd_fp32_n1k", "fwd", 1, 1, 1024, 64, dtype="fp32", b=64, m=64),
        # the short end of the 12-head, d = 64 layer sweep: serving-size latency
        _case("fwd_n4k_h12_d64", "fwd", 1, 12, 4096, 64),
        # the same layer with one split of the causal recursion
        _case("fwd_causal_n8k_h12_d64", "fwd", 1, 12, 8192, 64, causal=True),
        # sizes that no tile divides: block, sample count, heads and batch all odd
        _case("fwd_ragged_n6300_d128", "fwd", 3, 5, 6300, 128, b=100, m=77, r=6),
        # a 32-head long-context layer, unmasked (encoder, or prefill without a mask)
        _case("fwd_n32k_h32_d128", "fwd", 1, 32, 32768, 128),
        # clustered queries and keys, twice the samples, batch of two: the largest unmasked forward
        _case("fwd_mixture_n65k_d64", "fwd", 2, 32, 65536, 64, law="mixture", m=512),
        # long-context causal prefill of one layer: the benchmark's default
        _case("fwd_causal_n131k_h32_d128", "fwd", 1, 32, 131072, 128, causal=True),
        # Algorithm 2 as printed (caps), the option beside the main form, at the same layer
        _case("alg2_n32k_h32_d128", "alg2", 1, 32, 32768, 128, cap_scale=8.0, kappa=1.2, vnorm=False),
        # one training step's attention, forward and backward: a middle point of the sweep
        _case("train_n16k_h12_d64", "train", 1, 12, 16384, 64),
        # the same for fp32 tensors, causal, with small blocks
        _case("train_fp32_causal_n4k_d64", "train", 1, 4, 4096, 64, dtype="fp32", b=64, m=64, causal=True, n_min=1024),
        # exact attention with gradients at a length that no tile divides: the base the speed-ups are quoted against
        _case("exact_train_causal_n5000_d128", "exact_train", 1, 12, 5000, 128, causal=True),
        # the long-context causal layer in training: the largest case
        _case("train_causal_n131k_h32_d128", "train", 1, 32, 131072, 128, causal=True),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ones' ranges: both dtypes, both head sizes, masked and not, blocks of 32 to 512,
    up to 1024 samples, 1 to 64 heads in all, lengths from hundreds to 131072, at no more work than the largest."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["fwd", "fwd", "fwd", "train", "train", "exact", "exact_train", "alg2"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        d = rng.choice([64, 128])
        B, H = rng.choice([1, 1, 2, 3]), _log_int(rng, 1, 32)
        causal = rng.random() < 0.5
        b = rng.choice([64, 128, 256, 256, _log_int(rng, 32, 512)])
        m = rng.choice([64, 256, 256, _log_int(rng, 8, 1024)])
        r = rng.choice([7, 7, 6, 8])
        c = {"pass": kind, "B": B, "H": H, "d": d, "dtype": dtype, "b": b, "m": m, "r": r, "causal": causal, "n_min": 4096}
        c["law"] = "mixture" if kind == "fwd" and dtype == "bf16" and rng.random() < 0.3 else "iid"
        if kind in ("exact", "exact_train"):
            c["n"] = _log_int(rng, 500, 4000 if dtype == "fp32" else 16384)
        else:
            top = 16384 if dtype == "fp32" else 131072
            if causal:
                c["n_min"] = b * max(1, _log_int(rng, 512, 4096) // b)
                c["n"] = c["n_min"] << rng.randint(1, 5)
            else:
                c["n"] = b * max(2, _log_int(rng, 1024, top) // b)
            if c["n"] > top:
                continue
        if kind == "alg2":
            c.update(cap_scale=8.0, kappa=1.2, vnorm=rng.random() < 0.5)
            if dtype == "fp32" and c["n"] > 4096:
                continue
        # fp32 runs without the bf16 matrix cores: about a sixteenth of their rate
        if work(c)["flops"] * (16 if dtype == "fp32" else 1) <= most and B * H * c["n"] <= 1 << 22:
            return c


def _inputs(c, seed):
    """Q, K, V and the output's gradient, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, H, n, d = c["B"], c["H"], c["n"], c["d"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def randn(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    if c["law"] == "iid":
        qkv = [(randn(B, H, n, d) * d ** -0.25).to(dt) for _ in range(3)]
    else:
        centres = 2.0 * randn(B * H, 64, d)
        weight = torch.arange(1, 65, device="cuda", dtype=torch.float32) ** -1.1
        qkv = []
        for _ in range(2):
            which = torch.multinomial((weight / weight.sum()).expand(B * H, 64), n, replacement=True, generator=g)
            rows = torch.gather(centres, 1, which[:, :, None].expand(B * H, n, d))
            qkv.append((rows + 0.5 * randn(B * H, n, d)).view(B, H, n, d).to(dt))
        qkv.append(randn(B, H, n, d).to(dt))
    d_out = randn(B, H, n, d).to(dt) if c["pass"] in ("train", "exact_train") else None
    return qkv, d_out


def prepare(case, seed):
    c = dict(case)
    (Q, K, V), d_out = _inputs(c, seed)
    B, H, n, d = Q.shape
    s = {"c": c, "Q": Q, "K": K, "V": V, "d_out": d_out, "seed": seed, "out": torch.empty_like(Q),
         "lse": torch.empty((B, H, n), dtype=torch.float32, device="cuda")}
    shape = ha.make_shape(B, H, n, d, ha.HA_BF16 if c["dtype"] == "bf16" else ha.HA_FP32)
    params = ha.make_params(c["b"], c["m"], c["r"], c["causal"], c["n_min"], seed)
    kind = c["pass"]
    if kind in ("train", "exact_train"):
        s["out_f32"] = torch.empty(Q.shape, dtype=torch.float32, device="cuda") if c["dtype"] == "bf16" else None
        s["grads"] = tuple(torch.empty_like(Q) for _ in range(3))
    if kind in ("fwd", "train"):
        s["workspace"] = ha.alloc_workspace(shape, params)
    if kind == "train":
        s["bwd_workspace"] = ha.alloc_backward_workspace(shape, params)
    if kind == "exact_train":
        s["workspace"] = torch.empty(int(ha.lib().exact_attn_backward_workspace_bytes(shape)), dtype=torch.uint8, device="cuda")
    if kind == "alg2":
        s["workspace"] = torch.empty(int(ha.binding.ha_alg2_workspace_layout(shape, params).total_bytes), dtype=torch.uint8,
                                     device="cuda")
    return s


def run(s):
    c, kind = s["c"], s["c"]["pass"]
    Q, K, V, out, lse = s["Q"], s["K"], s["V"], s["out"], s["lse"]
    if kind in ("exact", "exact_train"):
        ha.exact_attn_forward(Q, K, V, causal=c["causal"], out=out, lse=lse, out_f32=s.get("out_f32"))
        if kind == "exact":
            return {"out": out, "lse": lse}
        dQ, dK, dV = ha.exact_attn_backward(Q, K, V, out, lse, s["d_out"], causal=c["causal"], workspace=s["workspace"],
                                            grads=s["grads"], out_f32=s["out_f32"])
        return {"out": out, "lse": lse, "dQ": dQ, "dK": dK, "dV": dV}
    alg = dict(causal=c["causal"], n_min=c["n_min"], seed=s["seed"])
    if kind == "alg2":
        ha.hyperattn_forward_alg2(Q, K, V, c["b"], c["m"], c["r"], cap_scale=c["cap_scale"], kappa=c["kappa"],
                                  vnorm_sampling=c["vnorm"], workspace=s["workspace"], out=out, lse=lse, **alg)
        return {"out": out, "lse": lse}
    ha.hyperattn_forward(Q, K, V, c["b"], c["m"], c["r"], workspace=s["workspace"], out=out, lse=lse,
                         out_f32=s.get("out_f32"), **alg)
    if kind == "fwd":
        return {"out": out, "lse": lse}
    dQ, dK, dV = ha.hyperattn_backward(Q, K, V, out, lse, s["d_out"], c["b"], c["m"], c["r"], fwd_workspace=s["workspace"],
                                       bwd_workspace=s["bwd_workspace"], grads=s["grads"], out_f32=s["out_f32"], **alg)
    return {"out": out, "lse": lse, "dQ": dQ, "dK": dK, "dV": dV}


def work(case):
    """Bytes: every input tensor read once, every result written once. Flops: two products (4 d flop) for every
    (query, key) pair that the method visits, five more (10 d) where gradients are taken: b + m keys per query row of
    every node, the causal half of every exact block; Algorithm 2's rows of T against every key of their node."""
    c = case
    kind, n, d, BH = c["pass"], c["n"], c["d"], c["B"] * c["H"]
    train = kind in ("train", "exact_train")
    if kind in ("exact", "exact_train"):
        pairs, tau = n * (n + 1) / 2 if c["causal"] else n * n, 0
    else:
        length = c["n_min"] if c["causal"] and n > c["n_min"] else n
        levels = int(round(math.log2(n / length))) if c["causal"] else 0
        rows = levels * (n // 2) if c["causal"] else n
        pairs = rows * (c["b"] + c["m"]) + ((n // length) * length * (length + 1) / 2 if c["causal"] else 0)
        # T: m rows of every node against its keys; a level's nodes hold n/2 keys together
        tau = c["m"] * rows if kind == "alg2" else 0
    esz = 2 if c["dtype"] == "bf16" else 4
    return {"bytes": BH * n * ((4 + (4 if train else 0)) * d * esz + 4),
            "flops": BH * (pairs * (14 if train else 4) * d + tau * 2 * d)}


def tolerance(case):
    """About four times what the paths differ by from the fp64 oracle (one to two heads of n = 1024 ... 8192, both head
    sizes, masked and not, both laws): bf16 1.7e-3 to 2.7e-3 relative, single elements up to 0.07 of the root mean square
    (one rounding of the result, softmax weights that enter the products in bf16); fp32 3e-7 to 9e-7, elements up to 3e-5."""
    return {"rel": 1e-2, "max": 0.3} if case["dtype"] == "bf16" else {"rel": 3e-6, "max": 1e-4}
