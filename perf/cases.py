"""What a user of the library has it do, as cases that can be timed and compared.

Four kinds of call, through the public entry points of paper_2310_01655_amd:

  forward    psf_causal_attn_fwd: the layer in evaluation, or a prompt's rows
  noncausal  psf_noncausal_attn_fwd: the same layer without a mask (an encoder)
  train      causal_polysketch_attention under autograd: output, then the gradients of Q, K, V
             (and of the networks' parameters with learned sketches)
  generate   psf_decode_prefill on a prompt, then psf_decode_step token by token

Sizes are those of the library's workloads (inputs.CONFIGS, the sweep over contexts 8k to 64k,
the serving shape of bench.py) and shorter or odd ones between them: contexts from 512, batches
and block sizes that are no round numbers, fp32 storage as a numerical check uses it.
"""
import math

import torch

from paper_2310_01655_amd import autograd
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs

_BASE = dict(kind="forward", batch=1, heads=12, n=1024, d=64, p=4, r=64, b=1024, dtype="bf16",
             local="exact", per_head=False, learned=False, dist="normal", prompt=0, tokens=0)


def _case(**changes):
    unknown = set(changes) - set(_BASE) - {"name"}
    assert not unknown, unknown
    return {**_BASE, **changes}


def listed():
    return [
        # one sequence being generated: latency of the single step, short prompt that ends inside
        # a block
        _case(name="generate_one", kind="generate", batch=1, n=32768, prompt=1500, tokens=24),
        # a server's batch: 64 sequences, 8k prompts; the tokens cross the end of a block, so
        # that one fold of a completed block is among them
        _case(name="generate_batch64", kind="generate", batch=64, n=32768, prompt=8180, tokens=24),
        # the numerical check: one head in fp32 with the small sketch (config 1)
        _case(name="forward_fp32_head", heads=1, n=1024, r=16, b=128, dtype="f32"),
        # the shortest context of the paper's tables, one sequence: launches and latency count
        _case(name="forward_short", n=512, r=32, b=256),
        # sequences whose length has no factor of 256: blocks of 200 tokens
        _case(name="forward_odd_blocks", batch=3, n=3000, r=32, b=200),
        # long context, the headline workload (config 3)
        _case(name="forward_long", batch=2, n=32768),
        # encoder: the layer without a mask
        _case(name="noncausal_medium", kind="noncausal", batch=5, n=4096, r=32, b=256),
        # training a GPT-2-small layer at 4k (config 2)
        _case(name="train_medium", kind="train", batch=8, n=4096, r=32, b=256, per_head=True),
        # training with sequences of odd length, blocks of 150 tokens
        _case(name="train_odd_blocks", kind="train", batch=2, n=1950, r=32, b=150),
        # training at long context (config 3)
        _case(name="train_long", kind="train", batch=2, n=32768),
        # training with learned sketches, parameters of the networks included
        _case(name="train_learned", kind="train", batch=4, n=8192, r=32, b=1024, learned=True),
        # training with wide heads and degree 8, heavy-tailed rows (config 5)
        _case(name="train_wide", kind="train", batch=1, heads=16, n=16384, d=128, p=8, b=512, dist="student_t3"),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["forward"] * 5 + ["train"] * 5 + ["generate"] * 3 + ["noncausal"] * 2)
    heads = rng.choice([1, 3, 8, 12, 12, 12, 16])
    dtype = "f32" if kind != "generate" and rng.random() < 0.15 else "bf16"
    p, d = rng.choice([4] * 7 + [8] * 2 + [2]), 128 if rng.random() < 0.2 else 64
    if p == 2:
        d = 64
    r = rng.choice([16, 32, 64]) if dtype == "f32" else rng.choice([32, 64])
    learned = kind in ("forward", "train") and p == 4 and d == 64 and dtype == "bf16" and rng.random() < 0.25
    odd = not learned and rng.random() < 0.35
    b = _log_int(rng, 48, 1000) if odd else rng.choice([256, 512, 1024])
    per_head = rng.random() < 0.25
    local = "sketch" if not learned and d == 64 and rng.random() < 0.15 else "exact"
    dist = rng.choice(["normal", "normal", "student_t3"])
    if kind == "generate":
        tokens, prompt = rng.randint(12, 40), _log_int(rng, 64, 12000)
        return _case(kind=kind, batch=_log_int(rng, 1, 96), heads=heads, n=16384 // b * b, d=d, p=p, r=r, b=b,
                     local=local, per_head=per_head, dist=dist, prompt=prompt, tokens=tokens)
    blocks = max(1, round(_log_int(rng, 512, 65536) / b))
    case = _case(kind=kind, batch=_log_int(rng, 1, 64), heads=heads, n=blocks * b, d=d, p=p, r=r, b=b, dtype=dtype,
                 local=local, per_head=per_head, learned=learned, dist=dist)
    # odd blocks and fp32 checks are smaller jobs than the long training runs
    most = 0.022e12 if odd or dtype == "f32" else 0.25e12 if learned else 1.0e12
    while work(case)["flops"] > most:
        if case["batch"] > 1:
            case["batch"] -= (case["batch"] + 2) // 3
        elif case["n"] > 2 * b:
            case["n"] = (case["n"] // b + 1) // 2 * b
        else:
            case["heads"] = max(1, case["heads"] // 2)
    return case


def _desc(c):
    return psf.make_desc(c["batch"], c["heads"], c["n"], c["d"], c["p"], c["r"], c["b"], c["dtype"],
                         local=psf.LOCAL_SKETCH if c["local"] == "sketch" else psf.LOCAL_EXACT,
                         per_head=c["per_head"], learned=c["learned"])


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 11)
    td = inputs.torch_dtype(c["dtype"])

    def rows(n, unit):
        x = torch.randn(c["batch"], c["heads"], n, c["d"], generator=g, device="cuda")
        if unit:
            if c["dist"] == "student_t3":                     # t = normal / sqrt(chi^2_3 / 3)
                chi = torch.zeros_like(x)
                for _ in range(3):
                    chi += torch.randn(x.shape, generator=g, device="cuda").square_()
                x /= chi.div_(3.0).sqrt_()
            x /= x.norm(dim=-1, keepdim=True)                 # rows reach the layer normalised
        return x.to(td)

    if c["p"] == 2:
        G = None
    elif c["learned"]:
        G = inputs.make_learned_params(c["heads"], c["d"], c["r"], c["p"], per_head=c["per_head"], seed=seed,
                                       dtype=c["dtype"]).cuda()
    else:
        sets = c["heads"] if c["per_head"] else 1
        G = torch.randn(sets, inputs.g_len(c["d"], c["r"], c["p"]), generator=g, device="cuda").to(td)
    desc = _desc(c)
    s = {"case": c, "desc": desc, "G": G}
    if c["kind"] == "generate":
        s["K"], s["V"] = rows(c["prompt"], True), rows(c["prompt"], False)
        s["steps"] = [(rows(1, True), rows(1, True), rows(1, False)) for _ in range(c["tokens"])]
        s["state"] = psf.decode_new_state(desc)
        return s
    s["Q"], s["K"], s["V"] = rows(c["n"], True), rows(c["n"], True), rows(c["n"], False)
    if c["kind"] == "train":
        for name in ("Q", "K", "V"):
            s[name].requires_grad_(True)
        if c["learned"]:
            G.requires_grad_(True)
        s["dO"] = rows(c["n"], False)
    else:
        s["workspace"] = (psf.alloc_noncausal_workspace if c["kind"] == "noncausal" else psf.alloc_workspace)(desc)
    return s


def run(state):
    s, c, desc = state, state["case"], state["desc"]
    if c["kind"] == "forward":
        return psf.psf_causal_attn_fwd(desc, s["Q"], s["K"], s["V"], s["G"], workspace=s["workspace"])
    if c["kind"] == "noncausal":
        return psf.psf_noncausal_attn_fwd(desc, s["Q"], s["K"], s["V"], s["G"], workspace=s["workspace"])
    if c["kind"] == "train":
        O = autograd.causal_polysketch_attention(
            s["Q"], s["K"], s["V"], s["G"], c["p"], c["r"], c["b"], local=desc.local, per_head=c["per_head"],
            learned=c["learned"])
        wrt = [s["Q"], s["K"], s["V"]] + ([s["G"]] if c["learned"] else [])
        return [O.detach(), *torch.autograd.grad(O, wrt, s["dO"])]
    psf.psf_decode_prefill(desc, s["K"], s["V"], s["G"], s["state"])      # starts from a reset state
    return [psf.psf_decode_step(desc, q, k, v, s["G"], c["prompt"] + i, s["state"])
            for i, (q, k, v) in enumerate(s["steps"])]


def _sketch_flops(c):
    """Flops of m(x) for one row."""
    d, r, p = c["d"], c["r"], c["p"]
    if p == 2:
        return 0
    if c["learned"]:
        net = lambda win: 2 * (win * 8 * r + 24 * r * r)
        return (p // 2) * net(d) + (p // 2 - 2) * net(r)
    return p // 2 * 2 * d * r + (p // 2 - 2) * 2 * r * r


def work(case):
    """Multiply-add = 2.  Features are counted as the distinct pairs of the symmetric phi', the
    in-block part as its causal triangle."""
    c = case
    units, n, d, b = c["batch"] * c["heads"], c["n"], c["d"], c["b"]
    m = d if c["p"] == 2 else c["r"]
    pairs = m * (m + 1) // 2
    size = 4 if c["dtype"] == "f32" else 2
    sets = c["heads"] if c["per_head"] else 1
    g_bytes = size * sets * (0 if c["p"] == 2 else
                             inputs.learned_len(d, c["r"], c["p"]) if c["learned"] else inputs.g_len(d, c["r"], c["p"]))
    sketch = _sketch_flops(c)
    state = lambda rows: 2 * rows * pairs * (d + 1)             # one product with [V | 1] or with the state
    if c["kind"] == "generate":
        steps, prompt = c["tokens"], c["prompt"]
        cached = sum((prompt + i) % b for i in range(steps))
        state_bytes = pairs * (d * size + 4)                    # read by every token
        return {"bytes": units * (2 * prompt * d * size + steps * (4 * d * size + state_bytes) +
                                  cached * 2 * d * size + state_bytes) + g_bytes,
                "flops": units * ((prompt + 2 * steps) * sketch + state(prompt + steps) + 4 * cached * d)}
    if c["kind"] == "noncausal":
        return {"bytes": units * n * 4 * d * size + g_bytes, "flops": units * (2 * n * sketch + 2 * state(n))}
    far = n - b                                                 # rows with a block before / after them
    near = n * (b + 1) // 2                                     # pairs inside blocks
    forward = 2 * n * sketch + 2 * state(far) + near * 2 * (2 * d + 1)
    if c["kind"] == "forward":
        return {"bytes": units * n * 4 * d * size + g_bytes, "flops": units * forward}
    # backward: the mirror state, its three contractions (dm(Q), dm(K), dV), five products per
    # pair inside blocks (scores, weight gradients, dQ, dK, dV), the sketches' reverse
    backward = 4 * state(far) + near * 2 * 5 * d + 2 * n * (2 if c["learned"] else 1) * sketch
    return {"bytes": units * n * 8 * d * size + g_bytes * (3 if c["learned"] else 1),
            "flops": units * (forward + backward)}


def tolerance(case):
    """About four times the distance to a float64 evaluation: 2e-6 in fp32 storage, 3e-3 to 5e-3
    where the operands of the products are bf16 (5e-3 to 7e-3 for gradients).  bf16 storage
    with odd blocks is computed in fp32 and differs by the rounding of the result."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] != "generate" and case["b"] % 256:
        return {"rel": 2e-3, "max": 5e-2}
    return {"rel": 2e-2 if case["kind"] == "train" else 1.2e-2}
