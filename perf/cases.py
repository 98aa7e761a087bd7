"""Work that a training program has this library do, for timing: optimizer steps through
`paper_2104_06069_amd.step.DeviceStep`, from lists of a few tensors, where a step is a handful of short
launches, to a flat buffer of 1.3e9 parameters.

A case is one pass over inputs that are resident in HBM:

  step "compress"  `period` consecutive compression-stage steps (Algorithm 1 lines 6-21), each with a
                   gradient of its own; with the variance in deferred form `period` steps are what it
                   takes until the variance array has been rewritten once, so every pass does the same
                   work.  What the other ranks send lies in the step's wire buffers beforehand.
  step "lamb"      one uncompressed LAMB step (eq. (1)), the warmup stage.

  form "compact"    1-bit momentum, errors in deferred form, ratio pass and update in one call, and for
                    period > 1 the variance in deferred form: what the README shows
  form "wait_free"  the same with OB_CFG_NO_BARRIERS, for programs that share the device
  form "plain"      DeviceStep's default arguments: every array of the state in its plain form

Tensor lists: BERT- and GPT-shaped ones (a word embedding, position table, and per block matrices,
biases and norms, tightly packed, so that tensors start and end anywhere), and `tensors` square ones.
"""
import math

import numpy as np
import torch

import paper_2104_06069_amd as ob
from paper_2104_06069_amd.step import DeviceStep

HYPER = dict(beta1=0.9, beta2=0.999, beta3=0.9, eta=1e-6, c_min=0.01, c_max=0.3, r_min=0.5,
             r_max=4.0, r_threshold=0.1, weight_decay=0.0)
LR = 1e-3
LOSS_SCALE = 1024.0      # of a binary16 gradient
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "none": None}


def _list(family, hidden, blocks, vocab, max_pos=512, ffn=0):
    return dict(family=family, hidden=hidden, ffn=ffn or 4 * hidden, blocks=blocks, vocab=vocab, max_pos=max_pos)


def _case(name, tensors, workers, step="compress", form="compact", period=4, grad="f32", x_copy="none",
          scaled=False, noise="normal"):
    return dict(name=name, step=step, form=form, period=period, workers=workers, grad=grad, x_copy=x_copy,
                scaled=scaled, noise=noise, **tensors)


MINI = _list("bert", 64, 2, 1000, 32)
BERT_BASE = _list("bert_fused_qkv", 768, 12, 30522)
BERT_LARGE = _list("bert", 1024, 24, 30528)
BERT_LARGE_FUSED_QKV = _list("bert_fused_qkv", 1024, 24, 30528)
GPT_1P3B = _list("gpt", 2048, 24, 50304, 2048)


def listed():
    return [
        # four 512x512 tensors among 4 workers, one step at a time: bound by launches and the host
        _case("tiny", _list("square", 512, 4, 0), 4, period=1),
        # a small model with tensors of 2 to 64000 elements; mixed precision with momentum scaling
        _case("mini_f16", MINI, 8, grad="f16", x_copy="f16", scaled=True, noise="student_t3"),
        # a model of 11 M parameters: between launch-bound and bandwidth-bound
        _case("small", _list("bert", 256, 4, 30522), 8),
        # the benchmark's models in its configuration
        _case("bert_base", BERT_BASE, 16, noise="layer_scaled"),
        _case("bert_large", BERT_LARGE, 64, noise="student_t3"),
        _case("gpt_1p3b", GPT_1P3B, 128, noise="sparse_layers"),
        # mixed precision with momentum scaling: how the large model is trained
        _case("bert_large_bf16", BERT_LARGE_FUSED_QKV, 64, grad="bf16", x_copy="bf16", scaled=True, noise="student_t3"),
        # more workers, and no kernel that waits for another workgroup
        _case("bert_large_w256_wait_free", BERT_LARGE, 256, form="wait_free", noise="student_t3"),
        # a program that takes DeviceStep as it comes, every array in its plain form
        _case("bert_base_plain", BERT_BASE, 16, form="plain", period=1, noise="layer_scaled"),
        # the warmup stage: a small ragged model in mixed precision, and the two large ones
        _case("lamb_small_f16", _list("bert", 192, 3, 8191, 256), 8, step="lamb", period=1, grad="f16", x_copy="f16"),
        _case("lamb_bert_large", BERT_LARGE, 64, step="lamb", period=1, noise="student_t3"),
        _case("lamb_gpt_1p3b_bf16", GPT_1P3B, 128, step="lamb", period=1, grad="bf16", x_copy="bf16", noise="sparse_layers"),
    ]


def draw(rng):
    """A model of 1e5 to 1.3e9 parameters, log-uniformly, with any number of workers and options."""
    while True:
        target = math.exp(rng.uniform(math.log(1e5), math.log(1.3e9)))
        family = rng.choice(["bert", "bert_fused_qkv", "gpt", "square"])
        if family == "square":
            blocks = rng.randint(2, 24)
            t = _list(family, max(16, round(math.sqrt(target / blocks))), blocks, 0)
        else:
            blocks = rng.choice([1, 2, 3, 4, 6, 8, 12, 18, 24])
            vocab = rng.choice([50304, 30522, 30528, rng.randint(300, 30000)])
            max_pos = rng.choice([32, 128, 512, 1000, 2048])
            # 12 hidden^2 per block and the embedding rows
            rows = vocab + max_pos
            h = (-rows + math.sqrt(rows * rows + 48.0 * blocks * target)) / (24.0 * blocks)
            h = round(h / 64) * 64 if h >= 256 else round(h)
            t = _list(family, max(16, h), blocks, vocab, max_pos)
        n = sum(_sizes(t))
        if 5e4 <= n <= 1.31e9:
            break
    step = rng.choice(["compress", "compress", "compress", "lamb"])
    form = rng.choice(["compact", "compact", "compact", "wait_free", "plain"])
    period = 1 if step == "lamb" or form == "plain" else rng.choice([1, 2, 4, 4]) if form == "compact" else rng.choice([2, 4])
    grad = rng.choice(["f32", "f32", "bf16", "f16"])
    workers = max(1, min(256, round(math.exp(rng.uniform(0.0, math.log(256.0))))))
    c = _case("", t, workers, step=step, form=form, period=period, grad=grad,
              x_copy=rng.choice(["none", grad]) if grad != "f32" else "none", scaled=rng.random() < 0.4,
              noise=rng.choice(["normal", "student_t3", "layer_scaled", "sparse_layers"]))
    del c["name"]
    return c


def _sizes(case):
    """Elements of each tensor, in list order."""
    H, F, V, P = case["hidden"], case["ffn"], case["vocab"], case["max_pos"]
    if case["family"] == "square":
        return [H * H] * case["blocks"]
    if case["family"] == "gpt":
        t = [V * H, P * H]
        for _ in range(case["blocks"]):
            t += [3 * H * H, 3 * H, H * H, H, H, H, H * F, F, F * H, H, H, H]
        return t + [H, H]
    t = [V * H, P * H, 2 * H, H, H]
    for _ in range(case["blocks"]):
        t += [3 * H * H, 3 * H] if case["family"] == "bert_fused_qkv" else [H * H, H] * 3
        t += [H * H, H, H, H, H * F, F, F * H, H, H, H]
    return t + [H * H, H, H * H, H, H, H, V, 2 * H, 2]


class _Inputs:
    """Arrays drawn on the device from the seed; the padding of every array is zero."""

    def __init__(self, sizes, n_pad, seed):
        self.sizes, self.n, self.n_pad = sizes, sum(sizes), n_pad
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.host = np.random.default_rng(seed)

    def normal(self, sigma):
        a = torch.randn(self.n_pad, generator=self.gen, device="cuda").mul_(sigma)
        a[self.n:] = 0
        return a

    def gradient(self, noise, dtype):
        g = self.normal(1e-3)
        if noise == "student_t3":
            chi = torch.zeros_like(g)
            for _ in range(3):
                w = torch.randn(self.n_pad, generator=self.gen, device="cuda")
                chi.addcmul_(w, w)
            g.div_(chi.div_(3.0).sqrt_())
        elif noise != "normal":     # a magnitude of its own per tensor, or hardly any gradient in a few of them
            L = len(self.sizes)
            kappa = np.random.default_rng(L).uniform(0.1, 10.0, L) if noise == "layer_scaled" else np.ones(L)
            if noise == "sparse_layers":
                kappa[:: 100] = 1e-6
            at = 0
            for k, s in zip(kappa.tolist(), self.sizes):
                if k != 1.0:
                    g[at:at + s].mul_(k)
                at += s
        if dtype == torch.float16:
            g.mul_(LOSS_SCALE)
        return g.to(dtype)

    def words(self, n):
        return torch.randint(-2 ** 31, 2 ** 31, (n,), generator=self.gen, device="cuda", dtype=torch.int32)

    def scales(self, n):
        return torch.from_numpy((1e-4 * self.host.uniform(0.5, 1.5, n)).astype(np.float32))


def prepare(case, seed):
    sizes = _sizes(case)
    offsets = np.concatenate([[0], np.cumsum(np.array(sizes, dtype=np.int64))])
    W, plain, lamb = case["workers"], case["form"] == "plain", case["step"] == "lamb"
    args = {} if plain else dict(packed_momentum=True, fused_apply=True, deferred_error=True,
                                 deferred_variance=case["period"] if case["period"] > 1 else 0)
    ds = DeviceStep(offsets, W, W // 2, x_lp_dtype=DTYPES[case["x_copy"]],
                    grad_scale=1.0 / LOSS_SCALE if case["grad"] == "f16" else 1.0,
                    flags=ob.OB_CFG_NO_BARRIERS if case["form"] == "wait_free" else 0, **args, **HYPER)
    a = _Inputs(sizes, ds.n_pad, seed)
    ds.t["m"].copy_(a.normal(1e-4))
    v = a.normal(1e-4).abs_().add_(1e-8)
    v[a.n:] = 0
    ds.load_state(dict(x=a.normal(0.02), m=ds.t["m"], v_fresh=v, v_frozen=v,
                       c_avg=a.host.uniform(0.5, 2.0, ds.L).astype(np.float32)))
    del v
    grads = [a.gradient(case["noise"], DTYPES[case["grad"]]) for _ in range(case["period"])]
    if not lamb:
        # the end of warmup and the first steps after it: from then on the momentum (compact forms) lies
        # in the wire buffers, each of which has been received into once
        if case["scaled"]:
            ds.momentum_scale()
        ds.packed_in.copy_(a.words(ds.packed_in.numel()))
        ds.scales_in.copy_(a.scales(W))
        for t in range(1 + ds.graph_period):
            ds.begin_step()
            ds.packed_all.copy_(a.words(ds.packed_all.numel()))
            ds.server_scales.copy_(a.scales(W))
            ds.step(grads[t % len(grads)], LR)
    torch.cuda.synchronize()
    return dict(ds=ds, grads=grads, lamb=lamb)


def run(state):
    ds = state["ds"]
    if state["lamb"]:
        ds.warmup_step(state["grads"][0], LR)
        out = {k: ds.t[k] for k in ("x", "m", "v_fresh", "c_avg", "coeff_c")}
    else:
        for g in state["grads"]:
            ds.begin_step()
            ds.step(g, LR)
        out = {k: ds.t[k] for k in ("x", "err_worker", "err_server", "r_prev", "coeff_c")}
        out.update(v_fresh=ds.v_fresh_dense(), packed_local=ds.packed_local, scales_local=ds.scales_local,
                   packed_all=ds.packed_all, server_scales=ds.server_scales)
        if not ds.packed_momentum:
            out["m"] = ds.t["m"]
    if ds.x_lp is not None:
        out["x_lp"] = ds.x_lp
    return out


def work(case):
    n, g, copy = sum(_sizes(case)), 4 if case["grad"] == "f32" else 2, 2 if case["x_copy"] != "none" else 0
    if case["step"] == "lamb":
        # gradient and 16-bit copy; m, v and x read and written
        return {"bytes": n * (g + copy + 24.0), "flops": 20.0 * n}
    # each step: the gradient and the 16-bit copy; error and x read and written; v_frozen and v_fresh
    # read; the words of this worker, of what its server receives and of what all servers send, and
    # the momentum; once per pass: v_fresh written
    momentum = 8.0 if case["form"] == "plain" else 0.125
    per_step = g + copy + 16.0 + 8.0 + 0.375 + momentum
    return {"bytes": n * (case["period"] * per_step + 4.0), "flops": 30.0 * n * case["period"]}


def tolerance(case):
    # The sums of squares are the only results that depend on an order of summation; they are
    # accumulated in binary64 and rounded once, so that another order can move a scale or norm by one
    # binary32 unit (6e-8) about once in 1e8; an element within that of zero may then change its sign.
    return {"rel": 5e-7, "max": 2e-5, "differ": 1e-6}
