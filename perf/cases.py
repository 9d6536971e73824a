"""The work that a fine-tuning program has this library do, as cases that can be timed and compared.

A case is one layer at one batch size; a pass is what a training or evaluation program asks of that layer for one batch,
through the public entry points of `paper_2505_14742_amd.binding`:

    op "train"  quaff_linear_fwd_step, then quaff_linear_bwd_step (input gradient and LoRA weight gradients)
    op "fwd"    quaff_linear_fwd_step alone (evaluation; the forward half of a step with recomputation)
    op "bwd"    quaff_linear_bwd_step alone (the backward half)
    op "dx"     quaff_linear_bwd_dx alone (a layer whose adapter is frozen or absent: only the gradient passes through)
    op "calls"  the four separate calls with bf16 results: quaff_scale_update, quaff_quant_act, quaff_linear_fwd_bf16,
                quaff_linear_bwd_dx_bf16 (a program that keeps activations and gradients in bf16)

`side` = True hands quaff_linear_bwd_step a second stream.  Sizes: t tokens, c_in x c_out weight, n outlier channels,
LoRA rank r; `tail` = True draws heavy-tailed activations (Student-t with three degrees of freedom).
"""
import math

import torch

from paper_2505_14742_amd import binding as q

DEV = "cuda"


def listed():
    return [
        # the smallest layer of the benchmark configurations: one short sequence, no adapter, evaluation
        _case("fwd_256x512x512", "fwd", 256, 512, 512, 8, 0, gamma=0.9),
        # a handful of tokens through a trained layer (scoring short prompts, generating in a batch of 16)
        _case("fwd_16x3072x9216", "fwd", 16, 3072, 9216, 31, 16),
        # a micro-batch of one 512-token sequence (gradient accumulation), hidden -> hidden projection
        _case("train_512x3072x3072", "train", 512, 3072, 3072, 31, 16),
        # the usual batch of four 512-token sequences: fused query/key/value projection, weight gradients on a second
        # stream as a training loop that has one passes it
        _case("train_2048x3072x9216", "train", 2048, 3072, 9216, 31, 16, side=True),
        # the same batch, MLP down-projection (long rows in, 0.5 % of them outliers), forward
        _case("fwd_2048x8192x3072", "fwd", 2048, 8192, 3072, 41, 16),
        # the same batch, fused gate/up projection: only the gradient passes through (adapter frozen)
        _case("dx_2048x3072x16384", "dx", 2048, 3072, 16384, 31, 16),
        # the paper's own outlier budget, 10 % of the channels of a down-projection, forward
        _case("fwd_2048x8192x3072_n819", "fwd", 2048, 8192, 3072, 819, 16),
        # hidden -> hidden projection with bf16 results through the separate calls
        _case("calls_2048x3072x3072", "calls", 2048, 3072, 3072, 31, 16),
        # an adapter of rank 64 on a 7B-sized hidden -> hidden projection, eight 512-token sequences
        _case("train_4096x4096x4096_r64", "train", 4096, 4096, 4096, 40, 64),
        # the backward half of a 7B-sized gate projection at rank 64
        _case("bwd_4096x4096x11008_r64", "bwd", 4096, 4096, 11008, 40, 64),
        # packed sequences of uneven length and a model whose widths are not multiples of a tile
        _case("train_1003x1040x2064_r32", "train", 1003, 1040, 2064, 13, 32),
        # long sequences, heavy-tailed activations: a 13B-sized gate projection, four 4096-token sequences
        _case("train_16384x5120x13824", "train", 16384, 5120, 13824, 64, 16, tail=True),
    ]


def draw(rng):
    """One more case of the same ranges: any token count from one to the longest batch, widths from 208 to 16384 (most
    models have multiples of 128, some of 64, a few only of 16), no outliers up to the paper's 10 %, every rank."""
    while True:
        op = rng.choice(["train", "train", "fwd", "fwd", "bwd", "dx", "calls"])
        t = _log(rng, 1, 16384)
        gran = rng.choice([128, 128, 128, 64, 64, 16])
        c_in, c_out = (max(gran, gran * round(_log(rng, 208, 16384) / gran)) for _ in range(2))
        n = rng.choice([0, 1, 2, 2, 2, 3])
        n = 0 if n == 0 else _log(rng, 1, min(64, c_in // 16)) if n < 3 else _log(rng, 1, c_in // 10)
        r = rng.choice([0, 16, 16, 16, 32, 48, 64, 64])
        if op in ("train", "bwd") and r == 0:
            continue
        if op == "calls" and (gran == 16 or n > 128):
            continue
        if t * c_in * c_out > 6e11:       # no more than half of the largest listed case
            continue
        c = _case("", op, t, c_in, c_out, n, r, gamma=rng.choice([0.2, 0.2, 0.9]),
                  side=op in ("train", "bwd") and rng.random() < 0.3, tail=rng.random() < 0.25)
        del c["name"]
        return c


def prepare(case, seed):
    t, c_in, c_out, n, r = (case[k] for k in ("t", "c_in", "c_out", "n", "r"))
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + t + c_in + c_out)
    f32, i8, bf16 = torch.float32, torch.int8, torch.bfloat16

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=DEV, dtype=f32)

    S = {"case": case}
    # frozen weight, outlier channels and adapter, prepared once per layer as a program does when it loads a model
    W = normal(c_in, c_out).mul_(0.02)
    O = torch.randperm(c_in, generator=gen, device=DEV)[:n].sort().values.to(torch.int32) if n else None
    S["O"] = O
    S["A"] = normal(c_in, r).div_(math.sqrt(c_in)).to(bf16) if r else None
    S["B"] = normal(r, c_out).mul_(0.02).to(bf16) if r else None
    n_p = q.padded_outliers(n)
    S["Wq"] = torch.empty(q.packed_weight_bytes(c_in, c_out), dtype=i8, device=DEV)
    S["delta_w"] = torch.empty(c_out, dtype=f32, device=DEV)
    S["W_O"] = torch.empty(n, c_out, dtype=f32, device=DEV) if n else None
    S["wmax"] = torch.empty(n, dtype=f32, device=DEV) if n else None
    q.prepare_weight(W, O, S["Wq"], S["delta_w"], S["W_O"], S["wmax"], None,
                     torch.empty(q.prepare_workspace_bytes(c_in, c_out), dtype=i8, device=DEV))
    del W
    # the batch: activations whose outlier channels are 20 to 100 times the others (50 to 500 with heavy tails)
    X = normal(t, c_in)
    if case["tail"]:
        X /= (sum(normal(t, c_in).square_() for _ in range(3)) / 3).sqrt_()
    if n:
        lo, hi = (50.0, 500.0) if case["tail"] else (20.0, 100.0)
        X[:, O.long()] *= lo * (hi / lo) ** torch.rand(n, generator=gen, device=DEV)
    S["X"] = X.to(bf16)
    del X
    if case["op"] != "fwd":
        S["dY"] = normal(t, c_out).mul_(2.0 ** -6).to(bf16)
    # per-layer state and buffers
    S["s"] = torch.ones(n, dtype=f32, device=DEV) if n else None
    S["colscale"] = torch.ones(c_in, dtype=f32, device=DEV)
    S["what"] = torch.zeros(c_out, n_p, dtype=i8, device=DEV) if n else None
    S["delta_what"] = torch.zeros(c_out, dtype=f32, device=DEV) if n else None
    S["Xq"] = torch.empty(t, c_in, dtype=i8, device=DEV)
    S["delta_x"] = torch.empty(t, dtype=f32, device=DEV)
    S["xq_O"] = torch.empty(t, n_p, dtype=i8, device=DEV) if n else None
    out = bf16 if case["op"] == "calls" else f32
    S["Y"] = torch.empty(t, c_out, dtype=out, device=DEV)
    S["dX"] = torch.empty(t, c_in, dtype=out, device=DEV)
    S["dA"] = torch.empty(c_in, r, dtype=f32, device=DEV)
    S["dB"] = torch.empty(r, c_out, dtype=f32, device=DEV)
    need = {
        "fwd": lambda: q.fwd_step_workspace_bytes(t, c_in, c_out, n, r),
        "train": lambda: max(q.fwd_step_workspace_bytes(t, c_in, c_out, n, r), q.bwd_step_workspace_bytes(t, c_in, c_out, r)),
        "bwd": lambda: q.bwd_step_workspace_bytes(t, c_in, c_out, r),
        "dx": lambda: q.workspace_bytes(t, c_in, c_out, n, r),
        "calls": lambda: q.workspace_bytes(t, c_in, c_out, n, r),
    }[case["op"]]()
    S["ws"] = torch.empty(need, dtype=i8, device=DEV)
    S["side"] = q.SideStream() if case["side"] else None
    return S


def run(S):
    op = S["case"]["op"]
    if op == "fwd":
        return _forward(S)
    if op == "bwd":
        return _backward(S)
    if op == "dx":
        return _input_gradient(S, False)
    if op == "calls":
        return {**_separate_forward(S), **_input_gradient(S, True)}
    return {**_forward(S), **_backward(S)}


def work(case):
    """Bytes and operations of a pass: X, dY, the weight codes, the retained outlier rows and the adapter read once in each
    direction, every output written once; multiply-adds of the integer products (int8) and of the adapter branch."""
    t, c_in, c_out, n, r, op = (case[k] for k in ("t", "c_in", "c_out", "n", "r", "op"))
    n_p = (n + 63) // 64 * 64
    el = 2 if op == "calls" else 4
    nbytes = flops = 0
    if op in ("fwd", "train", "calls"):
        nbytes += 2 * t * c_in + c_in * c_out + 4 * n * c_out + 2 * r * (c_in + c_out) + 4 * c_out
        nbytes += el * t * c_out + t * c_in + t * n_p + 4 * t + n_p * c_out + 4 * c_out
        flops += 2 * t * c_out * (c_in + n) + 2 * t * r * (c_in + c_out)
    if op in ("bwd", "train", "dx", "calls"):
        nbytes += 2 * t * c_out + c_in * c_out + 2 * r * (c_in + c_out) + 4 * c_out + el * t * c_in
        flops += 2 * t * c_out * c_in + 2 * t * r * (c_in + c_out)
    if op in ("bwd", "train"):
        nbytes += 2 * t * c_in + 4 * r * (c_in + c_out)
        flops += 2 * t * r * c_in + 2 * t * r * (c_in + c_out)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Codes and scales are exact.  fp32 results differ by the order of fp32 sums and by the 16 significant bits that the
    adapter's intermediate products are kept in; bf16 results where one rounds the other way.  Against the same pass in
    64 bits the library's own error is at most 1e-6 in Y and dX, 4e-6 in dA and dB (single values 1.5e-4) and, after
    rounding both to bf16, 4e-5 (single values one unit in the last place, 7.8e-3)."""
    if case["op"] == "calls":
        return {"rel": 1.6e-4, "max": 2.0 ** -6}
    if case["op"] in ("fwd", "dx"):
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 1.6e-5, "max": 6e-4}


def _case(name, op, t, c_in, c_out, n, r, gamma=0.2, side=False, tail=False):
    return {"name": name, "op": op, "t": t, "c_in": c_in, "c_out": c_out, "n": n, "r": r, "gamma": gamma, "side": side,
            "tail": tail}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _step_outputs(S):
    out = {"Y": S["Y"], "Xq": S["Xq"], "delta_x": S["delta_x"], "colscale": S["colscale"]}
    if S["O"] is not None:
        out.update(s=S["s"], what=S["what"], delta_what=S["delta_what"], xq_O=S["xq_O"])
    return out


def _forward(S):
    c = S["case"]
    q.linear_fwd_step(S["X"], S["O"], S["W_O"], S["wmax"], c["c_out"], c["gamma"], S["s"], S["colscale"], S["what"],
                      S["delta_what"], None, S["Xq"], S["delta_x"], S["xq_O"], S["Wq"], S["delta_w"], S["A"], S["B"],
                      c["r"], 1.0, S["Y"], S["ws"])
    return _step_outputs(S)


def _separate_forward(S):
    c = S["case"]
    q.scale_update(S["X"], S["O"], S["W_O"], S["wmax"], c["c_out"], c["gamma"], S["s"], S["colscale"], S["what"],
                   S["delta_what"], None, S["ws"])
    q.quant_act(S["X"], S["colscale"], S["O"], S["Xq"], S["delta_x"], S["xq_O"])
    q.linear_fwd(S["Xq"], S["delta_x"], S["xq_O"], S["Wq"], S["delta_w"], c["c_in"], c["c_out"], S["what"],
                 S["delta_what"], c["n"], S["X"] if c["r"] else None, S["A"], S["B"], c["r"], 1.0, S["Y"], S["ws"],
                 bf16_out=True)
    return _step_outputs(S)


def _input_gradient(S, bf16_out):
    c = S["case"]
    q.linear_bwd_dx(S["dY"], S["Wq"], S["delta_w"], c["c_in"], c["c_out"], S["A"], S["B"], c["r"], 1.0, S["dX"], S["ws"],
                    bf16_out=bf16_out)
    return {"dX": S["dX"]}


def _backward(S):
    c = S["case"]
    q.linear_bwd_step(S["dY"], S["X"], S["Wq"], S["delta_w"], c["c_in"], c["c_out"], S["A"], S["B"], c["r"], 1.0, S["dX"],
                      S["dA"], S["dB"], S["ws"], side=S["side"])
    return {"dX": S["dX"], "dA": S["dA"], "dB": S["dB"]}
