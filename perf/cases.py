"""Workloads of the SparseMoE layer whose speed is followed.

A case is one call (or one forward and backward) of a layer through ``MoELayerBuffers``:

  kind    "forward"  route ... combine: a decoding step, a prefill, an evaluation batch
          "train"    forward and backward of the expert path, logits given
          "block"    the drop-in block: router Linear layer in front, its backward behind
  path    "fold"     gate weights folded into the experts, rows gathered by the products
          "gather"   rows gathered by the products
          "plain"    the layer's default arguments: permuted rows are materialised
  T, d, E, k, f, e_begin, e_count, renormalize     the layer, as in ``workloads.MoEConfig``
  load    "even"     logits of a random router: every expert is about equally likely
          "zipf"     the same with the Zipf(1.2) bias of ``workloads.zipf_bias``: a few large experts, two without rows
"""
import math

import torch

from paper_2604_00785_amd import binding as B
from paper_2604_00785_amd import workloads as W

DEV = "cuda:0"

# the widest layer and the longest step of the listed cases bound what draw() may give
MAX_TRAIN_FLOP = 4.0e12
MAX_WEIGHT_BYTES = 1.1e9
MAX_ROW_BYTES = 1.6e9


def _case(name, kind, path, T, d, E, k, f, e_begin=0, e_count=None, renormalize=1, load="even"):
    return {"name": name, "kind": kind, "path": path, "T": T, "d": d, "E": E, "k": k, "f": f, "e_begin": e_begin,
            "e_count": E if e_count is None else e_count, "renormalize": renormalize, "load": load}


def _config(name, case_name, kind, path, **kw):
    c = W.CONFIGS[name]
    a = dict(T=c.T, d=c.d, E=c.E, k=c.k, f=c.f, e_begin=c.e_begin, e_count=c.n_local)
    a.update(kw)
    return _case(case_name, kind, path, **a)


def listed():
    return [
        # one decoding step of a single sequence: the smallest call, eight experts with a row each
        _config("olmoe", "decode_1", "forward", "fold", T=1),
        # one decoding step of a batch of sequences: nearly every expert is used, by a handful of rows
        _config("olmoe", "decode_48", "forward", "fold", T=48),
        # the tiny layer that the tests train, skewed load: launches and host work are what counts
        _config("tiny", "train_tiny_zipf", "train", "plain", load="zipf"),
        # a short prompt, gate weights not renormalised (the layer as the paper prints it), odd length
        _config("olmoe", "prefill_501", "forward", "gather", T=501, renormalize=0),
        # several prompts at once through a fine-grained layer
        _config("fine", "prefill_fine_4001", "forward", "fold", T=4001),
        # a training step on one sequence of the context length
        _config("olmoe", "train_2048", "train", "fold", T=2048),
        # the drop-in block of the 96-expert layer of the same width, two sequences with odd padding, skewed load
        _case("block_4099_zipf", "block", "fold", T=4099, d=2048, E=96, k=8, f=1024, load="zipf"),
        # the layer's default arguments (rows materialised, separate backward of the combine), a ragged batch
        _config("olmoe", "train_plain_6000", "train", "plain", T=6000),
        # the headline training step
        _config("olmoe", "train_olmoe", "train", "fold"),
        # many small groups
        _config("fine", "train_fine", "train", "fold"),
        # one rank's share of a wide layer under twelve-way expert parallelism
        _config("mula220b_ep12", "train_ep12", "train", "fold"),
        # one rank's share of the widest layer under eight-way expert parallelism: the largest
        _config("ep_share", "train_ep_share", "train", "fold"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["forward", "forward", "train", "train", "block"])
        E = _log_int(rng, 8, 240)
        e_count, e_begin = E, 0
        if E >= 16 and rng.random() < 0.3:                   # one rank's share of the experts
            e_count = max(1, E // rng.choice([2, 4, 8, 12]))
            e_begin = e_count * rng.randrange(E // e_count)
        c = {"kind": kind, "path": rng.choice(["fold", "fold", "gather", "plain"]),
             "T": _log_int(rng, 1, 32768) if kind == "forward" else _log_int(rng, 128, 32768),
             "d": 64 * _log_int(rng, 2, 64), "E": E, "k": rng.choice([1, 2, 4, 6, 8]), "f": 64 * _log_int(rng, 2, 32),
             "e_begin": e_begin, "e_count": e_count, "renormalize": rng.choice([0, 1, 1]),
             "load": rng.choice(["even", "even", "zipf"])}
        if work(dict(c, kind="train"))["flops"] <= MAX_TRAIN_FLOP and 6 * e_count * c["d"] * c["f"] <= MAX_WEIGHT_BYTES \
                and 2 * c["T"] * c["k"] * max(c["d"], c["f"]) <= MAX_ROW_BYTES:
            return c


def _normal(gen, shape, std, dtype=torch.bfloat16):
    t = torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32)
    return t.mul_(std).to(dtype)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    T, d, E, k, f, nl = c["T"], c["d"], c["E"], c["k"], c["f"], c["e_count"]
    s = {"kind": c["kind"]}
    s["x"] = _normal(gen, (T, d), 1.0)
    for n, shape in (("Wg", (nl, f, d)), ("Wu", (nl, f, d)), ("Wd", (nl, d, f))):
        s[n] = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
        for e in range(nl):
            s[n][e] = _normal(gen, shape[1:], 0.02)
    if c["kind"] != "forward":
        s["dout"] = _normal(gen, (T, d), 1.0)
    std = 0.02 * math.sqrt(d)            # of the logits that a N(0, 0.02) router gives on such rows
    if c["kind"] == "block":
        s["Wr"] = _normal(gen, (E, d), 0.02, torch.float32)
        if c["load"] == "zipf":          # a Linear layer has no bias: the first column of x is constant and carries it
            s["x"][:, 0] = 1.0
            s["Wr"][:, 0] = torch.from_numpy(W.zipf_bias(E, std)).to(DEV).clamp_(min=-64.0)
    else:
        s["logits"] = _normal(gen, (T, E), std, torch.float32)
        if c["load"] == "zipf":
            s["logits"] += torch.from_numpy(W.zipf_bias(E, std)).to(DEV)
    s["layer"] = B.MoELayerBuffers(T, d, E, k, f, c["e_begin"], nl, c["renormalize"], DEV,
                                   gather=c["path"] == "gather", fold=c["path"] == "fold")
    return s


def run(s):
    m = s["layer"]
    if s["kind"] == "forward":
        m.run_fwd(s["x"], s["logits"], s["Wg"], s["Wu"], s["Wd"])
        return {"out": m.out, "topk_idx": m.topk_idx, "topk_w": m.topk_w, "offsets": m.expert_offsets}
    if s["kind"] == "train":
        m.run_fwd_bwd(s["x"], s["logits"], s["dout"], s["Wg"], s["Wu"], s["Wd"])
        return {"out": m.out, "topk_idx": m.topk_idx, "topk_w": m.topk_w, "offsets": m.expert_offsets, "dx": m.dx,
                "dgate": m.dgate, "dWg": m.dWg, "dWu": m.dWu, "dWd": m.dWd}
    m.run_block_fwd_bwd(s["x"], s["Wr"], s["dout"], s["Wg"], s["Wu"], s["Wd"])
    return {"out": m.out, "topk_idx": m.topk_idx, "logits": m.logits, "dx": m.dx, "dlogits": m.dlogits, "dWr": m.dWr,
            "dWg": m.dWg, "dWu": m.dWu, "dWd": m.dWd}


def work(case):
    c = case
    T, d, E, k, f, nl = c["T"], c["d"], c["E"], c["k"], c["f"], c["e_count"]
    # expected share of local rows, and of experts that have a row at all (their weights must be read)
    p = [1.0 / E] * E
    if c["load"] == "zipf":
        w = [(e + 1.0) ** -1.2 for e in range(E - 2)]
        p = [v / sum(w) for v in w] + [0.0, 0.0]
    local = p[c["e_begin"]:c["e_begin"] + nl]
    rows = T * min(float(sum(min(1.0, k * v) for v in local)), float(k))
    used = sum(1.0 - (1.0 - min(1.0, k * v)) ** T for v in local)
    weights = 6.0 * used * d * f                       # Wg, Wu, Wd in bf16
    nbytes = 4.0 * T * E + 4.0 * T * d + weights + 8.0 * T * k      # logits, x and out, weights, topk_idx and topk_w
    flops = 6.0 * rows * d * f
    if c["kind"] != "forward":
        nbytes += 4.0 * T * d + 6.0 * nl * d * f + 4.0 * T * k      # dout and dx, weight gradients, dgate
        flops *= 3.0
    if c["kind"] == "block":
        nbytes += 8.0 * E * d + 4.0 * T * E                         # Wr and dWr, dlogits
        flops += 6.0 * T * E * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # results are bf16 and depend on intermediates that are bf16 (the saved g, u, h and the expert outputs);
    # routing is exact for given logits, while the block's logits are 32-bit sums: two correct ones may order
    # a nearly equal pair differently
    return {"rel": 1e-2, "differ": 1e-3 if case["kind"] == "block" else 0.0}
