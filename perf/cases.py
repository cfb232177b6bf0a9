"""Performance cases of the K-student forward.

A case is one call of ``Students.sp_forward`` on a packed batch that is already on the device, from the single request of
an idle server to the batch of a burst, for every student shape that the benchmark and the parity tests use.  The
loaded students are what a serving program keeps for its lifetime: they are loaded once per shape in a process.  What
changes from request to request, the token ids and the order of the sequence lengths, comes from the seed.
"""
from __future__ import annotations

import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2408_12526_amd import sp, synth

_BERT = dict(vocab=30522, max_pos=512, classes=2)
_SHAPES = {
    # the tiny fp32 group
    "tiny": dict(K=2, layers=2, hidden=128, heads=2, ffn=512, vocab=1000, max_pos=64, classes=2),
    # eight BERT-base-width students, two layers each: latency and burst workloads
    "base": dict(K=8, layers=2, hidden=768, heads=12, ffn=3072, **_BERT),
    # the paper's own student, 2 layers x 256
    "narrow": dict(K=3, layers=2, hidden=256, heads=4, ffn=1024, **_BERT),
    # BERT-large-width students
    "wide": dict(K=6, layers=2, hidden=1024, heads=16, ffn=4096, **_BERT),
    # the deeper student shapes
    "deep6": dict(K=2, layers=6, hidden=768, heads=12, ffn=3072, **_BERT),
    "deep12": dict(K=1, layers=12, hidden=1024, heads=16, ffn=4096, **_BERT),
}


def _case(name, shape, dtype, batch, k_active, kind, lo, hi, median=0):
    return dict(name=name, shape=shape, dtype=dtype, batch=batch, k_active=k_active, kind=kind, lo=lo, hi=hi, median=median)


def listed():
    return [
        # the tiny fp32 group on a handful of short sequences: launches and latency are all there is
        _case("tiny_fp32_b4", "tiny", "fp32", 4, 2, "uniform", 8, 32),
        # one request on an idle server, with the smallest and the largest active group
        _case("single_k1", "base", "bf16", 1, 1, "uniform", 64, 64),
        _case("single_k8", "base", "bf16", 1, 8, "uniform", 64, 64),
        # a full element of the length-aware buffer: four requests of one 8-token bin
        _case("element_b4_k2", "base", "bf16", 4, 2, "uniform", 41, 48),
        # a small dynamic batch between the latency and the throughput workloads
        _case("small_b12_k4", "base", "bf16", 12, 4, "lognormal", 8, 256, 48),
        # the batch-32 workload
        _case("batch32_k4", "base", "bf16", 32, 4, "uniform", 16, 128),
        # the burst workload with every student, and pruned to two
        _case("burst_k8", "base", "bf16", 256, 8, "lognormal", 8, 256, 48),
        _case("burst_k2", "base", "bf16", 256, 2, "lognormal", 8, 256, 48),
        # the same burst on quantised students
        _case("burst_fp8_k8", "base", "fp8", 256, 8, "lognormal", 8, 256, 48),
        # the paper's own student shape, its three-student ensemble, on the burst
        _case("narrow_b256_k3", "narrow", "bf16", 256, 3, "lognormal", 8, 256, 48),
        # BERT-large-width students on long sequences
        _case("wide_b64_k6", "wide", "bf16", 64, 6, "uniform", 64, 512),
        # one deep student on long sequences: the most work per call
        _case("deep12_b64", "deep12", "bf16", 64, 1, "uniform", 64, 512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A call of one of the shapes above: batches from one request to a burst's, any active prefix, lengths of any scale."""
    shape = rng.choice(["base"] * 6 + ["tiny", "narrow", "wide", "deep6", "deep12"])
    s = _SHAPES[shape]
    dtype = "fp32" if shape == "tiny" else "fp8" if shape == "base" and rng.random() < 0.25 else "bf16"
    batch = _log_int(rng, 1, 64 if shape in ("wide", "deep12") else 256)
    hi = min(s["max_pos"], rng.choice([64, 128, 256, 512]))
    if rng.random() < 0.5:
        lo = _log_int(rng, 4, hi)
        c = _case("", shape, dtype, batch, rng.randint(1, s["K"]), "uniform", lo, hi)
    else:
        c = _case("", shape, dtype, batch, rng.randint(1, s["K"]), "lognormal", 4, hi, _log_int(rng, 12, hi / 2))
    most = work(listed()[-1])
    while c["batch"] > 1 and (work(c)["flops"] > most["flops"] or _lengths(c).sum() > _lengths(listed()[-1]).sum()):
        c["batch"] = (c["batch"] + 1) // 2
    del c["name"]
    return c


def _lengths(case):
    """The batch's lengths, ascending: the quantiles of the named distribution, so that a case has one total."""
    u = (np.arange(case["batch"]) + 0.4) / case["batch"]
    lo, hi = case["lo"], case["hi"]
    if case["kind"] == "uniform":
        n = lo + np.floor(u * (hi - lo + 1))
    else:
        n = np.rint(case["median"] * np.exp(0.6 * np.array([NormalDist().inv_cdf(x) for x in u])))
    return np.clip(n, lo, hi).astype(np.int32)


_loaded = {}


def _students(case):
    key = (case["shape"], case["dtype"])
    if key not in _loaded:
        shape = synth.StudentShape(dtype=case["dtype"], **_SHAPES[case["shape"]])
        gen = torch.Generator(device="cuda").manual_seed(20)
        blob = np.empty(synth.blob_floats(shape), np.float32)
        for part in np.split(blob, shape.K):          # N(0, 0.02) everywhere, LayerNorm scale 1 and shift 0
            part[:] = torch.randn(part.size, generator=gen, device="cuda").mul_(0.02).cpu().numpy()
        for _, views in synth.iter_views(blob, shape):
            for name, v in views.items():
                if "ln" in name:
                    v[...] = 1.0 if name.endswith("_g") else 0.0
        _loaded[key] = sp.Students(sp.config_from_shape(shape), blob)
    return _loaded[key]


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    lengths = rng.permutation(_lengths(case))
    ids = synth.make_ids(rng, int(lengths.sum()), _SHAPES[case["shape"]]["vocab"])
    return dict(students=_students(case), ids=torch.from_numpy(ids).cuda(), cu=torch.from_numpy(sp.sp_pack(lengths)).cuda(),
                max_seqlen=int(lengths.max()), k_active=case["k_active"])


def run(state):
    return state["students"].sp_forward(state["ids"], state["cu"], state["max_seqlen"], state["k_active"])


def work(case):
    """Flops: every layer but the last for all tokens; of the last one only what the first token of each sequence needs
    (one query per sequence and head, folded through the key projection, on the token rows themselves); pooler and
    classifier.  Bytes: the active students' weights and the embedding rows of the tokens once, ids and offsets, logits."""
    s = _SHAPES[case["shape"]]
    H, F, C, A, k, B = s["hidden"], s["ffn"], s["classes"], s["heads"], case["k_active"], case["batch"]
    n = _lengths(case).astype(np.int64)
    T, full = int(n.sum()), s["layers"] - 1
    flops = k * full * (2 * T * (4 * H * H + 2 * H * F) + 4 * H * int((n * n).sum()))
    flops += k * (B * (2 * 4 * H * H + 4 * H * F) + 4 * T * A * H)
    flops += k * B * (2 * H * H + 2 * H * C)
    size = 4 if case["dtype"] == "fp32" else 2
    layer = 4 * H * H + 2 * H * F
    weights = layer * (full * (1 if case["dtype"] == "fp8" else size) + size) + (H * H + H * C) * size
    rows = (min(T, s["vocab"]) + int(n.max())) * H * size
    return {"bytes": k * (weights + rows) + 4 * (T + B + 1) + 4 * B * C, "flops": flops}


def tolerance(case):
    """fp32: sums in another order.  bf16: activations rounded to eight bits at other places.  fp8: three-bit mantissas."""
    return {"fp32": {"rel": 1e-5, "max": 1e-4}, "bf16": {"rel": 1e-2, "max": 6e-2},
            "fp8": {"rel": 3e-2, "max": 2e-1}}[case["dtype"]]
