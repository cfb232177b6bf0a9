"""Students of hidden width 256: the launches that make an encoder layer, at the edges of their tiles.  Needs an MI355X."""
import numpy as np
import pytest
import torch

from paper_2408_12526_amd import synth

pytestmark = pytest.mark.gpu


# the first call that takes them and tiles of 64 tokens with 1, 64 and fewer in the last (one block of FFN activations keeps the separate
# launches); on both sides of 8192 rows of all students (embedding and q|k|v in one launch)
@pytest.mark.parametrize("ffn,total,k", [(ffn, total, k) for ffn, first in ((256, 257), (512, 257), (768, 1280), (1024, 1664)) for total, k in (
    (first, 1), (first + 1, 1), (first + 63, 2), (first + 190, 3), (2730, 3), (2731, 3), (4096, 2), (8191, 1), (8193, 1))])
def test_layer_of_narrow_students(ffn, total, k):
    """q|k|v from the embedding rows and the layer's output from the attention output, against torch in fp64 on the weights as stored:
    operands, x1 and FFN activations in bf16, sums in fp32, one rounding of the output (the bound of the stage tests)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=3, layers=1, hidden=256, heads=4, ffn=ffn, vocab=100, max_pos=128, classes=2, dtype="bf16")
    rng = np.random.default_rng(total + ffn)
    lengths = []
    while sum(lengths) < total:
        lengths.append(int(min(rng.choice([1, 2, 15, 16, 17, 63, 64, 65, 100]), total - sum(lengths))))
    lengths = np.array(lengths, np.int32)
    ids, blob = synth.make_ids(rng, total, shape.vocab), synth.make_weights(rng, shape, std=0.06, ln_random=True)
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=True), blob)
    B, H = len(lengths), shape.hidden
    args = torch.from_numpy(ids).cuda(), torch.from_numpy(sp.sp_pack(lengths)).cuda(), int(lengths.max()), k
    x = st.read_activation(st.sp_forward_partial(*args, 0), "x", total, B, k)
    st.workspace(total, B).fill_(255)                       # (every 16-bit pattern in it a NaN)
    logits = st.sp_forward(*args)
    assert bool(torch.isfinite(logits).all())
    got = {n: torch.from_numpy(st.read_activation(st.workspace(total, B), n, total, B, k)) for n in ("qkv", "att", "x")}
    for m in range(k):
        v = {n: torch.from_numpy(a).bfloat16().double() if a.ndim == 2 else torch.from_numpy(a).double()
             for n, a in synth.student_views(blob, shape, m).items()}
        ln = lambda u, w: torch.nn.functional.layer_norm(u, (H,), v[f"l0.ln{w}_g"], v[f"l0.ln{w}_b"], shape.ln_eps)
        lin = lambda a, w, b: a @ v["l0." + w] + v["l0." + b]
        x0 = torch.from_numpy(x[m])
        x1 = ln(x0 + lin(got["att"][m], "Wo", "bo"), 1).bfloat16().double()
        g = torch.nn.functional.gelu(lin(x1, "W1", "b1")).bfloat16().double()
        want = {"qkv": torch.cat([lin(x0, "W" + p, "b" + p) for p in "qkv"], 1), "x": ln(x1 + lin(g, "W2", "b2"), 2)}
        for n, w in want.items():
            err = float((got[n][m] - w).abs().max() / w.abs().max())
            assert err < 1.2e-2, f"student {m} {n}: {err:.3e}"
    st.close()


# few rows for the FFN: the first and the last call that keep the separate launches, whose stages a whole forward leaves
@pytest.mark.parametrize("ffn,total,k", [(768, 257, 1), (768, 1279, 1), (768, 426, 3), (1024, 257, 1), (1024, 1663, 1), (1024, 831, 2)])
def test_layers_of_few_rows_keep_the_separate_launches(ffn, total, k):
    """x1, g and x of one layer on every token, each from the stage before it; bounds as above (one rounding of each)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=3, layers=1, hidden=256, heads=4, ffn=ffn, vocab=100, max_pos=128, classes=2, dtype="bf16")
    rng = np.random.default_rng(total + ffn)
    lengths = np.array([64] * (total // 64) + [total % 64], np.int32)
    ids, blob, B, H = synth.make_ids(rng, total, shape.vocab), synth.make_weights(rng, shape, std=0.06, ln_random=True), len(lengths), shape.hidden
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=True), blob)
    args = torch.from_numpy(ids).cuda(), torch.from_numpy(sp.sp_pack(lengths)).cuda(), 64, k
    x = st.read_activation(st.sp_forward_partial(*args, 0), "x", total, B, k)
    att = st.read_activation(st.sp_forward_partial(*args, 1), "att", total, B, k)
    st.workspace(total, B).fill_(255)
    st.sp_forward(*args)
    got = {n: torch.from_numpy(st.read_activation(st.workspace(total, B), n, total, B, k)) for n in ("x1", "g", "x")}
    st.close()
    for m in range(k):
        v = {n: torch.from_numpy(a).bfloat16().double() if a.ndim == 2 else torch.from_numpy(a).double()
             for n, a in synth.student_views(blob, shape, m).items()}
        ln = lambda u, w: torch.nn.functional.layer_norm(u, (H,), v[f"l0.ln{w}_g"], v[f"l0.ln{w}_b"], shape.ln_eps)
        lin = lambda a, w, b: a @ v["l0." + w] + v["l0." + b]
        want = {"x1": ln(torch.from_numpy(x[m]) + lin(torch.from_numpy(att[m]), "Wo", "bo"), 1), "g": torch.nn.functional.gelu(lin(got["x1"][m], "W1", "b1")),
                "x": ln(got["x1"][m] + lin(got["g"][m], "W2", "b2"), 2)}
        for n, w in want.items():
            err = float((got[n][m] - w).abs().max() / w.abs().max())
            assert err < 1.2e-2, f"student {m} {n}: {err:.3e}"


def test_deeper_narrow_students(oracle64):
    """Three layers, the last one on the first tokens and on all: q|k|v of a later layer from what the launch before left."""
    from oracle.sp_oracle import OracleConfig
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=3, layers=3, hidden=256, heads=4, ffn=512, vocab=100, max_pos=128, classes=3, dtype="bf16")
    rng = np.random.default_rng(8)
    lengths = rng.integers(1, 128, 48).astype(np.int32)
    ids, blob, cu = synth.make_ids(rng, int(lengths.sum()), shape.vocab), synth.make_weights(rng, shape, std=0.04, ln_random=True), sp.sp_pack(lengths)
    ow = torch.from_numpy(blob).to(torch.bfloat16).to(torch.float32).numpy()
    cfg = OracleConfig(shape.K, shape.layers, shape.hidden, shape.heads, shape.ffn, shape.vocab, shape.max_pos, shape.classes, shape.ln_eps)
    for k in (1, 3):
        want = oracle64.forward(cfg, ow, ids[:cu[4]], cu[:5], k)
        for all_tokens in (False, True):
            st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=all_tokens), blob)
            got = st.sp_forward(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k)[:4].double().cpu().numpy()
            err = np.abs(got - want).max() / max(np.abs(want).max(), 1e-3)
            assert err <= 3e-2, f"k_active {k}, all tokens {all_tokens}: {err:.3e}"
            st.close()
