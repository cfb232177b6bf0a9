"""Projections of launches of few tiles (bf16 path) at the edges of their tile rule.  Needs an MI355X."""
import numpy as np
import pytest
import torch

from paper_2408_12526_amd import synth

pytestmark = pytest.mark.gpu


# 257 tokens: the first call on the tile kernels; 768 and 1024 features of 256 or 512: 32 x 128 tiles, 64 x 128 ones and tiles of 256
# features on both sides of where they take over (256 workgroups), with a last tile that is partly filled
@pytest.mark.parametrize("total", [257, 320, 352, 1344, 1408, 2730, 2752])
@pytest.mark.parametrize("hidden,ffn,k", [(256, 1024, 1), (256, 1024, 2), (256, 128, 2), (512, 512, 1)])
def test_projections_of_few_tiles(hidden, ffn, k, total):
    """q|k|v, FFN up and what the residual projections leave, each from the rows that the previous kernel left, against torch in
    fp64 on the weights as stored: operands in bf16, sums in fp32, one rounding of the output (the bound of the stage tests)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=1, hidden=hidden, heads=hidden // 64, ffn=ffn, vocab=100, max_pos=64, classes=2, dtype="bf16")
    rng = np.random.default_rng(total + hidden)
    lengths = np.full(-(-total // 40), 40, np.int32)
    lengths[-1] -= lengths.sum() - total
    ids, blob = synth.make_ids(rng, total, shape.vocab), synth.make_weights(rng, shape, std=0.08, ln_random=True)
    st = sp.Students(sp.config_from_shape(shape), blob)
    B, H = len(lengths), hidden
    args = torch.from_numpy(ids).cuda(), torch.from_numpy(sp.sp_pack(lengths)).cuda(), int(lengths.max()), k
    x = st.read_activation(st.sp_forward_partial(*args, 0), "x", total, B, k)
    ws = st.sp_forward_partial(*args, 1)
    got = {n: st.read_activation(ws, n, total, B, k) for n in ("qkv", "att", "x1", "g", "x")}
    for m in range(k):
        v = {n: torch.from_numpy(a).bfloat16().double() if a.ndim == 2 else torch.from_numpy(a).double()
             for n, a in synth.student_views(blob, shape, m).items()}
        t = {n: torch.from_numpy(a[m]) for n, a in got.items()}
        ln = lambda u, w: torch.nn.functional.layer_norm(u, (H,), v[f"l0.ln{w}_g"], v[f"l0.ln{w}_b"], shape.ln_eps)
        lin = lambda a, w, b: a @ v["l0." + w] + v["l0." + b]
        x0 = torch.from_numpy(x[m])
        want = {"qkv": torch.cat([lin(x0, "W" + p, "b" + p) for p in "qkv"], 1), "x1": ln(x0 + lin(t["att"], "Wo", "bo"), 1),
                "g": torch.nn.functional.gelu(lin(t["x1"], "W1", "b1")), "x": ln(t["x1"] + lin(t["g"], "W2", "b2"), 2)}
        for n, w in want.items():
            err = float((t[n] - w).abs().max() / w.abs().max())
            assert err < 1.2e-2, f"student {m} {n}: {err:.3e}"
    st.close()
