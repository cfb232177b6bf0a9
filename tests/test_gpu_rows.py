"""The few-row projections (small calls and the first-token last layer) at the edges of their tiles.  Needs an MI355X."""
import numpy as np
import pytest
import torch

from oracle.sp_oracle import OracleConfig
from paper_2408_12526_amd import synth

pytestmark = pytest.mark.gpu


def _run(oracle64, shape, lengths, ks, seed):
    from paper_2408_12526_amd import sp
    rng = np.random.default_rng(seed)
    lengths = np.array(lengths, dtype=np.int32)
    ids = synth.make_ids(rng, int(lengths.sum()), shape.vocab)
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True)
    cu = sp.sp_pack(lengths)
    st = sp.Students(sp.config_from_shape(shape), blob)
    ow = torch.from_numpy(blob).to(torch.bfloat16).to(torch.float32).numpy()
    cfg = OracleConfig(shape.K, shape.layers, shape.hidden, shape.heads, shape.ffn, shape.vocab, shape.max_pos, shape.classes,
                       shape.ln_eps)
    pick = np.arange(len(lengths)) if len(lengths) <= 6 else np.unique(np.r_[0, len(lengths) - 1, rng.integers(0, len(lengths), 4)])
    sub_ids = np.concatenate([ids[cu[b]:cu[b + 1]] for b in pick])
    sub_cu = np.concatenate([[0], np.cumsum(lengths[pick])]).astype(np.int32)
    for k in ks:
        got = st.sp_forward(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k).double().cpu().numpy()
        want = oracle64.forward(cfg, ow, sub_ids, sub_cu, k)
        assert np.isfinite(got).all()
        err = np.abs(got[pick] - want).max() / max(np.abs(want).max(), 1e-3)
        assert err <= 3e-2, f"{shape}, lengths {lengths[:6]}, k_active {k}: {err:.3e}"
    st.close()


# every hidden width; reduction depths of one pass and of several, with and without unused steps in the last
@pytest.mark.parametrize("hidden,ffn", [(128, 128), (256, 1024), (384, 640), (512, 1536), (640, 2560), (768, 3072), (896, 2176), (1024, 4096)])
@pytest.mark.parametrize("lengths", [(1,), (15,), (16,), (17,), (5, 28), (57, 58), (64, 1, 63), (9,) * 20, (250, 6)])
def test_small_calls_on_every_width(oracle64, hidden, ffn, lengths):
    """Row blocks of sixteen just missed, met and passed, both sides of the fused LayerNorm's limit, one and several steps
    of the first-token attention."""
    shape = synth.StudentShape(K=5, layers=2, hidden=hidden, heads=hidden // 64, ffn=ffn, vocab=60, max_pos=256, classes=3,
                               dtype="bf16")
    _run(oracle64, shape, lengths, (1, 5), 7 * hidden + sum(lengths))


@pytest.mark.parametrize("nseq,length", [(33, 8), (64, 9), (255, 3), (256, 5), (257, 5), (300, 3), (300, 4), (511, 2), (600, 2), (1041, 3), (1500, 3)])
@pytest.mark.parametrize("hidden", [256, 512, 768, 1024])
def test_first_token_rows_of_many_sequences(oracle64, hidden, nseq, length):
    """The folded last layer at row blocks of every tile, on few and on many sequences; below 1024 tokens its rows share the
    buffers of the all-token layers."""
    shape = synth.StudentShape(K=3, layers=2, hidden=hidden, heads=hidden // 64, ffn=4 * hidden, vocab=60, max_pos=16, classes=2,
                               dtype="bf16")
    _run(oracle64, shape, (length,) * nseq, (1, 3), hidden + nseq)


@pytest.mark.parametrize("ffn,layers", [(128, 1), (512, 2), (768, 3)])
@pytest.mark.parametrize("lengths,k", [((1,), 1), ((2,), 2), ((3, 4), 2), ((27, 8, 32, 19), 2), ((64,) * 4, 2), ((64, 64, 64, 64, 1), 2),
                                       ((57,) * 9, 1)])
def test_fp32_layer_in_one_launch(oracle64, ffn, layers, lengths, k):
    """Two rows per workgroup: one row, odd counts, the last call on one launch per layer (512 rows of all students) and the
    first on separate ones; with and without a next layer.  fp32 sums of at most 768 terms, each within a few 1e-7 of its size."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=layers, hidden=128, heads=2, ffn=ffn, vocab=60, max_pos=64, classes=3, dtype="fp32")
    rng = np.random.default_rng(ffn + sum(lengths))
    lengths = np.array(lengths, dtype=np.int32)
    ids = synth.make_ids(rng, int(lengths.sum()), shape.vocab)
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True)
    cu = sp.sp_pack(lengths)
    st = sp.Students(sp.config_from_shape(shape), blob)
    got = st.sp_forward(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k).double().cpu().numpy()
    cfg = OracleConfig(shape.K, shape.layers, shape.hidden, shape.heads, shape.ffn, shape.vocab, shape.max_pos, shape.classes,
                       shape.ln_eps)
    want = oracle64.forward(cfg, blob, ids, cu, k)
    err = np.abs(got - want).max() / max(np.abs(want).max(), 1e-3)
    assert err <= 1e-5, f"{err:.3e}"
    st.close()


# the attention inside that launch: 32 keys of either wave and 64 of both just missed, met and passed, a second wave without keys, steps of
# which the last has few; rows' q|k|v in either of their two buffers; the narrowest FFN, whose own activations are smaller than those
@pytest.mark.parametrize("lengths,k", [((1, 31, 32, 33, 63, 64, 1), 2), ((65, 96, 97, 2), 1), ((127, 128, 129), 1), ((1, 320, 5), 1)])
@pytest.mark.parametrize("layers,ffn,all_tokens", [(1, 128, True), (2, 512, False), (3, 128, True), (4, 256, False)])
def test_fp32_layer_with_its_attention(oracle64, lengths, k, layers, ffn, all_tokens):
    """Sharp scores, a workspace full of NaN beforehand, and twice the same bits; bound as above."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=layers, hidden=128, heads=2, ffn=ffn, vocab=60, max_pos=320, classes=2, dtype="fp32")
    rng = np.random.default_rng(layers + sum(lengths))
    ids, cu = synth.make_ids(rng, sum(lengths), shape.vocab), sp.sp_pack(np.array(lengths, dtype=np.int32))
    assert len(ids) * k <= 512
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True, qk_std=0.3)
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=all_tokens), blob)
    st.workspace(len(ids), len(lengths)).fill_(255)
    args = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), max(lengths), k
    first = st.sp_forward(*args).clone()
    assert torch.equal(first, st.sp_forward(*args))
    st.close()
    cfg = OracleConfig(shape.K, shape.layers, shape.hidden, shape.heads, shape.ffn, shape.vocab, shape.max_pos, shape.classes, shape.ln_eps)
    want = oracle64.forward(cfg, blob, ids, cu, k)
    assert np.abs(first.double().cpu().numpy() - want).max() / max(np.abs(want).max(), 1e-3) <= 1e-5


# both buffers of the rows' q|k|v, in either order
@pytest.mark.parametrize("layers", [1, 2, 3, 4])
@pytest.mark.parametrize("all_tokens", [False, True])
def test_what_an_fp32_call_in_few_launches_leaves(layers, all_tokens):
    """The last layer's q|k|v, and its attention output and state in the rows that it computes, beside what the separate launches of a
    forward that stops behind it leave: sums of at most 256 fp32 terms in another order, over up to four layers."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=3, layers=layers, hidden=128, heads=2, ffn=256, vocab=60, max_pos=70, classes=2, dtype="fp32")
    rng, lengths = np.random.default_rng(layers), np.array((1, 70, 33, 2, 7), np.int32)
    cu, T, B = sp.sp_pack(lengths), int(lengths.sum()), len(lengths)
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=all_tokens), synth.make_weights(rng, shape, std=0.04, ln_random=True, qk_std=0.2))
    for k in (1, 3):
        args = torch.from_numpy(synth.make_ids(rng, T, shape.vocab)).cuda(), torch.from_numpy(cu).cuda(), 70, k
        ws = st.workspace(T, B).fill_(255)
        st.sp_forward(*args, workspace=ws)
        got = {n: st.read_activation(ws, n, T, B, k) for n in ("qkv", "att", "x")}
        ws = st.sp_forward_partial(*args, layers)
        rows = np.arange(T) if all_tokens else cu[:-1]
        for n, r in (("qkv", np.arange(T)), ("att", rows), ("x", rows)):
            want = st.read_activation(ws, n, T, B, k)[:, r]
            assert np.abs(got[n][:, r] - want).max() / np.abs(want).max() < 1e-5, (n, k)
    st.close()


# (embedding and q|k|v of hidden 256 in two launches and in one)
@pytest.mark.parametrize("hidden,ffn,layers,lengths,k,some", [
    (128, 256, 3, (5, 60, 33), 2, {"embed", "ffn_down", "last_first", "head"}),
    (128, 256, 3, (5, 60, 33), 1, {"embed", "ffn_down", "last_first"}),
    (256, 768, 2, (60,) * 20, 2, {"embed", "qkv", "attention", "ffn_down", "last_first", "head"}),
    (256, 768, 2, (60,) * 70, 2, {"embed", "attention", "ffn_down", "last_first", "head"})])
def test_phases_of_calls_in_few_launches(hidden, ffn, layers, lengths, k, some):
    """What sp_forward_profiled says of launches that cover several steps: the phases that it names have time, the others none."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=layers, hidden=hidden, heads=hidden // 64, ffn=ffn, vocab=60, max_pos=64, classes=2,
                               dtype="fp32" if hidden == 128 else "bf16")
    rng, cu = np.random.default_rng(k), sp.sp_pack(np.array(lengths, np.int32))
    st = sp.Students(sp.config_from_shape(shape), synth.make_weights(rng, shape))
    ms = st.sp_forward_profiled(torch.from_numpy(synth.make_ids(rng, sum(lengths), 60)).cuda(), torch.from_numpy(cu).cuda(), max(lengths), k)
    assert {n for n, t in ms.items() if t > 0} == some, ms
    st.close()


# one, two, three and eight rounds of 64 boundaries in the embedding of a whole call in few launches; 512 rows of all students and one more
@pytest.mark.parametrize("lengths,k", [((3,) * 64, 2), ((3,) * 65, 2), ((1, 2) * 64 + (5,), 2), ((1,) * 200, 2), ((1,) * 255 + (257,), 1), ((1,) * 512, 1),
                                       ((1,) * 513, 1)])
@pytest.mark.parametrize("classes", [1, 2])
def test_fp32_calls_of_many_sequences(oracle64, lengths, k, classes):
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=2, hidden=128, heads=2, ffn=256, vocab=60, max_pos=304, classes=classes, dtype="fp32")
    rng = np.random.default_rng(len(lengths))
    ids = synth.make_ids(rng, sum(lengths), shape.vocab)
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True)
    cu = sp.sp_pack(np.array(lengths, dtype=np.int32))
    st = sp.Students(sp.config_from_shape(shape), blob)
    got = st.sp_forward(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), max(lengths), k).double().cpu().numpy()
    st.close()
    cfg = OracleConfig(shape.K, shape.layers, shape.hidden, shape.heads, shape.ffn, shape.vocab, shape.max_pos, shape.classes,
                       shape.ln_eps)
    want = oracle64.forward(cfg, blob, ids, cu, k)
    assert np.abs(got - want).max() / np.abs(want).max() <= 1e-5         # (as in the test above)


# the pooler's share of the classifier (with one class its last lanes' weights are the matrix's end), the classifier behind the tile kernels, the
# one of the all-token last layer, the fp32 chain's
@pytest.mark.parametrize("hidden,lengths,dtype", [(128, (64,), "bf16"), (256, (17, 3), "bf16"), (768, (64, 1, 63), "bf16"), (1024, (250, 6), "bf16"),
                                                  (640, (90, 200, 13), "bf16"), (768, (30,) * 40, "bf16"), (256, (5,) * 3000, "bf16"),
                                                  (128, (9, 30), "fp32"), (256, (9, 30), "fp32")])
def test_one_class_is_the_first_of_two(hidden, lengths, dtype):
    """The same sums in the same order, so the same bits."""
    from paper_2408_12526_amd import sp
    one, two = (synth.StudentShape(K=3, layers=2, hidden=hidden, heads=hidden // 64, ffn=2 * hidden, vocab=60, max_pos=256, classes=c, dtype=dtype)
                for c in (1, 2))
    rng = np.random.default_rng(hidden + len(lengths))
    blob2 = synth.make_weights(rng, two, std=0.04, ln_random=True)
    blob1 = np.empty(synth.blob_floats(one), np.float32)
    for m in range(3):
        for (name, a), (_, b) in zip(synth.student_views(blob1, one, m).items(), synth.student_views(blob2, two, m).items()):
            a[...] = b if a.shape == b.shape else b[..., :1]
    ids = torch.from_numpy(synth.make_ids(rng, sum(lengths), one.vocab)).cuda()
    cu = torch.from_numpy(sp.sp_pack(np.array(lengths, np.int32))).cuda()
    got = []
    for shape, blob in ((one, blob1), (two, blob2)):
        st = sp.Students(sp.config_from_shape(shape), blob)
        got.append([st.sp_forward(ids, cu, max(lengths), k).cpu() for k in (1, 3)])
        st.close()
    for a, b in zip(*got):
        assert a.shape[1] == 1 and torch.isfinite(a).all() and a.abs().max() > 0 and torch.equal(a, b[:, :1])


# (hidden, ffn, layers, students, active, every token in the last layer): the attention-output projection splits its reduction and the
# FFN down-projection does not; the other way round with slices over the attention output; both; a call of few tokens
@pytest.mark.parametrize("hidden,ffn,layers,K,k,all_tokens,lengths",
                         [(512, 640, 3, 2, 2, False, (100, 37, 150, 62)), (768, 640, 2, 2, 2, True, (200, 90, 5)),
                          (1024, 128, 3, 1, 1, False, (64, 64, 64, 65, 64)), (256, 1024, 3, 4, 1, True, (90, 200, 13)),
                          (768, 3072, 3, 2, 1, True, (301, 12, 90)), (768, 384, 2, 5, 5, False, (100, 53)),
                          (384, 1536, 3, 2, 1, False, (301, 12, 90)), (640, 2560, 3, 1, 1, True, (77, 200, 13)),
                          # (short sequences alone, in a call of few tokens, and beside a longer one)
                          (768, 384, 2, 2, 2, False, (9,) * 33 + (5,)), (256, 512, 2, 3, 3, True, (31, 30, 3)),
                          (512, 640, 2, 4, 4, True, (5,) * 80 + (45,))])
def test_nothing_in_the_workspace_has_to_be_finite(oracle64, hidden, ffn, layers, K, k, all_tokens, lengths):
    """Padding rows reach attention with probability zero, which is no help against what is not a number: a workspace full of
    NaN gives what the oracle gives, for the last sequence too (token counts that are no multiple of eight)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=K, layers=layers, hidden=hidden, heads=hidden // 64, ffn=ffn, vocab=60, max_pos=304, classes=2,
                               dtype="bf16")
    rng = np.random.default_rng(hidden + ffn)
    lengths = np.array(lengths, dtype=np.int32)
    ids = synth.make_ids(rng, int(lengths.sum()), shape.vocab)
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True)
    cu = sp.sp_pack(lengths)
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=all_tokens), blob)
    ws = torch.full((sp.sp_workspace_bytes(st.cfg, len(ids), len(lengths)),), 0xff, dtype=torch.uint8, device="cuda")
    got = st.sp_forward(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k, workspace=ws)
    got = got.double().cpu().numpy()
    ow = torch.from_numpy(blob).to(torch.bfloat16).to(torch.float32).numpy()
    cfg = OracleConfig(K, layers, hidden, shape.heads, ffn, shape.vocab, shape.max_pos, shape.classes, shape.ln_eps)
    want = oracle64.forward(cfg, ow, ids, cu, k)
    assert np.isfinite(got).all()
    err = np.abs(got - want).max() / max(np.abs(want).max(), 1e-3)
    assert err <= 3e-2, f"{err:.3e}"
    st.close()


def _forks(hidden, layers, dtype, tokens, k):
    """Whether a call is expected to run as two groups: the rule beside which both sides are measured, stated once more."""
    work = tokens * k * hidden
    return (k >= 2 and tokens >= 8192 and work * (layers - 1 if k % 2 == 0 and layers > 2 else 1) >= 20 << 20 and
            (dtype == "fp8" or hidden < 512 or (k % 2 == 0 and work <= 64 << 20)))


# (hidden, students, sequences, tokens of each, layers): the first-token rows of all students and of a group, of the two groups of an odd
# number, or of few and of all students, lie on different sides of a limit between kernels; few tiles for one student
GROUP_SHAPES = [(768, 3, 153, 60, 2), (768, 4, 140, 60, 2), (768, 2, 230, 60, 2), (1024, 4, 138, 60, 2), (768, 5, 140, 60, 2),
                (1024, 6, 900, 16, 2), (256, 3, 460, 60, 2), (256, 5, 280, 60, 2), (256, 2, 150, 60, 6)]


@pytest.mark.parametrize("hidden,K,nseq,length,layers,dtype",
                         [s + (d,) for s in GROUP_SHAPES for d in ("bf16", "fp8") if (s[:2], d) != ((768, 3), "bf16")])
def test_one_group_of_students_or_two_give_the_same_bits(hidden, K, nseq, length, layers, dtype):
    """Which kernels a large call takes goes by its tokens and sequences and the model, not by the group of students at hand nor by
    how many are active: its logits are the same bits on one stream and on two, and the sum of the same terms for every k."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=K, layers=layers, hidden=hidden, heads=hidden // 64, ffn=1024, vocab=500, max_pos=64, classes=4, dtype=dtype)
    rng = np.random.default_rng(hidden + K)
    lengths = np.full(nseq, length, dtype=np.int32)
    ids = torch.from_numpy(synth.make_ids(rng, int(lengths.sum()), shape.vocab)).cuda()
    assert any(_forks(hidden, layers, dtype, ids.numel(), k) for k in range(1, K + 1))
    cu = torch.from_numpy(sp.sp_pack(lengths)).cuda()
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True)
    two = sp.Students(sp.config_from_shape(shape), blob)
    one = sp.Students(sp.config_from_shape(shape, single_stream=True), blob)
    two.sp_forward(ids, cu, length, K)
    z = torch.from_numpy(two.read_activation(two.workspace(ids.numel(), nseq), "z", ids.numel(), nseq, K)).float()
    total = torch.zeros(nseq, 4)
    for k in range(1, K + 1):
        total = total + z[k - 1]
        a, b = two.sp_forward(ids, cu, length, k).cpu(), one.sp_forward(ids, cu, length, k).cpu()
        assert torch.equal(a, b), f"k_active {k}: {(a - b).abs().max().item():.3e}"
        assert torch.equal(a, total), f"k_active {k}, terms: {(a - total).abs().max().item():.3e}"
    two.close()
    one.close()


def _stages(oracle64, shape, weights, m, x0, att, got):
    """Largest relative errors of x1, g and x of a one-layer student against the layer's pieces applied to what the GPU had."""
    v = {n[3:]: w for n, w in synth.student_views(weights, shape, m).items() if n.startswith("l0.")}

    def ln(u, which):
        return np.stack([oracle64.layernorm(r, v[f"ln{which}_g"], v[f"ln{which}_b"], shape.ln_eps) for r in u])

    def rel(a, b):
        return np.abs(a - b).max() / np.abs(b).max()

    g = torch.nn.functional.gelu(torch.from_numpy(oracle64.linear(got["x1"][m], v["W1"], v["b1"]))).numpy()
    return (rel(got["x1"][m], ln(x0[m] + oracle64.linear(att[m], v["Wo"], v["bo"]), 1)), rel(got["g"][m], g),
            rel(got["x"][m], ln(got["x1"][m] + oracle64.linear(got["g"][m], v["W2"], v["b2"]), 2)))


# one student of K: as many slices as the buffers of the others leave room for.  Slices of the two projections: 3 and 8, 3 and 6, 2
# and 3, 1 and 4 (an FFN that keeps the separate launches at this width), 1 and 6 (tiles of half the features), 1 and 2
@pytest.mark.parametrize("hidden,ffn,K", [(768, 3072, 8), (768, 3072, 2), (768, 3072, 1), (256, 2048, 2), (384, 1536, 2), (128, 512, 1)])
def test_split_reductions_stage_by_stage(oracle64, hidden, ffn, K):
    """A whole forward with every token in its one layer leaves x1, g and x of that layer: each against the oracle's piece applied
    to the stage before it (the attention output, which the slices overwrite, from a forward that stops after the layer)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=K, layers=1, hidden=hidden, heads=hidden // 64, ffn=ffn, vocab=60, max_pos=208, classes=2, dtype="bf16")
    rng = np.random.default_rng(hidden + K)
    lengths = np.array((101, 13, 199), dtype=np.int32)
    T, B = int(lengths.sum()), 3
    ids, blob, cu = synth.make_ids(rng, T, shape.vocab), synth.make_weights(rng, shape, std=0.05, ln_random=True), sp.sp_pack(lengths)
    weights = torch.from_numpy(blob).bfloat16().float().numpy()
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=True), blob)
    d_ids, d_cu = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda()
    x0 = st.read_activation(st.sp_forward_partial(d_ids, d_cu, 199, 1, 0), "x", T, B, 1)
    att = st.read_activation(st.sp_forward_partial(d_ids, d_cu, 199, 1, 1), "att", T, B, 1)
    st.workspace(T, B).fill_(255)                           # (nothing of the partial forwards is left: every 16-bit pattern in it a NaN)
    st.sp_forward(d_ids, d_cu, 199, 1)
    got = {n: st.read_activation(st.workspace(T, B), n, T, B, 1) for n in ("x1", "g", "x")}
    # (one bf16 rounding of each output: the operands are what the GPU had)
    assert max(_stages(oracle64, shape, weights, 0, x0, att, got)) < 1.2e-2
    st.close()


# K picks the tile heights: hidden 256 and 768 as in the test of the fp8 tiles; hidden 384 tiles of half the features, 32 tokens
# for the attention output and 64 for q|k|v at K = 1, 64 and 96 at K = 7
@pytest.mark.parametrize("tokens", [2049, 2111])
@pytest.mark.parametrize("hidden,ffn,K", [(256, 768, 1), (256, 768, 2), (256, 768, 3), (256, 768, 4), (768, 768, 1), (768, 768, 2),
                                          (768, 768, 3), (768, 768, 4), (384, 640, 1), (384, 640, 7)])
def test_tiles_of_every_height_at_their_edges(oracle64, hidden, ffn, K, tokens):
    """Every projection on the HIP path's own input, the last rows and a sample of the others: one row beyond a tile of any height,
    and one short of 64."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=K, layers=1, hidden=hidden, heads=hidden // 64, ffn=ffn, vocab=60, max_pos=128, classes=2, dtype="bf16")
    rng = np.random.default_rng(tokens + K)
    lengths = np.full(-(-tokens // 100), 100, dtype=np.int32)
    lengths[-1] = tokens - 100 * (len(lengths) - 1)
    B = len(lengths)
    ids, blob, cu = synth.make_ids(rng, tokens, shape.vocab), synth.make_weights(rng, shape, std=0.05, ln_random=True), sp.sp_pack(lengths)
    weights = torch.from_numpy(blob).bfloat16().float().numpy()
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=True), blob)
    d_ids, d_cu = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda()
    rows = np.unique(np.r_[np.arange(0, tokens, 61), np.arange(tokens - 130, tokens)])
    x0 = st.read_activation(st.sp_forward_partial(d_ids, d_cu, 100, K, 0), "x", tokens, B, K)[:, rows]
    ws = st.sp_forward_partial(d_ids, d_cu, 100, K, 1)
    got = {n: st.read_activation(ws, n, tokens, B, K)[:, rows] for n in ("qkv", "att", "x1", "g", "x")}
    for m in range(K):
        v = synth.student_views(weights, shape, m)
        qkv = oracle64.linear(x0[m], np.concatenate([v["l0.Wq"], v["l0.Wk"], v["l0.Wv"]], axis=1),
                              np.concatenate([v["l0.bq"], v["l0.bk"], v["l0.bv"]]))
        assert np.abs(got["qkv"][m] - qkv).max() / np.abs(qkv).max() < 1.2e-2
        assert max(_stages(oracle64, shape, weights, m, x0, got["att"], got)) < 1.2e-2
    st.close()


@pytest.mark.parametrize("hidden,K,nseq", [(768, 8, 68), (1024, 6, 68), (512, 13, 64), (1024, 24, 14)])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_calls_beside_a_capture_of_the_same_model(hidden, K, nseq, dtype):
    """While the model's second stream belongs to the capture of a large call, calls on another stream run eagerly with the single-stream
    bits: below 8192 tokens, which never fork however much work they are, and of a size that would fork.  A second forking call joins the
    capture.  The graph gives what the large calls give."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=K, layers=2, hidden=hidden, heads=hidden // 64, ffn=512, vocab=500, max_pos=64, classes=3, dtype=dtype)
    rng = np.random.default_rng(hidden + K)

    def call(n):
        ids = torch.from_numpy(synth.make_ids(rng, 63 * n, shape.vocab)).cuda()
        return ids, torch.from_numpy(sp.sp_pack(np.full(n, 63, dtype=np.int32))).cuda(), torch.empty(n, 3, device="cuda")
    ids, cu, out = call(nseq)
    assert ids.numel() < 8192 and ids.numel() * K * hidden >= 20 << 20
    large, large_cu, large_out = call((20 << 20) // (2 * hidden) // 63 + 1)
    assert _forks(hidden, 2, dtype, large.numel(), 2)
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True)
    two = sp.Students(sp.config_from_shape(shape), blob)
    one = sp.Students(sp.config_from_shape(shape, single_stream=True), blob)
    ws, large_ws = (torch.empty(sp.sp_workspace_bytes(two.cfg, i.numel(), c.numel() - 1), dtype=torch.uint8, device="cuda")
                    for i, c in ((ids, cu), (large, large_cu)))
    want = {k: one.sp_forward(ids, cu, 63, k).clone() for k in (K, K - 1)}
    want_large = one.sp_forward(large, large_cu, 63, 2).clone()
    two.sp_forward(large, large_cu, 63, 2, large_out, large_ws)
    torch.cuda.synchronize()
    side, other, graph = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    got, beside, again_out, beside_ws = ({k: torch.zeros_like(out) for k in (K, K - 1)}, torch.zeros_like(large_out),
                                         torch.zeros_like(large_out), torch.empty_like(large_ws))
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="thread_local"):
        two.sp_forward(large, large_cu, 63, 2, large_out, large_ws, stream=side)
        for k in (K, K - 1):
            two.sp_forward(ids, cu, 63, k, got[k], ws, stream=other)
        two.sp_forward(large, large_cu, 63, 2, beside, beside_ws, stream=other)
        two.sp_forward(large, large_cu, 63, 2, again_out, large_ws, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(beside, want_large)
    for k in (K, K - 1):
        assert torch.equal(got[k], want[k]), f"k_active {k}: {(got[k] - want[k]).abs().max().item():.3e}"
    for _ in range(3):
        large_out.zero_()
        again_out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(large_out, want_large) and torch.equal(again_out, want_large)
        two.sp_forward(large, large_cu, 63, 2, beside, large_ws)             # eager work between the replays, two groups again
        torch.cuda.synchronize()
        assert torch.equal(beside, want_large)
    two.close()
    one.close()


# 8192 tokens or more and enough work over the model's students: the folded last layer takes the rows before their LayerNorm
@pytest.mark.parametrize("hidden,dtype", [(256, "bf16"), (512, "bf16"), (768, "bf16"), (1024, "bf16"), (768, "fp8")])
@pytest.mark.parametrize("offset", [0.0, 6.0])
def test_folded_last_layer_on_rows_before_their_layernorm(oracle64, hidden, dtype, offset):
    """Against the oracle and the last layer on every token; a bias common to all features of the rows (their mean several times
    their deviation) must cancel but for the rounding of the rows themselves, which grows by that factor on either way."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=5 if hidden == 256 else 4, layers=2, hidden=hidden, heads=hidden // 64, ffn=256, vocab=60, max_pos=256, classes=3,
                               dtype=dtype)
    rng = np.random.default_rng(hidden)
    lengths = np.array((1, 2, 31, 32, 33, 64, 65, 256) + (60,) * 140, np.int32)
    T = int(lengths.sum())
    assert T >= 8192
    ids, blob = synth.make_ids(rng, T, shape.vocab), synth.make_weights(rng, shape, std=0.04, ln_random=True)
    for m in range(shape.K):
        synth.student_views(blob, shape, m)["l0.b2"][:] += offset
    cu, n = sp.sp_pack(lengths), 12                         # (the first twelve sequences against the oracle)
    args = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), shape.K
    st = sp.Students(sp.config_from_shape(shape), blob)
    got = st.sp_forward(*args).double().cpu().numpy()
    x = st.read_activation(st.workspace(T, len(lengths)), "x", T, len(lengths), shape.K)
    st.close()
    st = sp.Students(sp.config_from_shape(shape, last_layer_all_tokens=True), blob)
    full = st.sp_forward(*args).double().cpu().numpy()
    x_full = st.read_activation(st.sp_forward_partial(*args, 1), "x", T, len(lengths), shape.K)
    st.close()
    assert np.array_equal(x[:, :len(lengths)], x_full[:, cu[:-1]])       # the first tokens' rows are the LayerNorm's, bit for bit
    bound = {"bf16": 3e-2, "fp8": 1e-1}[dtype] * (1 if offset == 0 else 2)
    assert np.isfinite(got).all() and np.abs(got - full).max() / np.abs(full).max() < bound
    if dtype == "bf16":
        ow = torch.from_numpy(blob).bfloat16().float().numpy()
        cfg = OracleConfig(shape.K, shape.layers, shape.hidden, shape.heads, shape.ffn, shape.vocab, shape.max_pos, shape.classes, shape.ln_eps)
        want = oracle64.forward(cfg, ow, ids[:cu[n]], cu[:n + 1], shape.K)
        err = [np.abs(g[:n] - want).max() / np.abs(want).max() for g in (got, full)]
        assert err[0] < bound and err[1] < bound, err


# 8192 tokens or more, as above.  Scores spread about 4 (as in the stage test of the fold on normalised rows), first tokens that have all the
# weight (sequences of one token), and rows whose mean is several times their deviation
@pytest.mark.parametrize("hidden", [256, 512, 768, 1024])
@pytest.mark.parametrize("offset", [0.0, 6.0, 30.0])
def test_folded_attention_on_rows_before_their_layernorm_against_the_definition(hidden, offset):
    """Its attention output against keys and values formed in fp64 from the rows before their LayerNorm (what the FFN's stages left,
    rounded to bf16 as the fold reads them), and softmax attention of the HIP path's own queries over them."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=5, layers=2, hidden=hidden, heads=hidden // 64, ffn=256, vocab=300, max_pos=256, classes=2, dtype="bf16")
    rng = np.random.default_rng(hidden)
    lengths = np.array((1,) * 200 + (2, 31, 32, 33, 64, 65, 256, 129) + (60,) * 130, np.int32)
    T, B = int(lengths.sum()), len(lengths)
    assert T >= 8192
    ids = synth.make_ids(rng, T, shape.vocab)
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True, qk_std=1.92 / hidden ** 0.5)
    v = synth.student_views(blob, shape, 0)
    v["l0.b2"][:] += offset
    cu = sp.sp_pack(lengths)
    args = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), 256, 1
    st = sp.Students(sp.config_from_shape(shape), blob)
    st.sp_forward(*args)
    q, got, x_first = (st.read_activation(st.workspace(T, B), n, T, B, 1)[0][:B] for n in ("first_q", "first_att", "x"))
    ws = st.sp_forward_partial(*args, 1)
    x1, g, x_all = (st.read_activation(ws, n, T, B, 1)[0] for n in ("x1", "g", "x"))
    st.close()
    assert np.array_equal(x_first, x_all[cu[:-1]])           # (what such a call leaves in x)
    w = {n: (torch.from_numpy(a).bfloat16() if a.ndim == 2 else torch.from_numpy(a)).double().numpy() for n, a in v.items()}
    u64 = torch.from_numpy(x1 + g @ w["l0.W2"] + w["l0.b2"])
    u = u64.bfloat16().double().numpy()
    d = u - u.mean(1, keepdims=True)
    x = d / np.sqrt((d * d).mean(1, keepdims=True) + shape.ln_eps) * w["l0.ln2_g"] + w["l0.ln2_b"]
    keys, values = x @ w["l1.Wk"] + w["l1.bk"], x @ w["l1.Wv"] + w["l1.bv"]
    want = np.empty((B, hidden))
    for b in range(B):
        r = slice(cu[b], cu[b + 1])
        s = np.einsum("hd,thd->ht", q[b].reshape(-1, 64), keys[r].reshape(-1, shape.heads, 64)) / 8
        p = np.exp(s - s.max(1, keepdims=True))
        want[b] = np.einsum("ht,thd->hd", p / p.sum(1, keepdims=True), values[r].reshape(-1, shape.heads, 64)).reshape(-1)
    assert np.abs(got - want).max() / np.abs(want).max() < 1.2e-2
    # One token: its weight is one, so the output has two roundings to bf16 (weighted row, value), 2^-8 0.378 of a vector's norm each and
    # 2.1e-3 in quadrature.  One of the weight itself would be common to the whole vector: up to 3.9e-3 more.
    # (Rows of which fp32 sums, within 2^-20, may round another way than fp64 ones are not looked at: a step of a mean of 30 is large.)
    sure = ((u64 * (1 + 2.0 ** -20)).bfloat16() == (u64 * (1 - 2.0 ** -20)).bfloat16()).all(1).numpy()[:200]
    one = (np.linalg.norm(got[:200] - want[:200], axis=1) / np.linalg.norm(want[:200], axis=1))[sure]
    assert len(one) > 50 and one.max() < 3e-3, (len(one), one.max())


# one, two and three looks at the boundaries; a row and several rows per wave; runs of the shortest sequences, a last wave that is partly filled
@pytest.mark.parametrize("lengths", [(7,), (1,) * 64, (3, 1) * 32 + (2,), (1,) * 4095 + (9,), (1,) * 2500 + (5, 2) * 2100 + (64,) * 3, (63, 64, 1) * 100])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_embedding_finds_the_sequence_of_every_row(lengths, dtype):
    """Token row + position row, then LayerNorm, of every row in fp64; the bound of the stage tests (one rounding of the output)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=1, hidden=128, heads=2, ffn=128, vocab=100, max_pos=64, classes=2, dtype=dtype)
    rng = np.random.default_rng(len(lengths))
    cu, T, B = sp.sp_pack(np.array(lengths, np.int32)), sum(lengths), len(lengths)
    ids, blob = synth.make_ids(rng, T, shape.vocab), synth.make_weights(rng, shape, std=0.08, ln_random=True)
    st = sp.Students(sp.config_from_shape(shape), blob)
    x = st.read_activation(st.sp_forward_partial(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), max(lengths), 2, 0), "x", T, B, 2)
    pos = np.arange(T) - np.repeat(cu[:-1], lengths)
    for m in range(2):
        v = synth.student_views(blob, shape, m)
        tab = {n: (torch.from_numpy(v[n]).bfloat16() if dtype == "bf16" else torch.from_numpy(v[n])).double().numpy() for n in ("tok_emb", "pos_emb")}
        u = tab["tok_emb"][ids] + tab["pos_emb"][pos]
        d = u - u.mean(1, keepdims=True)
        want = d / np.sqrt((d * d).mean(1, keepdims=True) + shape.ln_eps) * v["emb_ln_g"] + v["emb_ln_b"]
        err = np.abs(x[m][:T] - want).max() / np.abs(want).max()
        assert err < (1.2e-2 if dtype == "bf16" else 2e-5), f"student {m}: {err:.3e}"
    st.close()


# few long sequences: parts of up to 128 tokens that are dealt evenly (one to eight of them, and a sequence of one part), on rows after
# their LayerNorm and (the last lengths) before it, at every width
@pytest.mark.parametrize("hidden", [256, 512, 768, 1024])
@pytest.mark.parametrize("lengths", [(1024, 128, 129, 255, 256, 257), (512, 513, 1), (383, 385, 640, 97, 96), (340,) * 31])
def test_folded_attention_of_sequences_in_parts(oracle64, hidden, lengths):
    """Logits against the oracle, and the attention output of the first tokens beside that of the same sequences in a call of many short
    ones, which takes each by one workgroup: rounded weights and rows on either side (the bound of the stage tests)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=4, layers=2, hidden=hidden, heads=hidden // 64, ffn=512 if hidden == 1024 else 256, vocab=60, max_pos=1024, classes=2,
                               dtype="bf16")
    n, T, item = len(lengths), sum(lengths), shape.heads * (hidden + 2) * 4
    # (what makes the first call split: few sequences of all students, a mean of 256 tokens, and room for the parts in the FFN's activations)
    assert 4 * n <= 128 and T >= max(1024, 256 * n) and (T // 128 + n) * item <= -(-T // 256) * 256 * shape.ffn * 2
    assert (T >= 8192 and T * 4 * hidden > (10 if hidden == 256 else 16) << 20) == (n == 31)        # (and the rows those before their LayerNorm)
    _run(oracle64, shape, lengths, (1, 4), hidden + len(lengths))
    rng = np.random.default_rng(hidden)
    both = lengths + (3,) * (4 * len(lengths))
    blob = synth.make_weights(rng, shape, std=0.04, ln_random=True, qk_std=1.92 / hidden ** 0.5)
    ids, out = synth.make_ids(rng, sum(both), shape.vocab), []
    assert sum(both) < 256 * len(both)
    for lens in (lengths, both):
        st, cu = sp.Students(sp.config_from_shape(shape), blob), sp.sp_pack(np.array(lens, np.int32))
        T, B = int(cu[-1]), len(lens)
        st.sp_forward(torch.from_numpy(ids[:T]).cuda(), torch.from_numpy(cu).cuda(), max(lens), shape.K)
        out.append(st.read_activation(st.workspace(T, B), "first_att", T, B, shape.K)[:, :len(lengths)])
        st.close()
    assert np.abs(out[0] - out[1]).max() / np.abs(out[1]).max() < 1.2e-2
