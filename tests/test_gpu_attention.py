"""All-token attention (bf16 path) at the edges of its key tiles and work items.  Needs an MI355X."""
import numpy as np
import pytest
import torch

from paper_2408_12526_amd import synth

pytestmark = pytest.mark.gpu

CASES = {
    # a tile's and an item's last token and the one behind it, behind sequences that shift the first key tile by 0 to 7 tokens
    "tile_edges": (1, 56, 57, 1, 58, 63, 64, 2, 65, 71, 72, 3, 120, 121, 127, 128, 129, 1, 136, 192, 193, 255, 256, 1, 257, 32, 33),
    # one, two and three looks at the boundaries; empty work items
    "64_sequences": (3, 130, 1, 40) * 16,
    "65_sequences": (3, 130, 1, 40) * 16 + (129,),
    "4097_sequences": (1,) * 2000 + (2,) * 2096 + (300,),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("qk_std", [0.12, 0.6])         # 0.6: scores that outgrow the first block's maximum by far more than 2^8
def test_attention_at_tile_and_item_edges(oracle64, name, qk_std):
    """Attention output against the oracle's attention on the queries, keys and values that the projection left: one rounding of
    the probabilities and one of the output, relative to the tensor's largest magnitude (the bound of the stage tests)."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=1, hidden=128, heads=2, ffn=128, vocab=100, max_pos=320, classes=2, dtype="bf16")
    lengths = np.array(CASES[name], np.int32)
    rng = np.random.default_rng(len(lengths))
    ids, blob = synth.make_ids(rng, int(lengths.sum()), shape.vocab), synth.make_weights(rng, shape, std=0.08, qk_std=qk_std)
    st = sp.Students(sp.config_from_shape(shape), blob)
    cu, k, H = sp.sp_pack(lengths), shape.K, shape.hidden
    T, B = int(cu[-1]), len(lengths)
    ws = st.sp_forward_partial(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k, 1)
    qkv, att = st.read_activation(ws, "qkv", T, B, k), st.read_activation(ws, "att", T, B, k)
    pick = range(B) if B < 200 else np.r_[0:50, 1980:2020, B - 50:B]
    for m in range(k):
        for b in pick:
            a = qkv[m][cu[b]:cu[b + 1]]
            want = oracle64.attention(a[:, :H], a[:, H:2 * H], a[:, 2 * H:], shape.heads)
            err = np.abs(att[m][cu[b]:cu[b + 1]] - want).max() / np.abs(want).max()
            assert err < 1.2e-2, f"student {m}, sequence {b} of {lengths[b]} tokens at {cu[b]}: {err:.3e}"
    st.close()


# pairs of student and head that an XCD has to itself and pairs left over: 2 and none, 2, 4 and none, 10, 18, 12 (four left), 24
@pytest.mark.parametrize("hidden,K", [(128, 1), (128, 2), (128, 4), (128, 5), (384, 3), (768, 1), (768, 2)])
@pytest.mark.parametrize("lengths", [(256,), (129, 127), (320, 1, 190, 2, 300, 128, 57, 250, 256, 31), (319,) * 27])
def test_long_sequences_by_pairs_of_student_and_head(oracle64, hidden, K, lengths):
    """Means of 128 tokens and more: every (student, head, item) is taken once, whichever way it reaches its XCD.  Bound as above."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=K, layers=1, hidden=hidden, heads=hidden // 64, ffn=128, vocab=100, max_pos=320, classes=2, dtype="bf16")
    lengths = np.array(lengths, np.int32)
    rng = np.random.default_rng(hidden + K)
    ids, blob = synth.make_ids(rng, int(lengths.sum()), shape.vocab), synth.make_weights(rng, shape, std=0.08, qk_std=1.36 / hidden ** 0.5)
    st = sp.Students(sp.config_from_shape(shape), blob)
    cu, H = sp.sp_pack(lengths), hidden
    T, B = int(cu[-1]), len(lengths)
    ws = st.sp_forward_partial(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), K, 1)
    qkv, att = st.read_activation(ws, "qkv", T, B, K), st.read_activation(ws, "att", T, B, K)
    for m in range(K):
        for b in range(B) if B < 20 else (0, 13, B - 1):
            a = qkv[m][cu[b]:cu[b + 1]]
            want = oracle64.attention(a[:, :H], a[:, H:2 * H], a[:, 2 * H:], shape.heads)
            err = np.abs(att[m][cu[b]:cu[b + 1]] - want).max() / np.abs(want).max()
            assert err < 1.2e-2, f"student {m}, sequence {b} of {lengths[b]} tokens at {cu[b]}: {err:.3e}"
    st.close()


# every length of the short part at every offset of the first key block, alone, beside longer sequences, and (few of them) in the general part
@pytest.mark.parametrize("hidden", [128, 384, 768])      # two, six and twelve heads: waves of a head group without a head
def test_short_sequences_alone_and_beside_longer_ones(oracle64, hidden):
    """Against the definition as above, and the same bits in each of the three: blocks of keys and their order are the same."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=1, hidden=hidden, heads=hidden // 64, ffn=128, vocab=100, max_pos=320, classes=2, dtype="bf16")
    rng = np.random.default_rng(hidden)
    few = np.array((9, 17, 25, 32, 31, 30, 29, 28, 27, 26, 24, 1), np.int32)             # 279 tokens, offsets 0 to 7
    short = np.r_[few, 1, rng.permutation(np.tile(np.arange(1, 33), 8))].astype(np.int32)
    calls = {"few, general": np.r_[few, 33], "alone": short, "mixed": np.r_[short, 33, 1, 200, 64, 3].astype(np.int32)}
    assert set((np.r_[0, np.cumsum(few)] & 7).tolist()) == set(range(8)) and calls["mixed"].sum() <= 32 * len(calls["mixed"])
    blob, ids = synth.make_weights(rng, shape, std=0.08, qk_std=1.36 / hidden ** 0.5), synth.make_ids(rng, int(calls["mixed"].sum()), shape.vocab)
    st = sp.Students(sp.config_from_shape(shape), blob)
    first, H, k = {}, hidden, shape.K
    for name, lengths in calls.items():
        lengths = lengths.astype(np.int32)
        cu, T, B = sp.sp_pack(lengths), int(lengths.sum()), len(lengths)
        ws = st.sp_forward_partial(torch.from_numpy(ids[:T]).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k, 1)
        qkv, att = st.read_activation(ws, "qkv", T, B, k), st.read_activation(ws, "att", T, B, k)
        first[name] = qkv[:, :279], att[:, :279]
        for m in range(k):
            for b in range(B):
                a = qkv[m][cu[b]:cu[b + 1]]
                want = oracle64.attention(a[:, :H], a[:, H:2 * H], a[:, 2 * H:], shape.heads)
                err = np.abs(att[m][cu[b]:cu[b + 1]] - want).max() / np.abs(want).max()
                assert err < 1.2e-2, f"{name}, student {m}, sequence {b} of {lengths[b]} tokens at {cu[b]}: {err:.3e}"
    for name in ("alone", "mixed"):
        assert all(np.array_equal(a, b) for a, b in zip(first[name], first["few, general"])), name
    st.close()


@pytest.mark.parametrize("copies", [1, 3])               # sixteen lanes per query; four
def test_fp32_attention_at_block_and_chunk_edges(oracle64, copies):
    """Blocks of eight keys, chunks of 64 and blocks of 16 or 64 queries just missed, met and passed; sharp scores.  fp32 sums of up
    to 129 terms against fp64: a few units of 2^-24 of the largest value."""
    from paper_2408_12526_amd import sp
    shape = synth.StudentShape(K=2, layers=1, hidden=128, heads=2, ffn=128, vocab=100, max_pos=160, classes=2, dtype="fp32")
    lengths = np.array((1, 7, 8, 9, 15, 16, 17, 63, 64, 65, 128, 129) * copies, np.int32)
    rng = np.random.default_rng(copies)
    ids, blob = synth.make_ids(rng, int(lengths.sum()), shape.vocab), synth.make_weights(rng, shape, std=0.08, qk_std=0.4)
    st = sp.Students(sp.config_from_shape(shape), blob)
    cu, k, H = sp.sp_pack(lengths), shape.K, shape.hidden
    T, B = int(cu[-1]), len(lengths)
    ws = st.sp_forward_partial(torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), int(lengths.max()), k, 1)
    qkv, att = st.read_activation(ws, "qkv", T, B, k), st.read_activation(ws, "att", T, B, k)
    for m in range(k):
        for b in range(B):
            a = qkv[m][cu[b]:cu[b + 1]]
            want = oracle64.attention(a[:, :H], a[:, H:2 * H], a[:, 2 * H:], shape.heads)
            err = np.abs(att[m][cu[b]:cu[b + 1]] - want).max() / np.abs(want).max()
            assert err < 2e-5, f"student {m}, sequence {b} of {lengths[b]} tokens: {err:.3e}"
    st.close()
