"""The whole-graph schedule of gnn_epoch against the partition-by-partition one: the same bits.

The sums of the two schedules are taken in the same order (partitions in schedule order, a
partition's rows in segments), so nothing is allowed to differ; the partition-by-partition epoch is
what the other tests hold against the oracle.
"""
import numpy as np
import pytest

from helpers import ring_of_blocks, small_graph
from synth import attention_vectors, features, glorot_weights, labels_and_mask, to_bf16_grid

pytestmark = pytest.mark.gpu
KEYS = ("act", "gact", "gW", "gWs", "gb")

CASES = [
    # (model, dims, n, m_draw, symmetric, k, mode, dtype, switches)
    ("gcn", (64, 64, 16), 10000, 100000, True, 4, "random", "f32", "tuned"),
    ("sage", (100, 256, 256, 47), 3000, 40000, True, 5, "lp", "f32", "tuned"),
    ("sage", (100, 256, 256, 47), 3000, 40000, True, 5, "lp", "f32", "default"),    # self terms inside the sums
    ("sage", (24, 40, 200, 9), 2000, 9000, False, 6, "random", "f32", "masked"),    # rows without entries, masked self
    ("gcn", (128, 128, 128, 172), 4000, 50000, False, 7, "lp", "f32", "tuned"),
    ("gcn", (7, 9, 5, 6), 300, 1500, True, 3, "random", "f32", "default"),          # rows of no whole vector
    ("sage", (33, 45, 61, 10), 900, 9000, False, 5, "random", "f32", "masked"),
    ("sage", (1028, 1030, 8), 200, 1500, True, 2, "random", "f32", "default"),      # column blocks, scalar rows
    ("gcn", (12, 520, 1028, 4), 300, 2500, True, 3, "random", "f32", "default"),    # column slices
    ("gcn", (36, 40, 8, 40, 12), 2500, 90000, True, 3, "lp", "f32", "tuned"),       # hubs cut into segments
    ("sage", (36, 40, 40, 12), 2500, 90000, True, 9, "lp", "f32", "default"),
    ("gcn", (64, 32, 8), 500, 4000, True, 500, "user", "f32", "tuned"),             # k = n
    ("sage", (16, 16, 8, 4), 480, 0, True, 12, "ring", "f32", "default"),           # partitions out of id order
    ("gcn", (64, 128, 64, 16), 3000, 30000, True, 4, "lp", "bf16", "tuned"),
    ("sage", (72, 136, 136, 8), 2000, 16000, True, 3, "random", "bf16", "default"),
    ("sage", (72, 136, 8), 2000, 16000, True, 3, "random", "bf16", "tuned"),
    ("gcn", (20, 50, 50, 7), 500, 3000, False, 2, "random", "bf16", "default"),     # odd widths
    ("gcn", (256, 264, 300, 16), 10000, 60000, True, 3, "random", "bf16", "default"),  # 256 x 256 tiles, ragged ends
    # attention; the model's heads per layer behind the colon
    ("gat:1x1x1", (24, 260, 30, 7), 3000, 40000, True, 5, "lp", "f32", "tuned"),
    ("gat:8x8x1", (100, 256, 256, 47), 3000, 60000, True, 4, "lp", "f32", "tuned"),  # heads side by side, in slots
    ("gat:3x2x1", (20, 36, 24, 7), 2500, 90000, True, 6, "random", "f32", "default"),  # side by side, head by head; hubs
    ("gat:4x5x1", (20, 20, 15, 7), 900, 7000, False, 7, "random", "f32", "default"),   # five and three columns a head
    ("gat:8x1", (16, 16, 5), 300, 900, True, 60, "random", "f32", "tuned"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%s-k%d-%s-%s" % (c[0], "x".join(map(str, c[1])), c[5], c[7], c[8]))
def test_whole_graph_epoch_gives_the_bits_of_the_partition_by_partition_epoch(monkeypatch, case):
    model, dims, n, m_draw, sym, k, mode, dtype, switches = case
    print("case whole %s" % (case,), flush=True)
    from paper_2605_11517_amd import Session
    model, _, heads = model.partition(":")
    user = None
    if mode == "ring":
        rowptr, colidx, user, _ = ring_of_blocks(k, n // k, seed=4)
        mode = "user"
    else:
        rowptr, colidx = small_graph(n, m_draw, seed=91, symmetric=sym, self_loops=(model == "gcn"))
        if mode == "user":
            user = np.arange(n, dtype=np.int32)[::-1].copy()
    X = features(n, dims[0], 5)
    y, _ = labels_and_mask(n, dims[-1], 0.5, 5)
    m = (np.random.default_rng(6).random(n) < 0.3).astype(np.uint8)
    w = glorot_weights(dims, 5, sage=(model == "sage"), bias_scale=0.1)
    if model == "gat":
        attention_vectors(w, 5)
        for layer, h in zip(w, heads.split("x")):
            layer["heads"] = int(h)
    if dtype == "bf16":
        X = to_bf16_grid(X)
    kw = {"tuned": dict(layer_order="auto", fuse_gather=True, masked_backward=True, keep_forward=True),
          "masked": dict(masked_backward=True), "default": {}}[switches]
    s = Session(model, dims, rowptr, colidx, k, mode, 3, X, w, y, m, dtype=dtype, user_part=user, **kw)
    out = {}
    for flag in ("0", "1"):
        monkeypatch.setenv("GNNMI_WHOLE", flag)
        s.scratch.fill_(0xFF)                       # NaN patterns: nothing may be read before it is written
        s.staging.fill_(0xFF)
        for t in s.gact + s.act:
            t.fill_(float("nan"))
        s.ctx.set_dropout(0.25, 11, 2)
        first = s.epoch()
        s.ctx.set_dropout(0.0, 0, 0)
        assert np.isfinite(first)
        out[flag] = (first, s.epoch(), s.results())
    assert out["0"][:2] == out["1"][:2]
    for key in KEYS:
        for l, (a, b) in enumerate(zip(out["0"][2][key], out["1"][2][key])):
            if a is None:
                continue
            assert np.isfinite(b).all(), (key, l)
            assert np.array_equal(a, b), (key, l, float(np.abs(a - b).max()))
