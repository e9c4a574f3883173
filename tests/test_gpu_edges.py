"""Edges of the decode kernel's tiles and hand-over, against the CPU oracle.

Attention works on tiles of 16 K/V rows over eight waves, with one, two or
three tiles per wave and pass (by head size and query group), and cuts every
fp32 query into three bf16 parts; a wave's weight stream runs on from one task
into the next, with rings shorter and longer than a task; a task's epilogue is
prepared ahead for up to 64 items.  Bar: the greedy token, and logits within
2e-4 of the largest logit, 5e-3 where decoding starts below position 8.  All
sums are fp32 (1e-7 to 4e-6 of the largest logit where nothing else differs);
what is left are appended K / V elements whose bf16 rounding the other order of
summation flips.  A flip is 2^-8 of one of the d elements of a row that weighs
about 1 / (pos + 1): some 2^-8 / sqrt(64) = 4.9e-4 of an attention output at
position 0, a few of them at once where wide inputs make flips more likely, and
2^-8 / sqrt(64) / 9 = 5e-5 from position 8 on.  The largest seen are 1.05e-3
(hidden 7232, position 3) and 1.05e-4 (hidden 7232, position 101)."""
import numpy as np
import pytest

import oracle
import synth
from synth.device import config_kwargs, kv_to_device, weights_to_device

pytestmark = pytest.mark.gpu

# name: heads, kv_heads, head_dim  (query groups 1, 3, 4, 5, 8 on both head sizes)
HEADS = {"g1_64": (2, 2, 64), "g3_64": (6, 2, 64), "g8_64": (8, 1, 64), "g4_128": (4, 1, 128), "g5_128": (5, 1, 128),
         "g8_128": (8, 1, 128)}


def shape_of(heads, hidden=256, inter=320, vocab=1000, layers=2, tied=False):
    nq, nkv, d = HEADS[heads]
    return synth.get("tiny").with_(name=f"edge_{heads}_{hidden}_{inter}_{vocab}", hidden=hidden, n_layers=layers,
                                   n_heads=nq, n_kv_heads=nkv, head_dim=d, intermediate=inter, vocab=vocab,
                                   tied_embeddings=tied)


def check(cfg, fmt, pos, tuning=None, group=0, steps=1, edit=None):
    import torch
    from paper_2606_09682_amd import amk
    w = synth.make_weights(cfg, seed=3)
    if fmt == "w8a16":
        synth.add_w8a16(w)
    if fmt == "w4a16":
        synth.add_w4a16(w, group=group)
    kv = synth.make_kv_cache(cfg, pos, seed=1, max_seq=pos + steps)
    dec = amk.Decoder(amk.make_config(**config_kwargs(cfg, fmt, pos + steps, group)), weights_to_device(w, fmt),
                      amk.amk_tuning_t(*tuning) if tuning else None)
    model = oracle.OracleModel(w, fmt, np.float32)
    if edit:
        edit(model, kv)
    dkv = kv_to_device(kv)
    logits = torch.empty((cfg.vocab + 3) // 4 * 4, dtype=torch.float32, device="cuda")
    ref_kv = kv.copy()
    tok = 1
    for i in range(steps):
        dec.step(tok, pos + i, dkv, logits)
        got = dec.next_token()
        ref = oracle.decode_step(model, tok, pos + i, ref_kv)
        err = float(np.max(np.abs(logits.cpu().numpy()[:cfg.vocab] - ref)) / np.max(np.abs(ref)))
        print(f"[edges] {cfg.name} {fmt} pos {pos + i}: relative logit error {err:.2e}", flush=True)
        assert err <= (2e-4 if pos >= 8 else 5e-3)
        assert got == oracle.argmax_first(ref)
        tok = got
    assert dec.status() == amk.AMK_OK
    dec.close()


@pytest.mark.parametrize("heads", list(HEADS))
@pytest.mark.parametrize("pos", [14, 15, 16, 126, 128, 255, 256, 383, 384, 800])
def test_attention_tile_edges(heads, pos):
    """One task holds all rows of a KV group (short schedule): whole and partial
    tiles, the last wave with a tile, one, two and more passes."""
    check(shape_of(heads), "bf16", pos, tuning=(0, 0, 0, 0, 1 << 30, -1, 0))


@pytest.mark.parametrize("heads", ["g3_64", "g8_64", "g4_128", "g8_128"])
@pytest.mark.parametrize("splits,pos", [(2, 31), (3, 400), (64, 500), (7, 700), (1, 40)])
def test_split_and_merge_edges(heads, splits, pos):
    """Split records of ragged lengths and their merge (long schedule); splits
    past the last row; rows loaded non-temporally (96 and more a split)."""
    check(shape_of(heads), "bf16", pos, tuning=(splits, 0, 0, 0, -1, -1, 0))


@pytest.mark.parametrize("fmt,group", [("bf16", 0), ("w8a16", 0), ("w4a16", 32), ("w4a16", 64)])
@pytest.mark.parametrize("hidden,inter,vocab", [(256, 320, 40), (1088, 4160, 3001), (7232, 1088, 520)])
def test_stream_and_epilogue_edges(fmt, group, hidden, inter, vocab):
    """Ranges shorter and longer than the ring, short last granules, LM-head
    tasks of one row and of several, and a hidden size whose RMSNorm gains do not
    all fit a wave's preload; steps from position 0 (tiny, then short schedule),
    and over a filled cache, under the bar of later positions."""
    check(shape_of("g3_64", hidden, inter, vocab), fmt, 0, group=group, steps=8)
    check(shape_of("g3_64", hidden, inter, vocab), fmt, 100, group=group, steps=2)


@pytest.mark.parametrize("rows", [2, 24, 64, 66, 128, 130])
@pytest.mark.parametrize("fmt", ["bf16", "w8a16"])
def test_task_size_edges(fmt, rows):
    """Many small tasks a queue, and gate/up tasks on both sides of the 64 items
    an epilogue is prepared for (a row pair is one item): 1, 8, 8, 33, 64 and 64
    or 65 of them under these row caps."""
    check(shape_of("g4_128", 512, 17408 if rows > 64 else 2048, 20000), fmt, 20, tuning=(0, 0, rows, 0, 0, 0, 0))


@pytest.mark.parametrize("fmt,group", [("bf16", 0), ("w8a16", 0), ("w4a16", 32)])
@pytest.mark.parametrize("pos", [3, 40])
@pytest.mark.parametrize("op,assign", [("qkv", 0), ("residual", 0), ("residual", 1)])
def test_large_task_epilogues(op, assign, pos, fmt, group):
    """q/k/v tasks of 96 row pairs (136 KV heads) and O / down tasks of 64 and 65
    rows (hidden 16416), in the tiny and the short schedule; with the queues
    assigned by cost, O and down tasks of one queue own different rows, so the
    residual is not the queue's own."""
    cfg = shape_of("g1_64", 16416 if op == "residual" else 256)
    if op == "qkv":
        cfg = cfg.with_(name="edge_136_heads", n_heads=136, n_kv_heads=136)
    check(cfg, fmt, pos, tuning=(0, 0, 0, 0, 0, 0, assign), group=group)


@pytest.mark.parametrize("pos", [40, 300])
def test_attention_scratch_in_activation_region(pos):
    """A SwiGLU width that leaves no room for the attention scratch beside the
    activation vector (row cap 2): it lies behind the queries inside it, for the
    inline attention and for splits and their merge."""
    check(shape_of("g1_64", 256, 35840, 1000, layers=1), "bf16", pos, tuning=(0, 0, 2, 0, 0, -1, 0))


def test_activation_past_the_room_for_a_task_is_refused():
    """Widths that were refused for lack of LDS stay refused."""
    from paper_2606_09682_amd import amk
    with pytest.raises(amk.AmkError) as e:
        check(shape_of("g1_64", 256, 30720, 1000, layers=1), "bf16", 40)
    assert e.value.status == amk.AMK_ERR_UNSUPPORTED


def mask_rows(model, kv, pos, rows):
    """Makes every query head of layer 0 score the cache rows `rows` minus infinity at `pos` (token 1): one
    element of each is an infinity, where all queries of the KV group have the same sign."""
    cfg, p = model.cfg, "layers.0."
    h = oracle.rmsnorm(model.embed_row(1), model.vec(p + "attn_norm"), cfg.rms_eps)
    q = oracle.linear(model.mat(p + "wq"), h).reshape(cfg.n_kv_heads, -1, cfg.head_dim)
    q = oracle.rope(q, pos, cfg.rope_theta)
    for g in range(cfg.n_kv_heads):
        least = np.where(np.abs(np.sign(q[g]).sum(0)) == len(q[g]), np.abs(q[g]).min(0), 0)
        d = int(np.argmax(least))
        assert least[d] > 1e-3
        kv[0, 0, g, rows, d] = 0xff80 if q[g, 0, d] > 0 else 0x7f80


@pytest.mark.parametrize("heads", ["g1_64", "g3_64", "g4_128", "g5_128"])
@pytest.mark.parametrize("rows", ["one", "some", "a tile", "a wave"])
def test_infinite_k_rows_have_no_weight(heads, rows):
    """A K row with a score of minus infinity has weight 0 and the others keep
    theirs, in one task of a KV group (short schedule)."""
    pos = 450
    which = {"one": [7], "some": list(range(0, pos, 3)), "a tile": list(range(16, 32)),
             "a wave": [r for r in range(pos) if r // 16 % 8 == 2]}[rows]
    check(shape_of(heads), "bf16", pos, tuning=(0, 0, 0, 0, 1 << 30, -1, 0),
          edit=lambda model, kv: mask_rows(model, kv, pos, which))


@pytest.mark.parametrize("heads", ["g1_64", "g3_64", "g4_128", "g5_128"])
@pytest.mark.parametrize("splits,masked", [(4, "a split"), (4, "across splits"), (16, "a split"), (16, "across splits")])
def test_infinite_k_rows_of_a_split_have_no_weight(heads, splits, masked):
    """A split whose rows all score minus infinity adds nothing to the merge
    (long schedule)."""
    pos = 450
    chunk = (pos + splits) // splits
    which = list(range(chunk, 2 * chunk)) if masked == "a split" else list(range(0, pos, 5))
    check(shape_of(heads), "bf16", pos, tuning=(splits, 0, 0, 0, -1, -1, 0),
          edit=lambda model, kv: mask_rows(model, kv, pos, which))


@pytest.mark.parametrize("heads", ["g1_64", "g3_64", "g4_128"])
@pytest.mark.parametrize("rows", [[0], [3], [0, 1, 2], [4, 6]])
def test_infinite_k_rows_at_the_first_positions(heads, rows):
    """The same in the tiny schedule, also before the first row with a weight."""
    check(shape_of(heads), "bf16", 7, tuning=(0, 0, 0, 0, 0, 8, 0),
          edit=lambda model, kv: mask_rows(model, kv, 7, rows))


def test_row_cap_that_fills_the_lds():
    """544 heads of 64 under a row cap of 384: the activation vector, a task of
    the row cap (192 q/k/v row pairs) and the staged records all fit."""
    cfg = synth.get("tiny").with_(name="edge_544_heads", hidden=256, n_layers=1, n_heads=544, n_kv_heads=136,
                                  head_dim=64, intermediate=320, vocab=1000)
    check(cfg, "bf16", 20, tuning=(0, 0, 384, 0, 0, 0, 0))


@pytest.mark.parametrize("heads", ["g1_64", "g4_128", "g8_128"])
@pytest.mark.parametrize("splits,pos", [(0, 65536), (0, 140001), (2, 140001)])
def test_contexts_past_an_offset_window(heads, splits, pos):
    """Rows are addressed by 32-bit offsets from bases that move on every 65536
    rows of a task: one task of a group (short schedule) and splits."""
    check(shape_of(heads, layers=1), "bf16", pos, tuning=(splits, 0, 0, 0, -1 if splits else 1 << 30, -1, 0))
