"""The projection GEMM's tile shapes on the GPU.  The launch picks a tile by
the output's size, so one prompt fed at growing lengths passes through all of
them: every length must give the oracle's logits and, position by position, the
bits of the longest prompt (each output is one ascending sum over k, whatever
the tile)."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import check_bf16, gpu_model, run_teacher_forced
from synthetic import model_weights, prompts, small_shape

pytestmark = pytest.mark.gpu

# tile edges (32, 64, 128, 256 tokens), one past and one before them
LENS = [1, 2, 31, 32, 33, 63, 65, 97, 128, 129, 255, 257, 390, 600]

SHAPES = {
    # K of an odd number of 32-deep units per K half (hidden and intermediate
    # 34 and 66 units in two halves): stages of one unit only; odd vocabulary
    "odd_units": ("1b", dict(layers=1, vocab=3001, hidden=1088, intermediate=2112)),
    # even units, biases, head dimension 128, N with a remainder in every tile
    "even_units_bias": ("7b", dict(layers=1, vocab=2016, hidden=1152, intermediate=1216)),
    # an output wide enough for the 256-token tiles
    "wide": ("1b", dict(layers=1, vocab=5000, hidden=512, intermediate=20480)),
}


@pytest.mark.parametrize("case", list(SHAPES))
def test_every_tile_shape_gives_the_same_bits_and_the_oracles_logits(case):
    base, ov = SHAPES[case]
    shape = small_shape(base, **ov)
    w = model_weights(shape, seed=41)
    ids = prompts(1, max(LENS), shape["vocab_size"], seed=42)[0]
    m = gpu_model(shape, w, max_batch=1, max_seq=max(LENS))
    flat = ids.to("cuda")
    full, _ = m.prefill(flat, [0, max(LENS)], all_logits=True)
    full = full.cpu()
    for n in LENS[:-1]:
        lg, nxt = m.prefill(flat[:n].contiguous(), [0, n], all_logits=True)
        lg = lg.cpu()
        assert torch.equal(lg, full[:n]), f"{n} tokens: {(lg - full[:n]).abs().max():.3e} off the longest prompt"
        assert int(nxt[0]) == int(lg[-1].argmax())
    m.close()
    n = 129
    w64 = oracle.weights_f64(w)
    exact = oracle.OracleDecoder(shape, w64).extend(0, ids[:n].numpy(), all_logits=True)
    b16 = oracle.OracleDecoder(shape, w64, io_round="bf16").extend(0, ids[:n].numpy(), all_logits=True)
    # the band around the bf16 storage error is the bar: at these widths that
    # error alone (mean 2.8e-3) is past the absolute 2e-3
    check_bf16(full[:n].double().numpy(), np.asarray(exact), np.asarray(b16), f"tiles {case}", absolute=False)


# decode batches above 64: the residual projections' K splits (the partials are
# summed by the next normalization) and the argmax over several column chunks;
# widths, K of even and odd unit counts, an odd vocabulary past two chunks
# (and, head dimension 128, decode attention of more workgroups than CUs)
WIDE = {
    "split_deep": (66, "1b", dict(layers=2, vocab=9001, hidden=512, intermediate=8192)),
    "odd_units": (129, "1b", dict(layers=2, vocab=4097, hidden=576, intermediate=1088)),
    "hd128_bias": (70, "7b", dict(layers=2, vocab=1000, hidden=512, intermediate=1024)),
}


@pytest.mark.parametrize("case", list(WIDE))
def test_decode_above_64_sequences(case):
    B, base, ov = WIDE[case]
    shape = small_shape(base, **ov)
    w = model_weights(shape, seed=43)
    V = shape["vocab_size"]
    ids = prompts(B, 6, V, seed=44).numpy()
    seqs = [ids[b, :1 + b % 4] for b in range(B)]
    forced = ids[:, 4:6]
    w64 = oracle.weights_f64(w)
    exact = oracle.teacher_forced(oracle.OracleDecoder(shape, w64), seqs, forced)
    b16 = oracle.teacher_forced(oracle.OracleDecoder(shape, w64, io_round="bf16"), seqs, forced)
    m = gpu_model(shape, w, max_batch=B, max_seq=8)
    got, toks = run_teacher_forced(m, seqs, forced)
    m.close()
    check_bf16(got, exact, b16, f"decode above 64 {case}", absolute=False)
    np.testing.assert_array_equal(toks.T, got.argmax(-1))


def test_split_decode_attention_of_many_workgroups():
    """33 sequences x 8 kv heads x 2 key splits: more workgroups than CUs (the
    4-wavefront form), contexts that end inside either split; the first and the
    last sequence against the oracle."""
    lens = [1700 if b in (0, 32) else 3 + b for b in range(33)]
    shape = small_shape("1b", layers=2, vocab=1000, hidden=512, intermediate=1024)
    w = model_weights(shape, seed=45)
    ids = prompts(33, 1702, shape["vocab_size"], seed=46).numpy()
    seqs, forced = [ids[b, :n] for b, n in enumerate(lens)], ids[:, 1700:1702]
    m = gpu_model(shape, w, max_batch=33, max_seq=3100)
    got, _ = run_teacher_forced(m, seqs, forced)
    m.close()
    pick = [0, 32]
    w64 = oracle.weights_f64(w)
    part = [seqs[b] for b in pick]
    exact = oracle.teacher_forced(oracle.OracleDecoder(shape, w64), part, forced[pick])
    b16 = oracle.teacher_forced(oracle.OracleDecoder(shape, w64, io_round="bf16"), part, forced[pick])
    check_bf16(got[:, pick], exact, b16, "split decode attention", absolute=False)
    assert np.all(np.isfinite(got))
