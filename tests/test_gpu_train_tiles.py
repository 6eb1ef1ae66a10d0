"""Edges of the training step's tiles, against the float64 oracle.

The attention backward's workgroups own 128 queries or keys of a sequence and
read 32-row tiles; the weight-gradient GEMM reads 32 token rows per k-tile
(its last one masked where the token count is no multiple of 32) and writes
256-row, 256-column tiles clipped to the weight; the logits projection leaves
softmax partials per 64 columns (the last one short where the vocabulary is no
multiple of 64); RMSNorm's backward holds a row in registers in four widths
(hidden up to 1024, 2048, 4096, 8192) and reads wider rows twice.  The shapes
stand on both sides of each of these.

The sizes of a real step take other forms of the GEMMs: 256 x 256 tiles for the
fused QKV, gate/up, logits and gated-activation-gradient epilogues, and weight
gradients split over the tokens, their partials summed in each of the three row
orders.  REACHES names these for the cases that stand for them (a CPU test holds
the launch rules to it).

The gradients' bars are those of the gradient test over ordinary shapes,
derived there, except the element-wise one of hidden 8256: its logits are the
largest (see the loss) and its tensors have up to 1.06M elements.  An element's
error is a sum of many independent roundings, so close to normal with the
tensor's relative L2 error as its spread; the largest of n such errors is about
sqrt(2 ln n) spreads, and with the L2 bar of 3e-2 that is 15.8% of the scale for
1.06M elements (measured 12.7%, at a relative L2 error of 1.7e-2).  The loss bar there (2e-3 at hidden 512 to 896) grows with
sqrt(hidden): a logit sums hidden products of a normalized activation (rms 1)
and a weight of fixed spread, each rounded with a relative error up to 2^-9,
so its error has a spread proportional to sqrt(hidden), and the loss averages
those of a few tens of tokens.  Measured: 8e-5 at 512, 6e-4 at 1088, 4.2e-3 at
8256 (bar 6.1e-3).
"""
import numpy as np
import pytest
import torch

import oracle
from parity_util import gpu_model, pack
from synthetic import model_weights, prompts, small_shape
from test_gpu_train import ULP, _targets, check_gradient, check_token_rows

pytestmark = pytest.mark.gpu

# name: base, heads, kv heads, hidden, intermediate, vocabulary, lengths
CASES = {
    "hd64_128_row_edges": ("1b", 8, 2, 512, 320, 1003, [127, 128, 129, 255, 2]),
    "hd128_128_row_edges": ("7b", 4, 2, 640, 192, 321, [129, 31, 257]),
    "hidden_1088": ("1b", 4, 4, 1088, 64, 130, [40, 5]),
    "hidden_2112": ("7b", 2, 1, 2112, 128, 191, [33, 30]),
    "hidden_4160": ("1b", 2, 1, 4160, 64, 129, [31, 1]),
    "hidden_8256": ("1b", 2, 2, 8256, 64, 65, [21, 12]),
    # odd token counts, no multiple of 32: the last of the token splits is masked
    "tiles_256_tied": ("1b", 8, 2, 512, 8192, 12001, [400, 301, 400]),
    "tiles_256_bias": ("7b", 40, 8, 512, 6144, 12001, [300, 257, 391, 301]),
    "token_splits_8": ("1b", 2, 1, 128, 128, 130, [258] * 15 + [257]),
}
# (part of a kernel's name, its K or token splits): GEMM epilogues 3 logits with
# softmax partials, 4 QKV with rotation, 6 gate/up, 7 gated-activation gradient;
# weight-gradient row orders 0 plain, 1 QKV, 2 gate/up
REACHES = {
    "tiles_256_tied": [("gemm_bf16_256_kernel<3, false, true>", 1), ("gemm_bf16_256_kernel<7, false, true>", 1)]
                      + [(f"gemm_tn_256_kernel<{r}", 2) for r in range(3)],
    "tiles_256_bias": [(f"gemm_bf16_256_kernel<{e}, false, true>", 1) for e in (3, 4, 6)]
                      + [(f"gemm_tn_256_kernel<{r}", 2) for r in range(3)],
    "token_splits_8": [(f"gemm_tn_256_kernel<{r}", 8) for r in range(3)],
}


def check_wide(name: str, g: np.ndarray, r: np.ndarray):
    """check_gradient with the largest of n normal errors as the element-wise bar."""
    assert np.all(np.isfinite(g)), name
    scale = np.full(r.shape, float(np.sqrt(np.mean(r * r))))
    if r.ndim == 2:
        scale = np.maximum(scale, np.sqrt(np.mean(r * r, axis=1, keepdims=True)))
    err = np.abs(g - r)
    assert np.all(err <= 3e-2 * np.sqrt(2 * np.log(r.size)) * scale + 4 * ULP * np.abs(r)), name
    rel = float(np.linalg.norm(g - r) / np.linalg.norm(r))
    assert rel < 3e-2, (name, rel)
    return rel, float((err / scale).max())


@pytest.mark.parametrize("case", list(CASES))
def test_tile_edges_against_oracle(case):
    base, heads, kv, hidden, inter, vocab, lens = CASES[case]
    shape = small_shape(base, layers=1, vocab=vocab, hidden=hidden, intermediate=inter)
    shape.update(num_attention_heads=heads, num_key_value_heads=kv)
    w = model_weights(shape, seed=81)
    ids = prompts(len(lens), max(lens), vocab, seed=82).numpy()
    seqs = [ids[i, :n] for i, n in enumerate(lens)]
    tg = _targets(seqs, vocab, seed=83)
    ref_loss, ref = oracle.loss_and_grads(shape, oracle.weights_f64(w), seqs, tg)
    m = gpu_model(shape, w, max_batch=len(lens), max_seq=max(lens))
    grads = {k: torch.full(tuple(v.shape), float("nan"), dtype=torch.float32, device="cuda") for k, v in w.items()}
    print(f"{case}: {sum(lens)} tokens", flush=True)
    loss = m.loss_and_grads(*pack(seqs), torch.as_tensor(np.concatenate(tg).astype(np.int32)).to("cuda"), grads)
    torch.cuda.synchronize()
    got = float(loss.item())
    print(f"{case}: loss {got:.6f} vs oracle {ref_loss:.6f}")
    assert abs(got - ref_loss) < 2e-3 * max(1.0, (hidden / 896) ** 0.5)
    for name, r in ref.items():
        rel, el = (check_wide if hidden > 8192 else check_gradient)(name, grads[name].cpu().double().numpy(), r)
        print(f"  {name}: relative L2 {rel:.2e}, largest element error {el:.2e} x scale")
    emb = "model.embed_tokens.weight"
    check_token_rows(grads[emb].cpu().double().numpy(), ref[emb], np.concatenate(seqs))
    m.close()
