"""The one-workgroup routing plan of a decode step and the router's K-split sum,
at their edges: the fewest and most experts and choices, one token, the last
batch of the small plan (512 choices) and the first past it (65 tokens, the
three-kernel plan).  Router weights are drawn 20 times as large, so that most
rows are clear of routing near-ties and can be held to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import check_bf16, gpu_model, run_teacher_forced
from synthetic import model_weights, prompts, small_shape
from test_gpu_moe import NEAR_TIE, _router_decisions

pytestmark = pytest.mark.gpu

# (experts, top k, sequences)
CASES = [(2, 1, 1), (5, 3, 63), (64, 6, 17), (256, 8, 64), (256, 8, 65), (130, 8, 33)]


@pytest.mark.parametrize("E,k,B", CASES)
def test_routing_plan_edges_against_oracle(E, k, B):
    shape = dict(small_shape("moe16b", layers=2, vocab=512, hidden=512, intermediate=512), n_routed_experts=E,
                 num_experts_per_tok=k, moe_intermediate_size=64, n_shared_experts=0, norm_topk_prob=True)
    w = model_weights(shape, seed=51)
    for n in w:
        if n.endswith("mlp.gate.weight"):
            w[n] = (w[n].float() * 20).to(torch.bfloat16)
    ids = prompts(B, 3, shape["vocab_size"], seed=52).numpy()
    seqs, forced = [ids[b, :1 + b % 2] for b in range(B)], ids[:, 2:3]
    w64 = oracle.weights_f64(w)
    exact = oracle.teacher_forced(oracle.OracleDecoder(shape, w64), seqs, forced)
    b16 = oracle.teacher_forced(oracle.OracleDecoder(shape, w64, io_round="bf16"), seqs, forced)
    dec = _router_decisions(shape, w64, seqs, forced)
    gaps = np.array([[min(d[1] for d in dec[st][b]) for b in range(B)] for st in range(2)]) if k < E else None
    m = gpu_model(shape, w, max_batch=B, max_seq=8)
    got, _ = run_teacher_forced(m, seqs, forced)
    m.close()
    assert np.all(np.isfinite(got))
    clear = gaps >= NEAR_TIE
    assert clear.any()
    check_bf16(got[clear], exact[clear], b16[clear], f"plan E {E} k {k} B {B}", absolute=False)


@pytest.mark.parametrize("E,k", [(64, 6), (256, 8)])
def test_nan_router_logits_stay_with_their_token(E, k):
    """A token whose router logits are NaN (its embedding row is) has no expert: its
    own logits are NaN and every other sequence's are bit for bit those of a
    model whose embedding is finite, through the small plan and the large one."""
    shape = dict(small_shape("moe16b", layers=2, vocab=512, hidden=512, intermediate=512), n_routed_experts=E,
                 num_experts_per_tok=k, moe_intermediate_size=64, n_shared_experts=0)
    w = model_weights(shape, seed=53)
    bad = 511
    ids = prompts(3, 60, bad, seed=54).numpy()
    ids[1, 3] = bad
    out = []
    for nan in (True, False):
        if nan:
            w = dict(w)
            good = w["model.embed_tokens.weight"]
            w["model.embed_tokens.weight"] = good.clone()
            w["model.embed_tokens.weight"][bad] = float("nan")
        else:
            w["model.embed_tokens.weight"] = good
        m = gpu_model(shape, w, max_batch=3, max_seq=64)
        print(f"E {E} k {k} nan {nan}", flush=True)
        for n in (2, 4, 60):  # 6 and 12 tokens: the small plan; 180: the large one
            got, _ = run_teacher_forced(m, [ids[b, :n] for b in range(3)], ids[:, n - 1:n])
            out.append(got)
        m.close()
    for a, b in zip(out[:3], out[3:]):
        assert np.all(np.isfinite(b))
        np.testing.assert_array_equal(a[:, [0, 2]], b[:, [0, 2]])
    np.testing.assert_array_equal(out[0], out[3])  # the token is not among the first two
    assert np.all(np.isnan(out[1][:, 1])) and np.all(np.isnan(out[2][:, 1]))
