"""What the library's host code launches, without a GPU: tests/recorded_hip.cpp
stands in for the HIP runtime, drives the C ABI through one scenario per run
and writes every launch, allocation and attribute call down."""
import os
import subprocess
from collections import namedtuple

import pytest

from paper_2608_19889_amd import axon, build
from synthetic import MODEL_SHAPES
from test_gpu_train_tiles import CASES, REACHES

HERE = os.path.dirname(os.path.abspath(__file__))
Launch = namedtuple("Launch", "device capture lds start stop gx gy kernel")
Limit = namedtuple("Limit", "device capture lds kernel")


@pytest.fixture(scope="session")
def recorder(tmp_path_factory):
    """scenario name -> its events: Launch and Limit tuples, and (kind, ...) tuples."""
    axon.lib()
    exe = str(tmp_path_factory.mktemp("recorded") / "recorded_hip")
    pkg = os.path.dirname(axon.LIB_PATH)
    subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f not in ("-O3", "-fPIC")], "--offload-host-only", "-x",
                    "hip", os.path.join(HERE, "recorded_hip.cpp"), "-rdynamic", "-o", exe, "-L" + pkg,
                    "-l:" + os.path.basename(axon.LIB_PATH), "-Wl,-rpath," + pkg],
                   check=True, capture_output=True, text=True)
    done = {}

    def run(*scenario):
        if scenario not in done:
            r = subprocess.run([exe, *map(str, scenario)], capture_output=True, text=True, timeout=60)
            assert r.returncode == 0 and r.stdout.endswith("done\n"), r.stdout[-500:] + r.stderr[-500:]
            done[scenario] = [_event(line) for line in r.stdout.splitlines()[:-1]]
        return done[scenario]
    return run


def _event(line):
    f = line.split(" ")
    if f[0] == "launch":
        return Launch(*map(int, f[1:8]), " ".join(f[8:]))
    if f[0] == "limit":
        return Limit(*map(int, f[1:4]), " ".join(f[4:]))
    if f[0] == "mark":
        return ("mark", line[5:])
    return (f[0], *map(int, f[1:]))


DEFAULT_LDS = 64 << 10  # dynamic LDS that a kernel may take without a raised limit


def test_lds_limits_are_raised_on_every_device_before_any_launch(recorder):
    """Two devices in one process: a kernel of more than 64 KB of dynamic LDS is
    launched only where its limit was raised on that device, and no call after
    axon_init_model (a graph's capture, the no-allocation step) raises one."""
    limits, large, step = {}, set(), ""
    for e in recorder("two_devices"):
        if isinstance(e, Limit):
            assert not e.capture and step.startswith("device"), (step, e)
            limits[e.device, e.kernel] = e.lds
        elif isinstance(e, Launch) and e.lds > DEFAULT_LDS:
            assert e.lds <= limits.get((e.device, e.kernel), DEFAULT_LDS), (step, e)
            large.add((e.device, e.kernel))
        elif e[0] == "mark":
            step = e[1]
    assert {d for d, _ in large} == {0, 1}
    assert {k for d, k in large if d == 0} == {k for d, k in large if d == 1}
    # the scenario reaches the 256-tile, ring, few-token and weight-gradient forms
    for part in ("gemm_bf16_256_kernel<", "gemm_ring_kernel<8", "gemm_ring_kernel<2", "gemm_tn_256_kernel<"):
        assert any(part in k for _, k in large), part


def test_float_rows_of_a_split_projection_are_never_accumulated(recorder):
    """A few-token projection to float rows leaves the raw partials of its K
    splits (GV_PART, one launch, enough workspace reported); storing rows (GV_F32)
    is the grouped experts' form and refused elsewhere, not run through the
    residual sum, which would add to what the rows held."""
    ev = [e for e in recorder("raw_rows") if isinstance(e, Launch) or e[0] == "mark"]
    seen = 0
    for i, e in enumerate(ev):
        if e[0] == "mark" and e[1].startswith("raw 5 "):
            assert ev[i + 1] == ("mark", "refused"), ev[i:i + 4]
        elif e[0] == "mark" and e[1].startswith("raw 4 "):
            assert "gemv_wide_kernel<" in ev[i + 1].kernel and ev[i + 1].gy == (1 if " 64 " in e[1] else 16), ev[i + 1]
            assert ev[i + 2] == ("mark", "launched")
            seen += 1
    assert seen == 8 and ("mark", "workspace too small") not in ev


def test_timed_weight_gradient_includes_the_sum_of_its_splits(recorder):
    """With kernel timing on, a weight gradient split over the tokens starts its
    event pair with the GEMM and stops it with the kernel that sums the splits."""
    launches = [e for e in recorder("timed_train") if isinstance(e, Launch)]
    split = [i for i, e in enumerate(launches) if "gemm_tn_256_kernel<" in e.kernel and e.gy > 1]
    assert {launches[i].kernel.split("<")[1][0] for i in split} == {"0", "1", "2"}  # every row order
    for i in split:
        gemm, total = launches[i], launches[i + 1]
        assert "wgrad_sum_kernel<" in total.kernel
        assert gemm.start and not gemm.stop and not total.start and total.stop == gemm.start + 1, (gemm, total)


def test_decode_splits_do_not_depend_on_an_earlier_training_step(recorder):
    """A decode step above 64 sequences takes the same launches (so the same order
    of sums, the same bits) whether or not the model has run a training step, which
    enlarges the shared buffer of partials: here the buffer a model starts with
    bounds the split of the down projection."""
    steps, inside = [], False
    for e in recorder("decode_after_training"):
        if e[0] == "mark":
            inside = e[1] == "decode"
            if inside:
                steps.append([])
        elif inside and isinstance(e, Launch):
            steps[-1].append((e.kernel, e.gx, e.gy))
    assert len(steps) == 2 and steps[0] == steps[1]
    assert any("gemm_" in k and gy > 1 for k, _, gy in steps[0])


def test_routing_rows_are_in_range_before_the_first_call(recorder):
    """Choices without an expert (NaN router logits) get no row in the plan, and
    what reads the plan then finds what its buffers held: token and row numbers of
    an earlier call, or zeros, never uninitialized memory."""
    ev = recorder("moe_init")
    size = 7 * 3 * 4  # max_tokens x top_k int32: choices, their weights, token and row of each choice
    at = [e[1] for e in ev if e[0] == "alloc" and e[2] == size]
    assert len(at) == 4
    filled = {e[1] for e in ev if e[0] == "fill" and e[2] == size}
    assert set(at[2:]) <= filled


@pytest.mark.parametrize("case", list(REACHES))
def test_training_cases_reach_the_kernels_they_stand_for(recorder, case):
    """The GPU test over the training step's tile edges takes the launches that it
    names, by the launch rules themselves."""
    base, heads, kv, hidden, inter, vocab, lens = CASES[case]
    shape = MODEL_SHAPES[base]
    launches = [e for e in recorder("train_step", hidden, heads, kv, shape["head_dim"], inter, vocab,
                                    int(shape["attention_bias"]), int(shape["tie_word_embeddings"]), *lens)
                if isinstance(e, Launch)]
    for kernel, splits in REACHES[case]:
        assert any(kernel in e.kernel and e.gy == splits for e in launches), (kernel, splits)


def test_partials_stay_inside_their_buffer(recorder):
    """Every launch that leaves partials for the next kernel (K splits, key splits,
    sums of squares, argmax) writes them inside one allocation of the model (or the
    fixed work array), for prompts of few and many tokens under few and many
    sequence slots: a prompt may have more tokens than the model has slots."""
    ends, step, seen = {}, "", 0
    for e in recorder("partials"):
        if isinstance(e, (Launch, Limit)):
            continue
        if e[0] == "alloc":
            ends[e[1]] = e[1] + e[2]
        elif e[0] == "mark":
            step = e[1]
        elif e[0] == "parts":
            base = max((b for b in ends if b <= e[1]), default=None)
            assert base is not None and e[1] + e[2] <= ends[base], (step, e, base and ends[base] - e[1])
            seen += 1
    assert seen > 100


def test_training_step_records_no_memset(recorder):
    """After the first call's set-up a training step (untied head: the embedding's
    gradient starts at zero) enqueues kernels only, so a caller may capture it: a
    memory-set node in a captured graph is not reliable on replays."""
    ev = recorder("train_twice")
    second = ev[ev.index(("mark", "second")):]
    assert any(isinstance(e, Launch) and "embed_bwd" in e.kernel for e in second)
    assert not any(e[0] in ("fill", "alloc") for e in second if not isinstance(e, (Launch, Limit)))
