"""When the weight-gradient products that wait are launched and in which tiles, for the models of test_gpu_waiting_weight_gradients.py,
test_gpu_grouped_weight_gradients.py and test_gpu_ragged_k.py: the schedule of a product on a stand-in runtime without a GPU.  A
change of a rule must not leave what the comments there name untested without notice."""
import re

import hip_standin as standin
import pytest

import test_gpu_grouped_weight_gradients as grouped
import test_gpu_ragged_k as ragged
import test_gpu_waiting_weight_gradients as waiting


def launches(tmp_path, model, batch):
    """The launches of the backward sweep, as (the adjoint of a norm that follows, what is launched): adjoints are named by their layer, m for
    the norm between its branches, x for the one whose result enters the layer below, and the last launch may have none behind it;
    "256 x n" is n blocks of that tile for products together, "one 128 x n" for one by itself."""
    enqueued, log = standin.run(tmp_path, "rc, c = create(desc, batch)\nassert rc == 0\nlog()\nr = hvp(c, batch, seq)\nshow([r, log()])",
                                desc=standin.desc(model), batch=batch, seq=model["max_seq"])
    assert enqueued == standin.ENQUEUED
    marks = ["final"] + [f"{l}{c}" for l in reversed(range(model["n_layer"])) for c in "mx"] + ["end"]
    out, done = [], 0
    for name, x, yz in standin.kernels(log):
        if "norm_bwd" in name:
            done += 1
        elif m := re.search(r"gemm_mfma_group_kernelILi(\d+)", name):
            out.append((marks[done], f"{m.group(1)} x {x}"))
        elif m := re.search(r"gemm_mfma_kernelILi(\d+).*Lb1ELb0E", name):
            out.append((marks[done], f"one {m.group(1)} x {x * yz}"))
    assert done == len(marks) - 1
    return out


WANT = {
    "many_products": [("2x", "128 x 318"), ("end", "128 x 189")],
    "inside_a_layer": [("0x", "256 x 584")],
    "odd_head": [("1x", "256 x 214"), ("end", "128 x 240")],
    "llama": [("2m", "128 x 234"), ("0m", "128 x 240"), ("end", "128 x 36")],
    "llama_grouped": [("1m", "128 x 112"), ("end", "128 x 84")],
    "cut": [("final", "one 128 x 1"), ("3x", "128 x 96"), ("end", "128 x 72")],
    "three_buffers": [("4x", "256 x 446"), ("1x", "256 x 444"), ("end", "128 x 432")],   # 4x writes where layer 6's adjoint is
    "two_buffers": [("3x", "128 x 1803"), ("1x", "128 x 1800"), ("end", "128 x 900")],   # 3x where layer 4's is
    "full_rounds": [("3m", "256 x 248"), ("2m", "256 x 246"), ("0x", "128 x 1014")],
}

GROUPED = {
    "128_whole": [("0x", "128 x 87")],
    "128_cut": [("final", "one 128 x 2"), ("0x", "128 x 168")],    # 84 tiles, two parts
    "256_whole": [("0x", "256 x 196")],
    "256_cut": [("final", "one 128 x 4"), ("0x", "256 x 216")],    # 72 tiles, three parts
}
# (products whose rows are no multiple of 16 bytes take a kernel that is not listed here: W_fc and W_proj of the ragged ones)
RAGGED = {
    "padded_65": [("0x", "128 x 201")],
    "ragged_65": [("1x", "one 128 x 3"), ("1x", "one 128 x 9"), ("1x", "one 128 x 24"), ("0x", "one 128 x 9"), ("0x", "one 128 x 24")],
    "ragged_llama_65": [("0x", "one 128 x 4")] * 3 + [("0x", "one 128 x 2")] * 2,
    "ragged_group_65": [("0m", "one 128 x 3"), ("0x", "128 x 30")],
    "ragged_group_129": [("1m", "one 128 x 3"), ("1x", "128 x 30"), ("0x", "128 x 30")],
}
ALL = [(n, waiting.SHAPES[n], w) for n, w in WANT.items()] + [(n, grouped.SHAPES[n], w) for n, w in GROUPED.items()] + \
      [(n, ragged.TOKENS[n], w) for n, w in RAGGED.items()]


@pytest.mark.parametrize("name,shape,want", ALL, ids=[a[0] for a in ALL])
def test_launches(tmp_path, name, shape, want):
    assert launches(tmp_path, *shape) == want


def test_every_model_is_held():
    assert set(WANT) == set(waiting.SHAPES) and set(GROUPED) == set(grouped.SHAPES)
