"""The matrix products of the compiled MLP kernels, read off this source's own
assembly.  A 16 x 16 x 16 product right behind a 16 x 16 x 32 one over the
same accumulator has given wrong sums: in the inference kernel, which has
both, at least 19 wait states (what the longest product asks for) must lie
between the two; the training kernels have the shorter kind alone."""
import os
import re
import subprocess

import pytest

from paper_1909_00573_amd import build as B


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instruction lines of each kernel."""
    if not os.path.exists(B.hipcc()):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("mlp") / "mlp.s")
    subprocess.run([B.hipcc()] + B.common_flags() + ["-S", "--offload-device-only",
                                                     os.path.join(B.CSRC, "neb_mlp.hip"), "-o", out],
                   check=True, capture_output=True)
    body, cur = {}, None
    for line in open(out):
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = body.setdefault(m.group(1), [])
        elif cur is not None:
            cur.append(line.strip())
    return body


def _one(kernels, name):
    found = [b for k, b in kernels.items() if name in k]
    assert len(found) == 1
    return found[0]


def test_inference_waits_between_the_kinds(kernels):
    waited, met, kinds = None, 0, set()
    for line in _one(kernels, "k_mlp_infer"):
        m = re.match(r"v_mfma_f32_16x16x(\d+)", line)
        if m:
            kinds.add(m.group(1))
            if m.group(1) == "32":
                waited = 0
            elif waited is not None:
                met += 1
                assert waited >= 19, line
            continue
        m = re.match(r"s_nop (\d+)", line)
        if m and waited is not None:
            waited += 1 + int(m.group(1))
    assert kinds == {"16", "32"} and met == 4  # one block of outputs each


@pytest.mark.parametrize("kernel", ["k_mlp_train_fb", "k_mlp_wgrad"])
def test_training_has_one_kind(kernels, kernel):
    kinds = {m.group(1) for m in (re.match(r"v_mfma_f32_16x16x(\d+)", line) for line in _one(kernels, kernel)) if m}
    assert kinds == {"16"}
