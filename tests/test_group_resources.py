"""Register budget of the group kernels and of the training step, read from the
compiler's resource report as in test_kernel_resources.py, and no packed
float32 arithmetic in them: the group inverter's only scratch is the frame of
the eigen fallback and its LDS lets eight waves share a CU, synthesis uses no
scratch, a training step's row kernel none with 16 rows per workgroup and 256
bytes per lane with 32."""
import os
import re
import subprocess

import pytest

from test_kernel_resources import CSRC, ROOT, _hipcc

SOURCES = ("group.hip", "mlp.hip")


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    from paper_0901_2702_amd import _build
    d = tmp_path_factory.mktemp("asm")
    procs = {src: subprocess.Popen(
        [_hipcc()] + _build.HIPCC_FLAGS + ["-I", CSRC, "-I", os.path.join(ROOT, "include"),
         "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", str(d / (src + ".s"))],
        stdout=subprocess.PIPE, stderr=subprocess.PIPE) for src in SOURCES}
    for src, p in procs.items():
        _, err = p.communicate()
        assert p.returncode == 0, (src, err[-2000:])
    return {src: (d / (src + ".s")).read_text() for src in SOURCES}


def _report(text, name):
    res = {}
    for m in re.finditer(r"^(_ZN5vfisv\w*%s\w*):" % name, text, re.M):
        seg = text[m.end():]
        res[m.group(1)] = {k: int(re.search(r"; %s: (\d+)" % k, seg).group(1))
                           for k in ("NumVgprs", "ScratchSize", "LDSByteSize")}
    return res


def test_group_inverter(asm):
    r = _report(asm["group.hip"], "lm_group_kernel")
    assert len(r) == 2
    for name, v in r.items():
        assert v["ScratchSize"] <= 96 and v["NumVgprs"] <= 256, (name, v)
        assert 8 * v["LDSByteSize"] <= 160 * 1024, (name, v)


def test_synthesis_by_waves(asm):
    r = _report(asm["group.hip"], "synth_group")
    assert len(r) == 4
    for name, v in r.items():
        assert v["ScratchSize"] == 0, (name, v)


def test_training_rows(asm):
    r = _report(asm["mlp.hip"], "train_rows_kernel")
    one = [v for k, v in r.items() if "ILi1E" in k]
    two = [v for k, v in r.items() if "ILi2E" in k]
    assert len(one) == len(two) == 1
    assert one[0]["ScratchSize"] == 0 and two[0]["ScratchSize"] <= 256, r


def test_no_packed_float32_arithmetic(asm):
    packed = re.compile(r"^\s*v_pk_(fma|mul|add)_f32\b", re.M)
    for src in SOURCES:
        assert not packed.search(asm[src]), src
    assert re.search(r"^\s*v_mfma_f32_16x16x4_f32\b", asm["group.hip"], re.M)
