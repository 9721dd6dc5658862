"""Waits of hand-written completion signals, read from the gfx950 code that
the build's own flags make (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2407_11290_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def copy_kernel(tmp_path_factory):
    """The instructions of k_copy_one, in order."""
    d = tmp_path_factory.mktemp("isa")
    src, out = d / "use.hip", d / "use.s"
    src.write_text('#include "tt_kernels.h"\n'
                   "void use(const double *s, double *t, int *f) { ttc::k_copy_one<<<1, 1024>>>(s, t, 5, f, 1); }\n")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([build.HIPCC, *flags, "-w", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
                    "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    body = re.search(r"^_ZN3ttcL10k_copy_one\w+:.*?\n(.*?)s_endpgm", out.read_text(), re.S | re.M).group(1)
    return [ln.split(";")[0].strip() for ln in body.splitlines() if ln.startswith("\t") and not ln.startswith("\t.")]


def _vm0(ins):
    return ins.startswith("s_waitcnt") and "vmcnt(0)" in ins


def test_core_copy_waits_for_every_store_before_its_flag(copy_kernel):
    """The host takes the copy for done when the flag arrives, so every
    wavefront's stores must be complete before the barrier (which does not
    wait for them), and written back to memory before the flag's store."""
    ins = copy_kernel
    bar = max(i for i, x in enumerate(ins) if x.startswith("s_barrier"))
    stores = [i for i, x in enumerate(ins) if re.match(r"(global|flat)_store_dwordx[24]", x)]
    flag = [i for i, x in enumerate(ins) if re.match(r"(global|flat)_store_dword ", x)]
    wb = [i for i, x in enumerate(ins) if x.startswith("buffer_wbl2")]
    assert stores and max(stores) < bar and len(flag) == 1
    assert any(_vm0(x) for x in ins[max(stores) + 1:bar])
    # one write-back, complete before the flag
    assert len(wb) == 1 and bar < wb[0] < flag[0] and "sc0 sc1" in ins[wb[0]]
    assert any(_vm0(x) for x in ins[wb[0] + 1:flag[0]])
    assert "sc0 sc1" in ins[flag[0]]
