"""What the compiler makes of the lane decoder (the listing of our own
kernels for gfx950), where an earlier form lost time on some alphabets only."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_17849_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def lane(tmp_path_factory):
    """Instructions of the lane decoder's forms, by bits per symbol."""
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    from paper_2602_17849_amd import build as qbuild   # the library's own flags
    out = str(tmp_path_factory.mktemp("listing") / "qlc_kernels.asm")
    cmd = [HIPCC] + [f for f in qbuild.HIPCC_FLAGS if f != "-fPIC"] + [
           "--cuda-device-only", "-S", os.path.join(CSRC, "qlc_kernels.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels, cur = {}, None
    for line in open(out):
        m = re.match(r"\S*8k_decodeILi(\d)E\S*:", line)
        if m:
            cur = []
            kernels.setdefault(int(m.group(1)), []).append(cur)
        elif cur is not None and line.startswith("\t") and not line.startswith("\t."):
            cur.append(line.strip())
            if line.strip().startswith("s_endpgm"):
                cur = None
    assert sorted(kernels) == [4, 6, 8]
    return kernels


def test_no_extension_again(lane):
    """A code-to-symbol entry is loaded extended to 32 bits: nothing masks it
    to 16 again on the way into the packed output."""
    for bits in (4, 6, 8):
        again = [i for form in lane[bits] for i in form if re.match(r"v_and_b32\S* v\d+, 0xffff, v", i)]
        assert len(again) < 8, bits


def test_store_policy(lane):
    """Runs that are whole lines, or aligned halves, go past the caches; for
    the 96-byte runs of 6-bit symbols there is a form of either kind."""
    for bits, op, kinds in ((4, "buffer_store_dwordx2", {True}),
                            (6, "buffer_store_dwordx3", {False, True}),
                            (8, "buffer_store_dwordx4", {True})):
        assert {" nt" in i for form in lane[bits] for i in form if i.startswith(op)} == kinds, bits
