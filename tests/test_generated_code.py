"""What the compiler must make of the kernels for them to work as designed, read from the assembly of the library's own sources."""
import os
import re
import subprocess

import pytest

from paper_2509_19128_amd import build as plbuild


@pytest.fixture(scope="module")
def attention(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "attn.s")
    r = subprocess.run([plbuild.HIPCC, *plbuild.COMMON, "-S", "--cuda-device-only", os.path.join(plbuild.CSRC, "kernels_attn.hip"), "-o", out],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    return open(out).read()


@pytest.mark.parametrize("rotate", [0, 1])
@pytest.mark.parametrize("hd", [32, 64, 128])
def test_decode_attention_reads_page_ids_by_scalar_loads(attention, hd, rotate):
    """In the loop over a sequence's runs a page id that comes by a vector load waits for all K/V loads in flight: no
    block of the kernel may load one value by vector and hand it to the scalar unit."""
    body = re.search(r"^(_ZN\S*attn_decode_kernelILi%dELi%dELb%dE\S*):(.*?)\.Lfunc_end" % (hd, 1 if rotate else 2, rotate), attention, re.S | re.M).group(2)
    assert "mfma" in body
    for block in re.split(r"^\.LBB\S+:", body, flags=re.M):
        loaded = set(re.findall(r"global_load_dword (v\d+),", block))
        assert not loaded & set(re.findall(r"v_readfirstlane_b32 s\d+, (v\d+)", block)), block[:400]
