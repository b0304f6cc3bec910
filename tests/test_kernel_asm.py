"""The direct-to-LDS loads (conv_stage.h) are inline assembly that sets m0, a
register that a clobber list cannot name: a compiler that kept a value of its own
there (for its own LDS loads, register indexing or messages) would not know of
it.  So the kernels that use them must have no other user of m0, which the
compiled code shows."""

import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2502_11618_amd import build as B

M0_USERS = re.compile(r"\bm0\b|_lds_dword|\blds\b|movrel|gpr_idx|sendmsg|gws|ds_direct")


def _outside_inline_asm(text):
    inside = False
    for line in text.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
            continue
        code = line.split(";")[0].strip()
        if not inside and code and not code.startswith("."):
            yield code


def test_users_of_m0_are_found():
    text = "\tv_mov_b32 v0, v1\n\t;;#ASMSTART\n\ts_mov_b32 m0, s1\n\t;;#ASMEND\n\ts_mov_b32 m0, s2 ; its own\n"
    assert [c for c in _outside_inline_asm(text) if M0_USERS.search(c)] == ["s_mov_b32 m0, s2"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")

    def one(src):
        dst = os.path.join(out, src + ".s")
        subprocess.run([B.hipcc()] + B.FLAGS + ["-x", "hip", "--offload-device-only", "-S",
                                                os.path.join(B.CSRC, src), "-o", dst],
                       check=True, capture_output=True)
        return open(dst).read()

    with ThreadPoolExecutor(2) as ex:
        return dict(zip(("conv16.hip", "unet.hip"), ex.map(one, ("conv16.hip", "unet.hip"))))


@pytest.mark.parametrize("src", ["conv16.hip", "unet.hip"])
def test_only_the_direct_loads_use_m0(assembly, src):
    text = assembly[src]
    assert text.count("global_load_lds_dwordx4") > 0
    assert [c for c in _outside_inline_asm(text) if M0_USERS.search(c)] == []
