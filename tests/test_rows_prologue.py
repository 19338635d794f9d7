"""Own tiles, as compiled for the GPU: what a wave does before its first matrix instruction. Zeros for results that the first tile overwrites
anyway do not stand in its way (64 registers of them and more once did), nor does code for block tables in kernels for contiguous caches."""
import os
import re
import subprocess

import pytest

from paper_2509_15235_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(channels, waves, row blocks, paged, read once, crowd) -> instructions."""
    to = tmp_path_factory.mktemp("rows") / "k.s"
    flags = [f for f in build.FLAGS if f != "-shared"]
    subprocess.check_call([build.HIPCC, "--offload-device-only", "-S"] + flags + [os.path.join(build.CSRC, "attention_mfma_rows.hip"), "-o", str(to)],
                          stderr=subprocess.DEVNULL)
    found, code = {}, None
    for line in to.read_text().splitlines():
        line = line.split(";")[0].strip()
        name = re.fullmatch(r"_ZN2vs.*attn_mfma_rows_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELb([01])ELb([01])E.*:", line)
        if name:
            code = found.setdefault(tuple(int(x) for x in name.groups()), [])
        elif line == "s_endpgm":
            code = None
        elif code is not None and line and not line.startswith(".") and not line.endswith(":"):
            code.append(line)
    return found


def test_all_kernels_are_here(kernels):
    assert set(kernels) == {(d, w, rb, paged, once, crowd) for d, w, rb in [(128, 8, 1), (128, 8, 2), (128, 4, 1), (64, 8, 1), (64, 4, 1)]
                            for paged, once, crowd in [(0, 0, 0), (0, 1, 0), (1, 0, 0), (0, 0, 1), (1, 0, 1)] if not crowd or (w, rb) == (8, 1)}


def test_no_zeros_for_the_results_before_the_first_tile(kernels):
    """Under half of the 32 registers a lane of the narrowest result; constants of addresses and predicates are some ten."""
    for name, code in kernels.items():
        first = next(i for i, line in enumerate(code) if line.startswith("v_mfma"))
        zeros = [line for line in code[:first] if re.fullmatch(r"v_mov_b(32_e32 v\d+|64_e32 v\[\d+:\d+\]), 0", line)]
        assert len(zeros) <= 16, (name, zeros)
