"""The loads into LDS that are written as inline assembly, compiled for the GPU in places where the compiler gives them no
room: the wait states behind a lane read that yields their address, and m0 between them and loads of the compiler's own."""
import re
import subprocess

import pytest

from paper_2509_15235_amd import build

SOURCE = """
#include "attn_mfma_common.h"
using namespace vs;
#define LANE_READ \\
    const int hi = t[threadIdx.x], lo = t[threadIdx.x + 64]; \\
    char* base = (char*)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, at) << 32) | (uint32_t)__builtin_amdgcn_readlane(lo, at))
#define KERNEL(name, load) \\
    extern "C" __global__ void name(int* t, int at) { \\
        __shared__ __attribute__((aligned(1024))) uint16_t s[1024]; \\
        LANE_READ; \\
        const uint32_t lds = (uint32_t)(uintptr_t)(lds_void*)s; \\
        load; \\
        wait_loads<0>(); \\
        t[threadIdx.x] = s[threadIdx.x]; \\
    }
KERNEL(k_base, load_to_lds(lds, base, threadIdx.x * 16))
KERNEL(k_four, load_to_lds4(lds, base, threadIdx.x * 4))
KERNEL(k_range, load_to_lds(lds, __builtin_amdgcn_make_buffer_rsrc(base, 0, 4096, 0x00027000), threadIdx.x * 16))
#define BETWEEN(name, load) \\
    extern "C" __global__ void name(int* t, int* base) { \\
        __shared__ __attribute__((aligned(1024))) uint16_t s[1024]; \\
        lds_void* const second = (lds_void*)(s + 512); \\
        const uint32_t lds = (uint32_t)(uintptr_t)(lds_void*)s; \\
        __builtin_amdgcn_global_load_lds(t + threadIdx.x * 4, second, 16, 0, 0); \\
        load; \\
        __builtin_amdgcn_global_load_lds(t + threadIdx.x * 4 + 256, second, 16, 0, 0); \\
        wait_loads<0>(); \\
        t[threadIdx.x] = s[threadIdx.x] + s[threadIdx.x + 512]; \\
    }
BETWEEN(m_base, load_to_lds(lds, base, threadIdx.x * 16))
BETWEEN(m_four, load_to_lds4(lds, base, threadIdx.x * 4))
BETWEEN(m_range, load_to_lds(lds, __builtin_amdgcn_make_buffer_rsrc(base, 0, 4096, 0x00027000), threadIdx.x * 16))
"""


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name -> its instructions."""
    at = tmp_path_factory.mktemp("lds_loads")
    (at / "k.hip").write_text(SOURCE)
    flags = [f for f in build.FLAGS if f != "-shared"]
    subprocess.check_call([build.HIPCC, "--offload-device-only", "-S"] + flags + [str(at / "k.hip"), "-o", str(at / "k.s")], stderr=subprocess.DEVNULL)
    found, name = {}, None
    for line in (at / "k.s").read_text().splitlines():
        line = line.split(";")[0].strip()
        if re.fullmatch(r"[km]_\w+:", line):
            name = line[:-1]
            found[name] = []
        elif name and line and not line.startswith(".") and not line.endswith(":"):
            found[name].append(line)
            if line == "s_endpgm":
                name = None
    return found


def _loads(code):
    return [i for i, line in enumerate(code) if re.match(r"global_load_lds_", line) or line.endswith(" lds")]


def _registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


@pytest.mark.parametrize("name", ["k_base", "k_four", "k_range"])
def test_wait_states_behind_a_lane_read(kernels, name):
    """Five between a vector instruction that writes a scalar register and the load that reads it."""
    code = kernels[name]
    (load,) = _loads(code)
    operands = code[load].split(None, 1)[1].replace(" offen", ",offen").split(",")
    asked = set().union(*(_registers(o.strip()) for o in operands))
    assert asked, code[load]
    for register in asked:
        states = 0
        for line in reversed(code[:load]):
            if " " in line and register in _registers(line.split(None, 1)[1].split(",")[0].strip()):
                assert line.startswith("s_") or states >= 5, code
                break
            states += int(line.split()[1]) + 1 if line.startswith("s_nop") else 1


@pytest.mark.parametrize("name", ["m_base", "m_four", "m_range"])
def test_loads_around_set_m0_again(kernels, name):
    code = kernels[name]
    loads = _loads(code)
    assert len(loads) == 3
    for first, second in zip(loads, loads[1:]):  # the three go to two places in turn
        assert any(re.match(r"s_\w+ m0,", line) for line in code[first + 1:second]), code
