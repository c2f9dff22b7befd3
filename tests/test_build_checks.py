"""What the build looks for in the device assembly."""
import importlib.util
import os
import re

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_15443_amd")


@pytest.fixture(scope="module")
def build():
    spec = importlib.util.spec_from_file_location("dc_build_checks", os.path.join(PKG, "build.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


@pytest.fixture(scope="module")
def assembly(build):
    return {source: build.device_assembly(os.path.join(PKG, "csrc", source)) for source in ("dc_decode.hip", "dc_encode.hip")}


LOOPED = """_Zkernel:
.LBB3_95:
\tv_readfirstlane_b32 s4, v28
\tv_cmp_eq_u64_e64 s[0:1], s[4:5], v[28:29]
\ts_and_saveexec_b64 s[0:1], s[0:1]
\tbuffer_store_dwordx4 v[50:53], v41, s[4:7], 0 offen
\ts_xor_b64 exec, exec, s[0:1]
\ts_cbranch_execnz .LBB3_95
"""


def test_loops_around_buffer_accesses_are_found(build):
    assert build.buffer_access_loops(LOOPED) == ["_Zkernel"]
    straight = LOOPED.replace("\ts_cbranch_execnz .LBB3_95\n", "\ts_endpgm\n")
    assert build.buffer_access_loops(straight) == []


def test_the_coders_stores_are_straight(build, assembly):
    asm = assembly["dc_encode.hip"]
    assert asm.count("buffer_store_dwordx4") >= 6
    assert build.buffer_access_loops(asm) == []


GENERIC = """_Zkernel:
\ts_mov_b64 s[8:9], src_shared_base
\ts_cmp_lg_u32 s9, -1
\ts_cselect_b32 s8, 0x1000, -1
.Lfunc_end0:
_Zother:
\ts_endpgm
"""


def test_lds_addresses_of_generic_pointers_are_found(build):
    assert build.generic_lds_addresses(GENERIC) == ["_Zkernel"]


@pytest.mark.parametrize("source", ["dc_decode.hip", "dc_encode.hip"])
def test_lds_addresses_are_constants(build, assembly, source):
    assert "ds_read_u16" in assembly[source]
    assert build.generic_lds_addresses(assembly[source]) == []


def test_decoders_lose_no_wavefronts_to_registers(assembly):
    # a compute unit has 160 KiB of LDS and four SIMDs of 512 registers a lane, given out by eights, and of eight wavefronts
    metadata = assembly["dc_decode.hip"].split("amdhsa.kernels:")[1]
    kernels, fewer = 0, []
    for kernel in metadata.split("\n  - ."):
        value = dict(re.findall(r"^\s*\.(\w+): +(\S+)$", kernel, re.M))
        if "dc_decode_kernel" not in value.get("name", ""):
            continue
        waves = (160 << 10) // int(value["group_segment_fixed_size"]) * (int(value["max_flat_workgroup_size"]) // 64)
        by_lds = min(8, (waves + 3) // 4)
        kernels += 1
        if by_lds * ((int(value["vgpr_count"]) + 7) // 8 * 8) > 512:
            fewer.append((value["name"], value["vgpr_count"], by_lds))
    assert kernels > 50 and not fewer
