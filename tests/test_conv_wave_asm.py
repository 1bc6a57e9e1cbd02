"""Static checks of the gfx950 code of the convolution kernel with one wave per pixel block."""
import os
import re

import pytest

from paper_2407_12075_amd import asm_check, build as hip_build

_INSTANCE = re.compile(r"conv_wave_kernelI([ft])Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELb([01])E")


@pytest.fixture(scope="module")
def instances():
    """(type, filters of a tile, taps, pixels, filter tiles, LDS pixels, runs, all bits) -> lines of the listing"""
    text = asm_check.compile_to_asm(os.path.join(hip_build.CSRC, "tbn_conv_wave.hip"))
    kernels = {_INSTANCE.search(name).groups(): body for name, body in asm_check._split_kernels(text).items() if _INSTANCE.search(name)}
    assert len(kernels) == 47
    return kernels


def test_runs_cost_no_64_bit_products(instances):
    """Addresses of the last channels are 32-bit offsets that grow by a plane: a run's instance multiplies 64-bit numbers no more often than the
    one that loads pixels or pairs (48 such products per wave once cost layers of one chunk more than runs gave them)."""
    products = lambda lines: sum(l.startswith(("v_mad_u64", "v_mad_i64")) for l in lines)
    runs = [key for key in instances if key[6] == "1"]
    assert len(runs) == 11
    for key in runs:
        assert products(instances[key]) <= products(instances[key[:6] + ("0",) + key[7:]]), key


def test_3x3_instances_keep_their_registers(instances):
    """Nothing of a 3x3 layer goes to scratch memory."""
    for key, lines in instances.items():
        if key[2] == "9":
            assert not any(l.startswith(("scratch_", "buffer_store", "buffer_load")) for l in lines), key
