"""CPU checks of layouts and rules in the library's sources, compiled for the
host only."""
import os
import subprocess

import pytest

from paper_2604_25459_amd import build


def _syntax(text, tmp_path):
    """Compiles `text` (host side, no code written) against the sources; returns the compiler's messages."""
    src = str(tmp_path / "t.hip")
    with open(src, "w") as f:
        f.write(text)
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-host-only", "-fsyntax-only", src], capture_output=True,
                       text=True)
    return r.returncode, r.stderr


@pytest.mark.parametrize("ts", [8, 16])
def test_lidar_quadratics_are_aligned_for_16_byte_reads(ts, tmp_path):
    rc, err = _syntax(f"""
#include <stddef.h>
#include "k_lidar.hip"
using Lds = gsr::LidarLds<{ts}>;
static_assert(offsetof(Lds, quad) % 16 == 0 && sizeof(Lds::quad[0]) % 16 == 0, "misaligned");
""", tmp_path)
    assert rc == 0, err


def test_lowest_bit_is_defined_for_every_mask(tmp_path):
    """Undefined results are no constant expressions: the mask without a bit,
    which every ray's walk ends with, has to have a value too."""
    rc, err = _syntax("""
#include "gsr_internal.h"
constexpr bool every_bit()
{
    for (uint32_t k = 0; k < 32; ++k)
        if (gsr::lowest_bit(1u << k) != k || gsr::lowest_bit(0xFFFFFFFFu << k) != k) return false;
    return true;
}
static_assert(every_bit(), "lowest set bit");
static_assert(gsr::lowest_bit(0u) == 31u, "an empty mask");
""", tmp_path)
    assert rc == 0, err
