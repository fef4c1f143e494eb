"""The default grid of the persistent launch holds the workgroups that are resident at once: as many
per compute unit as its registers and its LDS (160 KB, handed out in units of 1280 bytes) allow.
Host arithmetic of the built library, called by its C++ name; no GPU is used."""
import ctypes as C

import pytest

LDS = 160 * 1024
UNIT = 1280
SCRATCH = 512 * 8 + 64 * 4 + 64 + 4 * 8 + 16  # of a wave: sums, tags, entries in use, photons, start


def workgroups(nb, sides, waves, stack):
    from paper_1807_07094_amd import arc

    f = arc.lib()._ZN3arc28persistent_workgroups_per_cuEiiii
    f.restype, f.argtypes = C.c_int, [C.c_int] * 4
    return f(nb, sides, waves, stack)


def lds(nb, sides, waves, stack):
    terms = (4 * (sides + 6) + 15) // 16 * 16
    total = waves * SCRATCH + terms + waves * stack * 8 * (1 + nb)
    return (total + UNIT - 1) // UNIT * UNIT


@pytest.mark.parametrize("stack", [64, 128, 256])
@pytest.mark.parametrize("waves", [1, 2, 4, 8])
@pytest.mark.parametrize("nb", [1, 2, 3, 4])
def test_resident_workgroups(nb, waves, stack):
    by_registers = (16 if nb <= 3 else 12) // waves
    for sides in (3, 48, 768, 3072, 3696, 3712, 4128, 6144):
        got = workgroups(nb, sides, waves, stack)
        assert got == max(1, min(by_registers, LDS // lds(nb, sides, waves, stack))), sides


def test_where_the_lds_decides():
    assert workgroups(3, 3 * 256, 4, 64) == 4
    assert workgroups(3, 2048 + 1600 + 48, 4, 64) == 4
    assert workgroups(3, 2048 + 2048 + 32, 4, 64) == 3
    assert workgroups(3, 3 * 128, 4, 256) == 3
