"""Which sizes a launch accepts, on the host: the status of a plan belongs to
its own tile shape, whatever was asked before, and several generations are
taken for the sizes of their 256-cell (2-D) or 64-cell (3-D) tiles, however a
pass is cut."""
import pytest
import torch

from paper_2208_11617_amd import binding as smap


def wgs(n, threads):
    """Workgroups of an H step with 128-cell tiles, or the status that refuses it."""
    smap.set_tile(3, "ca3", 128, threads)
    try:
        return smap.plan_info(3, n, "ca3")["launched_wgs"]
    except smap.SimplexMapError as e:
        return e.status
    finally:
        smap.set_tile(3, "ca3", 0)


@pytest.mark.parametrize("first,n", [(128, 10000), (512, 10001)])
def test_status_of_a_tile_side_is_per_shape(first, n):
    """128 workgroups a tile are too many for this size, 32 are not: in both orders."""
    for threads in (first, 640 - first):
        got = wgs(n, threads)
        assert got == smap.ERANGE if threads == 128 else got > 0, (threads, got)


def steps_status(m, n, steps, layout=smap.LAYOUT_AUTO):
    """Status of a run of generations over a box far larger than any memory.
    The addresses are none of anybody's: a size that is not refused is only
    asked for where no GPU could run it."""
    smap.set_layout(3, layout)
    try:
        return smap.launch_steps_raw(m, n, "ca2" if m == 2 else "ca3", steps, 1 << 20, (1 << 21) + (n + 1) ** m)
    finally:
        smap.set_layout(3, smap.LAYOUT_AUTO)


@pytest.mark.parametrize("steps", [1, 8, 16, 17, 32, 100])
def test_steps_refuse_sizes_beyond_the_map(steps):
    """H numbers the 64-cell tiles of a 3-D box up to n of about 21500 (19000
    in the packed layout), the 256-cell tiles of a 2-D one up to about 990000."""
    for n in (23000, 30000, 65533, 65534, 100000):
        assert steps_status(3, n, steps) == smap.ERANGE, n
        assert steps_status(3, n, steps, smap.LAYOUT_PACKED) == smap.ERANGE, n
    for n in (1100000, 1500000, 20000000):
        assert steps_status(2, n, steps) == smap.ERANGE, n


@pytest.mark.skipif(torch.cuda.is_available(), reason="would launch on addresses that are no buffer's")
@pytest.mark.parametrize("steps", [1, 8, 16, 17, 23, 24, 32, 100])
def test_steps_take_sizes_of_their_tiles(steps):
    for n in (300000, 600000, 700000, 850000, 900000):
        assert steps_status(2, n, steps) != smap.ERANGE, n
    for n in (5000, 18000):
        assert steps_status(3, n, steps) != smap.ERANGE, n
