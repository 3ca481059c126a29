"""Which sizes a launch accepts, on the host: the status of a plan belongs to
its own tile shape, whatever was asked before."""
import pytest

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
