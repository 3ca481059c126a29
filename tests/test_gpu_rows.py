"""The two routes of ACCUM, HASH and EDM on 2-D tiles (whole tile rows, or
line-aligned parts of rows): at and around the sizes where one takes over
from the other, on boxes whose rows start at lines and on shifted ones, every
element against plain torch and everything outside the simplex kept."""
import pytest

import simplex_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def smap():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2208_11617_amd import binding
    binding.lib()
    return binding


def mul32(h, k):
    return (h * k) & 0xFFFFFFFF


def reference(op, n, src, y0, y1):
    """Rows y0 .. y1-1 in plain torch: int64 words, or float64 distances."""
    x = torch.arange(n + 1, device="cuda")
    y = torch.arange(y0, y1, device="cuda").view(-1, 1)
    if op == "accum":
        return (src.view(n + 1, n + 1)[y0:y1].long() + 1) & 0xFFFFFFFF
    if op == "edm":
        p = src.double()
        d = torch.zeros((y1 - y0, n + 1), dtype=torch.float64, device="cuda")
        for c in range(3):
            d += (p[:, c].view(1, -1) - p[n - y.view(-1), c].view(-1, 1)).square_()
        return d.sqrt_()
    h = mul32(0x811C9DC5 ^ x, 0x01000193)
    h = mul32(h ^ y, 0x01000193)
    h = mul32(h ^ (h >> 16), 0x85EBCA6B)
    h = mul32(h ^ (h >> 13), 0xC2B2AE35)
    return h ^ (h >> 16)


def check(smap, op, n, launch, off):
    words = (n + 1) ** 2
    src = {"accum": lambda: torch.randint(0, 1 << 31, (words,), dtype=torch.int32, device="cuda"),
           "hash": lambda: None,
           "edm": lambda: torch.from_numpy(si.points(n, 9600 + n)).cuda()}[op]()
    buf = torch.full((words + 64,), 7, dtype=torch.int32, device="cuda")
    launch(2, n, op, src, buf[off:off + words])
    torch.cuda.synchronize()
    assert bool((buf[:off] == 7).all()) and bool((buf[off + words:] == 7).all())
    got = buf[off:off + words].view(n + 1, n + 1)
    x = torch.arange(n + 1, device="cuda")
    for y0 in range(0, n + 1, 1024):
        y1 = min(n + 1, y0 + 1024)
        inside = x + torch.arange(y0, y1, device="cuda").view(-1, 1) <= n
        want, part = reference(op, n, src, y0, y1), got[y0:y1]
        assert bool((part[~inside] == 7).all())
        if op == "edm":
            # three rounded differences, squares and sums and a rounded root stay
            # within 3.5 ulp of the float32 result
            near = want.float()
            ulp = (torch.nextafter(near, torch.full_like(near, torch.inf)) - near).double()
            err = (part.view(torch.float32).double() - want).abs()
            assert bool((err <= 4 * ulp)[inside].all())
        else:
            assert bool(((part.long() & 0xFFFFFFFF) == want)[inside].all())


# the sizes from which H and BB take the row parts, per tile side
FROM = {"accum": {16: (3000, 2000), 32: (2200, 2000), 64: (6000, 5000), 128: (11000, 10000)},
        "hash": {16: (12000, 100), 32: (2000, 100), 64: (9000, 6000), 128: (12000, 12000)},
        "edm": {16: (13000, 2000), 32: (13000, 12500), 64: (5000, 4000), 128: (7000, 6000)}}


@pytest.mark.parametrize("kind", ["h", "bb"])
@pytest.mark.parametrize("rho", [16, 32, 64, 128])
@pytest.mark.parametrize("op", ["accum", "hash", "edm"])
def test_either_side_of_the_route(smap, op, rho, kind):
    first = FROM[op][rho][kind == "bb"]
    launch = smap.map_launch if kind == "h" else smap.bb_launch
    smap.set_shape(2, op, rho, 64 if rho == 16 else 256, 1)
    try:
        # either side of the line, a size past a tile's edge, one with rows on lines
        for n in (first - 1, first, first // rho * rho + rho, first // 32 * 32 + 31):
            for off in ((0, 5) if n <= first else (0,)):
                print(f"{op} rho={rho} {kind} n={n} offset {off}", flush=True)
                check(smap, op, n, launch, off)
    finally:
        smap.set_shape(2, op, 0)


@pytest.mark.parametrize("n", [31, 63, 127, 2047])
def test_rows_on_lines(smap, n):
    """Rows of whole lines: at a line's start and shifted by whole lines, half a
    line and one element, all tile sides."""
    for op in ("accum", "hash", "edm"):
        try:
            for rho in (16, 32, 64, 128):
                smap.set_tile(2, op, rho)
                for launch in (smap.map_launch, smap.bb_launch):
                    for off in (0, 32, 16, 1):
                        print(f"{op} rho={rho} n={n} offset {off}", flush=True)
                        check(smap, op, n, launch, off)
        finally:
            smap.set_tile(2, op, 0)
