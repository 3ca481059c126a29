"""Host checks of the expressions that the multi-generation kernels and the
distance matrix compute with (csrc/smap_ca2k.hpp, csrc/smap_ca3k.hpp,
csrc/smap_rows.hpp), each against its plain definition over every operand:
the byte packing by dot products, the masks of a word's cells, B3/S23 and
B6/S567 on unpropagated carries, and the rounding of a square root from a
neighbour of the right answer."""
import itertools
import random
from fractions import Fraction

import numpy as np

M32 = 0xFFFFFFFF


def maj(a, b, c):
    return (a & b) | (c & (a ^ b))


def test_pack16_every_byte_pattern():
    def udot4(a, b, acc):
        return acc + sum(((a >> 8 * k) & 255) * ((b >> 8 * k) & 255) for k in range(4))
    for bits in range(256):
        byte = [(bits >> k & 1) | 0xA4 for k in range(8)]        # only bit 0 of a byte counts
        lo, hi = (sum(v << 8 * k for k, v in enumerate(byte[o:o + 4])) & 0x01010101 for o in (0, 4))
        assert udot4(hi, 0x80402010, udot4(lo, 0x08040201, 0)) == bits


def test_word_masks():
    def clamp(v):
        return min(max(v, 0), 31)
    for x in range(-70, 40):
        left = 0 if x <= -32 else (M32 << clamp(-x)) & M32
        assert left == sum(1 << b for b in range(32) if x + b >= 0)
        for y, last in itertools.product((-2, -1, 0, 5), range(-4, 36)):
            past = (0xFFFFFFFE << clamp(last)) & M32
            none = M32 if (last < 0 or y < 0) else 0
            want = sum(1 << b for b in range(32) if x + b >= 0 and b <= last and y >= 0)
            assert left & ~past & ~none & M32 == want


def test_life_on_row_sums():
    for p, c, n, alive in itertools.product(range(4), range(4), range(4), (0, 1)):
        a, k = (p ^ c ^ n) & 1, maj(p & 1, c & 1, n & 1)
        b, m = (p ^ c ^ n) >> 1, maj(p >> 1, c >> 1, n >> 1)
        t3 = (k ^ b) & (1 - m)
        t4 = (1 - (k ^ b)) & (k ^ m)
        got = (a & t3) | ((1 - a) & (t4 & alive))
        t = p + c + n
        assert got == (t == 3 or (t == 4 and alive == 1)), (p, c, n, alive)


def test_b6s567_on_unpropagated_sums():
    reps = list(itertools.product((0, 1), repeat=4))             # q, k, t, m: q + 2 (k + t) + 4 m
    for A, B, C in itertools.product(reps, repeat=3):
        t0, u = A[0] ^ B[0] ^ C[0], maj(A[0], B[0], C[0])
        k, ck = A[1] ^ B[1] ^ C[1], maj(A[1], B[1], C[1])
        t, ct = A[2] ^ B[2] ^ C[2], maj(A[2], B[2], C[2])
        t1, cu = u ^ k ^ t, maj(u, k, t)
        m, cm = A[3] ^ B[3] ^ C[3], maj(A[3], B[3], C[3])
        v, cv = ck ^ ct ^ cu, maj(ck, ct, cu)
        t2, cw = m ^ v, m & v
        t3, t4 = cm ^ cv ^ cw, maj(cm, cv, cw)
        total = sum(q + 2 * (a + b) + 4 * d for q, a, b, d in (A, B, C))
        assert t0 + 2 * t1 + 4 * t2 + 8 * t3 + 16 * t4 == total
        e67, e89 = t1 & t2 & (1 - t3), (1 - t1) & (1 - t2) & t3
        born, stay = e67 & (1 - t0), e67 | (e89 & (1 - t0))
        for alive in (0, 1):
            got = (stay if alive else born) & (1 - t4)
            assert got == (total == 6 or (alive == 1 and total in (7, 8))), (A, B, C, alive)


def test_root_rounds_from_any_neighbour():
    rng = random.Random(11)
    xs = [np.float32(v) for v in (2.0 ** -96, 2.0 ** -95, 0.25, 1.0, 2.0, 3.0, 4.0, 3.4e38)]
    xs += [np.float32(np.uint32(rng.randrange(0x0F800000, 0x7F800000)).view(np.float32)) for _ in range(3000)]
    for root in (1.5, 1.9999999, 1.0000001, 1e-10, 7e15):          # squares and their neighbours
        sq = np.float32(np.float32(root) * np.float32(root))
        xs += [sq, np.nextafter(sq, np.float32(0)), np.nextafter(sq, np.float32(np.inf))]
    for x in xs:
        want = np.sqrt(x)
        for s in (np.nextafter(want, np.float32(0)), want, np.nextafter(want, np.float32(np.inf))):
            lo, hi = np.nextafter(s, np.float32(0)), np.nextafter(s, np.float32(np.inf))
            fx, fs = Fraction(float(x)), Fraction(float(s))
            r = lo if fx - Fraction(float(lo)) * fs <= 0 else s
            if fx - Fraction(float(hi)) * fs > 0:
                r = hi
            assert r == want, (x, s)
