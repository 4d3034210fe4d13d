"""What a product sent to the 256 x 256 kernels is cut into, without a device: wide tiles of the ring kernel, lower tiles of the persistent
one (only where rows of the output start on sectors of 64 bytes), or 256 x 256 ones."""
import re

import pytest

from tests.test_gemm_choice import choose, pytestmark  # noqa: F401

ONE_ROUND = [(3072, 4096), (3001, 4096), (2048, 5120), (768, 15104), (1536, 7168), (3584, 4096), (770, 15104)]


def test_lower_tiles_only_where_rows_start_on_sectors(choose):  # noqa: F811
    """... or where the contraction is long enough for them to pay all the same."""
    for M, N in ONE_ROUND:
        low = -(-M // 192) * -(-N // 256) <= 256
        for K in (512, 1024, 2048, 3456, 3584, 7040, 7168, 12288):
            want = "192 rows" if low else "224 rows" if K > 1024 else "256 rows"
            between = want if K >= (3584 if low else 7168) else "256 rows"
            for off, answer in zip((0, 32, 8, 16, 48, 56), choose(*[f"large {M} {N - o} {K}" for o in (0, 32, 8, 16, 48, 56)])):
                assert answer == (want if off % 32 == 0 else between), (M, N - off, K, answer)
            a = choose(f"slabs {M} {N} {K}", f"slabs {M} {N - 8} {K}")
            assert a == [want.replace("256", "0"), between.replace("256", "0")], (M, N, K, a)


def test_block_scaled_over_several_rounds(choose):  # noqa: F811
    heights = set()
    for M, N in ((4096, 14336), (8192, 8192), (5000, 8192), (14336, 4096), (6144, 4096), (6166, 7872)):
        for K in (1024, 2048, 2944, 3072, 4096, 6144, 8192):
            whole, half, odd, odder = (int(a.split()[0]) for a in choose(*[f"slabs {M} {n} {K}" for n in (N, N - 32, N - 8, N - 16)]))
            assert whole == half and (whole > 0 or K > 6144)
            assert odd == odder == (whole if K >= 3072 and whole != 256 else 0), (M, N, K)
            heights.add(odd)
    assert heights == {0, 192, 224}
    # forced forms stay forced
    assert choose("slabs 4096 14328 1024", GEMM_TILE_M=224) == ["224 rows"] and choose("slabs 300 264 1024", GEMM_STREAM=8) != ["0 rows"]


@pytest.mark.parametrize("cus", [64, 256])
def test_wide_tiles_in_one_round(choose, cus):  # noqa: F811
    """Products that the first choice leaves to the 256 x 256 kernels take a wide tile only where one round of it covers them."""
    seen = set()
    for K in (400, 1024, 4096, 10240):
        shapes = [(M, N) for M in (300, 514, 702, 782, 1400, 2261, 2816, 3072) for N in (2048, 3016, 3072, 4096, 4104, 6144, 11008, 24064)]
        for (M, N), first, wide, wide32 in zip(shapes, *(choose(*[f"{k} {M} {N} {K}" for M, N in shapes], cus=cus) for k in ("one", "large", "large32"))):
            for w in (wide, wide32):
                if m := re.match(r"ring (\d+)x(\d+)", w):
                    assert -(-M // int(m[1])) * -(-N // int(m[2])) <= cus, (M, N, K, w)
                    seen.add(f"{m[1]}x{m[2]}")
            assert first == "256x256" or first.startswith("ring")
    assert seen <= {"160x192", "192x192", "160x256", "224x192"} and len(seen) >= 3, seen
    if cus == 256:
        assert choose("one 702 11264 10112", "large 702 11264 10112") == ["256x256", "ring 192x192"]
        assert choose("large 782 11008 11920", "large 638 11008 4080") == ["ring 160x256", "ring 160x192"]
    assert not any(a.startswith("ring") for a in choose("large 702 11264 10112", "large 782 11008 11920", GEMM_STREAM=0))


def test_short_contractions_priced_with_their_operands(choose):  # noqa: F811
    """One round of 128 x 256 tiles of a short contraction is not left to rather few lower ones, which are slower there."""
    slower = ((820, 8576, 288), (329, 19744, 384), (560, 12864, 512), (834, 9056, 448))
    for kind in ("one", "f32"):
        for a in choose(*[f"{kind} {M} {N} {K}" for M, N, K in slower]):
            assert a.startswith(("ring 128x256", "ring 256x128")), (kind, a)
    faster = ((1294, 6688, 384), (475, 17760, 512), (4671, 2048, 512), (3072, 4096, 1024))
    assert choose(*[f"one {M} {N} {K}" for M, N, K in faster]) == ["256x256"] * 4
    assert choose(*[f"large {M} {N} {K}" for M, N, K in faster]) == ["192 rows"] * 4
