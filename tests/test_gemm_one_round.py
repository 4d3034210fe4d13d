"""The choice of tiles between the usual sizes, without a device: one product in one round, never pairs or several rounds."""
import re

import pytest

from tests.test_gemm_choice import choose, pytestmark  # noqa: F401

SIZES = [(M, N) for M in (65, 96, 160, 300, 777, 1400, 2500, 3001, 3072, 5000) for N in (64, 512, 1000, 2048, 3072, 4096, 6144, 11008, 28672)]
NEW = {"96x64", "64x192", "160x64", "96x128", "160x128", "192x128", "128x192", "160x192", "192x192", "160x256", "224x192"}


@pytest.mark.parametrize("kind", ["one", "own", "mx", "mxrows"])
@pytest.mark.parametrize("cus", [64, 256])
def test_only_in_one_round(choose, kind, cus):  # noqa: F811
    seen = set()
    for K in (128, 1024, 4096, 10240):
        for (M, N), a in zip(SIZES, choose(*[f"{kind} {M} {N} {K}" for M, N in SIZES], cus=cus)):
            m = re.match(r"ring (\d+)x(\d+)", a)
            if m and f"{m[1]}x{m[2]}" in NEW:
                seen.add(f"{m[1]}x{m[2]}")
                assert -(-M // int(m[1])) * -(-N // int(m[2])) <= cus, (M, N, K, a)
                assert "hint" not in a and not (M <= 256 and N * K >= 96 << 20)
    assert len(seen) >= 5, seen


def test_never_for_pairs(choose):  # noqa: F811
    for K in (256, 1024, 4096):
        for a in choose(*[f"two {M} {K} {N} {N} {K} {(M + 15) // 16 * 16}" for M, N in SIZES]):
            m = re.match(r"ring (\S+) together", a)
            assert a == "apart" or m[1] not in NEW, a


@pytest.mark.parametrize("M,N,K,tile", [(72, 14336, 4096, "96x64"), (3001, 2048, 4096, "192x128"), (2500, 2048, 8192, "160x128"), (1500, 2048, 4096, "96x128"),
                                        (1500, 4096, 2048, "192x128"), (2048, 3072, 4096, "128x192"), (512, 4096, 4096, "128x64"), (2048, 4096, 4096, "128x256")])
def test_the_tile_that_fills_the_round(choose, M, N, K, tile):  # noqa: F811
    assert choose(f"one {M} {N} {K}")[0].split()[1] == tile


def test_64x192_tiles_only_where_they_fetch_no_more(choose):  # noqa: F811
    """Beyond a short contraction not over rows that are no whole cache lines, nor over a few rows of tiles of an odd number."""
    def tile(kind, M, N, K):
        return choose(f"{kind} {M} {N} {K}")[0].split()[1]

    for M, N, K in ((172, 11216, 5296), (316, 8288, 6944), (105, 19784, 2080), (1222, 2136, 1264), (425, 6864, 2688), (576, 4496, 2048), (900, 3208, 12800)):
        assert tile("one", M, N, K) != "64x192", (M, N, K)
    for kind in ("mx", "mxrows"):
        for M, N, K in ((425, 6864, 2688), (576, 4496, 2048)):
            assert "64x192" not in choose(f"{kind} {M} {N} {K}")[0], (kind, M, N, K)
    for M, N, K in ((1222, 2136, 1024), (576, 4496, 1536), (128, 18776, 2432), (332, 7528, 1920), (1152, 2640, 2432)):
        assert tile("one", M, N, K) == "64x192", (M, N, K)


def test_a_weight_at_rest_is_not_fetched_more_often(choose):  # noqa: F811
    """Both sides of the lines; what the call itself has quantized is in the cache and keeps the fuller round."""
    def tiles(kind, *shapes):
        one, large = (choose(*[f"{k} {M} {N} {K}" for M, N, K in shapes]) for k in (kind, "large"))
        return [(b if a == "256x256" else a).split()[1] for a, b in zip(one, large)]

    slower = ((3520, 1856, 10416), (448, 14976, 7904), (953, 6784, 5840), (3502, 1808, 4384))
    assert tiles("one", *slower) == ["256x128"] * 4 and tiles("own", *slower) == ["160x192"] * 4
    # whole lines, a short contraction, clearly fewer tiles
    assert tiles("one", (3520, 1856, 10496), (448, 14976, 2544), (972, 6272, 3488)) == ["160x192"] * 3
    assert "128x192" not in tiles("one", (976, 4720, 10464), (4220, 1328, 10448), (975, 5384, 6640))
    assert tiles("one", (975, 5384, 6128), (975, 5384, 6656), (387, 11632, 10448)) == ["128x192"] * 3
    assert tiles("one", (279, 9208, 7168), (266, 10280, 15488), (281, 10496, 2064), (658, 4096, 16064), (644, 3784, 8576)) == ["128x128"] * 5
    assert tiles("own", (279, 9208, 7168)) == ["96x128"]
    assert tiles("one", (280, 9352, 2048), (185, 12224, 3072), (525, 4720, 3712)) == ["96x128"] * 3
