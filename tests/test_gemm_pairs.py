"""Which products of a backward step share a launch, without a device: compared with what the two take by themselves, one-round tiles
and all; forms that are forced; the time of tiles that the CUs take in turn."""
import pytest

from tests.test_gemm_choice import choose, pytestmark  # noqa: F401


def pair(M, K, N):
    return f"two {M} {K} {N} {N} {K} {(M + 15) // 16 * 16}"


def test_apart_where_one_round_of_each_is_clearly_less(choose):  # noqa: F811
    apart = [(3072, 3072, 3072), (4032, 2304, 3840), (7973, 1040, 7984), (4352, 2048, 5120), (6144, 1504, 5472), (1280, 2048, 6880), (2048, 4240, 2048), (9218, 1136, 5120),
             (2433, 1024, 5664)]
    together = [(1024, 2048, 1024), (2048, 5744, 1904), (3072, 3728, 3024), (1170, 4016, 2048), (1947, 2416, 4096), (512, 2528, 2048), (1792, 5120, 1024), (488, 2096, 5120),
                (4864, 1024, 14336), (1012, 4112, 2848), (875, 2656, 5120)]
    answers = choose(*[pair(*s) for s in apart + together])
    assert answers[:len(apart)] == ["apart"] * len(apart)
    for s, a in zip(together, answers[len(apart):]):
        assert " together " in a, (s, a)


def test_forced_tiles_are_shared_as_before(choose):  # noqa: F811
    for tile, name in ((4, "128x128"), (5, "128x256"), (15, "192x192")):
        for s in ((3072, 3072, 3072), (400, 400, 400)):
            assert choose(pair(*s), GEMM_RING=tile)[0].startswith(f"ring {name} together")
    assert choose(pair(400, 400, 400), PAIRS=0) == choose(pair(400, 400, 400), GEMM_VARIANT=4) == ["apart"]


@pytest.mark.parametrize("cus", [8, 64, 256])
def test_apart_or_together_for_every_size(choose, cus):  # noqa: F811
    """Extremes: one tile, one CU's worth more, contractions of one step and of thousands (the search ends)."""
    sizes = (16, 17, 33, 65, 300, 1040, 2064, 4112, 16384, 65536)
    queries = [pair(M, K, N) for M in sizes for K in (16, 272, 2048, 14336) for N in (16, 1040, 5120, 28672)]
    for q, a in zip(queries, choose(*queries, cus=cus)):
        assert a == "apart" or " together " in a, (q, a)
