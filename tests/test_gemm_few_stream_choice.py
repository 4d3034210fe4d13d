"""Which products of up to 16 rows go to persistent workgroups, and in which order those take their tiles, without a device: both sides
of every line of the rule."""
import pytest

from tests.test_gemm_choice import choose, pytestmark  # noqa: F401


def ask(choose, rows, **kw):
    """rows: (N, K) or (N, K, ld)"""
    return choose(*[("stream 16 %d %d" if len(r) == 2 else "streamld 16 %d %d %d") % tuple(r) for r in rows], **kw)


def test_sizes_that_fit(choose):  # noqa: F811
    assert choose("stream 16 20480 10240", "stream 17 20480 10240", "stream 1 20480 10240") == ["strided", "few-row", "strided"]
    assert ask(choose, [(10240, 10240), (9728, 10240)]) == ["strided", "few-row"]                    # 96 MiB
    assert ask(choose, [(8200, 16384), (8200, 16400)]) == ["strided", "few-row"]                     # eight wavefronts' registers of A
    assert ask(choose, [(131072, 1040), (131088, 1040)]) == ["strided", "few-row"]                   # 32 tiles of 16 rows a CU
    assert ask(choose, [(20480, 10240, 1 << 23), (20480, 10240, (1 << 23) - 128)]) == ["few-row", "strided"]


def test_rows_that_are_no_whole_lines(choose):  # noqa: F811
    assert ask(choose, [(16384, 7168), (16384, 7184), (16384, 7168, 7232), (16384, 7168, 7296)]) == ["few-row", "strided", "strided", "few-row"]


def test_few_tokens_over_two_tiles_a_workgroup(choose):  # noqa: F811
    for M, want in ((1, "few-row"), (4, "few-row"), (5, "strided"), (16, "strided")):
        assert choose(f"stream {M} 8192 12336", f"stream {M} 8200 12336") == [want, "strided"], M


def test_streams_a_multiple_of_4096_bytes_apart(choose):  # noqa: F811
    assert ask(choose, [(49152, 4096), (65504, 4096), (65536, 4096)]) == ["few-row", "few-row", "runs"]          # parts of 2048, 4096
    assert ask(choose, [(32736, 8192), (32768, 8192), (24576, 8192)]) == ["few-row", "strided", "few-row"]
    assert ask(choose, [(8192, 16384), (8192, 16256), (8192, 16384, 16512)]) == ["strided", "few-row", "few-row"]
    assert ask(choose, [(65536, 6144), (65536, 12288)]) == ["few-row", "strided"]


def test_rows_of_the_busiest_cu(choose):  # noqa: F811
    """few-row kernel / persistent: 32 / 32, 64 / 48, 64 / 64, 96 / 80, 128 / 112, 128 / 128 rows."""
    for K in (10240, 12288, 14336):
        assert ask(choose, [(8192 * 5 // 4, K), (12288, K), (14336, K), (16384, K), (16392, K), (20480, K), (24576, K), (28672, K), (32768, K)]) == \
            ["strided", "strided", "few-row", "few-row", "strided", "strided", "few-row", "strided", "few-row"], K
    # a seventh more does not pay for short rows
    assert ask(choose, [(28672, 6144), (28672, 6016), (28672, 4096), (36864, 4096), (32776, 4096), (20480, 5120)]) == ["runs", "few-row", "few-row", "runs", "runs", "runs"]


def test_order_of_tiles(choose):  # noqa: F811
    assert ask(choose, [(28672, 8192), (20480, 8192), (18432, 8192), (27648, 8320)]) == ["runs", "runs", "runs", "strided"]
    assert ask(choose, [(36864, 8192), (65536, 8192)]) == ["runs", "strided"]      # runs 2.25 and 8 times 256 KB apart
    assert ask(choose, [(20312, 6320), (40000, 2576)]) == ["strided", "strided"]


@pytest.mark.parametrize("cus", [64, 256])
def test_forced(choose, cus):  # noqa: F811
    rows = [(64, 128), (16 * cus, 128), (16 * cus + 8, 128), (5000, 4096)]
    assert ask(choose, rows, cus=cus, SKINNY_DMA=2) == ["strided"] * 4
    assert ask(choose, rows, cus=cus, SKINNY_DMA=3) == ["strided", "strided", "runs", "runs"]
    for v in (0, 1):
        assert ask(choose, [*rows, (20480, 10240)], cus=cus, SKINNY_DMA=v) == ["few-row"] * 5
