"""The choice of a kernel for an FP8 product, without a device: gemm_fp8.hip with stubs in place of the launchers behind it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_16099_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("choice") / "gemm_choice_check")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++20", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w", "-o", exe,
           os.path.join(ROOT, "tests", "gemm_choice_check.hip"), os.path.join(CSRC, "gemm_fp8.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(os.path.join(CSRC, "tuning.hpp")) as f:
        knobs = re.findall(r"^ +KNOB_(\w+)", f.read(), re.M)

    def ask(*queries, cus=256, **switches):
        args = [f"CUs={cus}"] + [f"{knobs.index(k)}={v}" for k, v in switches.items()]
        out = subprocess.run([exe, *args], input="\n".join(queries) + "\n", capture_output=True, text=True, timeout=60, check=True).stdout
        answers = out.splitlines()
        assert len(answers) == len(queries), (queries, out)
        return answers

    return ask


@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 64, 65, 300])
def test_ring_kernel_switched_off(choose, M):
    """GEMM_RING = 0 holds for every count of rows and width of weight."""
    queries = [f"{kind} {M} {N} {K}" for kind in ("one", "act") for N in (512, 8192, 10176, 10184, 28672) for K in (16, 1024, 8192)]
    assert any(a.startswith("ring") for a in choose(*queries))
    assert not any(a.startswith("ring") for a in choose(*queries, GEMM_RING=0))


def test_backward_of_few_tokens_compares_estimates(choose):
    """17 to 32 tokens against a wide layer: dX goes to the ring kernel, and shares a launch with dW where that is estimated to be
    faster, on the tile that is cheapest for both (not just where both by themselves take 64 x 64 tiles)."""
    def pair(M, K, N):
        return f"two {M} {K} {N} {N} {K} {(M + 15) // 16 * 16}"

    together = [(17, 10240, 128), (32, 11008, 256), (24, 14336, 256), (32, 28672, 64), (20, 16384, 384)]
    apart = [(32, 28672, 192), (17, 11008, 1024), (32, 11008, 11008)]
    answers = choose(*[pair(*s) for s in together + apart])
    for s, a in zip(together, answers):
        tiles = sum(-(-rows // int(t)) * -(-s[1] // int(u)) for t, u in re.findall(r"ring (\d+)x(\d+) together", a) for rows in (s[0], s[2]))
        assert 0 < tiles <= 512 and a.endswith(f"K={s[2]}"), (s, a)
    assert answers[len(together):] == ["apart"] * len(apart)


@pytest.mark.parametrize("N,K", [(28672, 3584), (28672, 8192), (16384, 6144)])
def test_streaming_hint_only_where_the_weight_is_read_once(choose, N, K):
    """One row of tiles: two fall out of step, and lines are fetched twice."""
    for M in (33, 64, 65, 128, 129, 160, 192, 193, 256, 257):
        for tile, rows in ((1, 64), (3, 64), (4, 128), (5, 128)):
            answer, = choose(f"one {M} {N} {K}", GEMM_RING=tile)
            assert ("hint" in answer) == (M <= rows), (M, answer)
        for tile in (2, 6):
            assert "hint" not in choose(f"one {M} {N} {K}", GEMM_RING=tile)[0]
    for tile in range(1, 7):      # smaller weights, and weights whose rows are not whole lines
        assert not any("hint" in a for a in choose(f"one 64 {N} 2048", f"one 64 {(96 << 20) // K - 8} {K}", f"one 64 {N} {K + 16}", GEMM_RING=tile))


@pytest.mark.parametrize("N,K", [(28672, 4096), (28672, 8192), (16384, 8192)])
def test_no_streaming_hint_on_tall_tiles_behind_the_weights_own_quantization(choose, N, K):
    """The codes are in the last-level cache."""
    for M in (33, 64, 65, 128, 193, 256):
        for tile in range(1, 7):
            one, own, strips = choose(f"one {M} {N} {K}", f"own {M} {N} {K}", f"strips {M} {N} {K}", GEMM_RING=tile)
            assert own == strips
            assert one.split()[1] == own.split()[1]
            assert ("hint" in own) == ("hint" in one and M <= 64 and tile <= 3), (M, tile, one, own)


def test_one_row_of_tiles_fetches_a_large_weight(choose):
    """129 to 256 rows: 256 x 128 tiles, on eight wavefronts up to 192 rows of a short contraction."""
    for M, K, waves in ((129, 4096, 8), (192, 6144, 8), (193, 4096, 4), (256, 4096, 4), (129, 6272, 4), (256, 8192, 4)):
        one, own = choose(f"one {M} 28672 {K}", f"own {M} 28672 {K}")
        assert one == f"ring 256x128 alone {waves} K={K}"
        assert own == f"ring 128x256 alone {8 if K <= 6144 else 4} K={K}"
    assert choose("one 200 28672 2048") == ["ring 128x256 alone 8 K=2048"]      # (a smaller weight)


@pytest.mark.parametrize("tile", [1, 4, 5, 6])
def test_wavefronts_of_the_widest_tiles(choose, tile):
    """Eight up to K = 6144, of a pair both."""
    for M, N in ((72, 1040), (256, 4096), (300, 1000), (128, 28672)):
        for kind in ("one", "mx"):
            a = choose(*[f"{kind} {M} {N} {K}" for K in (128, 6144, 6272)], GEMM_RING=tile)
            assert [re.search(r" (\d)(?: K=|$)", x)[1] for x in a] == (["8", "8", "4"] if tile >= 5 else ["4"] * 3), a
        a = choose(*[f"mxrows {M} {N} {K}" for K in (128, 1536, 1664)], GEMM_RING=tile)
        assert [x[-1] for x in a] == (["8", "8", "4"] if tile >= 5 else ["4"] * 3), a
    wide = 8 if tile >= 5 else 4
    assert choose("mx 256 28672 4096", GEMM_RING=tile)[0].endswith(f" {wide}")
    assert " together 4 " in choose("two 400 400 6144 400 400 6272", GEMM_RING=tile)[0]
    assert f" together {wide} " in choose("two 400 400 6144 400 400 6016", GEMM_RING=tile)[0]
    # rows of B that are no whole lines
    for K, waves in ((1520, wide), (1552, 4 if tile == 6 else wide)):
        assert f" alone {waves} " in choose(f"one 690 5968 {K}", GEMM_RING=tile)[0]
        assert f" together {waves} " in choose(f"two 690 5968 1024 690 5968 {K}", GEMM_RING=tile)[0]


@pytest.mark.parametrize("cus", [64, 256])
def test_half_of_the_cus_is_that_of_the_device(choose, cus):
    """The deeper ring of few rows and narrow strips are for grids of a part of the CUs, on a partition of the device too."""
    deep = choose(f"few 8 {8 * cus} 14336", f"few 8 {8 * cus + 8} 14336", f"few 9 {8 * cus} 14336", f"few 4 {12 * cus} 14336", f"few 4 {12 * cus + 8} 14336",
                  f"few 5 {12 * cus} 14336", f"few 4 {8 * cus} 10240", cus=cus)
    assert ["deep" in a for a in deep] == [True, False, False, True, False, False, False]
    assert choose(f"cols 2048 {cus // 2} 0", f"cols 2048 {cus // 2 + 1} 0", f"cols 1024 1 0", f"cols 4097 {cus} 0", cus=cus) == ["16", "32", "32", "16"]


def test_every_few_row_form_of_a_streamed_weight_has_the_hint(choose):
    """Weights of 96 MiB and more, of every width that the choice leaves to the few-row kernel."""
    shapes = [(M, N, -(-(96 << 20) // (16 * N)) * 16) for M in (1, 8, 16, 17, 32, 33, 48, 49, 64)
              for N in (16, 512, 3072, 6128, 6144, 8192, 8200, 10176, 16384, 65536, 262144, 1 << 20)]
    answers = choose(*[f"one {M} {N} {K}" for M, N, K in shapes])
    few = [s for s, a in zip(shapes, answers) if a == "few-row"]
    assert {M for M, _, _ in few} == {1, 8, 16, 17, 32, 33, 48, 49, 64}
    for s, a in zip(few, choose(*["few %d %d %d" % s for s in few])):
        assert a.endswith("hint"), (s, a)


def test_rounds_of_tiles_of_17_to_32_rows(choose):
    """A second round of 64 x 64 tiles that is hardly filled costs as much as a full one: wider tiles in one round, or the few-row kernel."""
    want = {(10176, 2048): "few-row", (10184, 512): "64x64", (16384, 8192): "64x64", (16392, 1008): "few-row", (16392, 1024): "64x128", (26176, 8192): "64x128",
            (26184, 8192): "64x64", (32768, 8176): "64x128", (32768, 4096): "few-row", (30720, 4096): "64x128", (32776, 4096): "few-row", (32776, 6144): "64x64", (65472, 4096): "few-row", (65536, 4096): "64x64",
            (128256, 2048): "few-row"}
    for M in (17, 32):
        for (N, K), w in want.items():
            answer, = choose(f"one {M} {N} {K}")
            assert w in answer, (M, N, K, answer)
    assert "64x128" in choose("one 20 8192 2048", cus=64)[0] and "64x64" in choose("one 20 4096 2048", cus=64)[0]


def test_low_tiles_over_several_rounds(choose):
    """What a low tile costs by itself in one round is not what it costs in several: wide products of a few hundred rows stay on 256 x 256 tiles, and pairs
    take larger tiles."""
    assert choose("one 319 24064 10240", "one 447 17280 12672", "one 182 34048 10368", "one 702 11264 10112") == ["256x256"] * 4
    assert choose("one 512 4096 8192")[0].split()[1] in ("128x64", "64x128")      # (one round)
    for M, K, N, tile in ((1286, 1024, 5120, "128x128"), (730, 6912, 656, "128x128"), (93, 14080, 256, "128x256"), (2048, 768, 11008, "128x128")):
        answer, = choose(f"two {M} {K} {N} {N} {K} {(M + 15) // 16 * 16}")
        assert answer.startswith(f"ring {tile} together"), (M, K, N, answer)


def test_few_rows_behind_the_weights_own_quantization(choose):
    """17 to 32 rows: codes just written go to the few-row kernel, unless in strips or beyond the size of a streamed weight."""
    for M in (17, 32):
        for N, K in ((10240, 4096), (16384, 1536), (20480, 2048)):
            assert choose(f"own {M} {N} {K}", f"strips {M} {N} {K}", f"one {M} {N} {K}")[0] == "few-row"
            assert choose(f"strips {M} {N} {K}") == choose(f"one {M} {N} {K}") != ["few-row"]
        assert choose(f"own {M} 28672 4096")[0].startswith("ring")
