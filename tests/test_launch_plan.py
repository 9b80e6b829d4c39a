"""Host checks of the launch rules (launch_plan.h): how a launch spreads its
packets over waves, chunks and lanes, for 256 compute units."""
import ctypes

import pytest

import lanesim

FIELDS = ("waves", "chunk", "lam_chunks", "n_chunks", "lanes", "threshold", "mixed", "sums", "own_chunks", "copies", "lone")


def plan(count, n_lambda=1, octree=False, point=True, direct=False, plain=True, chunk=0, chunk_shift=0, waves_per_cu=0,
         threshold=0, n_cu=256, cells=96):
    a = (ctypes.c_int64 * 12)(n_cu, count, n_lambda, octree, point, direct, plain, chunk, chunk_shift, waves_per_cu,
                              threshold, cells)
    out = (ctypes.c_int64 * 11)()
    lanesim.lib().ls_plan(a, out)
    return dict(zip(FIELDS, out))


@pytest.mark.parametrize("octree", [False, True])
@pytest.mark.parametrize("n_lambda", [1, 3])
@pytest.mark.parametrize("count", [32769, 60_000, 98_304, 98_305, 100_000, 131_072, 200_000, 1_000_000, 20_000_000])
def test_additions_of_direct_light(count, n_lambda, octree):
    """Above 32768 packets per wavelength the additions to the pixel of a point
    source's direct light keep their sizes: full waves, the queue's chunks of
    total / waves packets (32 to 256), the mixed loop with threshold 16, and one
    table where waves refill their lanes."""
    p = plan(count, n_lambda, octree, direct=True)
    chunk = min(256, max(32, count * n_lambda // 4096))
    chunks = -(-count // chunk) * n_lambda
    assert not p["sums"] and p["mixed"] and not p["own_chunks"] and p["copies"] == (chunk <= 32)
    assert (p["lanes"], p["threshold"], p["chunk"], p["n_chunks"]) == (64, 16, chunk, chunks)
    assert p["waves"] == min(4096, chunks)
    # no other launch is held to them
    assert plan(32768, n_lambda, octree, direct=True)["sums"]
    for other in (plan(count, n_lambda, octree), plan(count, n_lambda, octree, point=False),
                  plan(count, n_lambda, octree, direct=True, plain=False)):
        assert not other["mixed"] and not other["sums"] and other["copies"]


@pytest.mark.parametrize("octree", [False, True])
@pytest.mark.parametrize("kind", [dict(point=False), dict(), dict(direct=True), dict(direct=True, plain=False)])
def test_every_packet_has_a_wave(kind, octree):
    """Every chunk has a wave or the queue, and no launch is without one."""
    for count in (1, 2, 63, 64, 65, 2047, 2049, 3073, 12_289, 32_768, 32_769, 196_609, 5_000_000):
        for n_lambda in (1, 7, 64):
            p = plan(count, n_lambda, octree, **kind)
            assert p["lam_chunks"] * p["chunk"] >= count > (p["lam_chunks"] - 1) * p["chunk"]
            assert p["n_chunks"] == p["lam_chunks"] * n_lambda and 1 <= p["lanes"] <= 64
            assert 1 <= p["waves"] <= p["n_chunks"]
            assert p["waves"] == p["n_chunks"] or not p["own_chunks"]


@pytest.mark.parametrize("count", [1, 200, 500, 5000, 32_769, 1_000_000])
@pytest.mark.parametrize("tune", [dict(chunk=1), dict(chunk=16), dict(chunk=64), dict(chunk=256), dict(chunk=1024),
                                  dict(chunk_shift=1), dict(chunk_shift=3), dict(chunk_shift=6),
                                  dict(chunk=256, waves_per_cu=16), dict(chunk_shift=-2)])
@pytest.mark.parametrize("kind", [dict(), dict(point=False), dict(octree=True), dict(direct=True)])
def test_chunks_of_the_caller(kind, tune, count):
    """A wave has a lane for every packet of a chunk, up to 64."""
    p = plan(count, 2, **kind, **tune)
    assert p["lanes"] >= min(64, p["chunk"])
    if tune.get("chunk"):
        assert p["chunk"] == tune["chunk"]
    else:  # the automatic chunk's share of a shift does not change with the lanes
        auto, shift = plan(count, 2, **kind)["chunk"], tune["chunk_shift"]
        assert p["chunk"] == max(1, auto << shift if shift > 0 else auto >> -shift)


@pytest.mark.parametrize("count", [1, 500, 2048, 2049, 3072, 3073, 5000])
@pytest.mark.parametrize("cells", [3, 18, 29, 30, 300])
def test_lone_packets(cells, count):
    """The whole wave marches a packet where it has only one and rays are long."""
    for kind in (dict(), dict(point=False), dict(direct=True), dict(octree=True), dict(plain=False), dict(chunk=2)):
        p = plan(count, cells=cells, **kind)
        assert p["lone"] == (p["lanes"] == 1 and cells >= 30 and not kind.get("octree") and kind.get("plain", True))
    assert plan(count, cells=cells)["lanes"] == max(1, -(-count // 2048))
