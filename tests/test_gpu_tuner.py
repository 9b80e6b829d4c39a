"""GPU: a tuner whose search keeps what the options leave to each launch keeps
it automatic: in the sim, and as 0 in the cache; what it returns are the values
of the trial's launch, which can be set like any others."""
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu

# waves per compute unit and threshold of the automatic launch on 256 compute units
CASES = {"sphere": (2000, (8, 12), 64), "disk": (500, (12,), 64), "torus": (300, (16,), 48)}


def scene(kind):
    if kind == "torus":
        return scenes.torus(max_depth=4, torus_depth=3, n_lambda=2, npix=8, n_clumps=5)
    return scenes.disk((9, 7, 5), 2, 9) if kind == "disk" else scenes.sphere(n=12)


@pytest.mark.parametrize("kind", list(CASES))
def test_automatic_values_stay(kind, tmp_path):
    packets, waves, threshold = CASES[kind]
    cache = tmp_path / "tune.txt"
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, scene(kind), mcrt.FP32)
    t = mcrt.autotune([sim], [packets], seed=2, cache_path=str(cache))
    key, line = cache.read_text().strip().split("|")
    chunk, w, th, ms, default_ms, shift, slots = line.split()
    # a setting that the search took is not the automatic one under another name
    assert int(w) == 0 or int(w) in {8, 12, 16} - set(waves[:1])
    assert int(th) == 0 or int(th) in {8, 16, 24, 32, 48} - {threshold}
    assert int(slots) == 0 and t["deposit_slots"] == 16
    assert t["waves_per_cu"] in ((int(w),) if int(w) else waves) and t["threshold"] == (int(th) or threshold)

    # the automatic values from a cache: as an untuned sim runs
    cache.write_text(f"{key}|0 0 0 1.0 1.0 0 0\n")
    t = mcrt.autotune([sim], [packets], seed=2, cache_path=str(cache))
    assert t["from_cache"] and (t["chunk"], t["chunk_shift"], t["threshold"], t["deposit_slots"]) == (0, 0, threshold, 16)
    assert t["waves_per_cu"] in waves
    plain = mcrt.Sim(ctx, scene(kind), mcrt.FP32)
    a, b = sim.run(packets, seed=1).stats(), plain.run(packets, seed=1).stats()
    assert {k: v for k, v in a.items() if k != "kernel_ms"} == {k: v for k, v in b.items() if k != "kernel_ms"}

    # what was returned can be set; automatic values themselves cannot
    sim.set_tuning(t["chunk"], t["waves_per_cu"], t["threshold"], t["chunk_shift"], t["deposit_slots"])
    for w, th in ((0, threshold), (8, 0)):
        with pytest.raises(mcrt.MCRTError) as e:
            sim.set_tuning(0, w, th)
        assert e.value.code == mcrt.EINVAL
    for s in (sim, plain):
        s.close()
    ctx.close()


def test_batch_values(tmp_path):
    """A batch's automatic values are the same in every launch."""
    cache = tmp_path / "tune.txt"
    ctx = mcrt.Context(0)
    sims = [mcrt.Sim(ctx, scenes.sphere(n=n), mcrt.FP32) for n in (8, 10)]
    key = f"grid=cartesian prec=fp32 models=2 cells=2^{(8 ** 3 + 10 ** 3 - 1).bit_length()} lambda=1 ins=1"
    cache.write_text(f"{key}|0 0 0 1.0 1.0 0 0\n")
    t = mcrt.autotune(sims, [100, 100], cache_path=str(cache))
    assert t["from_cache"] and (t["waves_per_cu"], t["threshold"], t["deposit_slots"]) == (16, 24, 16)
    for s in sims:
        s.close()
    ctx.close()
