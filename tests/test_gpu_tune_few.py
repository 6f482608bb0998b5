"""The autotuner on levels of few work items: marches and cubes are candidates
alike, the choice (here given by the cache file) is what runs, and the reported
item depths say so.  Iterates are bit for bit the default's either way."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1104_1703_amd import gen  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def level(key):
    return int(key.split(":l")[1].split(":")[0])


# value of the cache per level (finest, 1, 2 and coarser) and the depths reported
CHOICES = {
    "few": ((-16, -4, -2), (16, 1, 1)),
    "few8": ((-8, -4, -2), (8, 1, 1)),
    "few32-march": ((-32, 2, -8), (32, 2, 1)),
    "march32-8-8": ((32, 8, 8), (32, 8, 8)),
    "march8-2-4": ((8, 2, 4), (8, 2, 4)),
    "cube": ((16, 1, 1), (16, 1, 1)),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(96, 64, 80), (128, 128, 128)], ids=lambda s: "x".join(map(str, s)))
def test_choice_of_the_tuner_is_what_runs(mg, tmp_path, monkeypatch, shape, precision):
    p = gen.holes_problem(n=128, seed=2) if shape == (128, 128, 128) else \
        gen.random_small_problem(shape, 9, active_frac=0.8, blur=2.0)
    print("tune few", shape, precision, flush=True)
    t = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    mask, rho, b = t(p.mask), t(p.rho), t(p.dirichlet)
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("MG_TUNE_CACHE", str(cache))
    with mg.Hierarchy(mask, p.h, precision=precision) as H:
        ref, rinfo = H.solve(rho, None, b, tol=1e-10)
        # a coarse level over cubes reports them; levels of the one-workgroup call keep their depth
        assert H.item_depths()[2][:2] == [16, 1]
    with mg.Hierarchy(mask, p.h, precision=precision, tune=1) as H:
        levels = H.nlevels(2)
    keys = [ln.split()[0] for ln in cache.read_text().splitlines()]
    assert {level(k) for k in keys} >= {0, 1} and all(k.endswith(":few") for k in keys)
    for name, (value, depth) in CHOICES.items():
        cache.write_text("".join(f"{k} {value[min(level(k), 2)]}\n" for k in keys))
        before = cache.read_text()
        with mg.Hierarchy(mask, p.h, precision=precision, tune=1) as H:
            assert cache.read_text() == before, name                   # taken from the file, not timed again
            for k in keys:
                o = int(k.split(":o")[1][0])
                assert H.item_depths()[o][level(k)] == depth[min(level(k), 2)], (name, k)
            assert H.nlevels(2) == levels
            got, info = H.solve(rho, None, b, tol=1e-10)
        assert (info["status"], info["cycles"], info["order_used"]) == \
            (rinfo["status"], rinfo["cycles"], rinfo["order_used"]), name
        assert torch.equal(got, ref), name
        ha, hb = np.array(info["history"]), np.array(rinfo["history"])
        if depth[0] == 16:
            assert np.array_equal(ha, hb), name
        else:  # other groups of partial sums: n terms' rounding at most
            assert np.all(np.abs(ha - hb) <= 1e-13 * np.abs(hb) + 1e-16 * info["r_ref"]), name


def test_entries_of_other_candidates_are_not_taken(mg, tmp_path, monkeypatch):
    """An entry written where cubes were no candidate does not decide such a level."""
    p = gen.sphere_problem(64)
    mask = torch.from_numpy(p.mask).cuda()
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("MG_TUNE_CACHE", str(cache))
    with mg.Hierarchy(mask, p.h, tune=1):
        pass
    lines = cache.read_text().splitlines()
    cache.write_text("".join(ln.split()[0][:-len(":few")] + " 32\n" for ln in lines if level(ln.split()[0]) == 0))
    with mg.Hierarchy(mask, p.h, tune=1):
        assert len(cache.read_text().splitlines()) == 1 + len(lines)
