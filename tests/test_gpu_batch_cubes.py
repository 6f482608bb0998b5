"""Batch launches of few live patches run over whole 8^3 cubes: bit for bit the
persistent engine (whose phases march over the work items), from one patch to
batches that start above the line and cross it as patches converge."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1104_1703_amd import gen  # noqa: E402


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def _patches(case):
    if case == "one":
        return [gen.random_small_problem((24, 40, 68), 5, active_frac=0.75, blur=1.5)]
    if case == "ragged":
        shapes = [(16, 16, 32), (24, 40, 68), (40, 72, 104), (12, 36, 20), (64, 64, 64)]
        return [gen.random_small_problem(s, 5 + i, active_frac=0.75, blur=1.5) for i, s in enumerate(shapes)]
    # 64 patches of 512 cubes: 32768 finest and 4096 level-1 cubes at the start
    one = [gen.holes_problem(n=64, seed=s, n_holes=8) for s in range(4)]
    return [one[i % 4] for i in range(64)]


@pytest.mark.parametrize("case", ["one", "ragged", "many"])
@pytest.mark.parametrize("opts", [dict(), dict(n_pre=1, n_post=1), dict(n_cycles=2), dict(n_pre=3, n_post=1, bc_order="first")],
                         ids=lambda o: "-".join(f"{k}={v}" for k, v in o.items()) or "default")
def test_cubes_equal_persistent_marches(mg, case, opts):
    print("batch cubes", case, opts, flush=True)
    probs = _patches(case)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
    B = mg.Batch([dev(p.mask) for p in probs], [p.h for p in probs], max_cycles=30, **opts)
    if B.phases(2) == 0:
        pytest.skip("the programs do not cover these options")
    assert B.validate()[0] == 0
    rhos, dirs = [dev(p.rho) for p in probs], [dev(p.dirichlet) for p in probs]
    out = {}
    for engine in ("persistent", "phased"):
        B.set_engine(engine)
        for _ in range(2):  # the second solve follows the first's boundary orders
            x, info, _ms = B.solve(rhos, None, dirs, tol=1e-9, check=False)
        out[engine] = x, info
        B.close()
        B = mg.Batch([dev(p.mask) for p in probs], [p.h for p in probs], max_cycles=30, **opts)
    B.close()
    (xp, ip), (xc, ic) = out["persistent"], out["phased"]
    for a, b, i, j in zip(xp, xc, ip, ic):
        assert (i["status"], i["cycles"], i["switched_at"], i["order_used"]) == \
            (j["status"], j["cycles"], j["switched_at"], j["order_used"])
        assert i["history"] == j["history"]
        assert torch.equal(a, b)
