"""Error paths under injected device-allocation failures
(sal_debug_fail_allocation): every allocation point of context creation,
surface-set creation, labeling and refinement fails once in turn; the call
that meets it reports out of memory, a refine round that fails leaves the
mesh as it was, and after disarming, the same objects (or new ones) give the
results of a run without failures."""
import numpy as np
import pytest

import synth
from oracle import kuhn

torch = pytest.importorskip("torch")
import paper_2203_10000_amd as sal  # noqa: E402

pytestmark = pytest.mark.gpu

OOM, DEVICE = 4, 5


@pytest.fixture(scope="module")
def case():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = synth.config_small("head", cells=8, subdiv=2)
    rng = np.random.default_rng(71)
    pts = synth.uniform_box(rng, 20000, -100, 100)
    return cfg, pts


def _run(cfg, pts, rule, state):
    """The sequence, resumable: creates what `state` lacks, then labels and
    refines.  Raises SalError at the first failure."""
    if "ctx" not in state:
        state["ctx"] = sal.Context(0)
    ctx = state["ctx"]
    if "ss" not in state:
        state["ss"] = sal.SurfaceSet(ctx, cfg.surfaces)
    if "labels" not in state:
        dev = torch.from_numpy(pts).to("cuda:0").contiguous()
        lab, _, _ = sal.label_points(ctx, state["ss"], dev)
        state["labels"] = lab.cpu().numpy()
    lat = cfg.lattice
    if "mesh" not in state:
        state["mesh"] = sal.TetMesh(ctx, lat.origin, lat.h, lat.cells)
    mesh = state["mesh"]
    while mesh.size()[1] < 2:
        mesh.refine_relabel(state["ss"], 1, rule=rule)
    e = mesh.export(keys=True, labels=True, centroids=False)
    return state["labels"], e["keys"].cpu().numpy(), e["labels"].cpu().numpy()


@pytest.mark.parametrize("rule", ["centroid", "four_nodes"])
def test_every_allocation_failure_is_reported_and_recoverable(case, rule):
    cfg, pts = case
    want = _run(cfg, pts, rule, {})
    failures = 0
    for k in range(1, 200):
        state = {}
        sal.lib().sal_debug_fail_allocation(k)
        try:
            got = _run(cfg, pts, rule, state)
            hit = False
        except sal.SalError as e:
            hit = True
            assert e.status in (OOM, DEVICE), (k, e.status, str(e))
            if "mesh" in state and "labels" in state:
                # a failed refine round changes nothing: leaves == N0 + 7 x split
                n, lv = state["mesh"].size()
                keys = state["mesh"].export(keys=True, labels=False, centroids=False)["keys"]
                assert len(keys) == n
        finally:
            sal.lib().sal_debug_fail_allocation(0)
        if not hit:
            # k is past the last allocation of the whole sequence
            assert failures > 0
            for a, b in zip(got, want):
                assert np.array_equal(a, b)
            break
        failures += 1
        got = _run(cfg, pts, rule, state)       # the same objects, disarmed
        for a, b in zip(got, want):
            assert np.array_equal(a, b), k
    else:
        pytest.fail("the sequence kept failing")
    assert failures >= 8


def test_a_failed_round_over_levels_of_unlike_sizes_changes_nothing(case):
    """A round that labels 373,248 points of one level, then 248,832 of the next
    coarser one: the second needs more tiles of the spatial order than the first,
    and every buffer has to be there before the first split."""
    nx, ny = 19, 18
    ctx = sal.Context(0)
    cfg = case[0]
    ss = sal.SurfaceSet(ctx, cfg.surfaces)
    k0 = kuhn.level0_keys((nx, ny, ny))
    deep = np.arange(len(k0)) // 6 % nx < 3          # three layers of cells along x, split once
    keys = np.concatenate([k0[~deep], kuhn.children(k0[deep], (nx, ny, ny)).reshape(-1)])
    labels = np.arange(len(keys)) % 5                # nearly every leaf has a neighbour of another label
    d_keys = torch.from_numpy(keys.view(np.int64)).cuda()
    d_labels = torch.from_numpy(labels.astype(np.int32)).cuda()
    failures = 0
    for k in range(1, 60):
        mesh = sal.TetMesh(ctx, (-95.0, -90.0, -90.0), 10.0, (nx, ny, ny))
        mesh.import_leaves(d_keys, d_labels)
        ctx2 = sal.Context(0)                        # (its labeling scratch is not there yet)
        mesh.ctx = ctx2
        before = mesh.size()
        sal.lib().sal_debug_fail_allocation(k)
        try:
            mesh.refine_relabel(ss, 1)
            hit = False
        except sal.SalError as e:
            hit = True
            assert e.status in (OOM, DEVICE), (k, e.status, str(e))
        finally:
            sal.lib().sal_debug_fail_allocation(0)
        if hit:
            assert mesh.size() == before, k
            left = mesh.export(keys=True, labels=True, centroids=False)
            assert int(left["labels"].min()) >= 0, k
            failures += 1
        mesh.close()
        ctx2.close()
        if not hit:
            break
    else:
        pytest.fail("the round kept failing")
    assert failures >= 8
