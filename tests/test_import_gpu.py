"""Device import of leaf sets at the edges of its range (a single cell, no
refinement, the deepest level, faults at the first and last leaf), and meshes
made and dropped in turn on two streams, whose buffers pass from one to the
other."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2203_10000_amd as sal  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sal.Context(0)


@pytest.mark.parametrize("cells,rounds", [((1, 1, 1), 0), ((1, 1, 1), 3), ((7, 3, 2), 1), ((5, 6, 4), 3)])
def test_import_of_an_export_gives_the_same_leaves(ctx, cells, rounds):
    ss = sal.SurfaceSet(ctx, synth.config_small("head", subdiv=2).surfaces)
    a = sal.TetMesh(ctx, (-100.0, -100.0, -100.0), 200.0 / max(cells), cells)
    a.refine_relabel(ss, rounds)
    e = a.export(centroids=False)
    perm = torch.randperm(len(e["keys"]), generator=torch.Generator().manual_seed(3)).cuda()
    b = sal.TetMesh(ctx, (-100.0, -100.0, -100.0), 200.0 / max(cells), cells)
    b.import_leaves(e["keys"][perm], e["labels"][perm])
    f = b.export(centroids=False)
    assert b.size() == a.size()
    order = lambda x: torch.argsort(x["keys"])  # noqa: E731
    oa, ob = order(e), order(f)
    assert torch.equal(e["keys"][oa], f["keys"][ob]) and torch.equal(e["labels"][oa], f["labels"][ob])
    # one fault at either end of the set: refused, and the mesh still fresh
    for at in (0, -1):
        keys, labels = e["keys"].clone(), e["labels"].clone()
        for bad_keys, bad_labels in ((torch.cat([keys[:at], keys[at:][1:]]), torch.cat([labels[:at], labels[at:][1:]])),
                                     (torch.cat([keys, keys[at:][:1]]), torch.cat([labels, labels[at:][:1]]))):
            c = sal.TetMesh(ctx, (-100.0, -100.0, -100.0), 200.0 / max(cells), cells)
            with pytest.raises(sal.SalError) as err:
                c.import_leaves(bad_keys, bad_labels)
            assert err.value.status == 1
            c.import_leaves(keys, labels)
            assert c.size() == a.size()


def test_meshes_in_turn_on_two_streams(ctx):
    cfg = synth.config_small("head", cells=12, subdiv=3)
    lat = cfg.lattice

    def leaves(c):
        mesh = sal.TetMesh(c, lat.origin, lat.h, lat.cells)
        ss = sal.SurfaceSet(c, cfg.surfaces)
        mesh.refine_relabel(ss, 2, rule="four_nodes")
        mesh.conform()
        mesh.smooth(max_iter_surface=2, max_iter_volume=2)
        out = mesh.export_conforming()
        return {k: v.clone() for k, v in out.items()}

    want = leaves(ctx)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    other = sal.Context(0, streams[0])
    moved = sal.Context(0, streams[0])
    for turn in range(3):
        moved.set_stream(streams[turn % 2])          # the same context, another stream
        for c, s in ((other, streams[0]), (moved, streams[turn % 2])):
            with torch.cuda.stream(s):
                got = leaves(c)
            s.synchronize()
            assert all(torch.equal(got[k], want[k]) for k in want)
