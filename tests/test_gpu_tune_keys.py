"""Which calls a tuned entry applies to: the kind of call it was timed on, and, for entries that
do not say (tables written before they did), every call of their precision."""
import json

import numpy as np
import pytest

from he_inputs import HE_STO3G_COEFS as C3, HE_STO3G_EXPS as E3, cluster_batch, pack_batch, random_cluster
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture
def hfk_dev():
    import torch
    import paper_2509_21039_amd as hfk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    hfk.clear_tuning()
    yield hfk, torch, torch.device("cuda:0")
    hfk.clear_tuning()


def _table(path, arch, single=(), batched=()):
    json.dump({"format": "hfk-tuning-2", "entries": [dict(arch=arch, **x) for x in single],
               "batched": [dict(arch=arch, **x) for x in batched]}, open(path, "w"))
    return str(path)


def _arch(torch):
    return torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]


def _batch_groups(hfk, torch, dev, systems, grad, atoms, g):
    off, xyz, dens = pack_batch(systems)
    e, c = np.array(E3[3 - g:]), np.array(C3[3 - g:])
    if atoms:
        e, c = np.tile(e, (off[-1], 1)), np.tile(c, (off[-1], 1))
    ws = hfk.new_workspace(hfk.batched_workspace_bytes(off, g, "fp64", grad, atoms), dev)
    hfk.fock_batched(off, torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev), e, c, 1e-10, "fp64",
                     with_grad=grad, workspace=ws)
    return hfk.read_stats(ws)["groups"]


def test_batched_entry_applies_to_its_kind_of_call(hfk_dev, tmp_path):
    hfk, torch, dev = hfk_dev
    systems = [random_cluster(n, 700 + n, box=8.0) for n in (3, 17, 30)]
    kinds = [(grad, atoms, g) for grad in (False, True) for atoms in (False, True) for g in (2, 3)]
    announce("batched tuning keys")
    untuned = {k: _batch_groups(hfk, torch, dev, systems, *k) for k in kinds}
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    one = dict(precision=0, gpc=1, block_items=0, owned_bound=-1, waves=8)
    hfk.load_tuning(_table(tmp_path / "kind.json", _arch(torch), batched=[dict(one, ngauss=3, grad=0, atoms=0)]))
    assert untuned[False, False, 3] > cus
    for k in kinds:
        want = cus if k == (False, False, 3) else untuned[k]
        assert _batch_groups(hfk, torch, dev, systems, *k) == want, k
    # an entry without the keys takes the place of every entry of its precision
    hfk.load_tuning(_table(tmp_path / "any.json", _arch(torch), batched=[one]))
    assert all(_batch_groups(hfk, torch, dev, systems, *k) == cus for k in kinds)


def test_tuning_one_kind_of_batch_does_not_slow_another(hfk_dev, tmp_path):
    hfk, torch, dev = hfk_dev
    systems = cluster_batch(nmol=120, seed=21)
    off, xyz, dens = pack_batch(systems)
    X, D, s = torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev), systems[0]
    ws = hfk.new_workspace(hfk.batched_workspace_bytes(off, 3, "fp64", True), dev)

    def timed(grad):
        best = 1e30
        for r in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            hfk.fock_batched(off, X, D, s.exps, s.coefs, s.tau, "fp64", with_grad=grad, workspace=ws)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1)) if r else best
        return best

    announce("batched fp64: untuned, then tuned forward only, then with the gradient")
    untuned = {grad: timed(grad) for grad in (False, True)}
    hfk.tune_batched(off, X, D, s.exps, s.coefs, s.tau, precision="fp64", with_grad=False)
    assert timed(True) <= 1.05 * untuned[True]
    path = str(tmp_path / "both.json")
    hfk.tune_batched(off, X, D, s.exps, s.coefs, s.tau, precision="fp64", with_grad=True, cache_path=path)
    assert all(timed(grad) <= 1.05 * untuned[grad] for grad in (False, True))
    entries = json.load(open(path))["batched"]
    assert sorted((x["ngauss"], x["grad"], x["atoms"]) for x in entries) == [(3, 0, 0), (3, 1, 0)]


def _tile(hfk, torch, dev, n, g):
    s = random_cluster(n, 40 + g, box=6.0)
    e, c = 0.2 * 3.0 ** np.arange(g - 1, -1, -1.0), np.linspace(0.2, 0.6, g)
    ws = hfk.new_workspace(hfk.workspace_bytes(n, g, "fp64"), dev)
    hfk.fock(torch.tensor(s.xyz, device=dev), torch.tensor(s.dens, device=dev), e, c, 1e-10, workspace=ws)
    return hfk.read_stats(ws)["tile_items"]


def test_entry_of_few_primitives_leaves_builds_of_many_their_default(hfk_dev, tmp_path):
    # five and six primitives on few atoms have a default of their own (one item per block)
    hfk, torch, dev = hfk_dev
    announce("tuning keys of the single-molecule build")
    gs = (1, 3, 4, 5, 6)
    untuned = {g: _tile(hfk, torch, dev, 20, g) for g in gs}
    entry = dict(precision=0, size_bucket=5, strategy=2, variant=1, gpc=4, group_bras=1024, ket_copies=8)
    hfk.load_tuning(_table(tmp_path / "g3.json", _arch(torch), single=[dict(entry, tile_items=16, ngauss=3)]))
    for g in gs:
        assert _tile(hfk, torch, dev, 20, g) == (16 if g <= 4 else untuned[g]), g
    hfk.load_tuning(_table(tmp_path / "g6.json", _arch(torch), single=[dict(entry, tile_items=4, ngauss=6)]))
    for g in gs:
        assert _tile(hfk, torch, dev, 20, g) == (16 if g <= 4 else 4), g
    # an entry without ngauss takes the place of every entry of its precision and size
    hfk.load_tuning(_table(tmp_path / "any.json", _arch(torch), single=[dict(entry, tile_items=2)]))
    assert all(_tile(hfk, torch, dev, 20, g) == 2 for g in gs)


def test_tuned_entry_names_its_primitives(hfk_dev, tmp_path):
    hfk, torch, dev = hfk_dev
    s = random_cluster(12, 3, box=6.0)
    X, D = torch.tensor(s.xyz, device=dev), torch.tensor(s.dens, device=dev)
    path = str(tmp_path / "t.json")
    announce("tuner: two contractions of one size")
    hfk.tune(X, D, s.exps, s.coefs, 1e-10, cache_path=path)
    hfk.tune(X, D, [6.0, 3.0, 1.5, 0.8, 0.4, 0.2], [0.1, 0.2, 0.3, 0.4, 0.3, 0.2], 1e-10, cache_path=path)
    assert [(x["size_bucket"], x["ngauss"]) for x in json.load(open(path))["entries"]] == [(4, 3), (4, 6)]
