"""Tuning tables on the host: entries with and without the kind of call they were timed on, and the
values that are refused."""
import json

import pytest

SINGLE = dict(arch="gfx950", precision=0, size_bucket=5, strategy=2, variant=1, gpc=4, tile_items=8, group_bras=1024,
              ket_copies=8)
BATCHED = dict(arch="gfx950", precision=1, gpc=2, block_items=0, owned_bound=-1, waves=8)
KIND = dict(ngauss=3, grad=1, atoms=0)


def _load(tmp_path, single=(), batched=()):
    import paper_2509_21039_amd as hfk
    path = tmp_path / "t.json"
    path.write_text(json.dumps({"format": "hfk-tuning-2", "entries": list(single), "batched": list(batched)}))
    try:
        hfk.load_tuning(str(path))
    finally:
        hfk.clear_tuning()


def test_entries_with_and_without_their_kind(tmp_path):
    _load(tmp_path, [SINGLE, dict(SINGLE, ngauss=6)], [BATCHED, dict(BATCHED, **KIND)])


@pytest.mark.parametrize("single,batched", [
    (dict(ngauss=0), None), (dict(ngauss=99), None), (None, dict(KIND, ngauss=0)), (None, dict(KIND, ngauss=99)),
    (None, dict(KIND, grad=2)), (None, dict(KIND, atoms=-1))])
def test_kinds_out_of_range_are_refused(tmp_path, single, batched):
    import paper_2509_21039_amd as hfk
    with pytest.raises(hfk.HfkError) as err:
        _load(tmp_path, [dict(SINGLE, **single)] if single else [], [dict(BATCHED, **batched)] if batched else [])
    assert err.value.status == hfk.HFK_EINVAL
