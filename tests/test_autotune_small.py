"""The autotuner knows the path that re-indexes a small mesh in one workgroup,
which only the library's default tuning takes."""
import json

import numpy as np
import pytest
import torch

import meshgen
from paper_2109_09812_amd import _lib
from paper_2109_09812_amd import autotune as at

DEFAULT = (0, 0, 0, 0)


def test_small_meshes_have_the_default_as_a_candidate(tmp_path):
    for vb in (4, 12, 64):
        shapes = len(_lib.tunings(vb))
        small = at.candidates(vb, 1689, False)
        assert small[0].as_key() == DEFAULT and len(small) == 2 * shapes + 1
        assert len(at.candidates(vb, 4096, False)) == 2 * shapes + 1
        assert len(at.candidates(vb, 4097, False)) == len(at.candidates(vb, 1689, True)) == 2 * shapes
    entries = {"k": {"tuning": list(DEFAULT)}, "flag": {"tuning": [0, 0, 0, 1]}}
    assert at.cached_tuning(entries, "k", 12).as_key() == DEFAULT
    assert at.cached_tuning(entries, "flag", 12) is None
    # a choice made before the default was among them is made again
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"schema": 3, "abi": _lib.load().mrx_abi_version(), "entries": entries}))
    assert at.load_cache(str(path)) == {}


@pytest.mark.gpu
def test_autotune_picks_one_workgroup_for_a_small_mesh(tmp_path):
    m = meshgen.grid_soup(16, 0.1, 4243, "small")
    v = torch.from_numpy(np.ascontiguousarray(m.vtx).view(np.int32)).to("cuda:0")
    i = torch.from_numpy(m.idx).to("cuda:0")
    print("[case] autotune", v.shape, flush=True)
    path = str(tmp_path / "t.json")
    t, report = at.autotune(v, i, reps=5, path=path)
    assert t.as_key() == DEFAULT, report
    assert at.autotune(v, i, path=path)[0].as_key() == DEFAULT
