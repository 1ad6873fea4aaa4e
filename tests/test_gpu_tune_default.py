"""The tuner's choices belong to the default kernel of the launches that they
were made for: small launches, whose default is another kernel, keep choices
of their own in a shared cache, whatever the size of the sample."""
import json

import numpy as np
import pytest

from paper_2303_13632_amd import eri, workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PRIM = 13


def test_cache_of_small_and_large_launches(tmp_path):
    cid = W.class_id(1, 1, 1, 1)
    cache = str(tmp_path / "tune.json")
    small = eri.Plan(*W.random_class_quartets(1, 1, 1, 1, 60, 1), bits=16)
    large = eri.Plan(*W.random_class_quartets(1, 1, 1, 1, 6000, 2), bits=16)
    assert small.class_tag[cid] == PRIM and large.class_tag[cid] != PRIM
    # an entry of another kernel's making is not taken: variant 1 for the large launches
    with open(cache, "w") as f:
        json.dump({"fp64:%d:16" % cid: 1}, f)
    small.tune(sample_quartets=60, trials=1, cache=cache)
    data = json.load(open(cache))
    assert set(data) == {"fp64:%d:16" % cid, "fp64:%d:d%d:16" % (cid, PRIM)} and data["fp64:%d:16" % cid] == 1
    assert small.class_variant[cid] == data["fp64:%d:d%d:16" % (cid, PRIM)]
    large.tune(sample_quartets=6000, trials=1, cache=cache)
    assert large.class_variant[cid] == 1


def test_sample_smaller_than_the_launches(tmp_path):
    """A sample of a size at which the default would be another kernel is timed
    against the kernel of the plan's launches."""
    cid = W.class_id(1, 1, 1, 1)
    cache = str(tmp_path / "tune.json")
    plan = eri.Plan(*W.random_class_quartets(1, 1, 1, 1, 6000, 2), bits=16)
    plan.tune(sample_quartets=60, trials=1, cache=cache)
    assert list(json.load(open(cache))) == ["fp64:%d:16" % cid]
    plan.set_variants(np.zeros(256, np.int32))
    assert plan.class_tag[cid] != PRIM
