"""What Ensemble.predict_many refuses before anything reaches a device: no items, and scenarios whose
coordinate arrays do not join."""
import dataclasses

import pytest

from paper_2009_10400_amd import surrogate
from paper_2009_10400_amd import workloads as W


@pytest.fixture
def ensemble():
    e = surrogate.Ensemble.__new__(surrogate.Ensemble)     # no networks: the refusals come first
    e.device, e.t_ref = 0, 300.0
    return e


def test_no_items(ensemble):
    with pytest.raises(ValueError, match="at least one array"):
        ensemble.predict_many([])


def test_coordinates_that_do_not_join(ensemble):
    (p, d), (q, e) = W.planning_scenarios(2, seed=3, lo=1000, hi=1500)
    with pytest.raises(ValueError, match="dimension"):
        ensemble.predict_many([(p, d), (dataclasses.replace(q, X=q.X[:, :2]), e)])
