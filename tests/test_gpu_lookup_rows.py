"""GPU parity of the prefill lookup that keeps a row's scores in registers, at the edges of its tiles of 32 clusters x 32 tokens, of
its eight waves and of the rule that gives long rows of few tokens to the sliced launches, against the oracle: masks and key counts
per query, masks of the averaged selection, clusters without keys whose centroids are not finite among them."""
import numpy as np
import pytest

from paper_2411_09688_amd import workload as wl
from test_gpu_prefill import compare_prefill, compare_prefill_mean, mean_thresholds, run_prefill_mean_step, run_prefill_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    from paper_2411_09688_amd import binding
    binding.lib()
    return binding


CASES = [
    dict(B=1, H=1, L=200, C=1, Lq=1),
    dict(B=1, H=3, L=500, C=31, Lq=31),
    dict(B=1, H=3, L=500, C=32, Lq=32),
    dict(B=2, H=2, L=600, C=33, Lq=33),
    dict(B=1, H=2, L=3000, C=256, Lq=65),             # one tile per wave
    dict(B=1, H=2, L=3000, C=257, Lq=64),             # and a tile of one cluster
    dict(B=1, H=2, L=5000, C=512, Lq=40),             # the longest row at any number of tokens
    dict(B=1, H=2, L=5000, C=513, Lq=40),             # sliced: too few tokens for a row of this length
    dict(B=1, H=63, L=2000, C=600, Lq=32),            # sliced: the most workgroups
    dict(B=1, H=64, L=2000, C=600, Lq=32),            # in registers: the fewest
    dict(B=2, H=32, L=2500, C=1024, Lq=30),           # the longest row; many clusters without keys
    dict(B=2, H=32, L=2500, C=1025, Lq=30),           # sliced
    dict(B=3, H=200, L=300, C=40, Lq=70),             # averaged: several blocks of tokens per workgroup
]


EMPTY = [
    dict(B=1, H=2, L=60, C=40, Lq=33),
    dict(B=1, H=2, L=900, C=500, Lq=40),
    dict(B=2, H=32, L=1500, C=1024, Lq=30),
    dict(B=1, H=2, L=1500, C=1024, Lq=40),            # sliced
]


def run(sq, oracle, w, centroids):
    per_query = wl.calibrate(w, oracle.scores).thresh
    averaged, stats = mean_thresholds(oracle, w)
    good = w.centroids
    w.thresh, w.centroids = per_query, centroids
    P = sq.upload(w)
    w.centroids = good
    run_prefill_step(sq, w, P)
    compare_prefill(oracle, w, P, "lookup", logits=False)
    w.thresh, w.centroids = averaged, centroids
    P = sq.upload(w)
    w.centroids = good
    compare_prefill_mean(oracle, w, P, run_prefill_mean_step(sq, w, P), stats, "lookup-mean")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B{B}H{H}L{L}C{C}Lq{Lq}".format(**c))
def test_lookup(sq, oracle, case):
    w = wl.make_workload("lookup_rows", seed=71, threads=4, U=3, keep_frac=0.25, causal_user=False, **case)
    run(sq, oracle, w, w.centroids)


@pytest.mark.parametrize("case", EMPTY, ids=lambda c: "B{B}H{H}L{L}C{C}Lq{Lq}".format(**c))
def test_clusters_without_keys_take_no_part(sq, oracle, case):
    """Whatever their centroids hold: the oracle sees finite ones, the library NaN and infinities."""
    w = wl.make_workload("lookup_empty", seed=72, threads=4, U=3, keep_frac=0.25, causal_user=False, **case)
    empty = w.sizes == 0
    assert empty.any(1).all()
    cent = w.centroids.copy()
    cent[empty] = np.resize(np.array([np.nan, np.inf, -np.inf], np.float16), (int(empty.sum()), 1))
    run(sq, oracle, w, cent)
