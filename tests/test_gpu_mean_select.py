"""GPU parity of the averaged selection that writes the key lists: sizes at the edges of its groups of 64 clusters, steps of 1024
and slices, against the oracle's averaged selection and attention."""
import numpy as np
import pytest

from paper_2411_09688_amd import workload as wl
from test_gpu_prefill import compare_prefill_mean, mean_thresholds, run_prefill_mean_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    from paper_2411_09688_amd import binding
    binding.lib()
    return binding


CASES = [
    dict(B=1, H=1, L=300, C=1, Lq=5),                 # one cluster, longer than a wave writes at once
    dict(B=1, H=2, L=900, C=64, Lq=20),               # one group, full
    dict(B=1, H=2, L=900, C=65, Lq=20),               # and one cluster of the next
    dict(B=1, H=3, L=5000, C=1024, Lq=65),            # one step, full; two parts of the sums
    dict(B=1, H=3, L=5000, C=1025, Lq=40),            # two steps, the second of one cluster
    dict(B=2, H=1, L=6000, C=4097, Lq=33),            # clusters without keys among them, two rounds of loads
    dict(B=1, H=1, L=3000, C=16384, Lq=9),            # the most clusters there are: slices of several groups
    dict(B=150, H=2, L=700, C=200, Lq=3),             # more rows than compute units: one slice each
    dict(B=150, H=2, L=1500, C=1100, Lq=2),           # ... of two steps: slices of at most 16 groups
]


@pytest.mark.parametrize("keep", ["some", "all"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "B{B}H{H}L{L}C{C}Lq{Lq}".format(**c))
def test_mean_step(sq, oracle, case, keep):
    w = wl.make_workload("mean_select", seed=61, threads=4, U=7, keep_frac=0.25, causal_user=False, **case)
    w.thresh, stats = mean_thresholds(oracle, w)
    if keep == "all":
        w.thresh = np.full(w.H, -1.0, np.float32)
    P = sq.upload(w)
    got = run_prefill_mean_step(sq, w, P)
    compare_prefill_mean(oracle, w, P, got, stats, f"mean-select {case} {keep}")
    if keep == "all":
        assert (got[3] == w.sizes.sum(1)[None]).all()
