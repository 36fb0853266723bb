"""GPU parity of the averaged selection that writes the key lists: sizes at the edges of its groups of 64 clusters, steps of 1024
and slices, against the oracle's averaged selection and attention."""
import numpy as np
import pytest
import torch

from gpu_util import ranges_from_keep, unpack_mask
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


ROUTES = [
    dict(B=1, H=3, L=2500, C=100, Lq=33, U=40),             # six shares of a few blocks
    dict(B=2, H=12, L=3001, C=99, Lq=333, U=333),
    dict(B=1, H=2, L=9000, C=2048, Lq=40, U=7),             # the most clusters that the attention launch selects from
    dict(B=1, H=2, L=9000, C=2049, Lq=40, U=7),             # and one more: a launch of its own
    dict(B=200, H=1, L=64 * 256, C=300, Lq=150, U=5),       # eight waves: the longest share, 256 blocks
    dict(B=200, H=1, L=64 * 256 + 1, C=300, Lq=150, U=5),   # and one block more
    dict(B=500, H=1, L=64 * 48, C=150, Lq=3, U=7),          # four waves: 48 blocks
    dict(B=500, H=1, L=64 * 48 + 1, C=150, Lq=3, U=7),
    dict(B=30, H=32, L=400, C=20, Lq=4, U=3),               # four waves: 15/8 of a round of workgroups
    dict(B=31, H=31, L=400, C=20, Lq=4, U=3),               # and one workgroup more
]


@pytest.mark.parametrize("keep", ["some", "all"])
@pytest.mark.parametrize("case", ROUTES, ids=lambda c: "B{B}H{H}L{L}C{C}Lq{Lq}".format(**c))
def test_step_equals_attention_over_its_set(sq, case, keep):
    """Whether the attention launch makes the kept set or a launch in front of it: the same bits as the call that is given the set's
    ranges, values that are not finite included, and all-kept rows keep everything."""
    w = wl.make_workload("mean_routes", seed=62, threads=4, keep_frac=0.25, causal_user=True, **case)
    w.thresh = np.full(w.H, -1.0 if keep == "all" else 0.6 / w.L, np.float32)   # (average scores are around 1 / L)
    P = sq.upload(w)
    P.V_fixed[:, ::7, 9] = np.inf
    P.V_user[:, :, 1, 77] = np.nan
    mask, _, _, nk = run_prefill_mean_step(sq, w, P)
    out, lse = P.out.clone(), P.lse.clone()
    kept = unpack_mask(mask, w.C)
    np.testing.assert_array_equal(nk, (kept * w.sizes[None]).sum(-1))
    if keep == "all":
        np.testing.assert_array_equal(nk, np.broadcast_to(w.sizes.sum(1), nk.shape))
    else:
        assert 0 < kept.sum() < kept.size
    ranges, nr = np.zeros((w.B, w.H, w.C, 2), np.int32), np.zeros((w.B, w.H), np.int32)
    for b in range(w.B):
        for h in range(w.H):
            ranges[b, h], nr[b, h] = ranges_from_keep(kept[b, h], w.offsets[h], w.sizes[h], w.C)
    t = lambda a: torch.from_numpy(a).to(P.q.device)  # noqa: E731
    P.out.fill_(7.0)
    sq.sq_sparse_attn_prefill_shared(P.shape, P.q, P.K_fixed, P.V_fixed, t(ranges), t(nr), t(nk), P.K_user, P.V_user, P.out, P.lse,
                                     sq.workspace(P.shape, sq.SQ_CALL_ATTN_PREFILL_SHARED, P.q.device))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), P.out.cpu().numpy())
    np.testing.assert_array_equal(lse.cpu().numpy(), P.lse.cpu().numpy())
