"""GPU parity of every form of the prefill attention kernels: workgroups of eight and of four waves, one and several shares of
the key blocks, block lists built in several rounds, walks longer than the entries held in registers.  Each case states the
division that sq_prefill_plan reports for it, so that a changed rule cannot leave a form untested unnoticed."""
import numpy as np
import pytest
import torch

from gpu_util import ATTN_ATOL, ranges_from_keep
from paper_2411_09688_amd import workload as wl
from test_gpu_prefill import banded_keep

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def sq():
    from paper_2411_09688_amd import binding
    binding.lib()
    return binding


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def sample_rows(w, n, seed):
    sel = np.zeros((w.B, w.H, w.Lq), bool)
    sel.ravel()[np.random.default_rng(seed).choice(sel.size, size=min(n, sel.size), replace=False)] = True
    sel[0, 0, 0] = sel[-1, -1, -1] = True
    return sel


def compare(oracle, w, P, ranges, nr, sel):
    out, lse = oracle.sparse_attn(w.q, w.K_fixed, w.V_fixed, ranges, nr, w.K_user, w.V_user, w.sm_scale,
                                  causal_user=w.causal_user, row_sel=sel)
    got, glse = P.out.cpu().numpy().astype(np.float64), P.lse.cpu().numpy()
    assert np.abs(got[sel] - out[sel]).max() <= ATTN_ATOL
    fin = np.isfinite(lse[sel])
    assert (np.isneginf(glse[sel]) == ~fin).all()
    np.testing.assert_allclose(glse[sel][fin], lse[sel][fin], atol=2e-4, rtol=1e-5)


def needed_share(w, gk, queries):
    """Share of the (wave, listed block) pairs with a kept key: a wave owns 32 queries, a workgroup lists what its waves need."""
    nblk, need, listed = (w.L + 63) // 64, 0, 0
    for h in range(w.H):
        cid = np.repeat(np.arange(w.C), w.sizes[h])
        for b in range(0, w.B, max(1, w.B // 8)):
            for g in range(0, w.Lq, queries):
                waves = [np.add.reduceat(gk[b, h, a:min(a + 32, g + queries)].any(0)[cid], np.arange(0, w.L, 64)) > 0
                         for a in range(g, min(g + queries, w.Lq), 32)]
                need += sum(int(v.sum()) for v in waves)
                listed += int(np.any(waves, axis=0).sum()) * len(waves)
    return need / listed


MASKED = [
    (8, 1, dict(B=200, H=1, L=64 * 600 + 9, C=300, Lq=150, U=5)),       # 601 blocks a share: the list is built in two rounds
    (4, 1, dict(B=500, H=1, L=64 * 300 + 7, C=150, Lq=3, U=70)),        # 301: two rounds of 256 threads
    (8, 5, dict(B=2, H=12, L=3001, C=99, Lq=333, U=333)),
    (4, 6, dict(B=2, H=40, L=4096, C=100, Lq=120, U=120)),
    (8, 2, dict(B=1, H=32, L=64 * 150, C=300, Lq=1000, U=64)),           # 75 listed blocks
    (4, 12, dict(B=1, H=40, L=20000, C=300, Lq=31, U=31)),               # the first tiles wait for the list
    (4, 12, dict(B=1, H=40, L=20000, C=300, Lq=32, U=32)),               # and leave before it
]


@pytest.mark.parametrize("waves,splits,case", MASKED)
@pytest.mark.parametrize("masks", ["random", "positions"])
def test_per_query_selection(sq, oracle, waves, splits, case, masks):
    """Explicit masks, drawn for every query by itself (every wave needs nearly every block) or in bands that 32 queries share."""
    w = wl.make_workload("prefill_forms", seed=51, threads=4, keep_frac=0.3, causal_user=True, **case)
    rng = np.random.default_rng(12)
    if masks == "random":
        gk = rng.random((w.B, w.H, w.Lq, w.C)) < 0.4
    else:
        gk = banded_keep(w, rng, max(4, w.C // 8), 1, qb=32)
    W = (w.C + 31) // 32
    bits = np.zeros((w.B, w.H, w.Lq, W * 32), bool)
    bits[..., :w.C] = gk
    words = (bits.reshape(w.B, w.H, w.Lq, W, 32) * (1 << np.arange(32, dtype=np.uint64))).sum(-1).astype(np.uint32)
    P = sq.upload(w)
    assert sq.sq_prefill_plan(P.shape) == (waves, splits)
    share = needed_share(w, gk, 32 * waves)
    assert share > 0.9 if masks == "random" else share < 0.7 or w.Lq <= 32
    P.keep_mask.copy_(torch.from_numpy(words.view(np.int32)))
    P.out.fill_(7.0)
    sq.sq_sparse_attn_prefill(P.shape, P.q, P.K_fixed, P.V_fixed, P.offsets, P.keep_mask, P.K_user, P.V_user, P.out, P.lse,
                              sq.workspace(P.shape, sq.SQ_CALL_ATTN_PREFILL, DEV))
    torch.cuda.synchronize()
    sel = sample_rows(w, 400, 13)
    cap = int(gk.sum(-1)[sel].max()) + 1
    ranges = np.zeros((w.B, w.H, w.Lq, cap, 2), np.int32)
    nr = np.zeros((w.B, w.H, w.Lq), np.int32)
    for b, h, i in np.argwhere(sel):
        ranges[b, h, i], nr[b, h, i] = ranges_from_keep(gk[b, h, i], w.offsets[h], w.sizes[h], cap)
    compare(oracle, w, P, ranges, nr, sel)


ONE_SET = [
    (8, 1, dict(B=200, H=1, L=64 * 300 + 9, C=300, Lq=150, U=5)),
    (4, 1, dict(B=500, H=1, L=64 * 200 + 7, C=150, Lq=3, U=70)),
    (8, 3, dict(B=2, H=12, L=3001, C=99, Lq=333, U=333)),
    (4, 11, dict(B=1, H=40, L=20000, C=600, Lq=33, U=33)),
]


@pytest.mark.parametrize("waves,splits,case", ONE_SET)
@pytest.mark.parametrize("share", [0.02, 0.6])
def test_one_kept_set(sq, oracle, waves, splits, case, share):
    w = wl.make_workload("prefill_forms_one", seed=52, threads=4, keep_frac=0.3, causal_user=True, **case)
    kept = np.random.default_rng(14).random((w.B, w.H, w.C)) < share
    P = sq.upload(w)
    assert sq.sq_prefill_plan(P.shape, one_set=True) == (waves, splits)
    ranges = np.zeros((w.B, w.H, w.C, 2), np.int32)
    nr = np.zeros((w.B, w.H), np.int32)
    for b in range(w.B):
        for h in range(w.H):
            ranges[b, h], nr[b, h] = ranges_from_keep(kept[b, h], w.offsets[h], w.sizes[h], w.C)
    nk = (kept * w.sizes[None]).sum(-1).astype(np.int32)
    P.out.fill_(7.0)
    sq.sq_sparse_attn_prefill_shared(P.shape, P.q, P.K_fixed, P.V_fixed, t(ranges), t(nr), t(nk), P.K_user, P.V_user, P.out,
                                     P.lse, sq.workspace(P.shape, sq.SQ_CALL_ATTN_PREFILL_SHARED, DEV))
    torch.cuda.synchronize()
    sel = sample_rows(w, 400, 15)
    cap = max(1, int(nr.max()))
    rr = np.ascontiguousarray(np.broadcast_to(ranges[:, :, None, :cap], (w.B, w.H, w.Lq, cap, 2)))
    nn = np.ascontiguousarray(np.broadcast_to(nr[:, :, None], (w.B, w.H, w.Lq)))
    compare(oracle, w, P, rr, nn, sel)


# Rows x shares on either side of the lines between the merges: one, two and eight half waves per row, one and several rounds.
MERGED = [
    (8, 12, dict(B=1, H=20, L=3000, C=99, Lq=60, U=3)),                  # 1200 rows: two half waves
    (8, 19, dict(B=1, H=4, L=6000, C=99, Lq=369, U=3)),                  # 1476 rows: two half waves, two rounds
    (4, 16, dict(B=1, H=32, L=9600, C=99, Lq=20, U=3)),                  # 640 rows
    (8, 24, dict(B=1, H=10, L=6000, C=99, Lq=100, U=3)),                 # 1000 rows: eight half waves
    (8, 46, dict(B=1, H=1, L=64 * 90, C=99, Lq=9, U=3)),                 # nine rows
    (8, 8, dict(B=1, H=5, L=4000, C=99, Lq=1000, U=3)),                  # one round of eight
    (8, 11, dict(B=1, H=6, L=4000, C=99, Lq=700, U=3)),                  # one half wave, rounds of six and five
    (8, 14, dict(B=1, H=6, L=8000, C=99, Lq=700, U=3)),                  # of seven
    (8, 16, dict(B=1, H=8, L=12000, C=99, Lq=512, U=3)),                 # of eight
    (8, 13, dict(B=1, H=3, L=4000, C=99, Lq=1000, U=3)),                 # two half waves, seven and six
    (8, 22, dict(B=1, H=2, L=4000, C=99, Lq=512, U=3)),                  # two rounds of six, five in the last
    (8, 32, dict(B=1, H=2, L=8000, C=99, Lq=512, U=3)),                  # of eight
    (8, 38, dict(B=1, H=2, L=12000, C=99, Lq=512, U=3)),                 # three rounds of seven, five in the last
    (8, 32, dict(B=1, H=1, L=4000, C=99, Lq=300, U=3)),                  # eight half waves, four shares each
    (8, 33, dict(B=1, H=1, L=2000, C=99, Lq=9, U=3)),                    # and one of them five
    (8, 53, dict(B=1, H=1, L=20000, C=99, Lq=700, U=3)),
    (8, 64, dict(B=1, H=1, L=4000, C=99, Lq=9, U=3)),                    # the most shares
]


@pytest.mark.parametrize("waves,splits,case", MERGED)
def test_merges(sq, oracle, waves, splits, case):
    test_per_query_selection(sq, oracle, waves, splits, case, "random")


@pytest.mark.parametrize("waves,splits,case", [(8, 9, dict(B=1, H=9, L=4000, C=99, Lq=100, U=3)),
                                               (8, 13, dict(B=1, H=1, L=64 * 90, C=99, Lq=9, U=3))])
def test_merges_one_kept_set(sq, oracle, waves, splits, case):
    test_one_kept_set(sq, oracle, waves, splits, case, 0.02)             # (shares without a key among them)


# (waves, shares on average, dealt in proportion).  The merge takes one half wave a row from 4096 rows on, two from 1024 on, else eight.
DEALT = [
    (8, 4, True, dict(B=1, H=32, L=64 * 512, C=300, Lq=300, U=300)),       # 64 units
    (8, 8, True, dict(B=2, H=8, L=64 * 1024 + 5, C=400, Lq=257, U=10)),    # 32 units, a unit of one query among every two
    (8, 62, False, dict(B=3, H=1, L=500000, C=200, Lq=200, U=0)),          # a little short of 16 blocks a share: even shares
    (8, 64, True, dict(B=3, H=1, L=524288, C=200, Lq=200, U=0)),           # three units, no user keys; 600 rows
    (8, 42, True, dict(B=3, H=1, L=524288, C=200, Lq=512, U=512)),         # 1536 rows
    (4, 61, True, dict(B=8, H=1, L=524288, C=200, Lq=5, U=5)),             # short prompts: eight rows a share, five of them queries
    (8, 61, True, dict(B=4, H=1, L=524288, C=200, Lq=40, U=40)),
    (4, 10, True, dict(B=5, H=2, L=64 * 2048, C=300, Lq=520, U=50)),       # four waves; 5200 rows
    (4, 32, True, dict(B=5, H=1, L=64 * 4096, C=300, Lq=257, U=0)),        # 1285 rows, a unit of one query among every three
    (4, 54, True, dict(B=3, H=1, L=524288, C=200, Lq=257, U=0)),           # 771 rows
]


@pytest.mark.parametrize("keep", ["some", "none"])
@pytest.mark.parametrize("waves,splits,dealt,case", DEALT, ids=lambda v: "B{B}H{H}L{L}Lq{Lq}".format(**v) if isinstance(v, dict) else str(v))
def test_shares_in_proportion(sq, oracle, waves, splits, dealt, case, keep):
    """Long contexts of few units: the shares follow the rows' numbers of kept keys, which go from none over one cluster to all; with
    nothing kept and no user keys, a unit's shares are those of units without a block."""
    w = wl.make_workload("prefill_dealt", seed=53, threads=4, keep_frac=0.3, causal_user=True, **case)
    rng = np.random.default_rng(16)
    share = np.resize([0.0, 0.02, 0.5, 1.0, 0.1], (w.B, w.H))
    kept = rng.random((w.B, w.H, w.C)) < share[..., None]
    kept[share == 0.02] = np.arange(w.C) == 7                 # one cluster
    if keep == "none":
        kept[:] = False
    P = sq.upload(w)
    assert sq.sq_prefill_plan(P.shape, one_set=True) == (waves, splits)
    assert sq.sq_prefill_form(P.shape, sq.SQ_CALL_ATTN_PREFILL_SHARED) == (sq.SQ_FORM_DEALT if dealt else 0)
    ranges, nr = np.zeros((w.B, w.H, w.C, 2), np.int32), np.zeros((w.B, w.H), np.int32)
    for b in range(w.B):
        for h in range(w.H):
            ranges[b, h], nr[b, h] = ranges_from_keep(kept[b, h], w.offsets[h], w.sizes[h], w.C)
    nk = (kept * w.sizes[None]).sum(-1).astype(np.int32)
    P.out.fill_(7.0)
    sq.sq_sparse_attn_prefill_shared(P.shape, P.q, P.K_fixed, P.V_fixed, t(ranges), t(nr), t(nk), P.K_user, P.V_user, P.out,
                                     P.lse, sq.workspace(P.shape, sq.SQ_CALL_ATTN_PREFILL_SHARED, DEV))
    torch.cuda.synchronize()
    sel = sample_rows(w, 300, 17)
    cap = max(1, int(nr.max()))
    rr = np.ascontiguousarray(np.broadcast_to(ranges[:, :, None, :cap], (w.B, w.H, w.Lq, cap, 2)))
    nn = np.ascontiguousarray(np.broadcast_to(nr[:, :, None], (w.B, w.H, w.Lq)))
    compare(oracle, w, P, rr, nn, sel)
