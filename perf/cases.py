"""The work that users of this library have it do, as measurable cases.

A case is one call of a step entry point on device-resident data, the way a serving loop (decode), a prompt (prefill) or
the offline preparation of a context (clustering) calls it.  Data follow the repository's own workload recipe: per head,
cluster centres ~ N(0, 1)^128, keys = centre + 0.3 N(0, 1) stored sorted by cluster, centroids the means of the keys,
values and user keys ~ N(0, 1), queries = a random centre + 0.3 N(0, 1), thresholds calibrated on queries of their own
to keep a target share of the keys.  Everything is drawn on the GPU from the seed alone.
"""
import math

import torch

from paper_2411_09688_amd import binding as sq

D = 128
NOISE = 0.3                      # keys and queries around their centre
COARSE_NOISE = 1.0               # fine centres around a coarse centre (two-level contexts)
N_CALIB = 32                     # calibration queries per head (decode and per-query prefill)
SM_SCALE = float(torch.tensor(1.0 / math.sqrt(D), dtype=torch.float32))
F16, F32, F64, I32 = torch.float16, torch.float32, torch.float64, torch.int32


def _case(name, kind, B, H, L, C, Lq, U, keep, G=1, C1=0, coarse_keep=0.0):
    return dict(name=name, kind=kind, B=B, H=H, L=L, C=C, Lq=Lq, U=U, keep=keep, G=G, C1=C1, coarse_keep=coarse_keep)


def listed():
    return [
        # One token over a short context with few heads: the smallest call, all launches and dependent reads.
        _case("decode_4k", "decode", B=1, H=4, L=4096, C=64, Lq=1, U=128, keep=1 / 4),
        # One token of a 7B-shaped layer over a 32K context: the headline workload.
        _case("decode_32k", "decode", B=1, H=32, L=32768, C=1024, Lq=1, U=512, keep=1 / 8),
        # A few sequences over a shared context of no round size, a handful of generated tokens.
        _case("decode_ragged_b3", "decode", B=3, H=20, L=20011, C=613, Lq=1, U=77, keep=0.1),
        # A full batch over one shared prefix: every sequence selects on its own, the union is streamed once.
        _case("decode_shared_b16", "decode", B=16, H=32, L=32768, C=1024, Lq=1, U=256, keep=1 / 8),
        # Grouped-query attention, 32 query heads over 8 K/V heads.
        _case("gqa_decode_32k", "gqa_decode", B=1, H=8, L=32768, C=1024, Lq=1, U=512, keep=1 / 8, G=4),
        # One token over a 512K context through the two-level lookup: the largest context.
        _case("hier_decode_512k", "hier_decode", B=1, H=32, L=524288, C=16384, Lq=1, U=1024, keep=1 / 16, C1=256,
              coarse_keep=1 / 8),
        # A 1024-token user prompt behind a 32K context, every token selecting for itself.
        _case("prefill_32k", "prefill", B=1, H=32, L=32768, C=1024, Lq=1024, U=1024, keep=1 / 8),
        # Two short prompts of no round length behind a short context, per-token selection.
        _case("prefill_ragged", "prefill", B=2, H=12, L=9001, C=281, Lq=333, U=333, keep=0.15),
        # The paper's prefill rule: scores averaged over the prompt, one kept set per head.
        _case("prefill_mean_32k", "prefill_mean", B=1, H=32, L=32768, C=1024, Lq=1024, U=1024, keep=1 / 8),
        # The same for a short question behind a context of no round size.
        _case("prefill_mean_ragged", "prefill_mean", B=1, H=20, L=20011, C=613, Lq=150, U=150, keep=0.1),
        # A prompt behind a 256K context, averaged selection through the two-level lookup.
        _case("hier_prefill_256k", "hier_prefill_mean", B=1, H=8, L=262144, C=16384, Lq=512, U=512, keep=1 / 16, C1=256,
              coarse_keep=1 / 8),
        # Offline: one Lloyd iteration over the 32K context of 32 heads.
        _case("kmeans_32k", "kmeans", B=1, H=32, L=32768, C=1024, Lq=1, U=0, keep=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode_shared", "gqa_decode", "hier_decode", "prefill", "prefill",
                       "prefill_mean", "prefill_mean", "hier_prefill_mean", "kmeans"])
    H = rng.choice([1, 2, 4, 5, 8, 12, 16, 20, 24, 32])
    L = _log_int(rng, 2000, 32768)
    C = max(16, L // rng.randint(20, 64))
    keep = round(rng.uniform(0.05, 0.3), 3)
    U = _log_int(rng, 1, 1024)
    Lq = _log_int(rng, 16, 1024)
    c = dict(kind=kind, B=1, H=H, L=L, C=C, Lq=1, U=U, keep=keep, G=1, C1=0, coarse_keep=0.0)
    if kind == "decode":
        c.update(B=rng.choice([1, 1, 2, 3, 5]))
    elif kind == "decode_shared":
        c.update(kind="decode", B=rng.randint(8, 16))
    elif kind == "gqa_decode":
        c.update(H=rng.choice([2, 4, 8]), G=rng.choice([2, 3, 4, 7, 8]), B=rng.choice([1, 1, 2, 4]))
    elif kind in ("hier_decode", "hier_prefill_mean"):
        L = _log_int(rng, 32768, 262144)
        C1 = _log_int(rng, 32, 256)
        c.update(L=L, C=min(16384, max(2 * C1, L // rng.randint(16, 48))), C1=C1, coarse_keep=round(rng.uniform(0.1, 0.4), 3),
                 keep=round(rng.uniform(0.03, 0.09), 3))
        if kind == "hier_prefill_mean":
            c.update(H=rng.choice([1, 2, 4, 8]), Lq=min(Lq, 512), U=min(Lq, 512))
    elif kind in ("prefill", "prefill_mean"):
        c.update(B=rng.choice([1, 1, 2]) if Lq <= 512 else 1, Lq=Lq, U=Lq)
    elif kind == "kmeans":
        c.update(U=0, keep=1.0)
    return c


# ---------------------------------------------------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------------------------------------------------
def _cut(score, weight, target):
    """Per row: threshold between the last score needed to cover `target` weight and the next one (geometric mean)."""
    s, order = torch.sort(score, dim=1, descending=True, stable=True)
    cum = torch.cumsum(weight.gather(1, order), dim=1, dtype=F64)
    k = (cum < target).sum(1, keepdim=True).clamp(max=s.shape[1] - 2)
    hi, lo = s.gather(1, k).double(), s.gather(1, k + 1).double()
    return torch.sqrt(hi * torch.maximum(lo, hi * 1e-3)).float().reshape(-1)


def _scores(q, cent, sizes, cand=None):
    """Eq. 1 scores of q [H, n, D] on cent [H, C, D]; cand [H, n, C]: the clusters that count for a query."""
    x = torch.matmul(q.float(), cent.float().transpose(1, 2).contiguous()) * SM_SCALE
    n = sizes.float().unsqueeze(1).expand_as(x)
    if cand is not None:
        n = torch.where(cand, n, torch.zeros_like(n))
    x = torch.where(n > 0, x, torch.full_like(x, -math.inf))
    m = x.amax(2, keepdim=True)
    e = torch.exp(x - torch.where(torch.isfinite(m), m, torch.zeros_like(m)))
    return e / (n * e).sum(2, keepdim=True).clamp_min(1e-30)


def _queries(g, centres, n):
    H, C, _ = centres.shape
    pick = torch.randint(0, C, (H, n), generator=g, device="cuda")
    c = torch.gather(centres, 1, pick.unsqueeze(-1).expand(H, n, D))
    return (c + NOISE * torch.randn(H, n, D, generator=g, device="cuda")).half()


def _context(case, g):
    """Keys sorted by cluster, values, centroids, sizes and offsets (and the coarse level) of one fixed context."""
    H, L, C, C1 = case["H"], case["L"], case["C"], case["C1"]
    rnd = lambda *s, **k: torch.randn(*s, generator=g, device="cuda", **k)  # noqa: E731
    t = {}
    if C1:
        coarse = rnd(H, C1, D)
        # every coarse cluster has at least one child; the others are dealt at random (variable fan-out)
        extra = torch.randint(0, C1, (H, C - C1), generator=g, device="cuda")
        parent = torch.cat([torch.arange(C1, device="cuda").expand(H, C1), extra], 1).sort(1).values
        fan = torch.zeros(H, C1, dtype=torch.int64, device="cuda").scatter_add_(1, parent, torch.ones_like(parent))
        centres = torch.gather(coarse, 1, parent.unsqueeze(-1).expand(H, C, D)) + COARSE_NOISE * rnd(H, C, D)
    else:
        centres = rnd(H, C, D)
    ids = torch.randint(0, C, (H, L), generator=g, device="cuda").sort(1).values
    sizes = torch.zeros(H, C, dtype=torch.int64, device="cuda").scatter_add_(1, ids, torch.ones_like(ids))
    offsets = torch.zeros(H, C + 1, dtype=torch.int64, device="cuda")
    offsets[:, 1:] = sizes.cumsum(1)
    K = torch.empty(H, L, D, dtype=F16, device="cuda")
    V = torch.empty(H, L, D, dtype=F16, device="cuda")
    cent = torch.empty(H, C, D, dtype=F16, device="cuda")
    widest = int(sizes.max())
    for h in range(H):
        K[h] = (centres[h][ids[h]] + NOISE * rnd(L, D)).half()
        V[h].normal_(generator=g)
        slot = ids[h] * widest + torch.arange(L, device="cuda") - offsets[h][ids[h]]
        padded = torch.zeros(C * widest, D, device="cuda")
        padded[slot] = K[h].float()
        mean = padded.view(C, widest, D).sum(1) / sizes[h].clamp(min=1).unsqueeze(1)
        cent[h] = torch.where(sizes[h].unsqueeze(1) > 0, mean, centres[h]).half()
    t.update(centres=centres, K_fixed=K, V_fixed=V, centroids=cent, sizes=sizes.int(), offsets=offsets.int())
    if C1:
        co = torch.zeros(H, C1 + 1, dtype=torch.int64, device="cuda")
        co[:, 1:] = fan.cumsum(1)
        onehot = torch.zeros(H, C1, C, device="cuda").scatter_(1, parent.unsqueeze(1), 1.0)
        t["centroids1"] = (torch.matmul(onehot, cent.float()) / fan.unsqueeze(-1)).half()
        t["sizes1"] = torch.zeros(H, C1, dtype=torch.int64, device="cuda").scatter_add_(1, parent, sizes).int()
        t["child_offsets"], t["parent"] = co.int(), parent
    return t


def _thresholds(case, t, g):
    H, L, keep = case["H"], case["L"], case["keep"]
    mean = case["kind"] in ("prefill_mean", "hier_prefill_mean")
    n = case["Lq"] if mean else N_CALIB
    qc = _queries(g, t["centres"], n)
    pool = lambda S: S.mean(1, keepdim=True) if mean else S  # noqa: E731
    rows = 1 if mean else n
    wide = lambda a: a.float().unsqueeze(1).expand(H, rows, a.shape[1]).reshape(H, -1)  # noqa: E731
    if not case["C1"]:
        t["thresh"] = _cut(pool(_scores(qc, t["centroids"], t["sizes"])).reshape(H, -1), wide(t["sizes"]), keep * rows * L)
        return
    S1 = pool(_scores(qc, t["centroids1"], t["sizes1"]))
    t["thresh1"] = _cut(S1.reshape(H, -1), torch.ones(H, S1[0].numel(), device="cuda"),
                        case["coarse_keep"] * rows * case["C1"])
    kept = S1 > t["thresh1"].view(H, 1, 1)
    T2 = []
    for h in range(H):                                     # a head at a time: the fine level is large
        cand = kept[h:h + 1][:, :, t["parent"][h]].expand(1, n, case["C"])
        S2 = pool(_scores(qc[h:h + 1], t["centroids"][h:h + 1], t["sizes"][h:h + 1], cand))
        T2.append(_cut(S2.reshape(1, -1), t["sizes"][h:h + 1].float().expand(rows, -1).reshape(1, -1), keep * rows * L))
    t["thresh"] = torch.cat(T2)


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)
    H, B, G, L, C, Lq, U = (case[k] for k in ("H", "B", "G", "L", "C", "Lq", "U"))
    if case["kind"] == "kmeans":
        # unsorted keys as a context delivers them, normalised, and C distinct keys as the seeding
        centres = torch.randn(H, C, D, generator=g, device="cuda")
        X = torch.empty(1, H, L, D, dtype=F16, device="cuda")
        init = torch.empty(1, H, C, D, dtype=F16, device="cuda")
        for h in range(H):
            ids = torch.randint(0, C, (L,), generator=g, device="cuda")
            k = centres[h][ids] + NOISE * torch.randn(L, D, generator=g, device="cuda")
            X[0, h] = (k / k.norm(dim=1, keepdim=True)).half()
            init[0, h] = X[0, h][torch.randperm(L, generator=g, device="cuda")[:C]]
        return dict(X=X, init=init)
    t = _context(case, g)
    n = B * G * Lq
    # [H, B, G or Lq, D] -> [B, H * G, Lq, D]
    q = _queries(g, t["centres"], n).view(H, B, G, Lq, D).permute(1, 0, 2, 3, 4)
    t["q"] = q.reshape(B, H * G, Lq, D).contiguous()
    t["K_user"] = torch.randn(B, H, U, D, generator=g, device="cuda").half()
    t["V_user"] = torch.randn(B, H, U, D, generator=g, device="cuda").half()
    _thresholds(case, t, g)
    return t


CALLS = dict(decode=sq.SQ_CALL_DECODE_STEP, gqa_decode=sq.SQ_CALL_GQA_DECODE_STEP, hier_decode=sq.SQ_CALL_HIER_DECODE_STEP,
             prefill=sq.SQ_CALL_PREFILL_STEP, prefill_mean=sq.SQ_CALL_PREFILL_MEAN_STEP,
             hier_prefill_mean=sq.SQ_CALL_HIER_PREFILL_MEAN_STEP, kmeans=sq.SQ_CALL_KMEANS_STEP)


def prepare(case, seed):
    kind, B, H, G, L, C, Lq, U = (case[k] for k in ("kind", "B", "H", "G", "L", "C", "Lq", "U"))
    t = _inputs(case, seed)
    for k in ("centres", "parent"):
        t.pop(k, None)
    shape = sq.make_shape(B, H, L, C, Lq, U, SM_SCALE, causal_user=Lq > 1)
    s = dict(kind=kind, G=G, C1=case["C1"], shape=shape, t=t, ws=sq.workspace(shape, CALLS[kind], "cuda:0"))
    e = lambda *sh, dtype: torch.empty(*sh, dtype=dtype, device="cuda")  # noqa: E731
    if kind == "kmeans":
        s.update(centers=e(1, H, C, D, dtype=F16), assign=e(1, H, L, dtype=I32), sizes=e(1, H, C, dtype=I32),
                 offsets=e(1, H, C + 1, dtype=I32), perm=e(1, H, L, dtype=I32))
        return s
    W = (C + 31) // 32
    per_row = kind in ("decode", "gqa_decode", "hier_decode", "prefill")
    s.update(out=e(B, H * G, Lq, D, dtype=F16), lse=e(B, H * G, Lq, dtype=F32),
             mask=e(B, H * G, Lq, W, dtype=I32) if per_row else e(B, H, W, dtype=I32))
    return s


def run(s):
    kind, t, shape, ws = s["kind"], s["t"], s["shape"], s["ws"]
    if kind == "kmeans":
        sq.sq_kmeans_step(shape, t["X"], t["init"], s["centers"], s["assign"], s["sizes"], s["offsets"], s["perm"], ws)
        return {k: s[k] for k in ("centers", "assign", "sizes", "offsets", "perm")}
    one = (t["q"], t["centroids"], t["sizes"], t["offsets"], t["thresh"], t["K_fixed"], t["V_fixed"], t["K_user"],
           t["V_user"], s["out"], s["lse"], s["mask"], None, ws)
    if kind == "decode":
        sq.sq_decode_step(shape, *one)
    elif kind == "gqa_decode":
        sq.sq_gqa_decode_step(shape, s["G"], *one)
    elif kind == "prefill":
        sq.sq_prefill_step(shape, *one)
    elif kind == "prefill_mean":
        sq.sq_prefill_mean_step(shape, *one)
    else:
        fn = sq.sq_hier_decode_step if kind == "hier_decode" else sq.sq_hier_prefill_mean_step
        fn(shape, s["C1"], t["q"], t["centroids1"], t["sizes1"], t["child_offsets"], t["thresh1"], *one[1:])
    return {"out": s["out"], "lse": s["lse"], "keep_mask": s["mask"]}


def work(case):
    """Each key that some row keeps read once (K and V), centroids, queries and user keys once, outputs once."""
    kind, B, H, G, L, C, Lq, U = (case[k] for k in ("kind", "B", "H", "G", "L", "C", "Lq", "U"))
    row = D * 2
    if kind == "kmeans":
        return dict(bytes=H * (L * row + 2 * C * row + 8 * L + 8 * C), flops=2.0 * H * L * C * D)
    rows = B * G * Lq                                      # query rows of a K/V head
    mean = kind in ("prefill_mean", "hier_prefill_mean")
    sets = B if mean else rows                             # kept sets of a K/V head
    keep = case["keep"]
    union = 1.0 - (1.0 - keep) ** sets
    seen = (U + 1) / 2 if Lq > 1 else U                    # user keys a query sees, on average
    cents = C if not case["C1"] else case["C1"] + case["coarse_keep"] * C
    W = (C + 31) // 32
    bytes_ = H * (2 * union * L * row + cents * row + 8 * cents) + B * H * 2 * U * row + H * rows * (2 * row + 4)
    bytes_ += H * sets * W * 4
    return dict(bytes=bytes_, flops=H * rows * (4.0 * D * (keep * L + seen) + 2.0 * D * cents))


def tolerance(case):
    # fp16 outputs of attention with fp16 probabilities on the matrix-core paths; the mask words that differ are those
    # of clusters whose score is within fp32 rounding of the threshold
    if case["kind"] == "kmeans":
        return {"rel": 1e-3, "max": 0.05, "differ": 1e-3}
    return {"rel": 2e-3, "max": 0.5, "differ": 2e-3}


# ---------------------------------------------------------------------------------------------------------------------
# The same in 64 bits, plain torch.
# ---------------------------------------------------------------------------------------------------------------------
def _keep64(x, sizes, T, cand=None, mean=False):
    """Kept clusters of logits x [n, C]: exp(x - m) / D > T, or its average over the rows."""
    ok = (sizes > 0).unsqueeze(0).expand_as(x)
    if cand is not None:
        ok = ok & cand
    x = torch.where(ok, x, torch.full_like(x, -math.inf))
    m = x.amax(1, keepdim=True)
    e = torch.exp(x - torch.where(torch.isfinite(m), m, torch.zeros_like(m)))
    S = e / (sizes.double() * e).sum(1, keepdim=True).clamp_min(1e-300)
    if mean:
        S = S.mean(0, keepdim=True)
    return (S > T) & (ok[:1] if mean else ok)


def exact(case, seed):
    t = _inputs(case, seed)
    kind, B, H, G, L, C, Lq, U = (case[k] for k in ("kind", "B", "H", "G", "L", "C", "Lq", "U"))
    if kind == "kmeans":
        centers = torch.empty(1, H, C, D, dtype=F64, device="cuda")
        for h in range(H):
            x, c = t["X"][0, h].double(), t["init"][0, h].double()
            a = (x @ c.T.contiguous() - 0.5 * (c * c).sum(1)).argmax(1)
            order = a.sort(stable=True)
            n = torch.bincount(a, minlength=C)
            widest = int(n.max())
            first = n.cumsum(0) - n
            padded = torch.zeros(C * widest, D, dtype=F64, device="cuda")
            padded[order.values * widest + torch.arange(L, device="cuda") - first[order.values]] = x[order.indices]
            mean = padded.view(C, widest, D).sum(1) / n.clamp(min=1).unsqueeze(1)
            centers[0, h] = torch.where(n.unsqueeze(1) > 0, mean, c)
        return dict(centers=centers, assign=None, sizes=None, offsets=None, perm=None)
    mean = kind in ("prefill_mean", "hier_prefill_mean")
    out = torch.zeros(B, H, G * Lq, D, dtype=F64, device="cuda")
    lse = torch.zeros(B, H, G * Lq, dtype=F64, device="cuda")
    q = t["q"].view(B, H, G * Lq, D)
    for h in range(H):
        sizes, T = t["sizes"][h], t["thresh"][h].double()
        ids = torch.repeat_interleave(torch.arange(C, device="cuda"), sizes.long())
        kt = t["K_fixed"][h].double().T.contiguous()
        v = t["V_fixed"][h].double()
        ct = t["centroids"][h].double().T.contiguous()
        for b in range(B):
            qb = q[b, h].double()
            cand = None
            if case["C1"]:
                c1 = t["centroids1"][h].double().T.contiguous()
                k1 = _keep64(qb @ c1 * SM_SCALE, t["sizes1"][h], t["thresh1"][h].double(), mean=mean)
                cand = k1[:, t["parent"][h]]
                cand = cand.expand(qb.shape[0], C) if mean else cand
            keep = _keep64(qb @ ct * SM_SCALE, sizes, T, cand, mean)
            x = qb @ kt * SM_SCALE
            x = torch.where(keep[:, ids].expand_as(x), x, torch.full_like(x, -math.inf))
            xu = qb @ t["K_user"][b, h].double().T.contiguous() * SM_SCALE
            if Lq > 1:
                future = torch.arange(U, device="cuda").unsqueeze(0) > torch.arange(Lq, device="cuda").unsqueeze(1)
                xu = torch.where(future, torch.full_like(xu, -math.inf), xu)
            z = torch.logsumexp(torch.cat([x, xu], 1), 1, keepdim=True)
            out[b, h] = torch.exp(x - z) @ v + torch.exp(xu - z) @ t["V_user"][b, h].double()
            lse[b, h] = z[:, 0]
    return dict(out=out.view(B, H * G, Lq, D), lse=lse.view(B, H * G, Lq), keep_mask=None)
