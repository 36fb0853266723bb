"""The C-ABI library loads, exports every symbol the header declares, and validates arguments on the
host (no GPU needed: invalid calls are rejected before anything is enqueued)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sq():
    from paper_2411_09688_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build_library()
    binding.lib()
    return binding


def test_every_declared_symbol_is_exported(sq):
    hdr = open(os.path.join(ROOT, "include", "squeezed_attention.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(sq_[a-z_0-9]+)\s*\(", hdr))
    assert {"sq_centroid_score", "sq_select", "sq_sparse_attn_decode", "sq_sparse_attn_prefill",
            "sq_hier_select"} <= declared
    L = sq.lib()
    for name in declared:
        assert hasattr(L, name), name
    assert set(sq.EXPORTS) == declared
    assert L.sq_version() >= 100


def test_every_entry_point_declares_its_parameters(sq):
    """The binding passes device pointers as integers: without argtypes ctypes would cut them to 32 bits."""
    hdr = open(os.path.join(ROOT, "include", "squeezed_attention.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    L = sq.lib()
    for name, params in re.findall(r"\b(sq_[a-z_0-9]+)\s*\(([^)]*)\)\s*;", hdr):
        kinds = [p.strip() for p in params.split(",") if p.strip() != "void"]
        if not kinds:
            continue
        types = getattr(L, name).argtypes
        assert types is not None and len(types) == len(kinds), name
        for p, t in zip(kinds, types):
            assert C.sizeof(t) == (4 if "*" not in p and p.split()[0] in ("int", "int32_t", "float") else 8), (name, p)


def test_workspace_sizes(sq):
    sh = sq.make_shape(1, 32, 32768, 1024, 1, 512, 0.0884)
    assert sq.workspace_bytes(sh, sq.SQ_CALL_CENTROID_SCORE) == 0
    assert sq.workspace_bytes(sh, sq.SQ_CALL_SELECT) == 0
    a = sq.workspace_bytes(sh, sq.SQ_CALL_ATTN_DECODE)
    b = sq.workspace_bytes(sh, sq.SQ_CALL_DECODE_STEP)
    assert a > 0 and b > 0 and a % 256 == 0 and b % 256 == 0
    # partials alone: 32 rows x (2 user + 128 fixed chunks) x 132 floats
    assert a >= 32 * 130 * 132 * 4
    bad = sq.make_shape(0, 32, 32768, 1024, 1, 512, 0.0884)
    assert sq.workspace_bytes(bad, sq.SQ_CALL_ATTN_DECODE) == 0


@pytest.mark.parametrize("H,L,Lq", [(32, 524288, 32768), (8, 2097152, 4096), (32, 262144, 131072), (1, 300000, 200), (32, 32768, 1024),
                                    (4, 100, 1)])
def test_prefill_workspace_is_bounded(sq, H, L, Lq):
    """Besides the block table (129 words per 64 keys and head) the masked prefill attention asks for partial results of at most
    two rounds of workgroups (512 of 256 tokens or 1024 of 128, 528 bytes a token), whatever the context's length is."""
    sh = sq.make_shape(1, H, L, 1024, Lq, Lq, 0.0884, causal_user=True)
    table = H * ((L + 63) // 64) * 129 * 4
    assert table <= sq.workspace_bytes(sh, sq.SQ_CALL_ATTN_PREFILL) <= table + 131072 * 528 + 1024


def test_shared_decode_workspace_holds_the_user_keys_once(sq):
    """User keys of a step over a shared context cost either 528 bytes of partial results per 64 keys and row (one query row per K/V
    head) or 1040 bytes of work items per 128 keys and row of a group of 16, never both."""
    for B, H, U in ((8, 8, 4096), (16, 8, 32768), (17, 4, 100)):
        with_u, none = (sq.make_shape(B, H, 32768, 1024, 1, u, 0.1) for u in (U, 0))
        more = {c: sq.workspace_bytes(with_u, c) - sq.workspace_bytes(none, c) for c in (sq.SQ_CALL_DECODE_STEP, sq.SQ_CALL_GQA_MEAN_DECODE_STEP)}
        assert more[sq.SQ_CALL_DECODE_STEP] <= B * H * ((U + 63) // 64) * 528 + 256
        assert more[sq.SQ_CALL_GQA_MEAN_DECODE_STEP] <= B * H * 16 * ((U + 127) // 128) * 1040 + 256


@pytest.mark.parametrize("B,H,C_,pieces", [(16, 32, 1024, 20 * 1024), (16, 8, 256, 14336), (9, 8, 700, 14336), (8, 32, 800, 20 * 800),
                                           (16, 8, 1025, 30720 + 13 * 1025), (12, 12, 4096, 30720 + 13 * 4096)])
def test_shared_decode_takes_user_keys_beside_the_selection_up_to_a_line(sq, B, H, C_, pieces):
    """The workspace shows which form a step takes: 528 bytes per row and 64 user keys, or 1040 per row of a group and 128."""
    last = pieces // (B * H) * 64
    for U, beside in ((last, True), (last + 1, False), (2 * last, False)):
        with_u, none = (sq.workspace_bytes(sq.make_shape(B, H, 32768, C_, 1, u, 0.1), sq.SQ_CALL_DECODE_STEP) for u in (U, 0))
        want = B * H * ((U + 63) // 64) * 528 if beside else H * 16 * ((U + 127) // 128) * 1040
        assert abs(with_u - none - want) <= 256, (U, beside)


@pytest.mark.parametrize("B,H,L,C_,U", [(20, 4, 190, 7, 7578), (32, 4, 80048, 1122, 3319), (9, 2, 3354, 579, 27181),
                                        (16, 8, 16384, 512, 8384), (16, 8, 16384, 512, 8448)])
def test_noalloc_step_takes_what_fits_with_work_items(sq, B, H, L, C_, U):
    """The step's intermediate state with its user keys in work items fits the built-in buffer: so does the step."""
    urows = (B + 15) // 16 * H
    tables = B * H * (C_ * 4 + 8 + (C_ + 31) // 32 * 4) + urows * (C_ * 16 + 20) + (768 + urows) * 16 * 528 + 12 * 256
    items = urows * (16 * ((U + 127) // 128) + (L + 127) // 128) * 1040
    assert tables + items <= sq.SQ_NOALLOC_SCRATCH_BYTES
    assert sq.workspace_bytes(sq.make_shape(B, H, L, C_, 1, U, 0.1), sq.SQ_CALL_DECODE_STEP) <= sq.SQ_NOALLOC_SCRATCH_BYTES


@pytest.mark.parametrize("B,H,L,C_,Lq,C1,inside", [
    (1, 32, 32768, 1024, 1024, 0, True), (1, 20, 20011, 613, 150, 0, True),
    (1, 1, 32768, 1024, 16384, 0, True),                      # one round of workgroups: any number of parts
    (480, 1, 2000, 100, 200, 0, True), (481, 1, 2000, 100, 200, 0, False),   # eight waves: 15/8 of a round
    (960, 1, 400, 20, 4, 0, True), (961, 1, 400, 20, 4, 0, False),           # four waves
    (1, 8, 8000, 400, 15360, 0, True),                        # 480 workgroups, 64 parts
    (1, 5, 16384, 1000, 20000, 0, False),                     # 395 workgroups, 102 parts
    (1, 32, 16384, 1024, 8192, 0, False), (1, 24, 16384, 1000, 4096, 32, True), (1, 32, 16384, 1000, 8192, 32, False),
])
def test_the_attention_launch_selects_in_about_one_round(sq, B, H, L, C_, Lq, C1, inside):
    sh = sq.make_shape(B, H, L, C_, Lq, 64, 0.1, causal_user=True)
    which = sq.SQ_CALL_HIER_PREFILL_MEAN_STEP if C1 else sq.SQ_CALL_PREFILL_MEAN_STEP
    assert bool(sq.sq_prefill_form(sh, which, C1) & sq.SQ_FORM_SELECTS) == inside, sq.sq_prefill_plan(sh, one_set=True)


@pytest.mark.parametrize("H,C_,Lq,C1,inside", [(8, 16384, 512, 256, True), (1, 3000, 40, 1024, True), (1, 3000, 40, 1025, False),
                                               (12, 2000, 64 * 128, 64, True), (12, 2000, 64 * 128 + 1, 64, False), (32, 1000, 16384, 32, False)])
def test_the_pass_over_the_candidates_lists_them_in_one_round(sq, H, C_, Lq, C1, inside):
    """Up to 768 workgroups (blocks of 128 tokens of all heads) and 1024 coarse clusters."""
    sh = sq.make_shape(1, H, 32768, C_, Lq, 64, 0.1, causal_user=True)
    assert bool(sq.sq_prefill_form(sh, sq.SQ_CALL_HIER_PREFILL_MEAN_STEP, C1) & sq.SQ_FORM_CHILDREN) == inside


@pytest.mark.parametrize("B,H", [(1, 8), (4, 1), (1, 2)])
def test_dealt_shares_hold_the_tokens_there_are(sq, B, H):
    """Shares in proportion to the kept keys: 528 bytes of partial results per share and query token, tokens rounded up to eight."""
    size = {}
    for Lq in (1, 8, 9, 16):
        sh = sq.make_shape(B, H, 524288, 16384, Lq, 1, 0.1)
        assert sq.sq_prefill_form(sh, sq.SQ_CALL_ATTN_PREFILL_SHARED) == sq.SQ_FORM_DEALT
        size[Lq] = sq.workspace_bytes(sh, sq.SQ_CALL_ATTN_PREFILL_SHARED)
    splits = sq.sq_prefill_plan(sh, one_set=True)[1]
    assert size[1] == size[8] and size[9] == size[16] and abs(size[16] - size[8] - B * H * splits * 8 * 528) <= 256


def test_host_side_validation(sq):
    L = sq.lib()
    buf = (C.c_char * 4096)()
    p = C.cast(buf, C.c_void_p)
    aligned = C.c_void_p((p.value + 255) & ~255)
    sh = sq.make_shape(1, 2, 64, 4, 1, 0, 0.1)
    rc = L.sq_centroid_score(C.byref(sh), None, aligned, aligned, aligned, aligned, aligned, None, 0, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"q is NULL" in L.sq_last_error()
    mis = C.c_void_p(aligned.value + 4)
    rc = L.sq_centroid_score(C.byref(sh), mis, aligned, aligned, aligned, aligned, aligned, None, 0, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"aligned" in L.sq_last_error()
    sh64 = sq.make_shape(1, 2, 64, 4, 1, 0, 0.1, d=64)
    rc = L.sq_centroid_score(C.byref(sh64), aligned, aligned, aligned, aligned, aligned, aligned, None, 0, None)
    assert rc == sq.SQ_ERR_UNSUPPORTED
    neg = sq.make_shape(1, 2, 64, -4, 1, 0, 0.1)
    rc = L.sq_select(C.byref(neg), *([aligned] * 10), None, 0, None)
    assert rc == sq.SQ_ERR_INVALID_ARG
    pre = sq.make_shape(1, 2, 64, 4, 3, 0, 0.1)
    rc = L.sq_sparse_attn_decode(C.byref(pre), *([aligned] * 10), aligned, 1 << 30, None)
    assert rc == sq.SQ_ERR_UNSUPPORTED and b"Lq == 1" in L.sq_last_error()
    rc = L.sq_sparse_attn_decode(C.byref(sh), *([aligned] * 10), None, 0, None)
    assert rc == sq.SQ_ERR_WORKSPACE
    rc = L.sq_decode_step(C.byref(sh), *([aligned] * 13), aligned, 16, None)
    assert rc == sq.SQ_ERR_WORKSPACE and b"needed" in L.sq_last_error()


def test_host_side_validation_of_the_offline_calls(sq):
    L = sq.lib()
    buf = (C.c_char * 4096)()
    aligned = C.c_void_p((C.cast(buf, C.c_void_p).value + 255) & ~255)
    sh = sq.make_shape(1, 2, 64, 4, 1, 0, 1.0)
    assert sq.workspace_bytes(sh, sq.SQ_CALL_KMEANS_STEP) > 0 and sq.workspace_bytes(sh, sq.SQ_CALL_CALIBRATE) > 0
    rc = L.sq_kmeans_step(C.byref(sh), None, *([aligned] * 6), aligned, 1 << 30, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"X is NULL" in L.sq_last_error()
    more = sq.make_shape(1, 2, 3, 4, 1, 0, 1.0)                  # more centres than keys
    rc = L.sq_kmeans_step(C.byref(more), *([aligned] * 7), aligned, 1 << 30, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"more centres" in L.sq_last_error()
    rc = L.sq_kmeans_step(C.byref(sh), *([aligned] * 7), aligned, 16, None)
    assert rc == sq.SQ_ERR_WORKSPACE
    rc = L.sq_cluster_layout(C.byref(sh), aligned, aligned, aligned, aligned, aligned, aligned, aligned, aligned, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"alias" in L.sq_last_error()
    other = C.c_void_p(aligned.value + 1024)
    rc = L.sq_cluster_layout(C.byref(sh), aligned, None, None, aligned, aligned, other, None, aligned, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"needs perm" in L.sq_last_error()
    rc = L.sq_cluster_nest(C.byref(sh), 9, *([aligned] * 8), aligned, 1 << 30, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"C1" in L.sq_last_error()
    rc = L.sq_calibrate_threshold(C.byref(sh), *([aligned] * 4), -1, aligned, aligned, 1 << 30, None)
    assert rc == sq.SQ_ERR_INVALID_ARG and b"negative" in L.sq_last_error()
    big = sq.make_shape(64, 2, 1 << 19, 4, 64, 0, 1.0)           # B * Lq * L = 2^31 pooled keys
    rc = L.sq_calibrate_threshold(C.byref(big), *([aligned] * 4), 5, aligned, aligned, 1 << 40, None)
    assert rc == sq.SQ_ERR_UNSUPPORTED and b"calibration queries" in L.sq_last_error()


def test_noalloc_step_rejects_oversized_shapes_on_the_host(sq):
    """sq_decode_step_noalloc checks the shape against its built-in buffer before it touches a device."""
    L = sq.lib()
    sh = sq.make_shape(4, 32, 32768, 1024, 1, 512, 0.0884)
    assert sq.workspace_bytes(sh, sq.SQ_CALL_DECODE_STEP) > sq.SQ_NOALLOC_SCRATCH_BYTES
    buf = (C.c_char * 4096)()
    p = C.c_void_p((C.cast(buf, C.c_void_p).value + 255) & ~255)
    rc = L.sq_decode_step_noalloc(C.byref(sh), p, p, p, p, p, p, p, p, p, p, None, None, None, None)
    assert rc == sq.SQ_ERR_WORKSPACE and b"built-in" in L.sq_last_error()
    fits = sq.make_shape(1, 32, 32768, 1024, 1, 512, 0.0884)
    assert sq.workspace_bytes(fits, sq.SQ_CALL_DECODE_STEP) <= sq.SQ_NOALLOC_SCRATCH_BYTES


@pytest.mark.parametrize("H,L,C_", [(32, 32768, 1024), (32, 32768, 1638), (8, 32768, 8192), (12, 32768, 8192), (32, 32769, 1900), (3, 256, 1), (1, 513, 65), (2, 513, 257)])
def test_kmeans_workspace_rows_of_whole_lines(sq, H, L, C_):
    """Counts of the parts: 16 bits in rows of whole 128-byte lines (of words below 256 centres) for parts of 256 keys, up to 32768 keys and 2^23 counts, and in any
    case room for 32 bits and parts of 512 keys (or 64 parts); a half norm per centre."""
    to, parts = 2 if C_ < 256 else 64, (L + 255) // 256
    row = (C_ + to - 1) // to * to
    want = H * ((L + 511) // 512 if L <= 32768 else (L + 767) // 768) * C_ * 4
    if parts <= 128 and H * parts * row <= 1 << 23:
        want = max(want, H * parts * row * 2)
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    assert sq.workspace_bytes(sq.make_shape(1, H, L, C_, 1, 0, 1.0), sq.SQ_CALL_KMEANS_STEP) == up(H * C_ * 4) + up(want)


def test_prefill_form_checks_its_arguments(sq):
    sh = sq.make_shape(1, 8, 262144, 16384, 512, 512, 0.1, causal_user=True)
    assert sq.sq_prefill_form(sh, sq.SQ_CALL_HIER_PREFILL_MEAN_STEP, 256) == sq.SQ_FORM_CHILDREN | sq.SQ_FORM_DEALT
    for which, C1 in ((sq.SQ_CALL_DECODE_STEP, 0), (sq.SQ_CALL_HIER_PREFILL_MEAN_STEP, 0), (sq.SQ_CALL_HIER_PREFILL_MEAN_STEP, 16385)):
        with pytest.raises(sq.SqError):
            sq.sq_prefill_form(sh, which, C1)
    assert sq.lib().sq_prefill_form(C.byref(sh), sq.SQ_CALL_PREFILL_MEAN_STEP, 0, None) == sq.SQ_ERR_INVALID_ARG
