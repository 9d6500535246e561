"""Every ring degree that a transform kernel is built for, end to end, and odd sizes of the decision.

The oracle tests pin the residues at some degrees; each other degree has its own register and exchange
layout, so each is run here: a wrong layout on either side of a product turns decryption into noise.  Inner
products must equal the exact plaintext products with |v - IP| <= 0.25 (the library's decryption bound), and
folds must lie within Appendix C.2's allowance of 0.02 plus the input's encryption error.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)
H = pytest.importorskip("paper_2601_17561_amd")

import hfe_synth as S  # noqa: E402


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _ternary(rng, n, d):
    return rng.integers(-1, 2, (n, d)).astype(np.int8)


def _check(keys, r, mq, mdb, what):
    v, ip = H.hfe_decrypt(keys, r)
    torch.cuda.synchronize()
    want = mq.astype(np.int64) @ mdb.astype(np.int64).T
    assert np.array_equal(ip.cpu().numpy(), want), what
    assert float(np.abs(v.cpu().numpy() - want).max()) <= 0.25, what


# two database chunks and three query chunks, the last ones ragged; both sides of the transforms' own sizes
@pytest.mark.parametrize("log_n", [5, 8, 9, 10, 11, 12, 13, 14])
@pytest.mark.parametrize("family", ["primes", "chain"])
def test_ccmm_decrypts_exactly_at_every_ring_degree(log_n, family):
    n = 1 << log_n
    d1 = n + 37 if log_n <= 12 else 40
    d2 = min(2 * n + 11, 9001)
    rng = np.random.default_rng(100 + log_n)
    mdb, mq = _ternary(rng, d1, d2), _ternary(rng, 3, d2)
    if family == "primes":
        keys, level, form = H.hfe_keygen(H.hfe_default_params(log_n, log_n, 2, d2, d1), 5), 2, H.HFE_FORM_RNS_I8
    else:
        keys = H.hfe_chain_keygen(H.hfe_chain_default_params(log_n, log_n, 5, 3, d2, d1), 5)
        level, form = 5, H.HFE_FORM_P2_I8
    _say(f"[gpu-sizes] {family} 2^{log_n} d1 {d1} d2 {d2}")
    db = H.hfe_encrypt_db(keys, torch.from_numpy(mdb).cuda(), 6, form)
    q = H.hfe_encrypt(keys, torch.from_numpy(mq).cuda(), level, 7)
    _check(keys, H.hfe_ccmm(db, q, 0, d1, form), mq, mdb, "all rows")
    lo, rows = d1 // 3, d1 // 2
    _check(keys, H.hfe_ccmm(db, q, lo, rows, form), mq, mdb[lo:lo + rows], "a row range")
    # enough columns that each workgroup takes every chunk of its column
    many = _ternary(rng, 200, d2)
    q = H.hfe_encrypt(keys, torch.from_numpy(many).cuda(), level, 8)
    _check(keys, H.hfe_ccmm(db, q, 0, d1, form), many, mdb, "many columns")


@pytest.mark.parametrize("log_n_q", [6, 9, 10, 11, 12, 13, 14])
def test_format_switch_decrypts_exactly_at_every_query_ring(log_n_q):
    n = 1 << log_n_q
    d1, d2 = 50, n + 9
    rng = np.random.default_rng(200 + log_n_q)
    mdb, mq = _ternary(rng, d1, d2), _ternary(rng, 3, d2)
    keys = H.hfe_keygen(H.hfe_default_params(7, log_n_q, 3, d2, d1), 5)
    _say(f"[gpu-sizes] format switch to 2^{log_n_q}")
    db = H.hfe_encrypt_db(keys, torch.from_numpy(mdb).cuda(), 6, H.HFE_FORM_RNS_I8)
    fk = H.hfe_fs_keygen(keys, 2, log_n_q + 1, 7)
    T = H.hfe_fs_encrypt(fk, torch.from_numpy(mq).cuda(), 8)
    q = H.hfe_format_switch(fk, T, 3)
    _check(keys, H.hfe_ccmm(db, q, 0, d1, H.HFE_FORM_RNS_I8), mq, mdb, "switched query")


@pytest.mark.parametrize("log_n", [6, 8, 9, 11, 12, 13])
def test_fold_matches_the_plain_values_at_every_ring_degree(log_n):
    from oracle import fold as OF
    w = S.FoldWorkload(f"fold_n{1 << log_n}", log_n, 4, 6, 1, 1100, (1 << log_n) // 2, S.BASE_SEED + 300 + log_n)
    ip, counts = S.fold_inputs(w)
    _say(f"[gpu-sizes] fold 2^{log_n}")
    fk = H.hfe_fold_keygen(w.log_n, w.k, w.rho, 5)
    ct = H.hfe_fold_encrypt(fk, torch.from_numpy(ip).cuda(), 6)
    got = H.hfe_fold_decrypt(fk, H.hfe_fold(fk, ct, torch.from_numpy(counts).cuda(), w.rho)).cpu().numpy()
    want = OF.fold_plain(ip.astype(np.int64), counts.astype(np.int64), w.rho, w.k)
    assert float(np.max(np.abs(got - want))) < 0.02 + 4 * 19 * w.k / 2.0 ** 20


def _match_by_hand(ip, qm, shifts, dm):
    rolled = np.stack([np.roll(qm, int(s), 1) for s in shifts], 1).reshape(-1, qm.shape[1]).astype(np.int64)
    ov = rolled @ dm.astype(np.int64).T
    dec = (ov > 0) & (ip.astype(np.int64) * 8 > 2 * ov)
    return dec.astype(np.uint8), dec.reshape(len(qm), -1).any(1).astype(np.uint8)


# code lengths around the 16-byte pieces and 64-bit words, unaligned rows, shifts beyond the code length; few and many
# columns (both column groups of the kernel)
@pytest.mark.parametrize("d2,rows,eyes,shifts", [(1, 3, 2, (0,)), (15, 5, 1, (0, 1)), (63, 65, 3, (-8, 7, 0)),
                                                 (64, 64, 2, (0, 5)), (65, 63, 2, (-1, 1)), (257, 300, 5, (0, -300, 1000)),
                                                 (1000, 4100, 34, tuple(range(-8, 8))), (1023, 257, 7, (3, -5, 9))])
def test_match_decisions_at_odd_lengths(d2, rows, eyes, shifts):
    rng = np.random.default_rng(d2 + rows)
    qm, dm = (rng.random((eyes, d2)) < 0.9).astype(np.uint8), (rng.random((rows, d2)) < 0.9).astype(np.uint8)
    qm[0], dm[0] = 0, 0  # no overlap
    qm[-1] |= (rng.integers(0, 128, d2) * 2).astype(np.uint8)  # only the lowest bit of a mask byte counts
    ip = rng.integers(-d2, d2 + 1, (eyes * len(shifts), rows)).astype(np.int32)
    ip[:, 1:] //= 3
    if eyes > 2:
        ip[len(shifts):2 * len(shifts)] = -1  # an eye without a match
    _say(f"[gpu-sizes] match d2 {d2} rows {rows} columns {eyes * len(shifts)}")
    dec, eye = H.hfe_match(torch.from_numpy(ip).cuda(), torch.from_numpy(qm).cuda(), list(shifts),
                           torch.from_numpy(dm).cuda())
    want, want_eye = _match_by_hand(ip, qm & 1, shifts, dm)
    assert np.array_equal(dec.cpu().numpy(), want) and np.array_equal(eye.cpu().numpy(), want_eye)


# K-blocks of 64: 145 (the last one ragged), so parts of unequal length; one row tile and three, one column and several
@pytest.mark.parametrize("rows,cols", [(37, 1), (37, 130), (300, 5)])
@pytest.mark.parametrize("form", ["i8", "rns", "p2", "chain"])
def test_contraction_split_along_the_code_length_gives_the_same_residues(form, rows, cols):
    d2 = 9219
    rng = np.random.default_rng(300 + rows + cols)
    if form == "chain":
        keys, level, f = H.hfe_chain_keygen(H.hfe_chain_default_params(6, 6, 5, 3, d2, rows), 5), 5, H.HFE_FORM_P2_I8
    else:
        keys, level = H.hfe_keygen(H.hfe_default_params(6, 6, 3, d2, rows), 5), 3
        f = {"i8": H.HFE_FORM_I8_MFMA, "rns": H.HFE_FORM_RNS_I8, "p2": H.HFE_FORM_P2_I8}[form]
    mdb, mq = _ternary(rng, rows, d2), _ternary(rng, cols, d2)
    db = H.hfe_encrypt_db(keys, torch.from_numpy(mdb).cuda(), 6, f)
    q = H.hfe_encrypt(keys, torch.from_numpy(mq).cuda(), level, 7)
    H.hfe_noalloc_init()
    _say(f"[gpu-sizes] split {form} rows {rows} cols {cols}")
    r = H.hfe_ccmm(db, q, 0, rows, f)
    got = H.hfe_export(r, 0)
    out = torch.zeros(got.size, dtype=torch.int64, device="cuda")
    H.hfe_ccmm_noalloc(db, q, 0, rows, f, out)  # one part: its region is fixed
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), got.astype(np.int64))
    _check(keys, r, mq, mdb, "split")


# rows several requests share (one job of both widths, cut at tile boundaries and beyond the last row), short ranges
# apart, one request alone; levels mixed so that each prime slot has its own set of requests
@pytest.mark.parametrize("spans", [
    [(0, 1500, 20, 3), (100, 900, 70, 1), (255, 2, 3, 2), (600, 900, 130, 2), (1499, 1, 1, 3), (0, 1500, 4, 3)],
    [(256 * i + 17, 40, 2 + i, 1 + i % 3) for i in range(5)],
    [(300, 1200, 33, 2)],
    [(0, 1500, 48, 1 + i % 3) for i in range(8)],
])
def test_batched_rns_jobs_give_every_request_its_single_result(spans):
    d1, d2 = 1500, 201
    rng = np.random.default_rng(400 + len(spans))
    keys = H.hfe_keygen(H.hfe_default_params(6, 6, 3, d2, d1), 5)
    mdb = _ternary(rng, d1, d2)
    db = H.hfe_encrypt_db(keys, torch.from_numpy(mdb).cuda(), 6, H.HFE_FORM_RNS_I8)
    items, mqs = [], []
    for i, (row0, rows, cols, level) in enumerate(spans):
        mqs.append(_ternary(rng, cols, d2))
        items.append((H.hfe_encrypt(keys, torch.from_numpy(mqs[-1]).cuda(), level, 50 + i), row0, rows))
    _say(f"[gpu-sizes] batched rns {spans}")
    outs = H.hfe_ccmm_batched(db, items, H.HFE_FORM_RNS_I8)
    for i, (q, row0, rows) in enumerate(items):
        one = H.hfe_ccmm(db, q, row0, rows, H.HFE_FORM_RNS_I8)
        assert np.array_equal(H.hfe_export(outs[i], 0), H.hfe_export(one, 0)), f"request {i}"
        _check(keys, outs[i], mqs[i], mdb[row0:row0 + rows], f"request {i}")


# the 32-column digit tile's last column, the next width's first; row tiles of 128 with a remainder of one row
@pytest.mark.parametrize("cols", [1, 31, 32, 33])
def test_few_columns_of_the_digit_form_equal_the_small_moduli(cols):
    d1, d2 = 193, 700
    rng = np.random.default_rng(500 + cols)
    keys = H.hfe_keygen(H.hfe_default_params(6, 7, 2, d2, d1), 5)
    mdb, mq = _ternary(rng, d1, d2), _ternary(rng, cols, d2)
    db = H.hfe_encrypt_db(keys, torch.from_numpy(mdb).cuda(), 6, H.HFE_FORM_I8_MFMA | H.HFE_FORM_RNS_I8)
    q = H.hfe_encrypt(keys, torch.from_numpy(mq).cuda(), 2, 7)
    _say(f"[gpu-sizes] digit form, {cols} columns")
    r = H.hfe_ccmm(db, q, 0, d1, H.HFE_FORM_I8_MFMA)
    assert np.array_equal(H.hfe_export(r, 0), H.hfe_export(H.hfe_ccmm(db, q, 0, d1, H.HFE_FORM_RNS_I8), 0))
    _check(keys, r, mq, mdb, "all rows")


# the digits' runs of 1, 4 and 8 coefficients, ratios of 8 and above, and polynomials split over several blocks
@pytest.mark.parametrize("log_n_q,log_n_t", [(7, 7), (7, 9), (7, 10), (7, 12), (10, 14), (11, 15)])
def test_format_switch_decrypts_exactly_at_every_ring_ratio(log_n_q, log_n_t):
    d1, d2 = 40, (1 << log_n_q) + 5
    rng = np.random.default_rng(700 + log_n_t)
    mdb, mq = _ternary(rng, d1, d2), _ternary(rng, 2, d2)
    keys = H.hfe_keygen(H.hfe_default_params(7, log_n_q, 3, d2, d1), 5)
    _say(f"[gpu-sizes] format switch 2^{log_n_t} to 2^{log_n_q}")
    db = H.hfe_encrypt_db(keys, torch.from_numpy(mdb).cuda(), 6, H.HFE_FORM_RNS_I8)
    fk = H.hfe_fs_keygen(keys, 2, log_n_t, 7)
    q = H.hfe_format_switch(fk, H.hfe_fs_encrypt(fk, torch.from_numpy(mq).cuda(), 8), len(mq))
    _check(keys, H.hfe_ccmm(db, q, 0, d1, H.HFE_FORM_RNS_I8), mq, mdb, "switched query")
