"""Calls under an allocator with a limit: what a call can do without must not cost it what it needs.

Buffers that only save time (the parts of a split contraction, errors drawn once for every modulus) are given up when
there is no memory for them, and the results are the same residues.  The limit is counted in the bytes that the
library asks for; the allocator behind it is torch's.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)
H = pytest.importorskip("paper_2601_17561_amd")


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


class _Limited:
    """The library's allocations inside the block: logged, and refused beyond `limit` bytes held at a time."""

    def __init__(self, limit=None):
        self.limit, self.live, self.log, self.peak = limit, {}, [], 0

    def __enter__(self):
        def alloc(n, stream):
            held = sum(self.live.values()) + n
            if self.limit is not None and held > self.limit:
                raise MemoryError
            p = torch.cuda.caching_allocator_alloc(n, stream=stream)
            self.live[p] = n
            self.log.append(n)
            self.peak = max(self.peak, held)
            return p

        def free(p, stream):
            self.live.pop(p, None)
            torch.cuda.caching_allocator_delete(p)

        H.hfe_set_allocator(alloc, free)
        return self

    def __exit__(self, *exc):
        H.use_torch_allocator()


def _ternary(rng, n, d):
    return torch.from_numpy(rng.integers(-1, 2, (n, d)).astype(np.int8)).cuda()


def _keys(family, log_n, d2, d1):
    if family == "chain":
        return H.hfe_chain_keygen(H.hfe_chain_default_params(log_n, log_n, 5, 3, d2, d1), 5), 5
    return H.hfe_keygen(H.hfe_default_params(log_n, log_n, 3, d2, d1), 5), 3


# 145 K-blocks and few tiles, so that every form cuts the code length into parts
@pytest.mark.parametrize("form", ["i8", "rns", "p2", "chain"])
def test_split_contraction_gives_its_parts_up_without_memory(form):
    rows, cols, d2 = 37, 130, 9219
    rng = np.random.default_rng(11)
    keys, level = _keys(form, 6, d2, rows)
    f = {"i8": H.HFE_FORM_I8_MFMA, "rns": H.HFE_FORM_RNS_I8}.get(form, H.HFE_FORM_P2_I8)
    db = H.hfe_encrypt_db(keys, _ternary(rng, rows, d2), 6, f)
    q = H.hfe_encrypt(keys, _ternary(rng, cols, d2), level, 7)
    with _Limited() as free:
        r = H.hfe_ccmm(db, q, 0, rows, f)
        want = H.hfe_export(r, 0)
        r.free()
    _say(f"[memory] split {form}: {free.log}")
    assert len(free.log) == 4  # query planes, contraction output, result, parts
    with _Limited(free.peak - 1):  # the parts have to go, whatever was asked for last
        r = H.hfe_ccmm(db, q, 0, rows, f)
        assert np.array_equal(H.hfe_export(r, 0), want)
        r.free()


# code lengths below three query rings, where the errors lie in a buffer that is free by then, and above
@pytest.mark.parametrize("d2,spare", [(700, True), (1600, False), (2500, False)])
@pytest.mark.parametrize("family", ["primes", "chain"])
def test_database_errors_need_no_memory_of_their_own(family, d2, spare):
    log_n, d1 = 9, 700
    m_db = _ternary(np.random.default_rng(12), d1, d2)
    keys, _ = _keys(family, log_n, d2, d1)
    forms = H.HFE_FORM_PLAIN_U64 | H.HFE_FORM_P2_I8
    with _Limited() as free:
        db = H.hfe_encrypt_db(keys, m_db, 6, forms)
        want = H.hfe_export(db, 0)
        db.free()
    errors = (d2 + (1 << log_n)) * d1
    _say(f"[memory] enrol {family} d2 {d2}: {free.log}, errors {errors}")
    assert (errors in free.log) == (not spare)
    if not spare:
        with _Limited(free.peak - 1):
            db = H.hfe_encrypt_db(keys, m_db, 6, forms)
            assert np.array_equal(H.hfe_export(db, 0), want)
            db.free()


# one column and chunk, several chunks side by side in small calls and one after the other in large ones
@pytest.mark.parametrize("d2,cols", [(301, 1), (1290, 5), (1290, 200)])
@pytest.mark.parametrize("family,level", [("primes", 1), ("primes", 3), ("chain", 5)])
def test_query_errors_need_no_memory_of_their_own(family, level, d2, cols):
    m_q = _ternary(np.random.default_rng(13), cols, d2)
    keys, _ = _keys(family, 9, d2, 64)
    with _Limited() as free:
        q = H.hfe_encrypt(keys, m_q, level, 7)
        want = H.hfe_export(q, 0)
        q.free()
    _say(f"[memory] encrypt {family} level {level} d2 {d2} columns {cols}: {free.log}")
    assert cols * d2 in free.log
    with _Limited(free.peak - 1):
        q = H.hfe_encrypt(keys, m_q, level, 7)
        assert np.array_equal(H.hfe_export(q, 0), want)
        q.free()


# a plan holds the batch's own query columns: the RNS contraction reads no padding
def test_rns_plan_holds_its_columns_only():
    d1, d2, level = 300, 500, 2
    rng = np.random.default_rng(14)
    keys = H.hfe_keygen(H.hfe_default_params(6, 6, level, d2, d1), 5)
    db = H.hfe_encrypt_db(keys, _ternary(rng, d1, d2), 6, H.HFE_FORM_RNS_I8)
    row = H.hfe_db_bytes(db, H.HFE_FORM_RNS_I8) // ((d1 + 64 + 63) // 64 * 64 + 256)  # every plane of one row
    items = [(H.hfe_encrypt(keys, _ternary(rng, c, d2), level, 7 + c), r0, rows)
             for c, r0, rows in ((5, 0, 300), (130, 0, 300), (3, 100, 90))]
    with _Limited() as free:
        plan = H.hfe_plan_create_for(db, items, H.HFE_FORM_RNS_I8)
        _say(f"[memory] plan {free.log}, a column {row}")
        assert 138 * row in free.log
        H.hfe_plan_run(plan, items, use_graph=False)
        for i, (q, row0, rows) in enumerate(items):
            one = H.hfe_ccmm(db, q, row0, rows, H.HFE_FORM_RNS_I8)
            assert np.array_equal(H.hfe_export(H.hfe_plan_result(plan, i), 0), H.hfe_export(one, 0))
            one.free()
        plan.free()
