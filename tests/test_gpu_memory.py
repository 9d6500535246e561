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
