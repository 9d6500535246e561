"""Batched RNS jobs whose columns lie in several narrow tiles (257 to 384 columns side by side)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)
H = pytest.importorskip("paper_2601_17561_amd")


def _ternary(rng, n, d):
    return torch.from_numpy(rng.integers(-1, 2, (n, d)).astype(np.int8)).cuda()


# one request, requests that fill the narrow tiles together, levels that leave a prime slot fewer columns, row ranges
# that share a part; the widths on both sides of the rule
@pytest.mark.parametrize("spans", [
    [(0, 700, 257, 2)],
    [(0, 700, 384, 2)],
    [(0, 700, 385, 1)],
    [(0, 700, 130, 1), (0, 700, 130, 2), (0, 700, 90, 3)],
    [(0, 500, 200, 2), (300, 400, 150, 2)],
])
def test_columns_in_several_narrow_tiles_equal_the_single_calls(spans):
    d1, d2 = 700, 201
    rng = np.random.default_rng(21)
    keys = H.hfe_keygen(H.hfe_default_params(6, 6, 3, d2, d1), 5)
    db = H.hfe_encrypt_db(keys, _ternary(rng, d1, d2), 6, H.HFE_FORM_RNS_I8)
    items = [(H.hfe_encrypt(keys, _ternary(rng, c, d2), level, 50 + i), row0, rows)
             for i, (row0, rows, c, level) in enumerate(spans)]
    print(f"[rns-jobs] {spans}", flush=True)
    sys.stdout.flush()
    outs = H.hfe_ccmm_batched(db, items, H.HFE_FORM_RNS_I8)
    for i, (q, row0, rows) in enumerate(items):
        one = H.hfe_ccmm(db, q, row0, rows, H.HFE_FORM_RNS_I8)
        assert np.array_equal(H.hfe_export(outs[i], 0), H.hfe_export(one, 0)), f"request {i}"
