"""What the binding refuses before it calls the library (no GPU needed: the library is replaced by a recorder)."""
import types

import pytest

torch = pytest.importorskip("torch")
H = pytest.importorskip("paper_2601_17561_amd")


class _Recorder:
    """Stands in for the library: counts residues as hfe_fs_transmit_count does and records every other call."""

    def __init__(self, per_column):
        self.per_column, self.called = per_column, []

    def hfe_fs_transmit_count(self, fk, d3, count):
        count._obj.value = self.per_column * d3
        return 0

    def __getattr__(self, name):
        def call(*args):
            self.called.append(name)
            return 0
        return call


@pytest.fixture
def fs(monkeypatch):
    rec = _Recorder(40)
    monkeypatch.setattr(H, "_lib", rec)
    monkeypatch.setattr(H, "_dev_ptr", lambda t, dtype: t.data_ptr())
    monkeypatch.setattr(H, "_stream", lambda stream: 0)
    return rec, types.SimpleNamespace(ptr=1)


# T is a bare pointer for the library: a column count above what T holds would read, or write, past the tensor
@pytest.mark.parametrize("held,asked,runs", [(3, 3, True), (4, 3, True), (3, 4, False), (0, 1, False)])
def test_transmission_tensors_shorter_than_their_columns_are_refused(fs, held, asked, runs):
    rec, fk = fs
    T = torch.zeros(40 * held, dtype=torch.int64)
    calls = [lambda: H.hfe_format_switch(fk, T, asked),
             lambda: H.hfe_fs_encrypt(fk, torch.zeros((asked, 8), dtype=torch.int8), 1, T)]
    for call, name in zip(calls, ("hfe_format_switch", "hfe_fs_encrypt")):
        rec.called.clear()
        if runs:
            call()
        else:
            with pytest.raises(ValueError):
                call()
        assert rec.called == ([name] if runs else [])
