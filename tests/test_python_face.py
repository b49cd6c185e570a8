"""The Python face names every entry point of the library that it wraps, and
counts steps as the library does."""
import types

import pytest

from paper_2504_14494_amd import _lib, gnn, lbm


def test_every_wrapped_entry_point_is_exported():
    for module in (lbm, gnn):
        wrapped = {n for n, f in vars(module).items() if isinstance(f, types.FunctionType)
                   and f.__module__ == module.__name__ and n in _lib.EXPORTS}
        assert wrapped and wrapped <= set(module.__all__), wrapped - set(module.__all__)


@pytest.mark.parametrize("nsteps,last", [(1, "b"), (2, "a"), (3.0, "b"), (2.5, "a")])
def test_lbm_steps_gnn_returns_the_buffer_of_the_steps_it_took(monkeypatch, nsteps, last):
    taken = []

    class Library:
        def lbm_steps_gnn(self, *args):
            taken.append(args[7])
            return 0

    class Buffer:
        def numel(self):
            return 0

    monkeypatch.setattr(gnn, "_gnn_step_args", lambda *args: (4, 4, None, Buffer()))
    monkeypatch.setattr(gnn._lib, "load", Library)
    monkeypatch.setattr(gnn, "_ptr", lambda t: None)
    monkeypatch.setattr(gnn, "_stream", lambda: None)
    assert gnn.lbm_steps_gnn("a", "b", 0.7, None, nsteps) == last
    assert taken == [int(nsteps)]
