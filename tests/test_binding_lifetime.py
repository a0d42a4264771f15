"""A context outlives the hierarchies and servers on it, in whatever order they
are closed or a collected garbage cycle finalises them (the library reads the
context when it destroys them).  The library's calls are recorded, not made."""
import gc
import itertools

import pytest

from paper_0904_4152_amd import _binding


class Recorder:
    def __init__(self):
        self.calls = []
        self.handles = itertools.count(1)

    def __getattr__(self, name):
        def call(*args):
            if "create" in name:
                args[-1]._obj.value = next(self.handles)
            self.calls.append(name)
            return _binding.MG_OK
        return call


@pytest.fixture
def calls(monkeypatch):
    r = Recorder()
    monkeypatch.setattr(_binding, "lib", lambda: r)
    return r.calls


def make():
    ctx = _binding.Context(0)
    return ctx, _binding.Hierarchy(ctx, 3, assemble=False), _binding.Server(ctx, 1, 1 << 20, 3)


def destroyed(calls):
    return [c for c in calls if c.endswith("_destroy")]


@pytest.mark.parametrize("order", list(itertools.permutations(range(3))))
def test_closed_in_any_order(calls, order):
    things = make()
    for i in order:
        things[i].close()
        things[i].close()
    got = destroyed(calls)
    assert sorted(got) == ["mg_context_destroy", "mg_hierarchy_destroy", "mg_server_destroy"]
    assert got[-1] == "mg_context_destroy"


@pytest.mark.parametrize("order", list(itertools.permutations(range(3))))
def test_collected_in_any_order(calls, order):
    # the finalisers called in every order, as a collector of a cycle may
    things = make()
    for i in order:
        things[i].__del__()
    del things
    gc.collect()
    got = destroyed(calls)
    assert len(got) == 3 and got[-1] == "mg_context_destroy"
