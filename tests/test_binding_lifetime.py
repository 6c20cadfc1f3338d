"""Objects of a context are freed before it, once each, whatever order Python
drops them in (the library's free functions use the context): recorded with a
stand-in for the library."""
import ctypes
import gc

import pytest

from paper_2203_14071_amd import rlf


class FakeLib:
    def __init__(self):
        self.calls, self.n = [], 0

    def __getattr__(self, name):
        def call(*args):
            if name in ("rlf_create", "rlf_mlp_create"):
                self.n += 1
                (args[0] if name == "rlf_create" else args[-1])._obj.value = self.n
            elif name.endswith("_free") or name == "rlf_destroy":
                self.calls.append((name, args[0].value))
            return 0
        return call


@pytest.fixture
def fake(monkeypatch):
    f = FakeLib()
    monkeypatch.setattr(rlf, "lib", lambda: f)
    return f


def _world():
    ctx = rlf.Context()
    return ctx, rlf.Facets(ctx, ctypes.c_void_p(11)), rlf.Pass(ctx, ctypes.c_void_p(12)), rlf.Mlp(ctx)


ALL = [("rlf_mlp_free", 2), ("rlf_pass_free", 12), ("rlf_facets_free", 11), ("rlf_destroy", 1)]


def test_closing_the_context_frees_what_is_left(fake):
    ctx, f, ps, net = _world()
    ctx.close()
    assert fake.calls == ALL
    f.free(), ps.free(), net.free(), ctx.close()
    assert fake.calls == ALL and not f.h and not ps.h and not net.h


def test_what_was_freed_is_not_freed_again(fake):
    ctx, f, ps, net = _world()
    f.free()
    ps.free()
    del net
    assert fake.calls == [("rlf_facets_free", 11), ("rlf_pass_free", 12), ("rlf_mlp_free", 2)]
    ctx.close()
    assert fake.calls[3:] == [("rlf_destroy", 1)]


@pytest.mark.parametrize("first", [0, 1, 2, 3])
def test_a_cycle_of_them_all(fake, first):
    objs = list(_world())
    objs = objs[first:] + objs[:first]
    frame = {"objs": objs}
    frame["self"] = frame
    del objs, frame
    gc.collect()
    assert sorted(fake.calls) == sorted(ALL) and fake.calls[-1] == ("rlf_destroy", 1)
