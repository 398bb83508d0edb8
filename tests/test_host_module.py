"""The host extension is an aid: without it, and without what it takes to build it, every call still goes through binding.py's own code."""
import threading
import time
import warnings

import pytest
import torch

import paper_2510_01450_amd as llla
from paper_2510_01450_amd import binding
from paper_2510_01450_amd import build


@pytest.fixture
def unloaded(monkeypatch):
    """A process that has made no call yet."""
    monkeypatch.setattr(binding, "_host", None)
    monkeypatch.setattr(binding, "_entries", {})


def _missing(monkeypatch, how, tmp_path):
    if how == "no compiler":
        monkeypatch.setattr(build, "host_is_current", lambda: False)
        monkeypatch.setattr(build, "CXX", str(tmp_path / "no-such-compiler"))
    elif how == "compiler fails":
        monkeypatch.setattr(build, "host_is_current", lambda: False)
        monkeypatch.setattr(build, "CXX", "false")
    elif how == "tree not writable":
        monkeypatch.setattr(build, "host_is_current", lambda: False)
        monkeypatch.setattr(build, "build_host", lambda verbose=False: open(str(tmp_path / "no-such-folder" / "llla_host.so"), "wb"))
    else:                                                      # a file that cannot be loaded
        bad = tmp_path / "llla_host.so"
        bad.write_bytes(b"not a library")
        monkeypatch.setattr(build, "host_is_current", lambda: True)
        monkeypatch.setattr(build, "LIB_HOST", str(bad))


@pytest.mark.parametrize("how", ["no compiler", "compiler fails", "tree not writable", "not a library"])
def test_calls_do_without_it(monkeypatch, unloaded, how, tmp_path):
    _missing(monkeypatch, how, tmp_path)
    with pytest.warns(RuntimeWarning, match="llla_host.so"):
        host = binding._load_host()
    assert host.forward(*range(14)) is NotImplemented and host.decode(*range(13)) is NotImplemented
    with warnings.catch_warnings():
        warnings.simplefilter("error")                         # told once, tried once
        assert binding._load_host() is host


def test_mistakes_load_nothing(monkeypatch, unloaded):
    def loads(*args):
        raise AssertionError("loaded for a call that is refused")
    monkeypatch.setattr(binding, "_load", loads)
    monkeypatch.setattr(binding, "_load_host", loads)
    t, q = torch.zeros(1, 1, 8, 16), torch.zeros(1, 1, 16)
    with pytest.raises(ValueError, match="device tensors"):
        llla.llla_forward(t, t, t, 0.1, 1.0)
    with pytest.raises(ValueError, match="device tensors"):
        llla.llla_decode(q, t, t, 0.1, 1.0)


def test_threads_build_it_once(monkeypatch, unloaded):
    built = []

    def slow_build(verbose=False):
        built.append(1)
        time.sleep(0.2)
        raise OSError("no compiler")
    monkeypatch.setattr(build, "host_is_current", lambda: False)
    monkeypatch.setattr(build, "build_host", slow_build)
    got = []
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        threads = [threading.Thread(target=lambda: got.append(binding._load_host())) for _ in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert len(built) == 1 and len(got) == 4 and all(h is got[0] for h in got)


def test_stamp_covers_the_flags(monkeypatch):
    before = build.host_hash()
    monkeypatch.setattr(build, "HOST_FLAGS", [f.replace("-O2", "-O3") for f in build.HOST_FLAGS])
    assert build.host_hash() != before


def test_kernels_are_built_before_it(monkeypatch):
    order = []
    monkeypatch.setattr(build, "_build_one", lambda lib, *a: order.append(lib))
    monkeypatch.setattr(build, "build_host", lambda verbose=False: order.append(build.LIB_HOST))
    build.build()
    assert order == [build.LIB, build.LIB_MEASURE, build.LIB_HOST]
