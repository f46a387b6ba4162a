"""The library's host side on the CPU, its kernels replaced by a record of what
they would add (tests/host_runtime.cpp): every push reaches a group's sums
exactly once and in order, also after a launch that was refused."""
import ctypes
import os
import subprocess
from types import SimpleNamespace

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stub_path(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host") / "libcorr_host.so")
    csrc = os.path.join(ROOT, "paper_2503_07526_amd", "csrc")
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
         "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=x", "-I/opt/rocm/include",
         os.path.join(csrc, "corr_runtime.cpp"), os.path.join(csrc, "corr_autotune.cpp"),
         os.path.join(ROOT, "tests", "host_runtime.cpp"), "-o", out])
    return out


class Host:
    """The binding over the recording library."""

    def __init__(self, corr):
        self.corr, self.L = corr, corr.lib()
        self.L.stub_reset()

    def context(self, groups, **kw):
        return self.corr.Correlator(groups, stream=SimpleNamespace(cuda_stream=0), **kw)

    def fail(self, name, after=0):
        self.L.stub_fail(name.encode(), after)

    def calls(self, name):
        return self.L.stub_calls(name.encode())

    def added(self, n_ch):
        """[(push number, its first sample)] added to the group of n_ch channels."""
        push, value = (ctypes.c_int64 * 4096)(), (ctypes.c_float * 4096)()
        n = self.L.stub_added(ctypes.c_int64(n_ch), push, value, 4096)
        return list(zip(push[:n], value[:n]))


@pytest.fixture
def host(stub_path, monkeypatch):
    import paper_2503_07526_amd.corr as c
    monkeypatch.setattr(c, "_lib", None)
    monkeypatch.setattr(c, "LIB_PATH", stub_path)
    monkeypatch.setenv("CORR_TUNE_CACHE", "/nonexistent/none")
    return Host(c)


def _frames(steps, *channels):
    """[steps][n] samples of every group; row s holds s + 1 everywhere."""
    return [np.repeat(np.arange(1, steps + 1, dtype=np.float32)[:, None], n, 1) for n in channels]


def _push(c, frames, s):
    c.push([f[s].ctypes.data for f in frames])


def _every_push_once(host, n_ch, steps):
    assert host.added(n_ch) == [(s, float(s)) for s in range(1, steps + 1)], f"{n_ch} channels"


@pytest.mark.parametrize("after", [0, 1])
@pytest.mark.parametrize("retry", ["push", "finalize"])
def test_refused_pass_of_waiting_pushes(host, after, retry):
    """A pass that the runtime refuses, for the first or the second of two
    groups, after 64 pushes or at a readout: a readout that needed it fails, no
    push is written past the rows, and after the next calls every push is in
    the sums of both groups once."""
    groups = [host.corr.GroupDesc(n, 3, 32, 2) for n in (5, 7)]
    steps = 200
    frames = _frames(steps, 5, 7)
    with host.context(groups) as c:
        s = refused = 0
        if retry == "finalize":
            for s in range(10):
                _push(c, frames, s)
            s = 10
            host.fail("multi_push", after)
            with pytest.raises(host.corr.CorrError):
                c.finalize(0)
            refused = 1
        else:
            host.fail("multi_push", after)
        while s < steps:
            try:
                _push(c, frames, s)
                s += 1
            except host.corr.CorrError:
                refused += 1
            assert c.n_pushes() == s
        c.finalize(0)
        assert refused == (retry == "finalize") and host.L.stub_out_of_range() == 0
        for n in (5, 7):
            _every_push_once(host, n, steps)


def test_passes_refused_several_times(host):
    """Passes refused several times in a row: pushes fail while no row is free
    and go on when the runtime takes launches again."""
    g = host.corr.GroupDesc(6, 3, 32, 2)
    frames = _frames(130, 6)
    with host.context([g]) as c:
        s = refused = 0
        while s < 130:
            if refused < 4:
                host.fail("multi_push")
            try:
                _push(c, frames, s)
                s += 1
            except host.corr.CorrError:
                refused += 1
            assert c.n_pushes() == s
        c.finalize(0)
        assert refused == 4 and host.L.stub_out_of_range() == 0
        _every_push_once(host, 6, 130)


@pytest.mark.parametrize("after", [0, 4, 5])
def test_refused_pass_of_a_history(host, after):
    """A pass over the rows of a history refused, for the first or the second of
    two groups: no readout of a group that is ahead of the count, and the rows
    that were not counted, given again, are in the sums once."""
    groups = [host.corr.GroupDesc(n, 3, 32, 2) for n in (5, 7)]
    hist = _frames(300, 5, 7)
    strides = (ctypes.c_int64 * 2)(*[h.strides[0] for h in hist])
    with host.context(groups) as c:
        for s in range(3):
            _push(c, hist, s)

        def steps(done):
            rows = (ctypes.c_void_p * 2)(*[h[done:].ctypes.data for h in hist])
            return host.L.corr_push_steps(c._h, 300 - done, rows, strides)

        host.fail("multi_push", after)
        assert steps(3) != 0
        done = c.n_pushes()
        assert done == (3 if after < 2 else 3 + 64)
        if after == 5:
            with pytest.raises(host.corr.CorrError):
                c.finalize(0)
        c.finalize(1)
        if after == 4:
            _push(c, hist, done)
            done += 1
        assert steps(done) == 0 and c.n_pushes() == 300
        c.finalize(0)
        for n in (5, 7):
            _every_push_once(host, n, 300)


def test_pending_error_is_reported_before_anything_is_issued(host):
    """An error that the caller's own HIP calls left behind: a push and a
    readout report it and issue nothing."""
    groups = [host.corr.GroupDesc(5, 3, 32, 2), host.corr.GroupDesc(7, 3, 8, 2), host.corr.GroupDesc(600, 3, 16, 2)]
    frames = _frames(70, 5, 7, 600)
    with host.context(groups) as c:
        for s in range(70):
            if s in (0, 10, 64):
                before = [host.calls(k) for k in ("keep_rows", "push_batched", "stage", "multi_push")]
                host.fail("last_error")
                with pytest.raises(host.corr.CorrError):
                    _push(c, frames, s)
                host.fail("last_error")
                with pytest.raises(host.corr.CorrError):
                    c.finalize(0)
                assert before == [host.calls(k) for k in ("keep_rows", "push_batched", "stage", "multi_push")]
            _push(c, frames, s)
        c.finalize(0)
        for n in (5, 7):
            _every_push_once(host, n, 70)


@pytest.mark.parametrize("n,pair,kw,single", [
    (98303, False, dict(points=32), "multi_push"), (98304, False, dict(points=32), "push_batched"),
    (65535, True, dict(points=16), "multi_push"), (65536, True, dict(points=16), "push_group"),
    (98304, False, dict(points=24, dtype="cf32", accum="kahan"), "multi_push")])
def test_single_push_of_a_large_group(host, n, pair, kw, single):
    """One push to add is added by the per-step kernel of a large group with
    narrow sums, else (and with another beside it) by a multi-step pass; from
    its row at a readout, and straight from a history."""
    g = host.corr.GroupDesc(n, 3, m=2, pair=pair, **kw)
    x = np.zeros((5, (2 if pair else 1) * n * (2 if "dtype" in kw else 1)), np.float32)
    x[:, 0] = [1, 2, 3, 4, 5]
    strides = (ctypes.c_int64 * 1)(x.strides[0])
    with host.context([g]) as c:
        _push(c, [x], 0)
        c.finalize(0)
        assert host.calls(single) == 1
        assert host.L.corr_push_steps(c._h, 1, (ctypes.c_void_p * 1)(x[1:].ctypes.data), strides) == 0
        assert host.calls(single) == 2 and (single == "multi_push" or host.calls("multi_push") == 0)
        _push(c, [x], 2)
        _push(c, [x], 3)
        c.finalize(0)
        assert host.calls("multi_push") == (3 if single == "multi_push" else 1)
        _push(c, [x], 4)
        host.fail(single)
        with pytest.raises(host.corr.CorrError):
            c.finalize(0)
        c.finalize(0)
        _every_push_once(host, n, 5)


def test_waiting_rows_only_where_pushes_wait(host):
    """Device memory of a group with multi-step passes: 64 rows of its pushes'
    samples where they wait there, none in a context with captured pushes (a
    captured run adds sample groups straight from the history)."""
    n, row = 5000, 5000 * 4 // 256 * 256 + 256
    host.L.stub_allocated.restype = ctypes.c_int64

    def bytes_of(**kw):
        before = host.L.stub_allocated()
        with host.context([host.corr.GroupDesc(n, 3, 32, 2)], **kw):
            return host.L.stub_allocated() - before

    plain = bytes_of(direct=True)
    assert bytes_of() - plain == 64 * row
    assert bytes_of(graph=True) == plain


@pytest.mark.parametrize("after", range(9))
def test_refused_fold(host, after):
    """A fold that the runtime refuses, in a push, in the rows of a short replay
    or at a readout that folds what is behind: after the call made again (from
    where the count stands) every subset of both groups has folded every block
    once, in order."""
    ns, T = (3 * 98304 - 5, 2 * 98304 - 7), 256
    groups = [host.corr.GroupDesc(n, 3, 16, 2) for n in ns]
    x = [np.zeros((T, n), np.float32) for n in ns]

    def check(c):
        q = c.n_pushes() // T
        for n, subsets in zip(ns, (3, 2)):
            out = (ctypes.c_int64 * 4096)()
            k = host.L.stub_folded(ctypes.c_int64(n), out, 4096)
            got = list(out[:k])
            for j in range(subsets):
                assert [v // 1000000 for v in got if v % 1000000 == j] == list(range(1, q + 1)), (n, j)
            assert len(got) == subsets * q

    with host.context(groups) as c:
        def steps(n):
            rows = (ctypes.c_void_p * 2)(*[a.ctypes.data for a in x])
            host.L.corr_push_steps(c._h, n, rows, (ctypes.c_int64 * 2)(*[a.strides[0] for a in x]))

        def again(f, n):
            """f to n more pushes, repeated for what is missing."""
            want, tries = c.n_pushes() + n, 0
            while c.n_pushes() < want:
                f(want - c.n_pushes())
                tries += 1
                assert tries < 4

        def push(n):
            for _ in range(n):
                try:
                    _push(c, x, 0)
                except host.corr.CorrError:
                    return

        host.fail("fold", after)
        again(push, T + 1)
        again(steps, 100)
        again(push, T - 101)       # up to a block's end
        try:
            c.finalize(0)
        except host.corr.CorrError:
            pass
        again(steps, 1)
        again(steps, 120)
        again(push, 3)
        again(steps, 200)
        for i in range(2):
            try:
                c.finalize(i)
            except host.corr.CorrError:
                c.finalize(i)
        check(c)


@pytest.mark.parametrize("others", [False, True])
@pytest.mark.parametrize("name,after", [("history_fold", 0), ("history_fold", 1), ("history_fold", 2), ("history_fold", 3),
                                        ("push_batched", 300), ("push_batched", 700)])
def test_refused_fold_of_a_history(host, others, name, after):
    """A whole-block fold straight from the history (or a push of the group
    beside it) refused: the call made again from where the count stands folds
    every block of both block-deferred groups once and pushes the others once."""
    n, T, steps = (300, 700), 256, 900
    x = [np.zeros((steps, k), np.float32) for k in n] + ([np.zeros((steps, 5), np.float32)] if others else [])
    for a in x:
        a[:, 0] = np.arange(1, steps + 1)
    groups = [host.corr.GroupDesc(k, 3, 16, 2) for k in n] + ([host.corr.GroupDesc(5, 3, 8, 2)] if others else [])
    with host.context(groups) as c:
        for s in range(3):
            _push(c, x, s)
        host.fail(name, after - 3 if name == "push_batched" else after)
        failed = 0
        while c.n_pushes() < steps:
            at = c.n_pushes()
            rows = (ctypes.c_void_p * len(x))(*[a[at:].ctypes.data for a in x])
            if host.L.corr_push_steps(c._h, steps - at, rows, (ctypes.c_int64 * len(x))(*[a.strides[0] for a in x])):
                failed += 1
                assert failed < 3
        for i in range(len(x)):
            c.finalize(i)
        out = (ctypes.c_int64 * 4096)()
        for k in n:
            got = out[:host.L.stub_folded(ctypes.c_int64(k), out, 4096)]
            assert [v // 1000000 for v in got] == list(range(1, steps // T + 1)), (k, failed)
        if others:
            _every_push_once(host, 5, steps)


def test_refused_push_between_scheduled_folds(host):
    """A replay that stops between the pushes at which two subsets fold: the
    subset whose push was counted folds at the next call."""
    n, T = 2 * 98304, 256
    x = [np.zeros((600, n), np.float32), np.zeros((600, 5), np.float32)]
    x[1][:, 0] = np.arange(1, 601)
    groups = [host.corr.GroupDesc(n, 3, 16, 2), host.corr.GroupDesc(5, 3, 8, 2)]
    with host.context(groups) as c:
        for s in range(T):
            _push(c, x, s)
        host.fail("push_batched", 2)
        for _ in range(2):
            at = c.n_pushes()
            rows = (ctypes.c_void_p * 2)(*[a[at:].ctypes.data for a in x])
            rc = host.L.corr_push_steps(c._h, T + 10 - at, rows, (ctypes.c_int64 * 2)(*[a.strides[0] for a in x]))
            assert (rc == 0) == (at > T) and c.n_pushes() == (T + 10 if at > T else T + 2)
        for s in range(T + 10, 600):
            _push(c, x, s)
        c.finalize(0)
        out = (ctypes.c_int64 * 64)()
        got = out[:host.L.stub_folded(ctypes.c_int64(n), out, 64)]
        for j in range(2):
            assert [v // 1000000 for v in got if v % 1000000 == j] == [1, 2], j
        _every_push_once(host, 5, 600)
