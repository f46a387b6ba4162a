"""GPU parity at the edges of the library's dispatch rules: the sizes at which
a launch takes another kernel, another split or another schedule, against the
FP64 oracle fed the same samples."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_helpers import TOL, ou_inputs, say

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def corrmod():
    import paper_2503_07526_amd.corr as m
    return m


def _check_channels(res, o, channels, tol, label):
    """Per-channel values of a finalize() slice [b, e) against oracle channels:
    channels = [(index in the slice, oracle channel)]."""
    t, c, n = o.readout()
    assert np.array_equal(res["t"], t) and np.array_equal(res["count"], n), label
    for i, ch in channels:
        _, cc, _ = o.readout(ch, ch + 1)
        err = np.max(np.abs(res["c_per_channel"][i] - cc)) / abs(cc[0])
        assert err <= tol, f"{label}: slice entry {i}: {err:.3e} > {tol:.1e}"


@pytest.mark.parametrize("n", [98303, 98304, 98305, 196608 + 700])
@pytest.mark.parametrize("graph", [False, True])
def test_fold_subsets(corrmod, n, graph):
    """Block-deferred groups of one, two and three fold subsets (98304 channels
    each): channels on both sides of every subset border, read out where no
    subset, one subset or every subset has folded the last block by itself and
    the readout folds the others."""
    say(f"[fold subsets] n={n} graph={graph}")
    rows, T = 40, 256
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((rows, n), generator=g, device="cuda")
    pick = sorted({0, 1, 98302, min(98304, n - 1), n - 2, n - 1})
    xs = x[:, pick].cpu().numpy().astype(np.float64)
    o = oracle.OracleCorrelator(len(pick), 5, 16, 2)
    buf = x[0].clone()
    with corrmod.Correlator([corrmod.GroupDesc(n, 5, 16, 2, dtype="f32", accum="kahan")],
                            graph=graph) as c:
        if graph:
            c.bind_input(0, buf)
        s = 0
        for stop in (T - 1, T, T + 1, T + 2, 2 * T + 1, 3 * T + 5):
            while s < stop:
                if graph:
                    buf.copy_(x[s % rows])
                    c.push()
                else:
                    c.push([x[s % rows]])
                o.push(xs[s % rows])
                s += 1
            for i, ch in enumerate(pick):
                r = c.finalize(0, slice_=(ch, ch + 1))
                _check_channels(r, o, [(0, i)], TOL[("f32", "kahan")], f"S={s} channel {ch}")


@pytest.mark.parametrize("accum", ["kahan", "f64", "f32"])
@pytest.mark.parametrize("block", [256, 128])
def test_readout_of_pending_pushes(corrmod, accum, block):
    """Readouts of a block-deferred group with 0 .. block - 1 pushes after the
    last block (both sides of every eight rows and of every chunk of 64), at
    counts where a level has its first lags (8 and 9 values) or none, over all
    channels, a channel range and a slice."""
    say(f"[pending readout] accum={accum} block={block}")
    n, levels = 197, 8
    stops = [1, 7, 8, 9, 16, 17, 63, 64, 65, 71, 72, 73, 127, 128, 129, 136, 191, 192, 193, 200,
             255, 256, 257, 264, 319, 320, 321, 383, 384, 447, 448, 511, 512, 513, 575, 576, 577]
    x = ou_inputs(31, 1, n, stops[-1], "f32")
    xt = torch.from_numpy(x).cuda()
    o = oracle.OracleCorrelator(n, levels, 16, 2)
    tuning = dict(tile_channels=256, chans_per_thread=2, lag_chunk=8, grid_blocks=0, fold_block=block)
    tol = TOL[("f32", accum)]
    with corrmod.Correlator([corrmod.GroupDesc(n, levels, 16, 2, dtype="f32", accum=accum)],
                            tuning=tuning) as c:
        s = 0
        for stop in stops:
            while s < stop:
                c.push([xt[s]])
                o.push(x[s].astype(np.float64))
                s += 1
            r = c.finalize(0, slice_=(60, 70))
            _check_channels(r, o, [(i, 60 + i) for i in range(10)], tol, f"S={s}")
            for b, e in ((0, n), (63, 130)):
                r = c.finalize(0, ch=(b, e))
                _, ref, _ = o.readout(b, e)
                err = np.max(np.abs(r["c"] - ref)) / abs(ref[0])
                assert err <= tol, f"S={s} channels [{b}, {e}): {err:.3e} > {tol:.1e}"


@pytest.mark.parametrize("source", ["rhok", "currents"])
@pytest.mark.parametrize("atoms", [127, 128, 129, 4097, 32768, 32769, 98305, 100001])
def test_producer_atom_blocks(corrmod, source, atoms):
    """Atom blocks of one 128-atom tile, of less than one, of two with a nearly
    empty second, and more blocks than compute units (small k-sets share
    them): C(0) of one push against the oracle's direct double sums, for a small
    k-set and one whose blocks need a compute unit each."""
    box = 40.0
    rng = np.random.default_rng(atoms)
    x = rng.uniform(0, box, (1, 3, atoms)).astype(np.float32)
    v = rng.standard_normal((1, 3, atoms)).astype(np.float32)
    for nk in (24, 900) if atoms < 5000 else (24,):
        say(f"[atom blocks] {source} atoms={atoms} nk={nk}")
        kv = synth.kvectors(nk)
        if source == "rhok":
            inp, ref = x, oracle.rhok(x[0], kv, box)
        else:
            inp = np.concatenate([x, v], 1)
            ref = oracle.currents(x[0], v[0], kv, box).reshape(-1)
        expect = np.abs(ref) ** 2 / atoms
        g = corrmod.GroupDesc(len(expect), 2, 4, 2, dtype="cf32", accum="f64", source=source, kvec=kv,
                              n_atoms=atoms, box=box)
        with corrmod.Correlator([g]) as c:
            c.push([torch.from_numpy(np.ascontiguousarray(inp[0])).cuda()])
            got = c.finalize(0, slice_=(0, len(expect)))["c_per_channel"][:, 0]
        err = np.max(np.abs(got - expect)) / np.max(expect)
        assert err < 2e-6, f"{source} atoms={atoms} nk={nk}: {err:.2e}"


def _same_readout(a, b, label):
    for k in ("t", "c", "count", "gk_running", "c_per_channel"):
        assert np.array_equal(a[k], b[k]), f"{label}: {k} differs"


@pytest.mark.parametrize("dtype,accum", [("f32", "kahan"), ("f32", "f64"), ("f32", "f32"), ("f64", "f64"),
                                         ("cf32", "kahan"), ("cf32", "f64"), ("cf32", "f32"), ("cf64", "f64")])
@pytest.mark.parametrize("pair", [False, True])
def test_multi_step_push(corrmod, dtype, accum, pair):
    """Waiting pushes added in passes of up to 64 against one push at a time
    (the per-group form): the same bits, for blocks of channels with and without
    a remainder, readouts at every kind of place in a pass, samples that
    are not 16-byte aligned and a caller's buffer that changes after each push;
    autocorrelations also against the oracle."""
    S, levels = 333, 7
    stops = (1, 2, 15, 31, 33, 63, 64, 65, 66, 127, 128, 192, 193, 250, 251, 333)
    for p, n in ((16, 33), (24, 64), (32, 7), (16, 100), (32, 129), (8, 40)):
        say(f"[multi-step] {dtype}/{accum} pair={pair} p={p} n={n}")
        x = ou_inputs(5 + p, 1, (2 if pair else 1) * n, S, dtype)
        xt = torch.from_numpy(x).cuda()
        cplx = np.iscomplexobj(x)
        o = oracle.OracleCorrelator(n, levels, p, 2, complex_=cplx)
        g = corrmod.GroupDesc(n, levels, p, 2, dtype=dtype, accum=accum, pair=pair)
        buf = torch.empty(xt.shape[1] + 1, dtype=xt.dtype, device="cuda")[1:]
        with corrmod.Correlator([g]) as c, corrmod.Correlator([g], per_group=True) as ref:
            s = 0
            for stop in stops:
                while s < stop:
                    buf.copy_(xt[s])
                    c.push([buf])
                    ref.push([xt[s]])
                    if not pair:
                        o.push(x[s].astype(np.complex128 if cplx else np.float64))
                    s += 1
                r = c.finalize(0, slice_=(0, n))
                if not (dtype == "f32" and p == 16 and not pair):  # (that one is block-deferred)
                    _same_readout(r, ref.finalize(0, slice_=(0, n)), f"p={p} n={n} S={s}")
                if not pair:  # (a pair's C(0) is no scale of its errors)
                    _check_channels(r, o, [(i, i) for i in (0, n // 2, n - 1)], TOL[(dtype, accum)], f"S={s}")


def test_multi_step_push_of_producers(corrmod):
    """Producers that write their waiting row, a momentum pair group and sample
    groups in one context, with the producers beside the other groups and on
    one stream: bit-identical to the per-group form."""
    N, nk, box, S = 700, 37, 30.0, 150
    kv = synth.kvectors(nk)
    rng = np.random.default_rng(4)
    pos = rng.uniform(0, box, (S, 3, N)).astype(np.float32)
    vel = rng.standard_normal((S, 3, N)).astype(np.float32)
    q = rng.standard_normal((S, 3)).astype(np.float32)
    both = np.concatenate([pos, vel], 1).reshape(S, -1)
    mom = np.concatenate([vel.reshape(S, -1), q, q], 1)
    st = rng.standard_normal((S, 9))
    inputs = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
              for a in (pos.reshape(S, -1), both, mom, st, q)]
    kw = dict(dtype="cf32", accum="kahan", kvec=kv, n_atoms=N, box=box)
    groups = [corrmod.GroupDesc(nk, 6, 32, 2, source="rhok", **kw),
              corrmod.GroupDesc(3 * nk, 6, 16, 2, source="currents", **kw),
              corrmod.GroupDesc(6, 6, 16, 2, dtype="f32", accum="kahan", source="momentum", n_atoms=N, box=box,
                                species=rng.integers(0, 2, N).astype(np.int32), masses=np.array([2.0, 3.0]),
                                pair=True),
              corrmod.GroupDesc(9, 8, 16, 2, dtype="f64", accum="f64"),
              corrmod.GroupDesc(3, 6, 16, 2, dtype="f32", accum="kahan")]
    with corrmod.Correlator(groups[:4], per_group=True) as ref:
        for s in range(S):
            ref.push([t[s] for t in inputs[:4]])
        want = [ref.finalize(i, slice_=(0, groups[i].n_channels)) for i in range(4)]
    for k in (4, 5):
        for overlap in (0, 1, 2):
            say(f"[multi-step producers] groups={k} overlap={overlap}")
            tuning = dict(tile_channels=256, chans_per_thread=2, lag_chunk=8, grid_blocks=0,
                          overlap_producers=overlap)
            with corrmod.Correlator(groups[:k], tuning=tuning) as c:
                for s in range(S):
                    c.push([t[s] for t in inputs[:k]])
                    if s in (0, 70):
                        c.finalize(1)
                for i in range(4):
                    _same_readout(c.finalize(i, slice_=(0, groups[i].n_channels)), want[i], f"group {i}")


@pytest.mark.parametrize("block", [256, 128])
@pytest.mark.parametrize("n", [1, 1021, 100003])
def test_replay_in_pieces(corrmod, block, n):
    """Histories replayed in calls of every kind of length (one push, up to a
    block boundary, across one, whole blocks, a remainder), single pushes and
    readouts in between, with rows that are and are not 16-byte aligned: the
    same bits as single pushes."""
    S = 6 * block
    say(f"[replay in pieces] n={n} block={block}")
    gen = torch.Generator(device="cuda").manual_seed(n)
    hist = torch.randn((S, n), generator=gen, device="cuda")
    small = torch.randn((S, 5), generator=gen, device="cuda", dtype=torch.float64)
    wide = torch.empty((S, n + 5), device="cuda")  # the same rows at another stride
    wide[:, :n] = hist
    d = corrmod.GroupDesc(n, 6, 16, 2, dtype="f32", accum="kahan")
    e = corrmod.GroupDesc(5, 6, 16, 2, dtype="f64", accum="f64")
    tuning = dict(tile_channels=256, chans_per_thread=2, lag_chunk=8, grid_blocks=0, fold_block=block)
    for groups, rows in (([d], [hist]), ([d], [wide[:, :n]]), ([d, e], [hist, small]), ([e], [small])):
        with corrmod.Correlator(groups, tuning=tuning) as c, corrmod.Correlator(groups, tuning=tuning) as ref:
            s = 0
            for k in (1, 63, block - 64, 1, block, 3, block + 200, block - 1, 40):
                k = min(k, S - s)
                if k == 3:
                    for j in range(s, s + k):
                        c.push([r[j] for r in rows])
                else:
                    c.push_steps([r[s:s + k] for r in rows])
                for j in range(s, s + k):
                    ref.push([r[j] for r in rows])
                s += k
                for i, g in enumerate(groups):
                    kw = dict(slice_=(max(0, g.n_channels - 3), g.n_channels))
                    if k not in (63, block - 1):  # (later folds and passes start in the middle of one)
                        _same_readout(c.finalize(i, **kw), ref.finalize(i, **kw), f"S={s} group {i}")
            assert c.n_pushes() == s


@pytest.mark.parametrize("overlap", [0, 1, 2])
@pytest.mark.parametrize("timing", [False, True])
@pytest.mark.parametrize("k", [1, 3, 5])
def test_captured_runs(corrmod, overlap, timing, k):
    """Captured runs of pushes (shorter and longer than a multi-step pass and
    than a fold block), each replayed several times with single pushes, other
    runs and readouts in between: the same bits as single pushes of the
    per-group form."""
    N, nk, box, R, n = 500, 30, 30.0, 150, 700
    say(f"[captured runs] overlap={overlap} timing={timing} groups={k}")
    kv = synth.kvectors(nk)
    gen = torch.Generator(device="cuda").manual_seed(3)
    pos = box * torch.rand((R, 3 * N), generator=gen, device="cuda")
    vel = torch.randn((R, 3 * N), generator=gen, device="cuda")
    q = torch.randn((R, 3), generator=gen, device="cuda")
    groups = [corrmod.GroupDesc(nk, 6, 32, 2, dtype="cf32", accum="kahan", source="rhok", kvec=kv, n_atoms=N, box=box),
              corrmod.GroupDesc(9, 8, 16, 2, dtype="f64", accum="f64"),
              corrmod.GroupDesc(n, 6, 16, 2, dtype="f32", accum="kahan"),
              corrmod.GroupDesc(6, 6, 16, 2, dtype="f32", accum="kahan", source="momentum", n_atoms=N, box=box,
                                species=np.arange(N, dtype=np.int32) % 2, masses=np.array([2.0, 3.0]), pair=True),
              corrmod.GroupDesc(40, 1, 600, 2, dtype="f32", accum="kahan")][:k]
    rows = [pos, torch.randn((R, 9), generator=gen, device="cuda", dtype=torch.float64),
            torch.randn((R, n), generator=gen, device="cuda"), torch.cat([vel, q, q], 1),
            torch.randn((R, 40), generator=gen, device="cuda")][:k]
    tuning = dict(tile_channels=256, chans_per_thread=2, lag_chunk=8, grid_blocks=0, overlap_producers=overlap,
                  fold_block=128)
    with corrmod.Correlator(groups, graph=True, timing=timing, tuning=tuning) as c, \
            corrmod.Correlator(groups, per_group=True, tuning=tuning) as ref:
        for b, e in ((0, 16), (0, 16), (0, 16), (3, 4), (10, 75), (10, 75), (0, 150), (0, 16), (0, 150), (5, 69)):
            c.push_steps([r[b:e] for r in rows])
            if e == 75:  # a push by itself between the runs
                c.push([r[7] for r in rows])
            for j in list(range(b, e)) + ([7] if e == 75 else []):
                ref.push([r[j] for r in rows])
            if b in (3, 10, 5) or e == 150:
                for i, g in enumerate(groups):
                    kw = dict(slice_=(0, min(g.n_channels, 40)))
                    _same_readout(c.finalize(i, **kw), ref.finalize(i, **kw), f"[{b}, {e}) group {i}")


@pytest.mark.parametrize("source", ["momentum", "rhok", "currents"])
@pytest.mark.parametrize("n,dtype", [(1, "f32"), (3, "f32"), (512, "f32"), (513, "f32"), (9, "f64"), (2049, "f64")])
def test_small_group_beside_a_producer(corrmod, source, n, dtype):
    """A small sample group whose copy the producer's final kernel carries (one
    tile of staging, a kept row of up to 16 KB; one channel more has its own
    launch): the same bits as the group by itself, the producer's as by itself."""
    N, box, S = 300, 20.0, 300
    say(f"[rider] {source} n={n} {dtype}")
    gen = torch.Generator(device="cuda").manual_seed(n)
    t = torch.float32 if dtype == "f32" else torch.float64
    flat = torch.randn((S * n + 1,), generator=gen, device="cuda", dtype=t)
    small = flat[1:].reshape(S, n)  # rows that are not 16-byte aligned
    d = corrmod.GroupDesc(n, 6, 16, 2, dtype=dtype, accum="kahan" if dtype == "f32" else "f64")
    kv = synth.kvectors(20)
    width = 6 if source == "currents" else 3
    big = box * torch.rand((S, width * N), generator=gen, device="cuda")
    if source == "momentum":
        p = corrmod.GroupDesc(6, 6, 16, 2, dtype="f32", accum="kahan", source=source, n_atoms=N, box=box,
                              species=np.arange(N, dtype=np.int32) % 2, masses=np.array([2.0, 3.0]))
    else:
        p = corrmod.GroupDesc(20 * width // 2 if source == "currents" else 20, 6, 32, 2, dtype="cf32", accum="kahan",
                              source=source, kvec=kv, n_atoms=N, box=box)
    with corrmod.Correlator([p, d]) as c, corrmod.Correlator([d]) as alone, corrmod.Correlator([p]) as prod:
        for s in range(S):
            c.push([big[s], small[s]])
            alone.push([small[s]])
            prod.push([big[s]])
            if s in (0, 70, 256, S - 1):
                kw = dict(slice_=(max(0, n - 4), n))
                _same_readout(c.finalize(1, **kw), alone.finalize(0, **kw), f"S={s + 1}")
                _same_readout(c.finalize(0, slice_=(0, 6)), prod.finalize(0, slice_=(0, 6)), f"S={s + 1} producer")


@pytest.mark.parametrize("graph", [False, True])
def test_error_left_by_the_caller(corrmod, graph):
    """A HIP call of the caller's own that failed before a push, a replay or a
    readout: the call that reports it, made again, does what it does without
    (pushes that wait, a fold subset behind at the readout, a window)."""
    say(f"[caller's error] graph={graph}")
    n, S = 98304 + 33, 270
    groups = [corrmod.GroupDesc(33, 6, 16, 2, dtype="f64", accum="f64"),
              corrmod.GroupDesc(n, 4, 16, 2, dtype="f32", accum="kahan"),
              corrmod.GroupDesc(40, 4, 8, 2, dtype="cf32", accum="kahan", pair=True),
              corrmod.GroupDesc(7, 1, 600, 2, dtype="f32", accum="f64")]
    rows = 20
    x = [torch.randn((rows, 33), device="cuda", dtype=torch.float64), torch.randn((rows, n), device="cuda"),
         torch.randn((rows, 80), device="cuda", dtype=torch.complex64), torch.randn((rows, 7), device="cuda")]

    def again(f, *a, **kw):
        assert corrmod.lib().hipSetDevice(1 << 20) != 0
        try:
            return f(*a, **kw)
        except corrmod.CorrError:
            return f(*a, **kw)
        finally:  # (a replayed graph does not look at it)
            corrmod.lib().hipGetLastError()

    with corrmod.Correlator(groups, graph=graph) as c, corrmod.Correlator(groups, graph=graph) as ref:
        for s in range(S):
            push = [t[s % rows] for t in x]
            again(c.push, push) if s % 50 in (0, 6) else c.push(push)
            ref.push(push)
            if s == 200:
                for _ in range(2):
                    again(c.push_steps, [t[3:10] for t in x])
                    ref.push_steps([t[3:10] for t in x])
            if s in (4, 70, 241, 242, S - 1):  # 14 more pushes after the replays
                for i, g in enumerate(groups):
                    kw = dict(slice_=(g.n_channels - 5, g.n_channels))
                    _same_readout(again(c.finalize, i, **kw), ref.finalize(i, **kw), f"S={s + 1} group {i}")
            assert c.n_pushes() == ref.n_pushes()


@pytest.mark.parametrize("dtype,accum,p,pair", [("f64", "f64", 16, False), ("f32", "kahan", 32, False),
                                                ("f32", "kahan", 24, True), ("cf32", "f32", 16, True)])
@pytest.mark.parametrize("graph", [False, True])
def test_single_pushes_of_large_groups(corrmod, dtype, accum, p, pair, graph):
    """Multi-step passes and per-step pushes of the same group in turn (one push
    to add takes the per-step kernel at these sizes): readouts after every kind
    of stretch, the same bits as one push at a time."""
    n = 65536 + 3 if pair else 98304 + 3
    say(f"[single pushes] {dtype}/{accum} p={p} pair={pair} graph={graph}")
    gen = torch.Generator(device="cuda").manual_seed(p)
    real = torch.float64 if dtype == "f64" else torch.float32
    x = torch.randn((66, (2 if pair else 1) * n * (2 if dtype == "cf32" else 1)), generator=gen, device="cuda", dtype=real)
    g = corrmod.GroupDesc(n, 5, p, 2, dtype=dtype, accum=accum, pair=pair)
    with corrmod.Correlator([g], graph=graph) as c, corrmod.Correlator([g], per_group=True) as ref:
        for k in (1, 2, 1, 1, 65, 1, 3, 64, 1, 1):
            c.push_steps([x[:k]])
            if not graph:  # one kept push as well
                c.push([x[65]])
            for r in list(range(k)) + ([] if graph else [65]):
                ref.push([x[r]])
            if k != 2:
                kw = dict(slice_=(n - 40, n))
                _same_readout(c.finalize(0, **kw), ref.finalize(0, **kw), f"after {k} pushes")
