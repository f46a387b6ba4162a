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
