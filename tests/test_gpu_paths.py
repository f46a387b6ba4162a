"""GPU parity at the edges of the library's dispatch rules: the sizes at which
a launch takes another kernel, another split or another schedule, against the
FP64 oracle fed the same samples."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_helpers import TOL, say

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
