"""Non-finite targets and received vectors in training: a sample acts from its
own step on, so the steps before it give what they give without it, in both
forms of training, and the flag is raised."""
import ctypes

import numpy as np
import pytest

import synth
import paper_2201_05024_amd as A
from parity_util import REL_TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"
K, M, P, CAP = 9, 4, 60, 96


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def train(rx, sym, p, blocks):
    """In blocks with scratch, step by step without: the packed form of this
    shape is smaller than a block."""
    m = A.Model(2 * M, K, CAP, DEV, 0.5)
    cp, keep = p._c()
    ws = torch.empty(A.library().apsm_train_scratch_bytes(ctypes.byref(cp), 2 * M, K, P, 1), dtype=torch.uint8,
                     device=DEV) if blocks else None
    rc = A.library().apsm_train_scratch(ctypes.byref(cp), 2 * M, K, rx.shape[0], 1, rx.data_ptr(), sym.data_ptr(),
                                        ctypes.byref(m._c()), ws.data_ptr() if blocks else None,
                                        ws.numel() if blocks else 0, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    return m.alpha.cpu().numpy(), m.w.cpu().numpy(), m.status()["flags"]


def same(a, b):
    """Equal up to rounding where finite, not finite at the same places."""
    np.testing.assert_array_equal(np.isfinite(a), np.isfinite(b))
    f = np.isfinite(a)
    assert np.abs(a[f] - b[f]).max() <= REL_TOL * max(np.abs(a[f]).max(), 1e-3)


# what the sample is, the set it has (0 slab, 1 plane, 2 upper, 3 lower), the
# step it comes at: in each half of a block, the first and the last of one
BAD = [("inf", 0), ("-inf", 0), ("nan", 0), ("inf", 2), ("-inf", 2), ("inf", 3), ("nan", 1), ("vector", 0),
       ("vector_inf", 0)]


@pytest.mark.parametrize("W,weights,extrapolate", [
    (1, "position", False), (16, "position", False), (20, "violation", False), (32, "position", False),
    (33, "position", False), (33, "active", False), (17, "violation", True), (32, "position", True)])
@pytest.mark.parametrize("what,kind", BAD)
def test_nonfinite_samples(what, kind, W, weights, extrapolate):
    print(f"[case] {what} kind={kind} W={W} {weights} ex={extrapolate}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=P, S=8, snr_db=12, seed=6500))
    for n in (32, 45, 63, 82):
        rx, sym = inst.rx_pilot.copy(), inst.sym_pilot.copy()
        st = np.zeros((P, K, 2), np.uint8)
        if what.startswith("vector"):
            rx[n // 2, 3] = np.inf if what == "vector_inf" else np.nan
        else:
            sym[n // 2, 2, n % 2] = float(what)
            st[n // 2, 2, n % 2] = kind
        p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=CAP, weights=weights,
                     extrapolate=extrapolate, set_types=cuda(st) if kind else None)
        steps = train(cuda(rx), cuda(sym), p, False)
        blocks = train(cuda(rx), cuda(sym), p, True)
        assert blocks[2] == steps[2] == A.FLAG_TRAIN_NONFINITE
        same(steps[0], blocks[0])
        same(steps[1], blocks[1])
