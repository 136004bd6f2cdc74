"""Training in blocks whose scratch holds a few blocks at a time: the ranges
of blocks follow one another in launches, with the lanes' state carried."""
import ctypes

import numpy as np
import pytest

import oracle as O
import synth
import paper_2201_05024_amd as A
from parity_util import REL_TOL, compare_soft, oracle_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def scratch_bytes(p, M2, K, P):
    cp, keep = p._c()
    return A.library().apsm_train_scratch_bytes(ctypes.byref(cp), M2, K, P, 1)


def c_train(rx, sym, p, m, scratch=None):
    """apsm_train_scratch on the current stream."""
    cp, keep = p._c()
    P, K = sym.shape[0], sym.shape[1]
    rc = A.library().apsm_train_scratch(ctypes.byref(cp), rx.shape[1], K, P, 1, rx.data_ptr(), sym.data_ptr(),
                                        ctypes.byref(m._c()), scratch.data_ptr() if scratch is not None else None,
                                        scratch.numel() if scratch is not None else 0,
                                        torch.cuda.current_stream().cuda_stream)
    assert rc == 0


def arrays(m):
    torch.cuda.synchronize()
    return [t.cpu().numpy().copy() for t in (m.dict, m.alpha, m.w, m.state)]


# several groups of users (K > 4), several ranges that are neither first nor last
@pytest.mark.parametrize("K,M,P,W,cap", [(5, 8, 200, 20, 128), (16, 64, 160, 32, 160), (9, 20, 170, 33, 400)])
def test_ranges_of_a_busy_gpu(K, M, P, W, cap):
    """The user groups of a launch start and end in any order: with detections
    on a second stream the model is the same as on an idle GPU, bit for bit."""
    print(f"[case] K={K} M={M} P={P} W={W} cap={cap}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=P, S=64, snr_db=12, seed=6100 + K))
    rx, sym, data = cuda(inst.rx_pilot), cuda(inst.sym_pilot), cuda(inst.rx_data)
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap)
    scratch = torch.empty(scratch_bytes(p, 2 * M, K, P) // 5, dtype=torch.uint8, device=DEV)
    idle = A.Model(2 * M, K, cap, DEV, 0.5)
    c_train(rx, sym, p, idle, scratch)
    want = arrays(idle)
    ref = O.detect_planar(O.train_from_pilots(inst.rx_pilot, inst.sym_pilot, oracle_params(p)), inst.rx_data)
    worst, _ = compare_soft(A.detect(idle, data)["soft"].cpu().numpy(), ref, "qpsk")
    print(f"[result] max scaled error {worst:.2e}", flush=True)
    assert worst <= REL_TOL
    other = A.train(rx, sym, p)
    many = data.repeat(1 << 11, 1).contiguous()
    soft = torch.empty((many.shape[0], K, 2), device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    busy = A.Model(2 * M, K, cap, DEV, 0.5)
    for _ in range(4):
        A.detect(other, many, modulation=None, soft=soft, stream=side)
    c_train(rx, sym, p, busy, scratch)
    for x, y in zip(arrays(busy), want):
        np.testing.assert_array_equal(x, y)
