"""Training in blocks of 32 steps: the edges of its rule (window 33, capacity
96) and of its blocks, against the FP64 oracle and between the ways it is
called: one block of pilots and a continued one, with a large, a small and no
scratch buffer, and in a batch."""
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


def model_bytes(m, rx):
    """The model and what its packed form detects (the form's padding is not
    defined)."""
    soft = A.detect(m, rx)["soft"]
    torch.cuda.synchronize()
    return [t.cpu().numpy().copy() for t in (m.dict, m.alpha, m.w, m.state, soft)]


def c_train(rx, sym, p, m, scratch=None):
    cp, keep = p._c()
    P, K = sym.shape[0], sym.shape[1]
    rc = A.library().apsm_train_scratch(ctypes.byref(cp), rx.shape[1], K, P, 1, rx.data_ptr(), sym.data_ptr(),
                                        ctypes.byref(m._c()), scratch.data_ptr() if scratch is not None else None,
                                        scratch.numel() if scratch is not None else 0,
                                        torch.cuda.current_stream().cuda_stream)
    del keep
    assert rc == 0


CASES = [
    # K, M, P, W, cap: one partial block, whole blocks, remainders; windows of
    # two and three lane rows; the capacity rule's edge; user groups of 1..4
    (1, 1, 3, 1, 96),
    (4, 8, 16, 16, 96),
    (5, 11, 60, 17, 97),
    (2, 20, 48, 18, 95),
    (9, 8, 100, 33, 96),
    (3, 8, 100, 34, 96),
    (16, 64, 81, 32, 128),
    (7, 33, 150, 32, 1000),
]


@pytest.mark.parametrize("K,M,P,W,cap", CASES)
def test_block_edges(K, M, P, W, cap):
    print(f"[case] K={K} M={M} P={P} W={W} cap={cap}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=2 * P, S=40, snr_db=12, seed=4000 + K * 31 + W))
    rx, sym, data = cuda(inst.rx_pilot), cuda(inst.sym_pilot), cuda(inst.rx_data)
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap,
                 pos_weights=list(np.linspace(1.0, 0.5, W)))
    m = A.train(rx[:P].contiguous(), sym[:P].contiguous(), p)
    # the rest of the pilots as a continued training
    q = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap, init="continue", pos_weights=p.pos_weights)
    first = model_bytes(m, data)
    A.train(rx[P:].contiguous(), sym[P:].contiguous(), q, model=m)
    o = A.detect(m, data)
    torch.cuda.synchronize()
    R, B = O.training_sequence(synth.planar_to_complex(inst.rx_pilot), synth.pair_to_complex(inst.sym_pilot))
    op = oracle_params(p)
    f = O.Trainer(R[:2 * P], B[:2 * P], op)
    for _ in range(2 * P):
        f.step()
    g = O.Trainer(R[2 * P:], B[2 * P:], op, f0=f.f, n0=2 * P)
    for _ in range(2 * P):
        g.step()
    worst, _ = compare_soft(o["soft"].cpu().numpy(), O.detect_planar(g.f, inst.rx_data), "qpsk")
    print(f"[result] max scaled error {worst:.2e}", flush=True)
    assert worst <= REL_TOL
    # no scratch (the room of the packed form: in chunks or, too little, step by step), and room for some blocks
    ref = O.detect_planar(f.f, inst.rx_data)
    worst, _ = compare_soft(first[-1], ref, "qpsk")
    assert worst <= REL_TOL
    for size in (None, 1 << 20):
        b = A.Model(2 * M, K, cap, DEV, 0.5)
        c_train(rx[:P].contiguous(), sym[:P].contiguous(), p, b,
                None if size is None else torch.empty(size, dtype=torch.uint8, device=DEV))
        again = model_bytes(b, data)
        worst, _ = compare_soft(again[-1], ref, "qpsk")
        print(f"[result] scratch {size}: max scaled error {worst:.2e}", flush=True)
        assert worst <= REL_TOL
        np.testing.assert_array_equal(again[0], first[0])
        np.testing.assert_array_equal(again[3], first[3])
    # a batch of one: the same bits, the model's arrays left alone until it trains
    b = A.Model(2 * M, K, cap, DEV, 0.5)
    for t in (b.dict, b.alpha, b.w, b.packed):
        t.fill_(7)
    b.state.copy_(torch.tensor([1, 2, 3, 4], dtype=torch.int32))
    before = [t.clone() for t in (b.dict, b.alpha, b.w, b.packed, b.state[:3])]
    batch = A.Batch(p, [A.BatchItem(model=b, rx_pilot=rx[:P].contiguous(), sym_pilot=sym[:P].contiguous(), sigma2=0.5)])
    batch.kernel_rows()
    for x, y in zip(before, (b.dict, b.alpha, b.w, b.packed, b.state[:3])):
        assert torch.equal(x, y)
    batch.train_prepared()
    if W <= 33 and cap >= 96:
        for x, y in zip(first, model_bytes(b, data)):
            np.testing.assert_array_equal(x, y)
