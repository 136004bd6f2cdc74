"""Batches with capacities past 8,192: a bounded workspace, the same models as
one detector at a time."""
import ctypes

import numpy as np
import pytest

import synth
import paper_2201_05024_amd as A
from test_abi import _fresh_model, _item, _params, needs_lib

torch = pytest.importorskip("torch")


@needs_lib
@pytest.mark.parametrize("n,P,cap", [(1, 100000, 65536), (40, 30000, 16384), (3, 700, 8193)])
def test_workspace_is_bounded(n, P, cap):
    L = A.library()
    one = _item(model=_fresh_model(M2=32, K=4, cap=cap), P=P, S=0)
    arr = (A._CBatchItem * n)()
    size = {"dict": 32 * cap * 4, "alpha": cap * 16, "w": 32 * 16, "state": 16,
            "packed": L.apsm_model_packed_bytes(32, 4, cap)}
    at = 1 << 40
    for c in arr:                           # arrays of their own
        ctypes.memmove(ctypes.byref(c), ctypes.byref(one), ctypes.sizeof(c))
        for f, b in size.items():
            setattr(c.model, f, at)
            at += (b + 255) // 256 * 256
    p, h = _params(), ctypes.c_void_p()
    assert L.apsm_batch_create(ctypes.byref(p), arr, n, ctypes.byref(h)) == 0
    try:
        block = 128 * cap + (64 << 10)      # of 32 steps
        assert L.apsm_batch_workspace_bytes(h) <= max(1 << 30, n * block) + (16 << 20)
    finally:
        L.apsm_batch_destroy(h)


@pytest.mark.gpu
def test_rounds_train_what_one_detector_trains():
    """Five detectors of two shapes whose blocks do not fit the bound at once,
    beside one that is prepared apart."""
    def cuda(x):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda()
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=16, dict_cap=1)
    items, want = [], []
    for i, (K, M, P, cap) in enumerate([(5, 4, 4096, 8193), (2, 4, 4000, 9000), (1, 2, 50, 100), (2, 4, 4100, 8300),
                                        (5, 4, 4096, 8193), (3, 2, 4300, 8500)]):
        print(f"[case] detector {i}: K={K} M={M} P={P} cap={cap}", flush=True)
        inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=P, S=8, snr_db=12, seed=6600 + i))
        rx, sym = cuda(inst.rx_pilot), cuda(inst.sym_pilot)
        m = A.Model(2 * M, K, cap, "cuda", 0.5)
        items.append(A.BatchItem(model=m, rx_pilot=rx, sym_pilot=sym, sigma2=0.5))
        want.append(A.train(rx, sym, A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=16, dict_cap=cap)))
    batch = A.Batch(p, items)
    assert batch.workspace.numel() <= (1 << 30) + (16 << 20)
    for _ in range(2):                      # a second training from the same workspace
        batch.train()
        torch.cuda.synchronize()
        for it, m in zip(items, want):
            for x, y in zip((it.model.dict, it.model.alpha, it.model.w, it.model.state),
                            (m.dict, m.alpha, m.w, m.state)):
                assert torch.equal(x, y)
