"""Trainings of one pilot, at the edges of the rule that runs their two steps
one by one."""
import numpy as np
import pytest

import oracle as O
import synth
import paper_2201_05024_amd as A
from parity_util import REL_TOL, compare_soft, oracle_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("K,M,cap,W", [(3, 8, 96, 1), (5, 8, 100, 33), (8, 16, 1024, 32), (8, 16, 1025, 32),
                                       (9, 16, 100, 32), (2, 17, 96, 8)])
def test_pilots_one_at_a_time(K, M, cap, W):
    """A pilot from zero, then continued pilot by pilot past the capacity
    where that is small."""
    n = 60 if cap < 128 else 8
    print(f"[case] K={K} M={M} cap={cap} W={W} pilots={n}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=n, S=40, snr_db=12, seed=6800 + K + cap))
    kw = dict(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap)
    zero, go_on = A.Params(**kw), A.Params(**kw, init="continue")
    rx, sym = cuda(inst.rx_pilot), cuda(inst.sym_pilot)
    m, f = None, None
    for i in range(n):
        m = A.train(rx[i:i + 1], sym[i:i + 1], go_on if i else zero, model=m)
        f = O.train_from_pilots(inst.rx_pilot[i:i + 1], inst.sym_pilot[i:i + 1], oracle_params(zero), f0=f, n0=2 * i)
    soft = A.detect(m, cuda(inst.rx_data))["soft"].cpu().numpy()
    worst, _ = compare_soft(soft, O.detect_planar(f, inst.rx_data), "qpsk")
    print(f"[result] max scaled error {worst:.2e}", flush=True)
    assert worst <= REL_TOL
    assert m.status() == {"size": min(2 * n, cap), "head": 2 * n % cap, "steps": 2 * n, "flags": 0}


def test_noalloc_is_a_batch_of_one():
    print("[case] one pilot without allocations", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=4, M=8, P=1, S=4, snr_db=12, seed=6810))
    rx, sym = cuda(inst.rx_pilot), cuda(inst.sym_pilot)
    p = A.Params(sigma2=0.5, window=16, dict_cap=256)
    a, b = A.Model(16, 4, 256, "cuda", 0.5), A.Model(16, 4, 256, "cuda", 0.5)
    A.train_noalloc(rx, sym, p, a)
    A.Batch(p, [A.BatchItem(model=b, rx_pilot=rx, sym_pilot=sym)]).train()
    torch.cuda.synchronize()
    for x, y in zip((a.dict, a.alpha, a.w, a.state), (b.dict, b.alpha, b.w, b.state)):
        assert torch.equal(x, y)
