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


# remainders of blocks, windows of one and two rows of lanes and of 33, an
# eviction in every block and none, set kinds and every choice of weights
RANGES = [
    # K, M, P, W, cap, init, weights, extrapolate, kinds
    (5, 8, 210, 16, 128, "zero", "position", False, False),
    (16, 64, 100, 32, 2000, "linear", "position", False, False),
    (3, 20, 130, 33, 97, "continue", "position", False, False),
    (6, 11, 150, 17, 128, "zero", "violation", False, True),
    (5, 8, 150, 32, 120, "zero", "active", True, True),
    (2, 16, 130, 33, 500, "zero", "violation", True, False),
    (9, 8, 140, 33, 128, "zero", "position", True, True),
    (4, 8, 140, 33, 100, "continue", "active", False, True),
]


@pytest.mark.parametrize("K,M,P,W,cap,init,weights,extrapolate,kinds", RANGES)
def test_the_same_bits_whatever_the_scratch(K, M, P, W, cap, init, weights, extrapolate, kinds):
    """One range of all blocks, several of a few and one block at a time give
    the same model, as does scratch that is too small for a block."""
    print(f"[case] K={K} M={M} P={P} W={W} cap={cap} {init} {weights} ex={extrapolate} kinds={kinds}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=2 * P, S=64, snr_db=12, seed=6300 + K + W))
    st = np.random.default_rng(6300 + K).integers(0, 4, (2 * P, K, 2)).astype(np.uint8) if kinds else None
    common = dict(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap, weights=weights, extrapolate=extrapolate)
    part = lambda x, lo, hi: cuda(x[lo:hi])  # noqa: E731
    q = A.Params(**common, init="zero", set_types=part(st, 0, P) if kinds else None)
    first = A.train(part(inst.rx_pilot, 0, P), part(inst.sym_pilot, 0, P), q)
    p = A.Params(**common, init=init, set_types=part(st, P, 2 * P) if kinds else None)
    rx, sym = part(inst.rx_pilot, P, 2 * P), part(inst.sym_pilot, P, 2 * P)
    whole = scratch_bytes(p, 2 * M, K, P)
    # an even share and room for what is kept per user: a block, not two
    one = whole // ((2 * P + 31) // 32) + 4 * K * (256 + 2 * M) + 1024
    want = None
    for size in (whole, whole // 2, whole // 4, one, 1000, 0):
        m = A.Model(2 * M, K, cap, DEV, 0.5)
        for a, b in ((m.dict, first.dict), (m.alpha, first.alpha), (m.w, first.w), (m.state, first.state)):
            a.copy_(b)
        m.pack()
        # (what is too small for a block leaves the room of the packed form,
        # which holds one from some 200 entries on)
        c_train(rx, sym, p, m, torch.empty(size, dtype=torch.uint8, device=DEV) if size else None)
        got = arrays(m)
        if want is None:
            want = got
            f = O.train_from_pilots(inst.rx_pilot[:P], inst.sym_pilot[:P], oracle_of(p), set_types=st[:P] if kinds else None)
            f0 = f if init == "continue" else linear_part(f) if init == "linear" else None
            g = O.train_from_pilots(inst.rx_pilot[P:], inst.sym_pilot[P:], oracle_of(p), f0=f0,
                                    n0=2 * P if init == "continue" else 0, set_types=st[P:] if kinds else None)
            assert m.status()["flags"] == 0
            worst, _ = compare_soft(A.detect(m, cuda(inst.rx_data))["soft"].cpu().numpy(),
                                    O.detect_planar(g, inst.rx_data), "qpsk")
            print(f"[result] max scaled error {worst:.2e}", flush=True)
            assert worst <= REL_TOL
        elif size >= one or cap >= 500:
            print(f"[result] scratch {size} of {whole}", flush=True)
            for x, y in zip(got, want):
                np.testing.assert_array_equal(x, y)


def oracle_of(p):
    q = oracle_params(p)
    q.weight_mode, q.extrapolate = p.weights, p.extrapolate
    return q


def linear_part(f):
    g = O.Filter(f.K, f.M2, f.sigma2)
    g.w = f.w.copy()
    return g


def test_noalloc_in_two_ranges_is_a_batch_of_one():
    """The largest trainings that the static array admits take two ranges of
    blocks, where a batch takes one."""
    K, M, P, W, cap = 5, 8, 7900, 32, 1024
    print(f"[case] noalloc K={K} M={M} P={P} W={W} cap={cap}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=P, S=16, snr_db=12, seed=6350))
    rx, sym = cuda(inst.rx_pilot), cuda(inst.sym_pilot)
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap)
    assert scratch_bytes(p, 2 * M, K, P) > 64 << 20
    a, b = A.Model(2 * M, K, cap, DEV, 0.5), A.Model(2 * M, K, cap, DEV, 0.5)
    A.train_noalloc(rx, sym, p, a)
    A.Batch(p, [A.BatchItem(model=b, rx_pilot=rx, sym_pilot=sym)]).train()
    for x, y in zip(arrays(a), arrays(b)):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("cap", [96, 300])
@pytest.mark.parametrize("seen", [0, 40])
def test_unused_slots_are_not_read(cap, seen):
    """A continued training does not read the slots that the model has not
    used yet, and leaves them zero."""
    print(f"[case] cap={cap} seen={seen}", flush=True)
    K, M, W = 5, 8, 8
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=70, S=16, snr_db=12, seed=6400 + cap))
    rx, sym = cuda(inst.rx_pilot), cuda(inst.sym_pilot)
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap)
    q = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap, init="continue")
    models = []
    for fill in (0.0, float("nan")):
        m = A.Model(2 * M, K, cap, DEV, 0.5)
        if seen:
            A.train(rx[:seen // 2].contiguous(), sym[:seen // 2].contiguous(), p, model=m)
        m.alpha[seen:] = fill
        m.dict[:, seen:] = fill
        A.train(rx[20:30].contiguous(), sym[20:30].contiguous(), q, model=m)
        models.append(arrays(m))
        A.train(rx[30:].contiguous(), sym[30:].contiguous(), q, model=m)
        models.append(arrays(m))
    for a, b in zip(models[0] + models[1], models[2] + models[3]):
        np.testing.assert_array_equal(a, b)
