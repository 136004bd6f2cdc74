"""Windows of 34 to 64 samples, which train step by step: the choices of start,
weights, relaxation and set kinds on each form of that kernel (dictionary in
registers, coefficients in LDS, both in the model buffers, kernel rows of a
batch), against the FP64 oracle."""
import numpy as np
import pytest

import oracle as O
import synth
import paper_2201_05024_amd as A
from test_gpu_extensions import check_detect, check_model, cuda, opar

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FORMS = {
    # K, M, P, cap, W
    "register_slots": (4, 8, 150, 256, 40),
    "lds_coefficients": (6, 16, 570, 1100, 34),
    "model_buffers": (16, 64, 120, 2200, 64),
    "rows_batch": (6, 16, 230, 400, 40),
}
CHOICES = [
    # weights, extrapolate, kinds, start
    ("position", False, False, "linear"),
    ("position", True, True, "zero"),
    ("violation", False, True, "continue"),
    ("violation", True, False, "zero"),
    ("active", False, False, "continue"),
    ("active", True, True, "linear"),
]


# Active-set weights jump where a member's distance crosses 1e-5.  Without the
# extrapolated relaxation members come to lie there: these instances are ones
# whose oracle coefficients move by less than 3e-5 of the largest when the
# pilots move by 2e-6 (others' by up to 1e-3).
SMOOTH = {"register_slots": 1, "lds_coefficients": 22, "model_buffers": 5}


def linear_part(f):
    g = O.Filter(f.K, f.M2, f.sigma2)
    g.w = f.w.copy()
    return g


@pytest.mark.parametrize("weights,extrapolate,kinds,start", CHOICES)
@pytest.mark.parametrize("form", FORMS)
def test_wide_windows(form, weights, extrapolate, kinds, start):
    K, M, P, cap, W = FORMS[form]
    batch = form == "rows_batch"
    if batch:                               # hyperslabs from zero or a linear part
        kinds, start = False, "linear" if start == "continue" else start
    print(f"[case] {form} W={W} {weights} ex={extrapolate} kinds={kinds} {start}", flush=True)
    first = 20 if start != "zero" else 0    # pilots of the model that is gone on from
    seed = 6900 + K + W + (1000 * SMOOTH.get(form, 0) if weights == "active" and not extrapolate else 0)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=first + P, S=100, snr_db=10.0, seed=seed))
    st = np.random.default_rng(6900 + K).integers(0, 4, (P, K, 2)).astype(np.uint8) if kinds else None
    base = dict(sigma2=0.5, eps=0.05, mu=1.0, window=W, dict_cap=cap)
    m, f0 = A.Model(2 * M, K, cap, "cuda", 0.5), None
    if first:
        A.train(cuda(inst.rx_pilot[:first]), cuda(inst.sym_pilot[:first]), A.Params(**base), model=m)
        f0 = O.train_from_pilots(inst.rx_pilot[:first], inst.sym_pilot[:first], opar(A.Params(**base)))
    p = A.Params(**base, weights=weights, extrapolate=extrapolate, init=start,
                 set_types=cuda(st) if kinds else None)
    rx, sym = cuda(inst.rx_pilot[first:]), cuda(inst.sym_pilot[first:])
    if batch:
        A.Batch(p, [A.BatchItem(model=m, rx_pilot=rx, sym_pilot=sym)]).train()
    else:
        A.train(rx, sym, p, model=m)
    torch.cuda.synchronize()
    assert m.status()["flags"] == 0
    f = O.train_from_pilots(inst.rx_pilot[first:], inst.sym_pilot[first:],
                            opar(p, weight_mode=weights, extrapolate=extrapolate),
                            f0=linear_part(f0) if start == "linear" else f0,
                            n0=2 * first if start == "continue" else 0, set_types=st)
    check_model(m, f, cap, form)
    check_detect(m, f, inst.rx_data, "qpsk", form)
