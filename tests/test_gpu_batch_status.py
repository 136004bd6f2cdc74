"""The flags word of batched training: training overwrites it with its own
flags, whatever was raised since its kernel values were computed."""
import numpy as np
import pytest

import synth
import paper_2201_05024_amd as A

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# the capacities take the two forms of training (in blocks, from kernel rows)
@pytest.mark.parametrize("K,M,cap", [(4, 8, 128), (9, 20, 200), (4, 8, 90)])
def test_training_overwrites_the_flags(K, M, cap):
    print(f"[case] K={K} M={M} cap={cap}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=60, S=40, snr_db=12, seed=6200 + cap))
    m = A.Model(2 * M, K, cap, "cuda", 0.5)
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=8, dict_cap=cap)
    batch = A.Batch(p, [A.BatchItem(model=m, rx_pilot=cuda(inst.rx_pilot), sym_pilot=cuda(inst.sym_pilot))])
    batch.train()
    rx = inst.rx_data.copy()
    rx[3, 1] = np.nan
    # raised by a detection between the two parts of a training
    batch.kernel_rows()
    A.detect(m, cuda(rx))
    assert m.status()["flags"] == A.FLAG_DETECT_NONFINITE
    batch.train_prepared()
    assert m.status()["flags"] == 0
    # a training repeated from the same kernel values
    m.state[3] = A.FLAG_TRAIN_NONFINITE
    batch.train_prepared()
    assert m.status()["flags"] == 0


def test_kernel_values_leave_the_flags():
    """Beside a detection with the model that the training will replace."""
    print("[case] flags raised before the kernel values", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=4, M=8, P=60, S=40, snr_db=12, seed=6210))
    m = A.Model(16, 4, 128, "cuda", 0.5)
    p = A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=8, dict_cap=128)
    batch = A.Batch(p, [A.BatchItem(model=m, rx_pilot=cuda(inst.rx_pilot), sym_pilot=cuda(inst.sym_pilot))])
    batch.train()
    m.state[3] = A.FLAG_DETECT_NONFINITE
    batch.kernel_rows()
    assert m.status()["flags"] == A.FLAG_DETECT_NONFINITE
