"""What the Python calls allocate when no workspace is given."""
import numpy as np
import pytest

import synth
import paper_2201_05024_amd as A

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def test_ball_projection_allocates_its_own_workspace_only():
    K, M, cap = 6, 16, 2048
    print(f"[case] ball K={K} M={M} cap={cap}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=40, S=8, snr_db=12, seed=6700))
    p = A.Params(sigma2=0.5, window=8, dict_cap=cap)
    m = A.train(cuda(inst.rx_pilot), cuda(inst.sym_pilot), p)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    A.project_ball(m, 1.0, p)
    torch.cuda.synchronize()
    need = A.library().apsm_ball_workspace_bytes(2 * M, K, cap)
    assert torch.cuda.max_memory_allocated() - before <= need + 4096
