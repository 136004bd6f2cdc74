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


@pytest.mark.parametrize("call", ["train", "train_batched", "pocs"])
def test_training_without_room_for_scratch(call, monkeypatch):
    """Scratch is an advantage, not a need: where the device has no room for
    it the training works in the models' own buffers, to the same bits."""
    K, M, P, cap = 5, 8, 150, 500
    print(f"[case] {call} K={K} M={M} P={P} cap={cap}", flush=True)
    inst = synth.make_instance(synth.InstanceSpec(K=K, M=M, P=P, S=8, snr_db=12, seed=6710))
    rx, sym = cuda(inst.rx_pilot), cuda(inst.sym_pilot)
    p = A.Params(sigma2=0.5, window=8, dict_cap=cap)
    # what is left of the device: the workspace of the projections, not the scratch
    room = A.library().apsm_ball_workspace_bytes(2 * M, K, cap)

    def run():
        if call == "train":
            ms = [A.train(rx, sym, p)]
        elif call == "train_batched":
            ms = A.train_batched(torch.stack([rx, rx]), torch.stack([sym, sym]), p)
        else:
            ms = [A.pocs(rx, sym, p, 2.0, 2)]
        torch.cuda.synchronize()
        return [t.clone() for m in ms for t in (m.dict, m.alpha, m.w, m.state)]

    want = run()
    alloc = A._device_bytes

    def full(nbytes, device, stream):
        if nbytes > room:
            raise torch.cuda.OutOfMemoryError("full")
        return alloc(nbytes, device, stream)

    monkeypatch.setattr(A, "_device_bytes", full)
    for x, y in zip(run(), want):
        assert torch.equal(x, y)
