"""Detection of few vectors (one wave a tile) gives the bits of the kernel for
many, tile by tile of 16 real vectors, at the line between the two."""
import numpy as np
import pytest

import paper_2201_05024_amd as A

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M2,K,D,cap", [
    (18, 3, 33, 40), (32, 6, 200, 200), (40, 9, 64, 70), (64, 12, 65, 65), (66, 5, 1, 33), (128, 16, 130, 192),
    (32, 2, 0, 16)])
def test_small_calls(M2, K, D, cap):
    print(f"[case] M2={M2} K={K} D={D}", flush=True)
    g = torch.Generator().manual_seed(M2 * 100 + K)
    m = A.Model(M2, K, cap, "cuda", 0.25 * M2)
    m.dict.copy_(torch.randn(m.dict.shape, generator=g))
    m.alpha.copy_(0.1 * torch.randn(m.alpha.shape, generator=g))
    m.w.copy_(0.1 * torch.randn(m.w.shape, generator=g))
    m.state[0] = D
    m.pack()
    line = 6 * torch.cuda.get_device_properties(0).multi_processor_count * 8     # received vectors
    rx = torch.randn(line + 1, M2, generator=g).cuda()
    truth = torch.zeros(line + 1, K, dtype=torch.uint8, device="cuda")
    many = A.detect(m, rx, modulation="qam16", truth=truth)
    ref_soft, ref_hard = many["soft"].cpu().numpy(), many["hard"].cpu().numpy()
    for S in (1, 7, 8, 9, 130, line):
        o = A.detect(m, rx[:S].contiguous(), modulation="qam16", truth=truth[:S].contiguous())
        whole = S - S % 8                     # a tile's scale is that of all its vectors
        np.testing.assert_array_equal(o["soft"].cpu().numpy()[:whole], ref_soft[:whole])
        hard = o["hard"].cpu().numpy()
        np.testing.assert_array_equal(hard[:whole], ref_hard[:whole])
        np.testing.assert_array_equal(o["errors"].cpu().numpy(), (hard != 0).sum(axis=0))
