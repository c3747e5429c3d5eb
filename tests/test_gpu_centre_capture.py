"""The centre of centred parameters under capture: host values are refused
(a graph would copy from memory that is gone at its replay), a device tensor
is captured, and outside a capture both give the same matrices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_centre_under_capture():
    import torch
    from paper_1909_10690_amd.autograd import centred_matrices
    rng = np.random.default_rng(3)
    params = torch.from_numpy(rng.normal(size=(4, 12))).cuda()
    centre = (31.5, -7.25, 12.0)
    on_device = torch.tensor(centre, dtype=torch.float64, device="cuda")
    want = centred_matrices(params, on_device)
    for host in (centre, list(centre), np.asarray(centre)):
        assert torch.equal(centred_matrices(params, host), want)
    torch.cuda.synchronize()
    graph, refused = torch.cuda.CUDAGraph(), []
    with torch.cuda.graph(graph):
        out = centred_matrices(params, on_device)
        for host in (centre, np.asarray(centre)):
            try:
                centred_matrices(params, host)
            except RuntimeError as e:
                refused.append(str(e))
    assert len(refused) == 2 and all("device tensor" in r for r in refused)
    for _ in range(3):
        params.add_(1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.allclose(out, centred_matrices(params, centre), rtol=1e-13, atol=1e-12)
