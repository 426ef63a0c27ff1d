"""Classification without a network, a record per thread: the bits of the
network kernel's box cuts for records outside the trained range, at the edges
of a workgroup, records that are no image among them."""
import pytest

import paper_1307_6489_amd as rta
from test_gpu_event_pass import make, network
from test_gpu_parity import torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 20000])
def test_equals_the_network_kernels_box_cuts(torch_dev, n):
    import torch
    m, bc = network()
    for k in range(10):
        bc.feat_lo[k], bc.feat_hi[k] = 1e30, 2e30  # nothing in range
    d = make(torch_dev, 600)[3][:n].clone()
    assert d.shape[0] == n
    d[::7, 0], d[3::11, 0], d[5::13, 3], d[2::17, 4] = 0.0, float("inf"), float("nan"), -1.0
    net, box = rta.classify(m, bc, d), rta.classify(None, bc, d)
    assert bool((net[:, 3] == 1).all())
    assert torch.equal(box.view(torch.int32), net.view(torch.int32))
