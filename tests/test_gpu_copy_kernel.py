"""The CU copy kernel's launches: what the statistics report of them."""
import pytest
import torch

import paper_2609_34334_amd as hc

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _fresh_config():
    saved = hc.get_config()
    yield
    hc.set_config(**saved)


@pytest.mark.parametrize("nbytes, budget", [(100, 0), (1 << 20, 0), ((64 << 20) + 5, 0), (1 << 20, 3)])
def test_statistics_hold_the_workgroups_launched(nbytes, budget):
    """A message of one tile takes one workgroup and one CU at most, a large
    one as many as it has tiles (of at least one 16-byte vector per thread)
    and every CU; a budget is what is launched."""
    hc.set_config(copy_path="kernel", workgroups_per_step=budget)
    x = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    hc.sendrecv([x, x], [None, torch.empty_like(x)], [1, -1])
    torch.cuda.synchronize()
    s = hc.last_stats()
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    most = -(-nbytes // (256 * 16))
    assert s["copy_kernel_launches"] == 1
    if budget:
        assert s["workgroups_per_step"] == budget and s["cus_used_max"] == budget
    else:
        assert 1 <= s["workgroups_per_step"] <= most, s
        assert s["cus_used_max"] == min(s["workgroups_per_step"], ncu)
    if nbytes > 64 << 20:
        assert s["cus_used_max"] == ncu
