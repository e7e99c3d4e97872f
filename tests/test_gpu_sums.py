"""What lies before a workgroup's tile or group, summed by the workgroup itself up to 1024 of them (four to a lane) and by a
kernel of its own beyond, against the CPU oracle."""
import numpy as np
import pytest

import paper_2111_09219_amd as J
from oracle import OracleImage, unstuff_bytes
from workloads import encode_jpeg, small_image

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [257 * 4096 + 5, 512 * 4096, 1024 * 4096 - 1, 1024 * 4096, 1024 * 4096 + 1])
def test_unstuffing_around_the_tiles_that_are_summed(n):
    import torch
    rng = np.random.default_rng(n)
    raw = rng.integers(0, 255, n, dtype=np.uint8)                     # no 0xFF
    at = np.flatnonzero(rng.random(n - 1) < 0.01)[::2]
    at = at[np.concatenate([[True], np.diff(at) > 1])]
    raw[at] = 255
    raw[at + 1] = 0
    want = unstuff_bytes(raw)
    d_in = torch.zeros((n + 15) // 16 * 16, dtype=torch.uint8)
    d_in[:n] = torch.from_numpy(raw)
    d_out = torch.full((n + 512,), 0xAA, dtype=torch.uint8, device="cuda")
    ws = torch.empty(4096 + 4 * (n // 4096 + 2), dtype=torch.uint8, device="cuda")
    k = J.jpgd_unstuff(d_in.cuda()[:n], d_out, ws)
    assert k == want.size and np.array_equal(d_out.cpu().numpy()[:k], want)


@pytest.mark.parametrize("h,ri,summed", [(500, 0, True), (560, 0, True), (1100, 100, True), (1700, 40, True), (1960, 0, True),
                                         (2200, 0, False), (2200, 225, False)])
def test_decoding_around_the_groups_that_are_summed(h, ri, summed):
    """128-bit subsequences: a group is as long as an unstuff tile.  With and without restart intervals, where the sums start
    anew; twice on a workspace that holds something else."""
    data = encode_jpeg(small_image(h, h, 1800, ncomp=1, sigma=60.0), 98, "gray", restart_interval=ri).data
    o = OracleImage(data)
    want = o.coefficients()
    batch = J.prepare_batch([data], J.Config.make(subseq_bits=128))
    for _ in range(2):
        batch.d_workspace.fill_(0xA5)
        launches = batch.decode().as_dict()["launches"]
        assert np.array_equal(batch.coefficients(0).cpu().numpy(), want)
        assert (launches["unstuff_scan"] == 0) == (launches["scan_prefix"] == 0) == summed
