"""Who clears the coefficients: the synchronisation kernels ahead of the write pass (calls of up to 320 MB of them), a kernel of
its own in front of a repeated write pass, the write pass's workgroups each their own stretch (beyond 320 MB), or nobody
where they are gathered in LDS (up to 128 workgroups of subsequences of up to 256 bits).  Always into buffers full of stale
values, against the encoder's coefficients."""
import numpy as np
import pytest

import paper_2111_09219_amd as J
from workloads import encode_jpeg, small_image

pytestmark = pytest.mark.gpu

CLEAR_AHEAD = 320 << 20


def _halves(h, w, ri=0):
    """Left half flat, right half noise: data units of a few bits beside units with a value in nearly every slot."""
    px = np.full((h, w, 3), 128, np.uint8)
    px[:, w // 2:] = np.random.default_rng(h).integers(0, 256, size=(h, w - w // 2, 3), dtype=np.uint8)
    return encode_jpeg(px, 92, "420", restart_interval=ri)


@pytest.mark.parametrize("sub,ri,L,overlap", [("420", 0, 128, None), ("444", 0, 128, 191), ("420", 0, 512, 191), ("420", 300, 128, None),
                                              ("420", 100, 256, 191)])
def test_a_repeated_write_pass_finds_cleared_coefficients(sub, ri, L, overlap):
    """Several inter-sequence rounds, so that the write pass has run once from states that were not settled and left what it
    made of them."""
    enc = encode_jpeg(small_image(16352, 620, 480, sigma=80.0), 100, sub, restart_interval=ri)
    batch = J.prepare_batch([enc.data], J.Config.make(subseq_bits=L, overlap=overlap))
    for fill in (0x7777, -1):
        batch.d_coef.fill_(fill)
        rep = batch.decode()
        assert rep.redo >= 1
        assert L > 256 or ri or (rep.n_subseq + 255) // 256 > 128   # not gathered in LDS: cleared ahead
        assert np.array_equal(batch.coefficients(0).cpu().numpy(), enc.coef)


@pytest.mark.parametrize("L,ri", [(128, 0), (1024, 0), (2048, 0), (128, 9), (1024, 9)])
def test_beyond_what_is_cleared_ahead(L, ri):
    import torch
    encs = [_halves(2040, 2056, ri), _halves(1024, 2056, ri)]
    files = [encs[k % 2].data for k in range(38)]
    batch = J.prepare_batch(files, J.Config.make(subseq_bits=L))
    assert batch.d_coef.numel() * batch.d_coef.element_size() > CLEAR_AHEAD
    batch.d_coef.fill_(0x7777)
    batch.d_pixels.fill_(0x5A)
    batch.decode()
    want = [torch.from_numpy(e.coef).cuda() for e in encs]
    for k in range(len(files)):
        assert torch.equal(batch.coefficients(k), want[k % 2]), k
    first = [batch.pixels(k).clone() for k in (0, 1)]
    for k in range(len(files)):
        assert torch.equal(batch.pixels(k), first[k % 2]), k


def test_beyond_what_is_cleared_ahead_with_a_repeated_write_pass():
    import torch
    enc = encode_jpeg(small_image(16352, 620, 480, sigma=80.0), 100, "444")
    n = 190
    batch = J.prepare_batch([enc.data] * n, J.Config.make(subseq_bits=128))
    assert batch.d_coef.numel() * batch.d_coef.element_size() > CLEAR_AHEAD
    batch.d_coef.fill_(0x7777)
    assert batch.decode().redo >= 1
    want = torch.from_numpy(enc.coef).cuda()
    for k in range(n):
        assert torch.equal(batch.coefficients(k), want), k
