"""Components that share their Huffman tables in other ways than the usual one (luma 0/0, chroma 1/1), against the CPU oracle:
the kernels know data units by the pair of tables they take, of which an image has up to three."""
import numpy as np
import pytest

import paper_2111_09219_amd as J
import jpegfile as jf
from oracle import OracleImage
from workloads import encode_jpeg, small_image

pytestmark = pytest.mark.gpu

# DC and AC table of the three components: one kind of data unit, two, three in four tables, five and six tables
PAIRINGS = [((0, 0, 0), (1, 1, 1)), ((0, 1, 0), (0, 1, 1)), ((1, 1, 0), (0, 1, 1)), ((0, 0, 0), (0, 1, 2)),
            ((0, 1, 2), (1, 1, 1)), ((0, 1, 1), (0, 1, 2)), ((0, 1, 2), (0, 1, 2))]


def _records_are_the_oracles(batch, rep, o, L):
    rec = J.jpgd_read_sync_info(batch.d_workspace, 0, rep.n_subseq + 8)
    bs = o.boundary_states(L)
    n = len(bs["p"])
    live = np.cumsum(bs["units"]) < o.total_units
    for name in ("p", "u", "z", "units"):
        assert np.array_equal(rec[name][:n][live].astype(np.int64), bs[name][live].astype(np.int64)), name
    assert np.array_equal(rec["dcsum"][:n][live].astype(np.int16), bs["dcsum"][live].astype(np.int16))


@pytest.mark.parametrize("td,ta", PAIRINGS)
@pytest.mark.parametrize("split", [0, 2])
@pytest.mark.parametrize("L", [128, 1024])
def test_pairings_of_tables(td, ta, split, L):
    """One kernel and two (which no call with more than four tables takes); records, coefficients, and the image among
    others.  Noise at quality 97: the rounds with a wavefront per chain have work in every sequence."""
    enc = encode_jpeg(small_image(77, 640, 720, sigma=30.0), 97, "420")
    data = jf.written_with_tables(enc, td, ta)
    other = encode_jpeg(small_image(3, 120, 200, sigma=9.0), 85, "444", True).data
    batch = J.prepare_batch([data], J.Config.make(subseq_bits=L, sync_split=split))
    rep = batch.decode()
    tables = len(set(td)) + len(set(ta))
    assert rep.launches[J.KERNELS.index("sync_tail")] == (1 if split == 2 and tables <= 4 else 0)
    assert np.array_equal(batch.coefficients(0).cpu().numpy(), enc.coef)
    _records_are_the_oracles(batch, rep, OracleImage(data), L)
    batch = J.prepare_batch([other, data, other], J.Config.make(subseq_bits=L, sync_split=split))
    batch.decode()
    assert np.array_equal(batch.coefficients(1).cpu().numpy(), enc.coef)
    for i in (0, 2):
        assert np.array_equal(batch.coefficients(i).cpu().numpy(), OracleImage(other).coefficients())


@pytest.mark.parametrize("td,ta", [((0, 1, 0), (0, 1, 1)), ((0, 1, 2), (1, 1, 1)), ((0, 1, 2), (0, 1, 2))])
@pytest.mark.parametrize("split", [0, 2])
def test_three_kinds_over_several_inter_sequence_rounds(td, ta, split):
    enc = encode_jpeg(small_image(16352, 303, 231, sigma=80.0), 100, "420")
    data = jf.written_with_tables(enc, td, ta)
    batch = J.prepare_batch([data], J.Config.make(subseq_bits=128, sync_split=split))
    rep = batch.decode()
    assert rep.inter_rounds >= 2
    assert np.array_equal(batch.coefficients(0).cpu().numpy(), enc.coef)
    _records_are_the_oracles(batch, rep, OracleImage(data), 128)
