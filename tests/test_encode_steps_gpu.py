"""The encoder's steps of 64 numbers against the oracle: steps of one- and
two-byte numbers, steps in which some or all are longer, tiles whose code
starts at every byte of a 16-byte piece of the output, and outputs cut inside
a piece."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_11456_amd as ad

pytestmark = pytest.mark.gpu


def encode_into(idx, out):
    lib = ad.library()
    d_idx = torch.from_numpy(idx).cuda()
    ws = torch.empty(lib.delta_leb128_encode_workspace_bytes(idx.size), dtype=torch.uint8,
                     device="cuda")
    nb = torch.zeros(1, dtype=torch.int64, device="cuda")
    st = lib.delta_leb128_encode(d_idx.data_ptr(), idx.size, None, None, 0, out.data_ptr(),
                                 out.numel(), nb.data_ptr(), None, None, ws.data_ptr(),
                                 ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return int(nb.item())


@pytest.mark.parametrize("at", range(16))
@pytest.mark.parametrize("long", ["none", "one", "all"])
def test_steps(at, long):
    count = 6 * 4096 + 64 * at + 7
    r = np.random.default_rng(at)
    gaps = r.integers(1, 1 << 14, count, dtype=np.int64)
    gaps[:4096] = r.integers(1, 128, 4096)
    if long != "none":   # one lane of every third step, or every lane of it
        k = np.arange(count)
        pick = (k // 64 % 3 == 1) & ((k % 64 == (7 * (k // 64)) % 64) | (long == "all"))
        gaps[pick] = np.int64(1) << (14 + 5 * (k[pick] % 8))
    idx = np.cumsum(gaps)
    ref, n = oracle.leb128_encode(idx)
    for room in (n, n - 1, n - 17, 5):
        buf = torch.full((room + 48,), 0xA5, dtype=torch.uint8, device="cuda")
        assert encode_into(idx, buf[at:at + room]) == n
        got = buf.cpu().numpy()
        np.testing.assert_array_equal(got[at:at + room], ref[:room])
        assert (got[:at] == 0xA5).all() and (got[at + room:] == 0xA5).all()
