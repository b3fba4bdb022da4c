"""The decoder around the edges of its pieces (16 bytes a lane, 1 KiB a
wavefront, 4 KiB a tile): a number of every length ending at, before and
across an edge, segments that open there, and code at any alignment.  The
expected indices are numpy's running sums of the gaps; the bytes are the
oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_11456_amd as ad

pytestmark = pytest.mark.gpu

EDGES = [16, 1024, 4096, 8192]


def encode(idx):
    return oracle.leb128_encode(idx)[0]


def leb_len(g):
    n = np.ones(g.size, dtype=np.int64)
    for b in range(7, 63, 7):
        n += g >= (1 << b)
    return n


def gaps_with(at, length, rng, two_bytes):
    """Gaps whose code has a number of `length` bytes starting at byte `at`,
    small numbers before it and after it, 9000-odd bytes in all."""
    def small(nbytes):
        out, left = [], nbytes
        while left:
            if two_bytes and left >= 2 and rng.random() < 0.5:
                out.append(int(rng.integers(128, 16384)))
                left -= 2
            else:
                out.append(int(rng.integers(1, 128)))
                left -= 1
        return out
    lo = 1 if length == 1 else 1 << (7 * (length - 1))
    big = lo + int(rng.integers(0, 50))
    return np.array(small(at) + [big] + small(9011 - at), dtype=np.int64)


def device_code(code, shift):
    buf = torch.zeros(code.size + shift, dtype=torch.uint8, device="cuda")
    buf[shift:] = torch.from_numpy(np.ascontiguousarray(code)).cuda()
    return buf[shift:]


@pytest.mark.parametrize("edge", EDGES)
@pytest.mark.parametrize("length", [1, 2, 3, 4, 9])
def test_number_across_an_edge(edge, length):
    rng = np.random.default_rng(edge + length)
    for back in range(0, length + 1):
        for two in (False, True):
            gaps = gaps_with(edge - back, length, rng, two)
            idx = np.cumsum(gaps)
            code = encode(idx)
            assert leb_len(gaps).sum() == code.size
            got = ad.delta_leb128_decode(device_code(code, back % 4))
            np.testing.assert_array_equal(got.cpu().numpy(), idx)


@pytest.mark.parametrize("edge", EDGES)
@pytest.mark.parametrize("length", [1, 2, 3])
def test_segment_opens_at_an_edge_and_apply(edge, length):
    """Three segments, the second opening with the number at the edge, the
    third one entry later; decoded, and applied straight from the code."""
    rng = np.random.default_rng(31 * edge + length)
    for back in range(-1, length + 1):
        gaps = gaps_with(edge - back, length, rng, True)
        starts = np.cumsum(leb_len(gaps)) - leb_len(gaps)
        e = int(np.flatnonzero(starts == edge - back)[0])
        offs = np.array([0, e, e + 1, gaps.size], dtype=np.int64)
        local = [np.cumsum(gaps[a:b]) for a, b in zip(offs, offs[1:])]
        numels = [int(x[-1]) + 5 for x in local]
        bases = np.cumsum([0] + numels[:-1])
        idx = np.concatenate([b + x for b, x in zip(bases, local)])
        code = np.concatenate([encode(x) for x in local])
        dev = device_code(code, (back + 1) % 4)
        got = ad.delta_leb128_decode(dev, offs, bases)
        np.testing.assert_array_equal(got.cpu().numpy(), idx)
        val = rng.integers(0, 1 << 16, idx.size, dtype=np.uint16)
        want = np.zeros(sum(numels), dtype=np.uint16)
        oracle.apply_(want, idx, val)
        for fill in (0, 100 * sum(numels)):   # dense, then sparse over a longer last tensor
            flat = torch.zeros(sum(numels) + fill, dtype=torch.int16, device="cuda")
            w = list(flat.split([numels[0], numels[1], numels[2] + fill]))
            ad.delta_apply_leb128_multi(w, dev, offs, None, torch.from_numpy(val.view(np.int16)).cuda(),
                                        check=True)
            np.testing.assert_array_equal(flat[:want.size].cpu().numpy().view(np.uint16), want)
            assert not bool(flat[want.size:].any())


@pytest.mark.parametrize("nbytes", [1, 15, 16, 17, 1023, 1024, 1025, 4095, 4096, 4097])
def test_stream_lengths(nbytes):
    rng = np.random.default_rng(nbytes)
    idx = np.cumsum(rng.integers(1, 128, nbytes))
    dev = device_code(encode(idx), nbytes % 5)
    np.testing.assert_array_equal(ad.delta_leb128_decode(dev).cpu().numpy(), idx)
    dev = dev.clone()
    dev[-1] |= 0x80   # ends inside a number
    with pytest.raises(ad.DeltaError):
        ad.delta_leb128_decode(dev)
