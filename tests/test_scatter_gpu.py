"""The scatter of an index stream against the oracle: entry counts around
the pieces a wavefront (128 entries), a workgroup (512) and the eight XCDs
take, tensor lists around the sizes at which the tensor search changes form
(64 and 512 tensors), any order of the entries, and entries outside."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_11456_amd as ad

pytestmark = pytest.mark.gpu


def _case(rng, tensors, count, empty):
    sizes = rng.integers(1, 9, tensors) + count // tensors + 1
    sizes[rng.random(tensors) < empty] = 0
    sizes[rng.integers(tensors)] += count
    total = int(sizes.sum())
    idx = rng.choice(total, count, replace=False).astype(np.int64)
    val = rng.integers(0, 1 << 16, count, dtype=np.uint16)
    words = rng.integers(0, 1 << 16, total, dtype=np.uint16)
    return [int(s) for s in sizes], idx, val, words


@pytest.mark.parametrize("tensors", [1, 2, 63, 64, 65, 512, 513, 1500])
@pytest.mark.parametrize("count", [1, 127, 129, 511, 513, 4096 + 1, 9 * 512 + 77])
@pytest.mark.parametrize("order", ["sorted", "shuffled"])
def test_multi(tensors, count, order):
    rng = np.random.default_rng(tensors * 7919 + count)
    sizes, idx, val, words = _case(rng, tensors, count, 0.2)
    if order == "sorted":
        idx.sort()
    expect = words.copy()
    bad = oracle.apply_(expect, idx, val)
    assert bad == 0
    flat = torch.from_numpy(words.view(np.int16).copy()).cuda()
    w = list(flat.split(sizes))
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ad.delta_apply_multi(w, torch.from_numpy(idx).cuda(),
                         torch.from_numpy(val.view(np.int16)).cuda(), error_flag=flag)
    assert int(flag.item()) == 0
    assert np.array_equal(flat.cpu().numpy().view(np.uint16), expect)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("count", [1, 128, 512, 513, 8 * 512 + 1, 20011])
def test_single(dtype, count):
    rng = np.random.default_rng(count)
    _, idx, val, words = _case(rng, 1, count, 0.0)
    expect = words.copy()
    oracle.apply_(expect, idx.astype(dtype), val)
    w = torch.from_numpy(words.view(np.int16).copy()).cuda()
    ad.delta_apply(w, torch.from_numpy(idx.astype(dtype)).cuda(),
                   torch.from_numpy(val.view(np.int16)).cuda(), check=True)
    assert np.array_equal(w.cpu().numpy().view(np.uint16), expect)


@pytest.mark.parametrize("tensors", [1, 70, 600])
def test_outside(tensors):
    """Entries outside the list are skipped and flagged, wherever they sit;
    the others are written."""
    rng = np.random.default_rng(tensors)
    sizes, idx, val, words = _case(rng, tensors, 3000, 0.2)
    total = sum(sizes)
    for p, g in ((0, -1), (64, total), (700, np.iinfo(np.int64).max),
                 (2999, np.iinfo(np.int64).min)):
        idx[p] = g
    expect = words.copy()
    assert oracle.apply_(expect, idx, val) == 4
    flat = torch.from_numpy(words.view(np.int16).copy()).cuda()
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ad.delta_apply_multi(list(flat.split(sizes)), torch.from_numpy(idx).cuda(),
                         torch.from_numpy(val.view(np.int16)).cuda(), error_flag=flag)
    assert int(flag.item()) != 0
    assert np.array_equal(flat.cpu().numpy().view(np.uint16), expect)
