"""Reductions that add their results in the launch itself, with adding blocks that give up before what they wait for
is there: the sum then comes from a block that ends later, with the same bits.  The launchers take the number of
looks and the place of the adding blocks from here; every wait ends."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


class Late(ctypes.Structure):
    _fields_ = [("patience", ctypes.c_uint32), ("grace", ctypes.c_uint32), ("ahead", ctypes.c_uint32)]


class TensorArgs(ctypes.Structure):
    _fields_ = [("io", ctypes.c_void_p), ("packed", ctypes.c_void_p), ("gmin", ctypes.c_void_p), ("gscale", ctypes.c_void_p),
                ("n", ctypes.c_int64), ("seed_lo", ctypes.c_uint32), ("seed_hi", ctypes.c_uint32),
                ("blk_base_lo", ctypes.c_uint32), ("meta", ctypes.c_uint32)]


class ReduceArgs(ctypes.Structure):
    _fields_ = [("a", ctypes.c_void_p), ("b", ctypes.c_void_p), ("n", ctypes.c_int64), ("dtype", ctypes.c_int32),
                ("pad", ctypes.c_int32)]


# (patience, grace, ahead): the library's own; no patience, adding blocks behind the others and in front of them; these
# with so little grace that they are gone before a long grid has ended (and far more than a block takes that has begun)
LATE = [(1 << 14, 1 << 20, 0), (0, 1 << 20, 0), (0, 1 << 20, 1), (0, 512, 1)]
TAG = 0x9E3779B97F4A7C15


def counted(period, n):
    return torch.arange(period, device="cuda", dtype=torch.uint8).repeat(n // period + 1)[:n]


@pytest.mark.parametrize("late", LATE)
@pytest.mark.parametrize("blocks", (1, 2, 511, 513, 4096, 4097, 36865, 300001))
def test_sensitivity(gact, blocks, late):
    n = blocks * 8192 - 5
    g0 = counted(7, n).to(torch.bfloat16)
    g1 = torch.full((1,), 2.0, device="cuda", dtype=torch.bfloat16).expand(n).contiguous()
    full, rest = divmod(n, 7)
    want = float(full * sum((i - 2) ** 2 for i in range(7)) + sum((i - 2) ** 2 for i in range(rest)))   # whole numbers: exact
    fn = gact.lib.gact_launch_diff_sq
    fn.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_uint, ctypes.c_void_p, ctypes.c_int, ctypes.c_uint64,
                                           ctypes.c_double, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    table = torch.from_numpy(np.frombuffer(bytes(ReduceArgs(g0.data_ptr(), g1.data_ptr(), n, gact.GACT_BF16, 0)), np.uint8).copy()).cuda()
    first = torch.tensor([0, blocks], dtype=torch.int32, device="cuda")
    partial = torch.full((2 * blocks + 8,), -1, dtype=torch.int64, device="cuda")
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    how = Late(*late)
    for turn in range(3):
        assert fn(None, table.data_ptr(), first.data_ptr(), 1, blocks, partial.data_ptr(), 1, TAG + 2 * turn + (blocks << 20),
                  1.0, out.data_ptr(), torch.cuda.current_stream().cuda_stream, ctypes.addressof(how)) == 0
        assert out.item() == want, turn
        out.zero_()
    assert bool((partial[2 * blocks:] == -1).all())


@pytest.mark.parametrize("late", LATE)
@pytest.mark.parametrize("blocks,ns", [(2, 3), (2, 257), (513, 0), (513, 256), (2049, 1), (2049, 32768), (40001, 3)])
def test_compressor_with_a_footprint(gact, blocks, ns, late):
    G, bits = 256, 2
    n = blocks * 8192 - 77
    x = counted(251, n).float()
    want = gact.gact_compress_footprint(x, G, bits, 5, ns)
    assert want[3][1:].cpu().tolist() == [float(j * n // ns % 251) for j in range(ns)]
    p, mn, sc = gact.alloc_compressed(n, G, bits, x.device)
    t = TensorArgs(x.data_ptr(), p.data_ptr(), mn.data_ptr(), sc.data_ptr(), n, 5, 0, 0, bits | gact.GACT_F32 << 8)
    lpg, lds = G // 32, 64 * 32
    geo = (ctypes.c_int32 * 8)(lpg, 64 // lpg * lpg, 1, 64 // lpg, 3, -2**31, 65536 // lpg + 1, lds)
    fn = gact.lib.gact_launch_compress_sum
    fn.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint, ctypes.c_void_p, ctypes.c_int, ctypes.c_uint64,
                   ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    partial = torch.full((2 * blocks + 8,), -1, dtype=torch.int64, device="cuda")
    fp = torch.zeros(1 + ns, dtype=torch.float64, device="cuda")
    how = Late(*late)
    for turn in range(3):
        assert fn(ctypes.addressof(t), ctypes.addressof(geo), blocks, partial.data_ptr(), 1, TAG + 2 * turn + (blocks << 20),
                  ns, fp.data_ptr(), torch.cuda.current_stream().cuda_stream, ctypes.addressof(how)) == 0
        assert all(torch.equal(a, b) for a, b in zip((p, mn, sc, fp), want)), turn
        for u in (p, mn, sc, fp):
            u.zero_()
    assert bool((partial[2 * blocks:] == -1).all())


@pytest.mark.parametrize("patience", (1 << 14, 0))
@pytest.mark.parametrize("blocks", (32769, 600001))
def test_sums_added_by_several_blocks_of_a_launch_behind(gact, blocks, patience):
    n = blocks * 8192 - 5
    x = counted(9, n).to(torch.bfloat16)
    full, rest = divmod(n, 9)
    fn = gact.lib.gact_launch_footprint
    fn.argtypes = [ctypes.c_void_p, ctypes.c_uint, ctypes.c_void_p, ctypes.c_uint64, ctypes.c_int, ctypes.c_void_p,
                   ctypes.c_void_p, ctypes.c_void_p]
    r = ReduceArgs(x.data_ptr(), None, n, gact.GACT_BF16, 0)
    partial = torch.full((blocks + 8,), -1, dtype=torch.int64, device="cuda")
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    how = Late(patience, 1 << 20, 0)
    for turn in range(3):
        assert fn(ctypes.addressof(r), blocks, partial.data_ptr(), TAG + blocks, 0, out.data_ptr(),
                  torch.cuda.current_stream().cuda_stream, ctypes.addressof(how)) == 0
        assert out.item() == float(36 * full + rest * (rest - 1) // 2), turn
        out.zero_()
    assert bool((partial[blocks:] == -1).all())
