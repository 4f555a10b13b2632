"""The sequence map where its kernels meet: direct counting up to 256 sequences (64 without a work list),
chunks above. The tables are read back from the workspaces of elis_attention (with a work list) and
elis_pool_head (without one) and compared with plain numpy; the lengths spread over many buckets or tie."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2505_09142_amd import _elis as E
from paper_2505_09142_amd.device import DeviceWeights
from tests.gpu_util import dev, note, ok, stream, workspace
from tests.test_attention_worklist import RPB, bucket, capacity
from workloads import TINY, make_weights

pytestmark = pytest.mark.gpu


def tables(buf, base, n):
    """status, start, len and tile_off at the front of the workspace, and the offset behind them."""
    host = buf.cpu().numpy()[base - buf.data_ptr():]
    at, out = 0, []
    for count in (1, n, n, n + 1):
        out.append(host[at:at + 4 * count].view(np.int32))
        at += (4 * count + 255) // 256 * 256
    return host, out, at


def batch(n, spread):
    rng = np.random.default_rng(n + spread)
    lens = rng.integers(1, 700 if spread else 3, n)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    tiles = (lens + RPB - 1) // RPB
    return lens, cu, np.concatenate([[0], np.cumsum(tiles)])


def check(got, cu, lens, tile_off):
    status, start, length, offs = got
    assert status[0] == 0 and np.array_equal(start, cu[:-1]) and np.array_equal(length, lens) and np.array_equal(offs, tile_off)


@pytest.mark.parametrize("spread", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 255, 256, 257, 300])
def test_tables_and_work_list(n, spread):
    note(f"sequence map n={n} spread={spread}")
    lens, cu, tile_off = batch(n, spread)
    T = int(cu[-1])
    qkv = torch.zeros((T, 3 * 32), dtype=torch.bfloat16, device="cuda")
    out = torch.empty((T, 32), dtype=torch.bfloat16, device="cuda")
    buf, ws, wsb = workspace(E.elis_attention_workspace_bytes(n, T))
    buf.fill_(0xEE)
    ok(E.elis_attention(qkv.data_ptr(), dev(cu).data_ptr(), n, T, int(lens.max()), 1, 32, out.data_ptr(), ws, wsb, stream()))
    torch.cuda.synchronize()
    host, got, at = tables(buf, ws, n)
    check(got, cu, lens, tile_off)
    cap = capacity(n, T)
    work = host[at:at + 16 * cap].view(np.int32).reshape(cap, 4)
    first = sorted(range(n), key=lambda s: (-bucket(int(lens[s])), s))
    want = [(cu[s], lens[s], q * RPB, s) for s in first for q in range((int(lens[s]) + RPB - 1) // RPB)]
    assert np.array_equal(work[:len(want)], np.array(want, np.int32))
    assert np.all(work[len(want):, 1] == 0)


@pytest.mark.parametrize("n", [1, 64, 65, 256, 257])
def test_tables_without_a_work_list(n):
    note(f"sequence map of the head n={n}")
    lens, cu, tile_off = batch(n, 0)
    shape = dataclasses.replace(TINY, n_layers=0)
    W = make_weights(shape, 3)
    dw = DeviceWeights(shape, {k: v for k, v in W.device.items() if k.startswith("head_")})
    T = int(cu[-1])
    hidden, pred = torch.zeros((T, shape.d_model), device="cuda", dtype=torch.float32), torch.empty(n, device="cuda", dtype=torch.float32)
    buf, ws, wsb = workspace(E.elis_pool_head_workspace_bytes(dw.cfg, n, int(lens.max())))
    buf.fill_(0xEE)
    ok(E.elis_pool_head(dw.struct, hidden.data_ptr(), dev(cu).data_ptr(), n, T, int(lens.max()), pred.data_ptr(), ws, wsb, stream()))
    torch.cuda.synchronize()
    check(tables(buf, ws, n)[1], cu, lens, tile_off)
