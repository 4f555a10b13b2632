"""The head takes rows at any float's address: with hidden states and weights off 16 bytes by one to three
floats its matrix-core layers load through registers instead of straight into LDS, with the same bits."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

from paper_2505_09142_amd import _elis as E
from paper_2505_09142_amd.device import DeviceWeights
from tests.gpu_util import dev, note, ok, stream, workspace
from workloads import TINY_HEAD8, make_weights

pytestmark = pytest.mark.gpu


def shifted(t, floats):
    out = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")[floats:floats + t.numel()]
    out.copy_(t.reshape(-1))
    assert out.data_ptr() % 16 == 4 * floats
    return out


@pytest.mark.parametrize("hidden_width", [64, 128])  # four and eight waves
@pytest.mark.parametrize("pooling", [E.ELIS_POOL_CLS, E.ELIS_POOL_MEAN])
@pytest.mark.parametrize("layers", [2, 4])
def test_same_bits_at_any_float_address(hidden_width, pooling, layers):
    shape = dataclasses.replace(TINY_HEAD8, n_layers=0, pooling=pooling, head_hidden=hidden_width, head_layers=layers)
    W = make_weights(shape, 5)
    dw = DeviceWeights(shape, {k: v for k, v in W.device.items() if k.startswith("head_")})
    lens = [5, 1, 33, 64, 17] * 4
    n, T = len(lens), sum(lens)
    cu = dev(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    gen = torch.Generator(device="cuda").manual_seed(layers)
    hidden = torch.randn((T, shape.d_model), generator=gen, device="cuda", dtype=torch.float32)
    w1 = dev(W.device["head_w1"])
    mids = [dev(m) for m in W.device.get("head_mid_w", [])]
    assert len(mids) == layers - 2
    outs = []
    for h_off, w_off in ((0, 0), (1, 0), (0, 2), (3, 1)):
        note(f"head rows off by {h_off} and {w_off} floats: width {hidden_width}, pooling {pooling}, {layers} layers")
        keep = [shifted(hidden, h_off), shifted(w1, w_off)] + [shifted(m, w_off) for m in mids]
        dw.struct.head_w1 = keep[1].data_ptr()
        if mids:
            table = (ctypes.c_void_p * len(mids))(*[k.data_ptr() for k in keep[2:]])
            dw.struct.head_mid_w = ctypes.cast(table, ctypes.POINTER(ctypes.c_void_p))
        out = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
        buf, ws, wsb = workspace(E.elis_pool_head_workspace_bytes(dw.cfg, n, max(lens)))
        ok(E.elis_pool_head(dw.struct, keep[0].data_ptr(), cu.data_ptr(), n, T, max(lens), out.data_ptr(), ws, wsb, stream()))
        torch.cuda.synchronize()
        outs.append(out)
    assert all(torch.equal(outs[0], o) for o in outs[1:]) and not torch.isnan(outs[0]).any()
