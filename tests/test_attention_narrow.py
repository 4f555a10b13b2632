"""Attention in launches of few work-groups (one 16-query block per wave) gives the bits of the wide form.

The same sequences run alone, where the launch is small, and packed with enough others that it is not;
lengths at the edges of 16-query blocks, 64-query work-groups, key tiles and 128-query items."""
import numpy as np
import pytest
import torch

from paper_2505_09142_amd import _elis as E
from tests.gpu_util import dev, note, ok, stream, workspace

pytestmark = pytest.mark.gpu


def attend(qkv, lens, heads, dh):
    T = int(sum(lens))
    cu = dev(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    out = torch.full((T + 8, heads * dh), 7.0, dtype=torch.bfloat16, device="cuda")
    buf, ws, wsb = workspace(E.elis_attention_workspace_bytes(len(lens), T))
    ok(E.elis_attention(qkv.data_ptr(), cu.data_ptr(), len(lens), T, max(lens), heads, dh, out.data_ptr(), ws, wsb, stream()))
    torch.cuda.synchronize()
    assert E.elis_read_status(ws, stream()) == (E.ELIS_OK, 0) and bool((out[T:] == 7.0).all())
    return out[:T].view(torch.int16)


@pytest.mark.parametrize("dh,heads", [(64, 12), (32, 4)])
@pytest.mark.parametrize("lens", [[1], [15, 16, 17], [63, 64, 65], [127, 128, 129], [191, 192, 193, 1], [700, 33]])
def test_same_bits_alone_and_in_a_large_batch(lens, dh, heads):
    note(f"attention alone and packed lens={lens} dh={dh}")
    extra = [200] * 500  # more than any threshold of a small launch
    T, D = int(sum(lens)), heads * dh
    gen = torch.Generator(device="cuda").manual_seed(T + dh)
    qkv = torch.randn((T + sum(extra), 3 * D), generator=gen, device="cuda", dtype=torch.float32)
    qkv[:, :D] *= 4.0  # sharp enough that running maxima move
    qkv = qkv.to(torch.bfloat16)
    alone = attend(qkv, lens, heads, dh)
    packed = attend(qkv, lens + extra, heads, dh)
    assert torch.equal(alone, packed[:T])
