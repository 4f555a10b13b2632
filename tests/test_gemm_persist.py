"""The persistent 256 x 256 product kernel: a CPU mirror of its addresses, and its bits on the GPU.

The mirror re-evaluates, over all work-groups, waves and lanes, which tiles a work-group walks, what
the direct loads fetch into which place of LDS, what the fragment reads take from there, and which
output bytes the epilogue stores (rows past the end must fall outside the buffer resource). On the
GPU every size is compared bit for bit with 128 x 128 tiles: one tile and several per work-group,
ragged rows, odd and even slab counts, and the depths the kernel hands on (k = 64).
"""
import numpy as np
import pytest

from paper_2505_09142_amd import _elis as E

GROUP_M, CUS = 8, 256


def tiles_of(bid, grid, tiles):
    """Tile indices of one work-group: its XCD's contiguous range, dealt out to the XCD's work-groups."""
    xcd, per, rem = bid & 7, tiles >> 3, tiles & 7
    count = per + (xcd < rem)
    end = xcd * per + min(xcd, rem) + count
    return list(range(end - count + (bid >> 3), end, (grid - xcd + 7) >> 3))


@pytest.mark.parametrize("tiles", [1, 2, 7, 8, 9, 63, 255, 256, 257, 282, 1092, 4368])
def test_every_tile_is_walked_once(tiles):
    grid = min(tiles, CUS)
    walked = [tiles_of(b, grid, tiles) for b in range(grid)]
    assert all(walked)  # a work-group's first tile always exists
    assert sorted(sum(walked, [])) == list(range(tiles))


def swz(row):
    return (row >> 1) & 7


def test_loads_and_fragment_reads_agree():
    """Each half-slab is filled once, and a fragment read of (row, k) sees that element of the tile."""
    lane = np.arange(64)
    for operand, row_of in (("a", lambda h, r: (r >> 6) * 128 + h * 64 + (r & 63)), ("b", lambda h, r: (r >> 5) * 64 + h * 32 + (r & 31))):
        for h in (0, 1):
            lds = np.full((128 * 8, 2), -1)  # 16-byte unit of the half-slab -> (tile row, logical chunk)
            for w in range(8):
                for i in (0, 1):
                    r = w * 16 + i * 8 + (lane >> 3)
                    unit = (w * 16 + i * 8) * 8 + lane  # the load writes lane i's 16 bytes at base + 16 i
                    assert np.all(lds[unit] == -1)
                    lds[unit, 0], lds[unit, 1] = row_of(h, r), (lane & 7) ^ swz(r)
            assert np.all(lds >= 0) and len({tuple(x) for x in lds}) == 128 * 8
            for w in range(8):  # wave block: rows 128 (w / 4) + 64 h + 32 i, columns 64 (w % 4) + 32 h
                for i in range(2 if operand == "a" else 1):
                    for ks in range(4):
                        rl, kg = lane & 31, lane >> 5
                        first = (w >> 2) * 64 + i * 32 if operand == "a" else (w & 3) * 32
                        unit = (first + rl) * 8 + ((ks * 2 + kg) ^ swz(rl))
                        want = (w >> 2) * 128 + h * 64 + i * 32 + rl if operand == "a" else (w & 3) * 64 + h * 32 + rl
                        assert np.array_equal(lds[unit, 0], want) and np.array_equal(lds[unit, 1], ks * 2 + kg)


@pytest.mark.parametrize("M", [1, 31, 128, 255, 256, 257, 511])
@pytest.mark.parametrize("f32", [False, True])
def test_stores_cover_the_output_once(M, f32):
    N, eb = 512, 4 if f32 else 2
    lane = np.arange(64)
    ch, rr0 = lane & 7, lane >> 3
    out = np.zeros((M * N * eb) // 16, int)
    for m0 in range(0, M, 256):
        rows = min(256, M - m0)
        for n0 in range(0, N, 256):
            size, base = (rows * N - n0) * eb, (m0 * N + n0) * eb
            for w in range(8):
                wm, wn = w >> 2, w & 3
                for i in range(4):
                    for j in range(2 if f32 else 1):
                        for rr in range(4):
                            row = wm * 128 + i * 32 + rr * 8 + rr0
                            off = (row * N + wn * 64) * eb + ch * 16
                            keep = off < size  # the resource drops the others, with and without the scalar offset
                            assert np.array_equal(keep, off < size - j * 128) and np.array_equal(keep, row < rows)
                            np.add.at(out, (base + off[keep] + j * 128) // 16, 1)
    assert np.all(out == 1)


@pytest.mark.gpu
@pytest.mark.parametrize("epi", [E.ELIS_EPI_BIAS_BF16, E.ELIS_EPI_BIAS_GELU_BF16, E.ELIS_EPI_BIAS_RES_F32])
@pytest.mark.parametrize("m,n,k", [(1, 256, 128), (257, 256, 64), (300, 512, 192), (513, 768, 256), (65793, 256, 128),
                                   (25000, 768, 320)])
def test_same_bits_as_small_tiles(m, n, k, epi):
    import torch
    from tests.gpu_util import note, ok, stream
    note(f"persistent product m={m} n={n} k={k} epi={epi}")
    gen = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn((m, k), generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    w = (0.05 * torch.randn((n, k), generator=gen, device="cuda", dtype=torch.float32)).to(torch.bfloat16)
    bias = torch.randn(n, generator=gen, device="cuda", dtype=torch.float32)
    f32 = epi == E.ELIS_EPI_BIAS_RES_F32
    res = torch.randn((m, n), generator=gen, device="cuda", dtype=torch.float32) if f32 else None
    guard = 4096  # elements past the output that must stay as they are
    outs = []
    for tile in ((256, 256, 1), (128, 128, 2)):
        out = torch.full((m * n + guard,), 7.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
        ok(E.elis_linear_with_plan(x.data_ptr(), w.data_ptr(), bias.data_ptr(), res.data_ptr() if f32 else None, m, n, k, epi,
                                   (*tile, m, 0, 0, 0), out.data_ptr(), stream()))
        torch.cuda.synchronize()
        assert bool((out[m * n:] == 7.0).all())
        outs.append(out[:m * n].view(torch.int32 if f32 else torch.int16))
    assert torch.equal(outs[0], outs[1])


@pytest.mark.gpu
@pytest.mark.parametrize("epi", [E.ELIS_EPI_BIAS_BF16, E.ELIS_EPI_BIAS_GELU_BF16, E.ELIS_EPI_BIAS_RES_F32])
@pytest.mark.parametrize("m,n,k", [(1, 128, 64), (31, 128, 128), (32, 256, 448), (33, 384, 512), (65, 128, 576), (193, 768, 3072),
                                   (512, 1024, 320)])
def test_few_rows_same_bits_as_small_tiles(m, n, k, epi):
    """32 x 32 tiles, from one slab to more than the ring of eight (1, 2, 5, 7, 8, 9 and 48), against 64 x 64
    tiles and the library's own choice."""
    import torch
    from tests.gpu_util import note, ok, stream
    note(f"few rows m={m} n={n} k={k} epi={epi}")
    gen = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn((m, k), generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    w = (0.05 * torch.randn((n, k), generator=gen, device="cuda", dtype=torch.float32)).to(torch.bfloat16)
    bias = torch.randn(n, generator=gen, device="cuda", dtype=torch.float32)
    f32 = epi == E.ELIS_EPI_BIAS_RES_F32
    res = torch.randn((m, n), generator=gen, device="cuda", dtype=torch.float32) if f32 else None
    outs = []
    for plan in ((32, 32, 2, m, 0, 0, 0), (64, 64, 2, m, 0, 0, 0), None):
        out = torch.full((m * n + 4096,), 7.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
        args = (x.data_ptr(), w.data_ptr(), bias.data_ptr(), res.data_ptr() if f32 else None, m, n, k, epi)
        ok(E.elis_linear(*args, out.data_ptr(), stream()) if plan is None else E.elis_linear_with_plan(*args, plan, out.data_ptr(), stream()))
        torch.cuda.synchronize()
        assert bool((out[m * n:] == 7.0).all())
        outs.append(out[:m * n].view(torch.int32 if f32 else torch.int16))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.gpu
@pytest.mark.parametrize("d,d_ff,heads,sizes", [(256, 320, 4, (8003, 33001, 65537)), (512, 1024, 8, (2000, 8000, 16001, 33003, 66001))])
def test_residual_norm_epilogues_same_bits_in_every_tile(d, d_ff, heads, sizes):
    """The epilogues that rebuild a LayerNorm output as the residual (out-projection and second feed-forward
    product) are reached through the encoder only: the same sequences' final hidden states, alone (32 x 32 tiles) and at
    both ends of batches whose products run in every other tile, the persistent one over one and several tiles
    per work-group and with a ragged last tile among them. Alone they are checked against the oracle."""
    import torch

    import oracle
    from paper_2505_09142_amd.device import DeviceWeights, Predictor, upload_batch
    from tests.gpu_util import note
    from workloads import make_weights, pack
    from workloads.configs import EncoderShape
    shape = EncoderShape("residual_norm", 2, d, heads, d_ff, 1000, 512, 1, 0, True)
    W = make_weights(shape, d)
    pr = Predictor(DeviceWeights(shape, W.device))
    rng = np.random.default_rng(d)
    own = [rng.integers(1, 1000, L).astype(np.int32) for L in (61, 1, 33)]
    rows = sum(len(s) for s in own)

    def hidden(seqs):
        b = pack(seqs)
        ids, cu, _ = upload_batch(b)
        pred, hid = pr.predict(ids, cu, b.max_seqlen, want_hidden=True)
        assert pr.status() == (E.ELIS_OK, 0)
        return b, pred, hid

    b, pred, alone = hidden(own)
    ref_p, ref_h = oracle.oracle_forward(b.token_ids, b.cu_seqlens, W.master, shape)
    assert float(np.abs(alone.cpu().numpy() - ref_h).max()) <= 5e-2 and np.all(np.abs(pred.cpu().numpy() - ref_p) <= 2e-2 * np.maximum(np.abs(ref_p), 1))
    tiles = set()
    for T in (rows,) + sizes:
        for k in (d, d_ff):
            p = E.elis_linear_plan(T, d, k, E.ELIS_EPI_BIAS_RES_F32)[1]
            tiles |= {p[:2]} | ({p[4:6]} if p[3] < T else set())
    assert {(32, 32), (64, 64), (256, 256)} <= tiles
    for T in sizes:
        note(f"residual-norm epilogues d={d} T={T}")
        fill, extra = T - 2 * rows, []
        while fill > 0:
            extra.append(rng.integers(1, 1000, min(fill, 500)).astype(np.int32))
            fill -= len(extra[-1])
        _, _, hid = hidden(own + extra + own)
        assert torch.equal(hid[:rows], alone) and torch.equal(hid[T - rows:], alone), T
