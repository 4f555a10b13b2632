"""The job table where its launches change: packs at and past 1,024 jobs (one launch or two), selects that
gather by themselves (up to 1,024 candidates), rank a gathered list (8,192) and select over the device,
and appends that wrap the ring, start a job, or carry nothing, by work-groups and (past 8,192 jobs of few tokens)
by tokens; against plain numpy."""
import numpy as np
import pytest
import torch

from paper_2505_09142_amd import _elis as E
from paper_2505_09142_amd.device import JobTable
from tests.gpu_util import dev, note

pytestmark = pytest.mark.gpu


def expected_input(tokens, max_pos):
    return tokens if len(tokens) <= max_pos else np.concatenate([tokens[:1], tokens[len(tokens) - (max_pos - 1):]])


@pytest.mark.parametrize("max_pos", [2, 16, 33])
@pytest.mark.parametrize("n", [1, 255, 256, 257, 1023, 1024, 1025, 2049, 8192, 8193])
def test_append_and_pack(n, max_pos):
    note(f"jobs append + pack n={n} max_pos={max_pos}")
    rng = np.random.default_rng(n + max_pos)
    t = JobTable(n + 3, max_pos)
    slots = rng.permutation(n + 3)[:n].astype(np.int32)
    d_slots = dev(slots)
    t.start(d_slots, dev(np.arange(n, dtype=np.int64)))
    held = [np.zeros(0, np.int32) for _ in range(n)]
    for step in range(3):
        cnt = rng.integers(1 if step == 0 else 0, 3 * max_pos + 300 if n < 300 else 40, size=n)
        off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
        tok = rng.integers(1, 1 << 20, size=int(off[-1])).astype(np.int32)
        held = [np.concatenate([h, tok[a:b]]) for h, a, b in zip(held, off, off[1:])]
        t.append(d_slots, dev(off), dev(tok) if len(tok) else torch.zeros(1, dtype=torch.int32, device="cuda"), int(off[-1]))
        want = [expected_input(h, max_pos) for h in held]
        lens = np.array([len(x) for x in want])
        ids = torch.full((int(lens.sum()) + 16,), -7, dtype=torch.int32, device="cuda")
        cu = torch.full((n + 1 + 16,), -7, dtype=torch.int32, device="cuda")
        t.pack(d_slots, int(lens.sum()), int(lens.max()), ids, cu)
        torch.cuda.synchronize()
        got, gcu = ids.cpu().numpy(), cu.cpu().numpy()
        assert np.array_equal(gcu[:n + 1], np.concatenate([[0], np.cumsum(lens)])) and np.all(gcu[n + 1:] == -7)
        assert np.array_equal(got[:len(got) - 16], np.concatenate(want)) and np.all(got[-16:] == -7)
        assert t.status() == (E.ELIS_OK, 0)
    t.pack(d_slots, int(lens.sum()) + 1, int(lens.max()), torch.empty(int(lens.sum()) + 1, dtype=torch.int32, device="cuda"), cu)
    assert t.status()[1] & E.ELIS_DEV_PACK_SIZE


@pytest.mark.parametrize("aging", [None, 10.0])
@pytest.mark.parametrize("a", [1, 16, 17, 63, 64, 65, 1023, 1024, 1025, 4096, 4097, 8192, 8193, 20001])
def test_select_over_the_table(a, aging):
    note(f"jobs select a={a} aging={aging}")
    rng = np.random.default_rng(a)
    t = JobTable(a + 5, 4)
    slots = rng.permutation(a + 5)[:a].astype(np.int32)
    arr = rng.integers(0, max(2, a // 3), size=a).astype(np.int64)
    pred = np.round(rng.standard_normal(a) * 100 + 250, -1).astype(np.float32)
    pred[rng.random(a) < 0.05] = np.nan
    wait = (rng.random(a) * 20).astype(np.float32)
    d_slots = dev(slots)
    t.start(d_slots, dev(arr))
    t.store_pred(d_slots, dev(pred))
    key = pred if aging is None else (pred.astype(np.float64) - aging * wait.astype(np.float64)).astype(np.float32)
    order = np.lexsort((np.arange(a), arr, np.where(np.isnan(key), np.inf, key), np.isnan(key)))
    for cap in sorted({0, 1, min(a, 37), min(a, 8192), min(a + 4, 8192)}):
        out = torch.full((cap + 8,), -1, dtype=torch.int32, device="cuda")
        count = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        t.select(d_slots, cap, out, count, wait=None if aging is None else dev(wait), aging=aging or 0.0)
        torch.cuda.synchronize()
        m = min(cap, a)
        assert int(count.item()) == m
        got = out.cpu().numpy()
        assert np.array_equal(got[:m], slots[order[:m]]) and np.all(got[m:] == -1)
    assert t.status() == (E.ELIS_OK, 0)


@pytest.mark.parametrize("a", [3, 64, 65, 2000])
def test_bad_slots_are_flagged_and_rank_last(a):
    note(f"jobs select with a bad slot a={a}")
    t = JobTable(a, 4)
    slots = np.arange(a, dtype=np.int32)
    t.start(dev(slots), dev(np.arange(a, dtype=np.int64)))
    t.store_pred(dev(slots), dev(np.ones(a, np.float32)))
    bad = slots.copy()
    bad[0] = a + 9
    out = torch.empty(a, dtype=torch.int32, device="cuda")
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    t.select(dev(bad), a, out, count)
    assert t.status()[1] & E.ELIS_DEV_BAD_SLOT
    assert np.array_equal(out.cpu().numpy(), np.concatenate([slots[1:], [a + 9]]))
