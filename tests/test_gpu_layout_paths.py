"""The layout on either side of its dispatch rules, against the oracle bit for bit: one
kernel or two, top-k with rows in registers (1, 2, 4, 8) or general, 4- or 16-wave rank
workgroups, runs of one tile shared by several workgroups, one or several counters per
expert, expert counts not a multiple of four, a routing array that is not 16-byte aligned,
the window layout; and a bad id and a repeated expert in the first and the last row.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_40093_amd as ep
from gpu_cases import routing, say

pytestmark = pytest.mark.gpu
DEV = "cuda"
ONE = 20480  # entries up to which one kernel does the layout (k of 1, 2, 4, 8)

CASES = [(T, E, k) for k in (1, 2, 4, 8) for T, E in ((ONE // k - 1, 96), (ONE // k, 257), (ONE // k + 1, 130))]
CASES += [(1365, 60, 3), (1366, 60, 3), (683, 513, 6), (7, 600, 5),            # general rows, at one tile's end
          (131072 // 8 + 3, 256, 8), (131072 // 4, 64, 4), (40001, 33, 3),     # 4- and 16-wave runs
          (100000, 160, 3), (36864, 512, 8),                                   # a tile's last run ends with the tile
          (60000, 300, 8), (9000, 2047, 8), (33001, 2048, 2), (300, 2048, 64), (70, 100, 96)]


def device(idx, misaligned):
    if not misaligned:
        return torch.from_numpy(idx).to(DEV)
    flat = torch.empty(idx.size + 1, dtype=torch.int32, device=DEV)[1:]
    return flat.copy_(torch.from_numpy(idx.reshape(-1)).to(DEV)).view(idx.shape)


@pytest.mark.parametrize("T,E,k", CASES)
def test_layout_paths(T, E, k):
    R = next(r for r in (8, 5, 4, 3, 2, 1) if E % r == 0)
    idx = routing("skewed" if (T + E) % 2 else "random", T, E, k, seed=T + E)
    want = oracle.layout(idx, E, R)
    assert want.status == oracle.OK
    for misaligned in (False, True):
        say(f"layout T={T} E={E} k={k} R={R} misaligned={misaligned}")
        lay = ep.dispatch_layout(device(idx, misaligned), E, R)
        ep.layout_validate(lay)
        for key in ("expert_counts", "expert_offsets", "rank_counts", "rank_offsets", "slot_pos", "row_src"):
            assert np.array_equal(getattr(lay, key).cpu().numpy(), getattr(want, key)), (key, misaligned)
    lo, hi = E // 3, min(E, E // 3 + max(1, E // 4))
    local = oracle.local_layout(idx, E, lo, hi)
    say(f"window layout [{lo}, {hi})")
    got = ep.dispatch_layout_local(device(idx, False), E, lo, hi)
    assert np.array_equal(got.slot_pos.cpu().numpy(), local.slot_pos)
    assert np.array_equal(got.local_offsets.cpu().numpy(), local.local_offsets)
    rows = int(local.local_offsets[-1])
    assert np.array_equal(got.row_src.cpu().numpy()[:rows], local.row_src[:rows])


@pytest.mark.parametrize("T,E,k", [c for c in CASES if c[2] > 1])
@pytest.mark.parametrize("row", [0, -1])
def test_bad_routing_is_found(T, E, k, row):
    idx = routing("random", T, E, k, seed=5)
    for what, slot, value in (("id past the experts", k - 1, E), ("negative id", 0, -7),
                              ("repeated expert", k - 1, idx[row, 0])):
        bad = idx.copy()
        bad[row, slot] = value
        say(f"layout with a {what}: T={T} E={E} k={k} row {row}")
        with pytest.raises(ep.EPError, match="repeated" if what.startswith("rep") else "outside"):
            ep.layout_validate(ep.dispatch_layout(device(bad, False), E, 1))
    twice = idx.copy()
    twice[row, :2] = E + 3  # a repeated id that names no expert is only out of range
    lay = ep.dispatch_layout(device(twice, False), E, 1)
    torch.cuda.synchronize()
    assert int(lay.workspace[:4].view(torch.int32)) == 1


@pytest.mark.parametrize("T,E,k", [(1366, 60, 3), (8003, 250, 7), (1301, 130, 63), (700, 2048, 64), (1000, 96, 65),
                                   (90, 700, 130), (40001, 33, 3)])
def test_general_rows_are_checked_wherever_they_lie(T, E, k):
    """Top-k without rows in registers: a repeated expert is found in rows that two tiles share,
    at both ends of a wave's rows and in any two slots; equal slots of two rows are no repeat."""
    idx = routing("random", T, E, k, seed=11)
    idx[1::7] = idx[0]  # neighbouring rows with the same experts
    clean = ep.dispatch_layout(device(idx, False), E, 1)
    ep.layout_validate(clean)
    per_wave = max(1, 64 // k)
    rows = {0, 1, per_wave - 1, per_wave, T // 2, T - 1}
    rows |= {entry // k for entry in range(1024, T * k, 1024)}  # tiles end at multiples of 1024 (or of 256)
    rng = np.random.default_rng(k)
    for row in sorted(r for r in rows if r < T)[:48]:
        a, b = sorted(rng.choice(k, 2, replace=False))
        bad = idx.copy()
        bad[row, b] = bad[row, a]
        say(f"repeat in slots {a}, {b} of row {row}: T={T} E={E} k={k}")
        lay = ep.dispatch_layout(device(bad, False), E, 1)
        torch.cuda.synchronize()
        assert int(lay.workspace[:4].view(torch.int32)) == 2, row
        if E > 300:
            local = ep.dispatch_layout_local(device(bad, False), E, 5, 9)
            torch.cuda.synchronize()
            assert int(local.workspace[:4].view(torch.int32)) == 2, row


def test_a_long_row_costs_no_more_per_id_than_a_short_one():
    """The layout of 400000 entries in rows of 64 ids takes at most twice that in rows of 8 (16 and
    14 us; a check that reloads every earlier id of a row makes it 58)."""
    us = {}
    for k in (8, 64):
        T, E = 400000 // k, 128
        table = routing("random", 512, E, k, seed=k)
        idx = device(table[np.random.default_rng(k).integers(0, 512, T)], False)
        lay = ep.dispatch_layout(idx, E, 1)
        say(f"layout time T={T} E={E} k={k}")
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(100):
                ep.dispatch_layout(idx, E, 1, out=lay)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 10)
        us[k] = min(times)
    assert us[64] <= 2 * us[8], us
