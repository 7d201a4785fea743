"""The combine with slots that have no row, over every batch length (k = 1..8 in one batch,
9 and 16 in several), chunk length and row remainder, bf16 and fp32 results.

Reference: the sum in float64 over the slots with a row.  The kernel does n fp32 FMAs from
+0 (n slots with a row), each with a relative rounding of 2^-24 of its result, and every
partial sum is at most S = sum |w y| (1 + n 2^-24): the fp32 result is within n 2^-24 S
(taken as (n + 1) 2^-24 S), a bf16 result within half a bf16 step more (a step is 2^-7 of
the power of two below the value, so half a step is at most 2^-8 of the value).
A token without any row is +0, bit for bit.
"""
import numpy as np
import pytest
import torch

import paper_2609_40093_amd as ep
from gpu_cases import say
from paper_2609_40093_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H", [8, 512, 520, 1024, 2048, 3072, 6152, 7168])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 16])
def test_slots_without_rows(k, H):
    T, rows = 129, 97
    rng = np.random.default_rng([k, H])
    y = synth.normal_bf16_rows(np.random.SeedSequence([k, H]), rows, H)
    w = rng.standard_normal((T, k)).astype(np.float32)
    pos = rng.integers(0, rows, (T, k)).astype(np.int32)
    # tokens with every slot, with about half and with few; -1 and rows past the last one
    missing = rng.random((T, k)) < np.array([0.0, 0.5, 0.9])[np.arange(T) % 3][:, None]
    pos[missing] = rng.choice(np.array([-1, rows, rows + 7, 2**31 - 1], np.int32), int(missing.sum()))
    has = ~missing
    yf = synth.bf16_bits_to_f32(y).astype(np.float64)
    terms = np.where(has[:, :, None], w.astype(np.float64)[:, :, None] * yf[np.where(has, pos, 0)], 0.0)
    exact, size = terms.sum(axis=1), np.abs(terms).sum(axis=1)
    bound = (has.sum(axis=1)[:, None] + 1) * 2.0**-24 * size
    say(f"combine_rows with missing slots: k={k} H={H}")
    args = [torch.from_numpy(a).to(DEV) for a in (y.view(np.int16), pos.reshape(-1), w)]
    for dt, extra in ((torch.float32, 0.0), (torch.bfloat16, 2.0**-8)):
        out = torch.full((T, H), 7.0, dtype=dt, device=DEV)
        ep.combine_rows(args[0], args[1], args[2], out)
        got = out.double().cpu().numpy()
        assert (np.abs(got - exact) <= bound + extra * (np.abs(exact) + bound)).all()
        empty = ~has.any(axis=1)
        assert not out.view(torch.int32 if dt == torch.float32 else torch.int16).cpu().numpy()[empty].any()


@pytest.mark.parametrize("k,H,dtype", [(8, 7168, torch.bfloat16), (6, 6152, torch.bfloat16), (5, 3072, torch.float32),
                                       (7, 3592, torch.float32), (8, 4096, torch.float32)])
def test_missing_slots_in_large_outputs(k, H, dtype):
    """Slots without rows above 44 MiB of output and more than four slots, where a combine of a
    whole layout also reserves LDS: through ep_combine and ep_combine_rows, the same bits."""
    T, rows = 4096, 5000
    gen = torch.Generator(device=DEV).manual_seed(k * H)
    y = torch.empty((rows, H), device=DEV, dtype=torch.bfloat16).normal_(generator=gen)
    w = torch.randn((T, k), device=DEV, generator=gen)
    pos = torch.randint(0, rows, (T, k), device=DEV, generator=gen, dtype=torch.int32)
    share = torch.tensor([0.0, 0.5, 0.9], device=DEV)[torch.arange(T, device=DEV) % 3]
    missing = torch.rand((T, k), device=DEV, generator=gen) < share[:, None]
    pos[missing] = torch.where(torch.rand(int(missing.sum()), device=DEV, generator=gen) < 0.5, -1, T * k + 3).to(torch.int32)
    assert T * H * (2 if dtype == torch.bfloat16 else 4) > 44 << 20
    exact = torch.zeros((T, H), dtype=torch.float64, device=DEV)
    size = torch.zeros_like(exact)
    for j in range(k):
        term = torch.where(missing[:, j], 0.0, w[:, j].double())[:, None] * y[pos[:, j].clamp(0, rows - 1).long()].double()
        exact += term
        size += term.abs()
    bound = ((~missing).sum(dim=1)[:, None] + 1) * 2.0**-24 * size
    if dtype == torch.bfloat16:
        bound = bound + 2.0**-8 * (exact.abs() + bound)
    st = ep.Staging("hbm", T * k, H, 1, num_buffers=1)
    st.write_device("recv", y.view(torch.int16))
    flat = pos.reshape(-1).contiguous()
    say(f"combine of {T} tokens with missing slots: k={k} H={H} {dtype}")
    out = ep.combine(st, flat, w, out=torch.full((T, H), 7.0, dtype=dtype, device=DEV))
    assert (out.double() - exact).abs().le(bound).all()
    say("and from the caller's rows")
    assert torch.equal(ep.combine_rows(y, flat, w, torch.full((T, H), 7.0, dtype=dtype, device=DEV)), out)
    st.close()


@pytest.mark.parametrize("H,dtype", [(7168, torch.bfloat16), (3584, torch.float32)])
def test_store_policies_agree(H, dtype):
    """The combine stores by its output's bytes and by how its rows were dispatched (one kernel,
    two, a caller's own positions): 56 MiB of output, the same bits each way."""
    T, E, k, R = 4096, 64, 2, 4
    gen = torch.Generator(device=DEV).manual_seed(H)
    idx = torch.rand((T, E), device=DEV, generator=gen).topk(k, dim=1).indices.to(torch.int32)
    w = torch.rand((T, k), device=DEV, generator=gen)
    x = torch.randint(-2**15, 2**15, (T, H), device=DEV, dtype=torch.int16, generator=gen)
    y = torch.empty((T * k, H), device=DEV, dtype=torch.bfloat16).normal_(generator=gen)
    st = ep.Staging("hbm", T * k, H, R, num_buffers=2)
    outs = []
    for buf, one in ((0, True), (1, False), (1, True), (0, False)):
        say(f"combine after a dispatch in {'one kernel' if one else 'two'}: buffer {buf} H={H} {dtype}")
        if one:
            lay = ep.dispatch_fused(x, idx, E, R, st, buf=buf, epoch=1)
        else:
            lay = ep.dispatch_layout(idx, E, R)
            ep.dispatch(x, lay.slot_pos, st, topk=k, buf=buf, epoch=1, rank_offsets=lay.rank_offsets)
        assert torch.equal(ep.pack(x, lay.slot_pos, torch.empty_like(y.view(torch.int16)), topk=k),
                           st.read_device("send", T * k, buf=buf))
        st.write_device("recv", y.view(torch.int16), buf=buf)
        outs.append(ep.combine(st, lay.slot_pos, w, out=torch.empty((T, H), dtype=dtype, device=DEV), buf=buf, epoch=1))
    outs.append(ep.combine_rows(y, lay.slot_pos, w, torch.empty((T, H), dtype=dtype, device=DEV)))
    terms = w.double()[:, :, None] * y[lay.slot_pos.long()].view(T, k, H).double()
    exact, bound = terms.sum(dim=1), (k + 1) * 2.0**-24 * terms.abs().sum(dim=1)
    if dtype == torch.bfloat16:
        bound = bound + 2.0**-8 * (exact.abs() + bound)
    assert (outs[0].double() - exact).abs().le(bound).all()
    for out in outs[1:]:
        assert torch.equal(out, outs[0])
    st.close()
