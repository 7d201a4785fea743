"""The pack on either side of its rules -- slots per workgroup, chunk lengths, rows that are
no whole number of 64-vector groups, 64-byte pieces or chunks, the store policies by bytes
packed -- byte for byte against the definition, with slots that have no row left unwritten.
"""
import pytest
import torch

import paper_2609_40093_amd as ep
from gpu_cases import say

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [(T, H, k) for k in (1, 2, 3, 5, 7, 16, 17) for T, H in ((37, 8), (65, 520), (33, 2888), (700, 1536))]
CASES += [(1025, 7176, 3),       # 15 groups, partly filled, enough waves for whole rows
          (400, 2512, 3), (400, 2520, 3), (400, 2504, 3),  # the lead reaches the last two groups
          (300, 8712, 2),        # 18 groups
          (600, 9736, 6),        # 20 groups
          (130, 8640, 4),        # 17 groups: no divisor, chunks of 16 and 1
          (2500, 2056, 4), (5200, 2056, 4),    # rows of 16-byte ends
          (4100, 4128, 4), (4100, 4096, 4)]    # 64-byte and whole-line rows, past 128 MiB packed


# through ep_dispatch, where whole rows of top-1 and of top-2 below 80 MiB take a wave per token
DISPATCH = [(T, H, k) for k in (1, 2, 3) for T, H in ((1, 512), (37, 6144), (1025, 1536), (300, 9216), (65, 17408))]
DISPATCH += [(3413, 6144, 2), (3414, 6144, 2), (700, 520, 2), (700, 520, 1), (11000, 6144, 1)]  # the last: 129 MiB


@pytest.mark.parametrize("T,H,k,by", [(*c, "pack") for c in CASES] + [(*c, "dispatch") for c in DISPATCH])
def test_pack_rows(T, H, k, by):
    gen = torch.Generator(device=DEV).manual_seed(T * 31 + H + k)
    x = torch.randint(-2**15, 2**15, (T, H), device=DEV, dtype=torch.int16, generator=gen)
    rows = T * k
    pos = torch.randperm(rows, device=DEV, generator=gen).to(torch.int32)
    missing = torch.rand(rows, device=DEV, generator=gen) < 0.2
    beyond = missing & (torch.arange(rows, device=DEV) % 2 == 0)
    given = torch.where(missing, torch.where(beyond, rows + pos, -1 - pos), pos).to(torch.int32)
    out = torch.full((rows + 1, H), 0x5A5A, dtype=torch.int16, device=DEV)  # a row more than max_rows
    say(f"{by} T={T} H={H} k={k}")
    if by == "pack":
        ep.pack(x, given, out[:rows], topk=k)
    else:
        st = ep.Staging("hbm", rows, H, 1, num_buffers=1)
        st.write_device("send", out[:rows])
        ep.dispatch(x, given, st, topk=k)
        out[:rows] = st.read_device("send", rows)
        st.close()
    want = torch.full_like(out, 0x5A5A)
    keep = ~missing
    want[pos[keep].long()] = x.repeat_interleave(k, dim=0)[keep]
    assert torch.equal(out, want)
