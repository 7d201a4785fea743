"""ep_dispatch_fused: layout and pack in one call (one kernel up to 256 experts and top-8).

Its outputs must equal the oracle's layout and pack, and the two-call path's
(ep_dispatch_layout then ep_dispatch) bit for bit: counts, offsets, rank counts and
offsets, slot_pos, row_src and the packed rows, also with routing errors.  The trace
shows which kernel ran, so the fused kernel's cases are known to have used it and the
fallback cases to have used the two kernels.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_40093_amd as ep
from gpu_cases import TOL_MAX_ABS, TOL_MEAN_ABS, combine_errors, from_config, make_case, say

pytestmark = pytest.mark.gpu

DEV = "cuda"
LAYOUT_KEYS = ("expert_counts", "expert_offsets", "rank_counts", "rank_offsets", "slot_pos", "row_src")


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def run_fused(idx_d, x_d, E, R, staging, buf=0, epoch=1):
    ep.trace_reset()
    ep.trace_enable(True)
    lay = ep.dispatch_fused(x_d, idx_d, E, R, staging, buf=buf, epoch=epoch)
    ep.trace_enable(False)
    torch.cuda.synchronize()
    kernels = set(ep.trace_read())
    return lay, kernels


def run_two_calls(idx_d, x_d, E, R, staging, k, buf=0, epoch=1):
    lay = ep.dispatch_layout(idx_d, E, R)
    ep.dispatch(x_d, lay.slot_pos, staging, topk=k, buf=buf, epoch=epoch, rank_offsets=lay.rank_offsets)
    torch.cuda.synchronize()
    return lay


def layout_np(lay):
    return {key: getattr(lay, key).cpu().numpy() for key in LAYOUT_KEYS}


FUSED_CASES = [
    # name, T, H, E, k, R, routing; every case fits the fused kernel (workgroups of 4 waves
    # up to 4096 entries, 8 up to 8192, 16 above: all three sizes appear)
    ("k2_e8_rows8", 4096, 4096, 8, 2, 4, "skewed"),
    ("k2_e16_rows2", 128, 1024, 16, 2, 4, "random"),
    ("k1_e4_rows1_ragged_tokens", 1001, 512, 4, 1, 2, "random"),
    ("k4_e32_rows4", 3000, 2048, 32, 4, 8, "skewed"),
    ("k2_e3_odd_experts", 17, 512, 3, 2, 3, "random"),
    ("k2_rows16", 300, 8192, 8, 2, 2, "random"),
    ("single_token", 1, 1024, 8, 2, 4, "random"),
    ("k4_empty_experts", 999, 512, 16, 4, 4, "firstk"),
    ("k2_limit_65536_slots", 32768, 512, 32, 2, 8, "random"),   # 8 tokens per wave
    ("k4_limit_65536_slots", 16384, 512, 16, 4, 4, "skewed"),
    ("k1_limit_65536_slots", 65536, 512, 2, 1, 1, "random"),    # 16 tokens per wave
    ("e33", 2000, 1024, 33, 2, 3, "random"),
    ("eight_wave_groups_ragged", 3001, 2048, 16, 2, 4, "skewed"),   # 6002 entries: 8-wave workgroups
    ("eight_wave_groups_k1", 5000, 1024, 8, 1, 2, "random"),
    ("one_expert", 100, 512, 1, 1, 1, "random"),
    ("ids_shorter_than_one_group", 3, 512, 4, 1, 2, "random"),      # no whole 4-id group
    # each side of the workgroup-size and count-loop switches (4096, 8192, 16384 entries)
    ("entries_4096", 2048, 512, 8, 2, 4, "random"),
    ("entries_4098", 2049, 512, 8, 2, 4, "random"),
    ("entries_8194", 4097, 512, 8, 2, 4, "random"),
    ("entries_16384", 8192, 512, 16, 2, 4, "skewed"),
    ("entries_16386", 8193, 512, 16, 2, 4, "skewed"),
    ("e64_r64_one_expert_per_rank", 5000, 2048, 64, 2, 64, "skewed"),
    ("e64_k4", 7000, 512, 64, 4, 8, "random"),
    # above 64 experts (four per lane in the scan) and top-8 (a row spans two 4-id
    # groups), up to 16384 entries (8192 for rows over 8 KiB); rows of 14 groups (H = 7168)
    ("decode_shape_k8_e256_rows14", 256, 7168, 256, 8, 8, "skewed"),
    ("k8_e16", 300, 512, 16, 8, 4, "random"),
    ("k8_e64_r64", 500, 1024, 64, 8, 64, "skewed"),
    ("k8_e128_8192", 1024, 512, 128, 8, 8, "random"),           # 8-wave workgroups
    ("k8_e128_limit_16384", 2048, 2048, 128, 8, 8, "random"),   # 16-wave workgroups
    ("e256_k2_limit_16384", 8192, 512, 256, 2, 8, "skewed"),    # 2 tokens per wave
    ("k8_rows14_limit_8192", 1024, 7168, 256, 8, 8, "random"),
    ("k8_ragged_tokens", 333, 512, 32, 8, 4, "random"),
    ("e65", 500, 512, 65, 2, 5, "random"),
    ("e128_k4", 2000, 1024, 128, 4, 8, "skewed"),
    ("e256_k1_limit_8192", 8192, 512, 256, 1, 8, "random"),     # 2 tokens per wave
    ("e256_r256_one_expert_per_rank", 300, 512, 256, 2, 256, "random"),
    ("e255_odd_wide", 200, 512, 255, 4, 5, "random"),
    ("e200_empty_experts", 999, 512, 200, 4, 4, "firstk"),
    ("rows14_k2", 200, 7168, 16, 2, 4, "random"),
    ("rows14_e128_k1", 600, 7168, 128, 1, 4, "random"),
    # below 1024 tokens a row is split over waves: 14 waves of one group each, two tokens
    # of 7 waves each (the ids need 14 waves' loads), and each side of the 1024-token switch
    ("split14_rows14", 100, 7168, 16, 2, 4, "random"),
    ("split7_two_tokens_per_group", 1000, 7168, 256, 8, 8, "skewed"),
    ("split_tokens_1023", 1023, 1024, 8, 2, 4, "random"),
    ("split_k1_four_tokens_per_group", 300, 2048, 16, 1, 4, "random"),  # m*k kept a multiple of 4
    ("split_tokens_1024", 1024, 1024, 8, 2, 4, "random"),
    # top-1: 4-wave workgroups below 2048 tokens, 8-wave ones from there up
    ("k1_tokens_2047", 2047, 512, 8, 1, 2, "random"),
    ("k1_tokens_2048", 2048, 512, 8, 1, 2, "random"),
    # under the limits of bytes packed (17406 entries: also the count loop with rows of 8 groups)
    ("k2_under_136_mib_packed", 8703, 4096, 8, 2, 4, "skewed"),
    ("k4_under_120_mib_packed", 3839, 4096, 16, 4, 4, "random"),
]


@pytest.mark.parametrize("spec", FUSED_CASES, ids=[c[0] for c in FUSED_CASES])
def test_fused_matches_oracle_and_two_calls(spec):
    name, T, H, E, k, R, kind = spec
    case = make_case(name, T, H, E, k, R, kind, seed=len(name))
    say(f"fused {name}: T={T} H={H} E={E} k={k} R={R}")
    ref = oracle.layout(case.topk_idx, E, R)
    assert ref.status == oracle.OK
    packed_ref = oracle.pack(case.x, ref.slot_pos, k)
    idx_d, x_d = to_dev(case.topk_idx), to_dev(case.x.view(np.int16))
    st = ep.Staging("hbm", T * k, H, R, num_buffers=2)
    lay, kernels = run_fused(idx_d, x_d, E, R, st, buf=1)
    assert "layout_pack" in kernels and "layout" not in kernels and "pack" not in kernels, kernels
    ep.layout_validate(lay)
    got = layout_np(lay)
    for key in LAYOUT_KEYS:
        assert np.array_equal(got[key], getattr(ref, key)), f"{key} differs from the oracle"
    packed = st.read_device("send", T * k, buf=1).cpu().numpy().view(np.uint16)
    assert packed.tobytes() == packed_ref.tobytes(), "packed rows differ from the oracle"
    # the two-call path on the other buffer set gives the same bytes
    lay2 = run_two_calls(idx_d, x_d, E, R, st, k, buf=0)
    for key in LAYOUT_KEYS:
        assert np.array_equal(getattr(lay2, key).cpu().numpy(), got[key]), f"{key}: fused != two calls"
    assert st.read_device("send", T * k, buf=0).cpu().numpy().tobytes() == packed.tobytes()
    st.close()


def test_fused_workloads_tiny_and_coarse():
    for name in ("tiny", "coarse"):
        case = from_config(name)
        say(f"fused workload {name}")
        ref = oracle.layout(case.topk_idx, case.E, case.R)
        st = ep.Staging("hbm", case.slots, case.H, case.R, num_buffers=1)
        lay, kernels = run_fused(to_dev(case.topk_idx), to_dev(case.x.view(np.int16)), case.E, case.R, st)
        assert "layout_pack" in kernels
        ep.layout_validate(lay)
        assert np.array_equal(lay.slot_pos.cpu().numpy(), ref.slot_pos)
        assert np.array_equal(lay.rank_offsets.cpu().numpy(), ref.rank_offsets)
        packed = st.read_device("send", case.slots).cpu().numpy().view(np.uint16)
        assert packed.tobytes() == oracle.pack(case.x, ref.slot_pos, case.k).tobytes()
        st.close()


def test_fused_repeated_calls_reuse_buffers():
    """Rounds on one layout object and staging: each round's routing and rows are new."""
    T, H, E, k, R = 2048, 1024, 8, 2, 4
    st = ep.Staging("hbm", T * k, H, R, num_buffers=2)
    lay = None
    for r in range(4):
        case = make_case(f"round{r}", T, H, E, k, R, "skewed" if r % 2 else "random", seed=100 + r)
        say(f"fused round {r}")
        lay = ep.dispatch_fused(to_dev(case.x.view(np.int16)), to_dev(case.topk_idx), E, R, st, buf=r % 2,
                                epoch=r + 1, out=lay)
        ep.layout_validate(lay)
        ref = oracle.layout(case.topk_idx, E, R)
        assert np.array_equal(lay.slot_pos.cpu().numpy(), ref.slot_pos), f"round {r}"
        assert np.array_equal(lay.expert_counts.cpu().numpy(), ref.expert_counts), f"round {r}"
        packed = st.read_device("send", T * k, buf=r % 2).cpu().numpy().view(np.uint16)
        assert packed.tobytes() == oracle.pack(case.x, ref.slot_pos, k).tobytes(), f"round {r}"
    st.close()


FALLBACK_CASES = [
    # outside the fused kernel's limits: the two kernels run
    ("e257_too_many_experts", 300, 512, 257, 2, 1),
    ("k8_over_16384_entries", 2049, 512, 16, 8, 4),
    ("e65_over_16384_entries", 8193, 512, 65, 2, 5),
    ("k8_rows14_over_8192_entries", 1025, 7168, 16, 8, 4),
    ("k3", 300, 512, 16, 3, 4),
    ("rows12", 200, 6144, 16, 2, 4),
    ("h520_not_whole_groups", 100, 520, 8, 2, 2),
    ("slots_over_limit", 40000, 512, 8, 2, 4),
    ("k2_136_mib_packed", 8704, 4096, 8, 2, 4),
    ("k4_120_mib_packed", 3840, 4096, 16, 4, 4),
]


@pytest.mark.parametrize("spec", FALLBACK_CASES, ids=[c[0] for c in FALLBACK_CASES])
def test_fallback_runs_two_kernels(spec):
    name, T, H, E, k, R = spec
    case = make_case(name, T, H, E, k, R, "random", seed=7)
    say(f"fused fallback {name}")
    ref = oracle.layout(case.topk_idx, E, R)
    st = ep.Staging("hbm", T * k, H, R, num_buffers=1)
    lay, kernels = run_fused(to_dev(case.topk_idx), to_dev(case.x.view(np.int16)), E, R, st)
    assert "layout_pack" not in kernels and {"layout", "pack"} <= kernels, kernels
    ep.layout_validate(lay)
    assert np.array_equal(lay.slot_pos.cpu().numpy(), ref.slot_pos)
    packed = st.read_device("send", T * k).cpu().numpy().view(np.uint16)
    assert packed.tobytes() == oracle.pack(case.x, ref.slot_pos, k).tobytes()
    st.close()


def test_misaligned_routing_falls_back():
    T, H, E, k, R = 512, 512, 8, 2, 4
    case = make_case("misaligned_idx", T, H, E, k, R, "random", seed=8)
    big = np.zeros((T + 1, k), np.int32)
    big[1:] = case.topk_idx
    idx_d = to_dev(big)[1:]                     # 8 bytes past a 16-byte boundary
    assert idx_d.data_ptr() % 16 != 0
    say("fused with a misaligned routing array")
    st = ep.Staging("hbm", T * k, H, R, num_buffers=1)
    lay, kernels = run_fused(idx_d, to_dev(case.x.view(np.int16)), E, R, st)
    assert "layout_pack" not in kernels
    ep.layout_validate(lay)
    ref = oracle.layout(case.topk_idx, E, R)
    assert np.array_equal(lay.slot_pos.cpu().numpy(), ref.slot_pos)
    st.close()


@pytest.mark.parametrize("k,E", [(1, 16), (2, 16), (4, 16), (8, 16), (2, 128), (8, 128)])
def test_fused_routing_errors_match_two_calls(k, E):
    """Ids outside [0,E) get no row and are reported; a repeated expert is reported and
    still ranked; the fused kernel and the layout kernel agree on every output."""
    T, H, R = 700, 512, 4   # at most 5600 entries: every case fits the fused kernel
    case = make_case(f"errors_k{k}_e{E}", T, H, E, k, R, "random", seed=9)
    idx = case.topk_idx.copy()
    idx[5, 0] = E
    idx[321, k - 1] = -7
    if k > 1:
        idx[600, 1] = idx[600, 0]
    say(f"fused routing errors k={k} E={E}")
    idx_d, x_d = to_dev(idx), to_dev(case.x.view(np.int16))
    st = ep.Staging("hbm", T * k, H, R, num_buffers=2)
    lay, kernels = run_fused(idx_d, x_d, E, R, st, buf=0)
    assert "layout_pack" in kernels
    with pytest.raises(ep.EPError) as ei:
        ep.layout_validate(lay)
    assert ei.value.status == 2
    msg = str(ei.value)
    assert "outside" in msg and (k == 1 or "repeated" in msg), msg
    got = layout_np(lay)
    assert got["slot_pos"][5 * k] == -1 and got["slot_pos"][321 * k + k - 1] == -1
    lay2 = run_two_calls(idx_d, x_d, E, R, st, k, buf=1)
    with pytest.raises(ep.EPError):
        ep.layout_validate(lay2)
    for key in LAYOUT_KEYS:
        if key == "row_src":   # rows no slot maps to are left unwritten by both paths
            continue
        assert np.array_equal(getattr(lay2, key).cpu().numpy(), got[key]), f"{key}: fused != two calls"
    valid = got["slot_pos"] >= 0
    rows = got["slot_pos"][valid]
    a = st.read_device("send", T * k, buf=0).cpu().numpy()[rows]
    b = st.read_device("send", T * k, buf=1).cpu().numpy()[rows]
    assert a.tobytes() == b.tobytes()
    # the next good routing on the same workspace clears the status
    lay = ep.dispatch_fused(x_d, to_dev(case.topk_idx), E, R, st, out=lay)
    ep.layout_validate(lay)
    st.close()


@pytest.mark.parametrize("first,second", [(1, 2), (1, 6), (3, 4), (7, 0)],
                         ids=["same_half", "across_halves", "halves_edge", "last_and_first"])
def test_fused_k8_repeated_expert(first, second):
    """A top-8 row naming one expert twice, within one of its 4-id halves or across them
    (the halves sit in neighbouring lanes): reported, and equal to the two-call path."""
    T, H, E, R = 300, 512, 32, 4
    case = make_case("k8_repeat", T, H, E, 8, R, "random", seed=12)
    idx = case.topk_idx.copy()
    idx[123, second] = idx[123, first]
    say(f"fused top-8 repeated expert at slots {first} and {second}")
    idx_d, x_d = to_dev(idx), to_dev(case.x.view(np.int16))
    st = ep.Staging("hbm", T * 8, H, R, num_buffers=2)
    lay, kernels = run_fused(idx_d, x_d, E, R, st, buf=0)
    assert "layout_pack" in kernels
    with pytest.raises(ep.EPError, match="repeated"):
        ep.layout_validate(lay)
    lay2 = run_two_calls(idx_d, x_d, E, R, st, 8, buf=1)
    with pytest.raises(ep.EPError, match="repeated"):
        ep.layout_validate(lay2)
    for key in LAYOUT_KEYS:
        assert np.array_equal(getattr(lay2, key).cpu().numpy(), getattr(lay, key).cpu().numpy()), key
    st.close()


def test_fused_pinned_default_mode_host_leg():
    """Pinned staging, default mode: the fused kernel, then the SDMA leg and its flags."""
    case = make_case("pinned_fused", 1024, 2048, 8, 2, 4, "random", seed=10)
    say("fused dispatch with pinned staging")
    st = ep.Staging("pinned", case.slots, case.H, case.R, num_buffers=2)
    lay, kernels = run_fused(to_dev(case.topk_idx), to_dev(case.x.view(np.int16)), case.E, case.R, st,
                             buf=1, epoch=5)
    assert "layout_pack" in kernels
    st.status()
    ref = oracle.layout(case.topk_idx, case.E, case.R)
    assert np.array_equal(lay.slot_pos.cpu().numpy(), ref.slot_pos)
    sent = st.host_array("send", 1)[:case.slots]
    assert sent.tobytes() == oracle.pack(case.x, ref.slot_pos, case.k).tobytes()
    flags = st.host_array("send_flags", 1)
    assert flags[0] == 5
    st.close()


def test_fused_exchange_mode_falls_back():
    case = make_case("pinned_exchange", 512, 1024, 8, 2, 4, "random", seed=11, gates="uniform")
    say("fused dispatch with an exchange mode")
    st = ep.Staging("pinned", case.slots, case.H, case.R, num_buffers=1)
    st.set_mode(ep.MODE_PER_SENDER, 0)
    peers = ep.SimPeers(st, echo=True)
    peers.post(0, 3, case.slots)
    lay, kernels = run_fused(to_dev(case.topk_idx), to_dev(case.x.view(np.int16)), case.E, case.R, st, epoch=3)
    assert "layout_pack" not in kernels and "pack" in kernels
    w = to_dev(case.topk_w)
    out32 = ep.combine(st, lay.slot_pos, w, out_dtype=torch.float32, epoch=3, rank_offsets=lay.rank_offsets)
    st.status()
    peers.drain()
    ref = oracle.layout(case.topk_idx, case.E, case.R)
    assert np.array_equal(lay.slot_pos.cpu().numpy(), ref.slot_pos)
    sent = st.host_array("send", 0)[:case.slots]
    assert sent.tobytes() == oracle.pack(case.x, ref.slot_pos, case.k).tobytes()
    # identity experts (the peers echo the rows) and gates of 1/2: combine returns x exactly
    xf = torch.from_numpy(case.x.view(np.int16)).view(torch.bfloat16).float()
    assert torch.equal(out32.cpu(), xf)
    peers.close()
    st.close()


def test_fused_argument_errors_enqueue_nothing():
    case = make_case("fused_args", 64, 512, 8, 2, 4, "random", seed=12)
    idx_d, x_d = to_dev(case.topk_idx), to_dev(case.x.view(np.int16))
    say("fused argument checks")
    small = ep.Staging("hbm", case.slots - 1, 512, 4, num_buffers=1)
    with pytest.raises(ep.EPError, match="exceed"):
        ep.dispatch_fused(x_d, idx_d, 8, 4, small)
    st = ep.Staging("hbm", case.slots, 512, 4, num_buffers=1)
    with pytest.raises(ep.EPError, match="E % R"):
        ep.dispatch_fused(x_d, idx_d, 8, 3, st)
    with pytest.raises(ep.EPError, match="buffer"):
        ep.dispatch_fused(x_d, idx_d, 8, 4, st, buf=1)
    flat = torch.zeros(64 * 512 + 8, dtype=torch.int16, device=DEV)
    with pytest.raises(ep.EPError, match="aligned"):
        ep.dispatch_fused(flat[1:1 + 64 * 512].view(64, 512), idx_d, 8, 4, st)
    small.close()
    st.close()


def test_trace_percentiles():
    """The trace's percentiles lie between the minimum and the maximum, in order."""
    case = make_case("trace", 2048, 1024, 8, 2, 4, "random", seed=13)
    idx_d, x_d = to_dev(case.topk_idx), to_dev(case.x.view(np.int16))
    st = ep.Staging("hbm", case.slots, case.H, case.R, num_buffers=1)
    say("trace percentiles")
    ep.trace_reset()
    ep.trace_enable(True)
    lay = None
    for _ in range(25):
        lay = ep.dispatch_fused(x_d, idx_d, case.E, case.R, st, out=lay)
    ep.trace_enable(False)
    s = ep.trace_read()["layout_pack"]
    assert s["count"] == 25
    assert 0 < s["min_ms"] <= s["p10_ms"] <= s["p50_ms"] <= s["p90_ms"] <= s["max_ms"]
    st.close()


def test_fused_dispatch_and_combine_replay_in_a_graph():
    """The benchmark's step (one-kernel dispatch, then combine; HBM staging) captured once
    in a HIP graph and replayed with new rows, a new routing and new gates written into the
    captured inputs each time: every replay's layout, packed rows and combine match the
    oracle's for its inputs."""
    T, H, E, k, R = 1024, 2048, 8, 2, 4
    base = make_case("fused_graph", T, H, E, k, R, "random", seed=40)
    st = ep.Staging("hbm", T * k, H, R, num_buffers=1)
    x = to_dev(base.x.view(np.int16))
    idx = to_dev(base.topk_idx)
    w = to_dev(base.topk_w)
    y = to_dev(base.y.view(np.int16))
    st.write_device("recv", y)
    out = torch.empty((T, H), dtype=torch.bfloat16, device=DEV)
    lay = ep.dispatch_fused(x, idx, E, R, st)
    ep.combine(st, lay.slot_pos, w, out=out)
    torch.cuda.synchronize()
    say("fused step: graph capture")
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            ep.dispatch_fused(x, idx, E, R, st, out=lay)
            ep.combine(st, lay.slot_pos, w, out=out)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    for rep in range(4):
        say(f"fused step: graph replay {rep}")
        case = make_case("fused_graph_rep", T, H, E, k, R, "skewed" if rep % 2 else "random", seed=50 + rep)
        x.copy_(to_dev(case.x.view(np.int16)))
        idx.copy_(to_dev(case.topk_idx))
        w.copy_(to_dev(case.topk_w))
        g.replay()
        torch.cuda.synchronize()
        ep.layout_validate(lay)
        ref = oracle.layout(case.topk_idx, E, R)
        for key in LAYOUT_KEYS:
            assert np.array_equal(getattr(lay, key).cpu().numpy(), getattr(ref, key)), f"replay {rep}: {key}"
        packed = st.read_device("send", T * k).cpu().numpy().view(np.uint16)
        assert packed.tobytes() == oracle.pack(case.x, ref.slot_pos, k).tobytes(), f"replay {rep}: packed"
        exact, _, _ = oracle.combine(base.y, ref.slot_pos, case.topk_w)
        mx, mean = combine_errors(out.view(torch.int16).cpu().numpy().view(np.uint16), exact)
        assert mx <= TOL_MAX_ABS and mean <= TOL_MEAN_ABS, f"replay {rep}: combine {mx} {mean}"
    st.close()


def _random_fused_shapes(n=48, seed=2024):
    """Seeded shapes inside the one kernel's limits: every k, expert counts from 1 to 256
    with a rank count dividing them, every row length, token counts up to each limit."""
    rng = np.random.default_rng(seed)
    shapes = []
    while len(shapes) < n:
        k = int(rng.choice([1, 2, 4, 8]))
        E = int(rng.integers(max(k, 1), 257))
        divisors = [r for r in range(1, min(E, 32) + 1) if E % r == 0]
        R = int(rng.choice(divisors))
        G = int(rng.choice([1, 2, 4, 8, 14, 16]))
        H = 512 * G
        limit = 65536 if (E <= 64 and k <= 4) else (16384 if H <= 4096 else 8192)
        T = int(rng.integers(1, min(limit // k, 20000) + 1))
        if T * H * 2 * (k + 1) > (1 << 28):   # keep each case under 256 MiB of rows
            continue
        kind = str(rng.choice(["random", "skewed", "firstk"]))
        shapes.append((f"r{len(shapes)}_T{T}_H{H}_E{E}_k{k}_R{R}_{kind}", T, H, E, k, R, kind))
    return shapes


@pytest.mark.parametrize("spec", _random_fused_shapes(), ids=lambda c: c[0])
def test_fused_random_shapes(spec):
    name, T, H, E, k, R, kind = spec
    case = make_case(name, T, H, E, k, R, kind, seed=len(name) + T)
    say(f"fused random shape {name}")
    ref = oracle.layout(case.topk_idx, E, R)
    st = ep.Staging("hbm", T * k, H, R, num_buffers=1)
    lay, kernels = run_fused(to_dev(case.topk_idx), to_dev(case.x.view(np.int16)), E, R, st)
    assert "layout_pack" in kernels, kernels
    ep.layout_validate(lay)
    for key in LAYOUT_KEYS:
        assert np.array_equal(getattr(lay, key).cpu().numpy(), getattr(ref, key)), f"{key} differs"
    packed = st.read_device("send", T * k).cpu().numpy().view(np.uint16)
    assert packed.tobytes() == oracle.pack(case.x, ref.slot_pos, k).tobytes(), "packed rows differ"
    st.close()
