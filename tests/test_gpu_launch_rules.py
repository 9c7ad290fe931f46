"""The launch rules at their edges, each step (fused and as three calls)
against the oracle: one workgroup per (request, KV head) with as many waves
as it has tiles, and grouped-head workgroups of fewer waves where that keeps
every one resident."""

import random

import pytest
import torch

from oracle import step as ostep
from paper_2609_19702_amd import binding as B
from paper_2609_19702_amd import synth
from tests.gpu_util import (DEV, c_replay_states, check_layer_vs_oracle, fp8_request_arrays,
                            launches, request_arrays, say, states_to_buffer)
from tests.test_gpu_mfma_tiles import positions, run

pytestmark = pytest.mark.gpu

CASES = [
    # name, B, Hq, Hkv, d, L_p, grid, N_r, N_att, sinks, splits > 1, waves
    # one query head per KV head: 16-row tiles at d = 128, 40-row ones at d = 64
    ("wide_no_prompt", 12, 2, 2, 128, 0, 8, 20, 6, 0, False, 1),
    ("wide_16_tiles", 12, 3, 3, 128, 225, 12, 60, 16, 0, False, 16),
    ("wide_18_tiles", 12, 4, 4, 128, 256, 24, 256, 29, 4, False, 16),
    ("wide_512_rows", 33, 2, 2, 128, 103, 40, 600, 409, 0, False, 16),
    ("wide_513_rows", 33, 2, 2, 128, 104, 40, 600, 409, 0, True, 4),
    ("few_448_rows", 8, 2, 2, 128, 70, 40, 600, 378, 4, False, 16),
    ("few_449_rows", 8, 2, 2, 128, 71, 40, 600, 378, 4, True, 2),
    ("wide_d64", 12, 5, 5, 64, 121, 20, 130, 41, 4, False, 6),
    ("wide_256_pairs", 16, 16, 16, 64, 41, 12, 60, 9, 0, False, 3),
    ("pairs_257", 257, 1, 1, 64, 41, 12, 60, 9, 0, False, 2),
    # grouped heads: up to 10 tiles of 32 rows, or at least 64 pairs
    ("mfma_10_tiles", 12, 8, 2, 128, 256, 24, 200, 64, 0, False, 8),
    ("mfma_11_tiles", 12, 8, 2, 128, 257, 24, 200, 64, 0, True, 2),
    ("mfma_63_pairs", 21, 6, 3, 64, 300, 24, 200, 90, 4, True, 4),
    ("mfma_64_pairs", 16, 32, 4, 64, 300, 24, 200, 90, 4, False, 8),
    # more workgroups than CUs: four waves while every workgroup is resident,
    # then three (d = 64) and two
    ("mfma_257_pairs", 257, 2, 1, 64, 70, 12, 60, 9, 0, False, 4),
    ("mfma_513_pairs", 513, 2, 1, 64, 70, 12, 60, 9, 0, False, 4),
    ("mfma_769_pairs", 769, 2, 1, 64, 70, 12, 60, 9, 0, False, 3),
    ("mfma_1025_pairs", 1025, 2, 1, 64, 70, 12, 60, 9, 0, False, 2),
    ("mfma_d128_512_pairs", 512, 2, 1, 128, 70, 12, 60, 9, 0, False, 4),
    ("mfma_d128_513_pairs", 513, 2, 1, 128, 70, 12, 60, 9, 0, False, 2),
    # skip lists of 1024 entries, and longer ones (no kept lists)
    ("skips_1024", 17, 4, 4, 64, 20, 40, 1324, 300, 0, False, 9),
    ("skips_1025", 17, 4, 4, 64, 20, 40, 1325, 300, 0, False, 9),
    ("long_skips_d128", 17, 4, 4, 128, 20, 40, 1500, 310, 4, False, 16),
    ("long_skips_mfma", 17, 8, 4, 128, 40, 40, 1500, 310, 4, False, 8),
    ("long_skips_split", 17, 4, 4, 64, 20, 48, 1999, 560, 4, True, 4),
    # selections outside the decode kernel: windows of 257 and of over 512 keys,
    # and one whose softmaxes do not fit in LDS (2100 keys of eight heads)
    ("select_257_g2", 12, 4, 2, 64, 300, 30, 500, 257, 0, True, 3),
    ("select_600_g4", 12, 8, 2, 128, 40, 36, 1100, 600, 4, True, 3),
    ("select_600_g1", 12, 2, 2, 128, 40, 36, 1100, 600, 4, True, 3),
    ("select_2100_g8", 12, 8, 1, 64, 30, 48, 2300, 2100, 0, True, 5),
    ("mfma_g8_528_pairs", 33, 128, 16, 64, 70, 12, 100, 40, 4, False, 4),
]


@pytest.mark.parametrize("kv_type", ["bf16", "fp8"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_launch_rule_edges_match_oracle(case, kv_type):
    name, Bn, Hq, Hkv, d, Lp, grid, N_r, N_att, sinks, split, waves = case
    L = grid * grid
    p = B.make_params(Lp, grid, grid, N_r, N_att, B.MODE_DIAGONAL, sinks)
    s = B.make_shape(Bn, Hq, Hkv, d)
    info = B.launch_info(p, s)
    say("launch rule", name, kv_type, "splits", info.max_splits, "waves", info.waves_per_group)
    assert (info.max_splits > 1) == split and info.waves_per_group == waves
    ts = positions(Bn, L, N_r, N_att, seed=Bn + d)
    rng = random.Random(N_att * 13 + Hkv)
    w = synth.Workload(name, 1, Bn, Hq, Hkv, d, Lp, grid, grid, N_r, outlier_frac=0.01)
    kv = synth.layer_kv(w, 0, DEV)
    arrays_of = lambda b: request_arrays(kv, b, Lp)  # noqa: E731
    if kv_type == "fp8":
        kv = synth.to_fp8(kv)
        arrays_of = lambda b: fp8_request_arrays(kv, b, Lp, Hkv)  # noqa: E731
    q = synth.layer_query(w, 0, DEV)
    # the oracle's states count steps from the first position after the sinks
    states, _ = c_replay_states(N_r, N_att - sinks, L, [t - sinks for t in ts], Hkv, rng)
    st0 = states_to_buffer(p, s, states, ts)
    pos = torch.tensor(ts, dtype=torch.int32, device=DEV)
    lay = B.kv_layout(kv.k, k_scale=kv.k_scale, v_scale=kv.v_scale)
    arrays = [arrays_of(b) for b in range(Bn)]
    got = []
    for fused in (True, False):
        bufs, st = run(p, s, q, kv, pos, st0, fused, lay)
        forced = check_layer_vs_oracle(p, s, q, arrays, ts, states, bufs.plan, bufs.out, st,
                                       bufs.logits if kv_type == "bf16" else None)
        assert forced <= 2
        got.append((bufs, st))
    (fb, fst), (sb, sst) = got
    assert torch.equal(fb.out, sb.out) and torch.equal(fst, sst)
    assert torch.equal(fb.logits, sb.logits)
    cnt, flg, idx = B.plan_views(p, s, fb.plan)
    rcnt, rflg, ridx = B.plan_views(p, s, sb.plan)
    assert torch.equal(cnt, rcnt) and torch.equal(flg, rflg) and torch.equal(idx, ridx)


WINDOW_CASES = [
    # name, B, Hq, Hkv, d, L_p, grid, N_att, sinks, splits > 1
    ("wide", 12, 3, 3, 128, 225, 12, 16, 0, False),
    ("mha_split", 12, 2, 2, 64, 500, 12, 40, 4, True),
    ("mfma_10_tiles", 12, 8, 2, 128, 256, 14, 64, 0, False),
    ("mfma_11_tiles", 12, 8, 2, 128, 257, 14, 64, 4, True),
    ("mfma_513_pairs", 513, 2, 1, 64, 70, 12, 9, 0, False),
]


@pytest.mark.parametrize("kv_type", ["bf16", "fp8"])
@pytest.mark.parametrize("case", WINDOW_CASES, ids=[c[0] for c in WINDOW_CASES])
def test_launch_rule_edges_in_window_mode(case, kv_type):
    name, Bn, Hq, Hkv, d, Lp, grid, N_att, sinks, split = case
    L = grid * grid
    p = B.make_params(Lp, grid, grid, N_att, N_att, B.MODE_WINDOW, sinks)
    s = B.make_shape(Bn, Hq, Hkv, d)
    assert (B.launch_info(p, s).max_splits > 1) == split
    ts = positions(Bn, L, N_att, N_att, seed=Bn + d)
    w = synth.Workload(name, 1, Bn, Hq, Hkv, d, Lp, grid, grid, N_att, outlier_frac=0.01)
    kv = synth.layer_kv(w, 0, DEV)
    arrays_of = lambda b: request_arrays(kv, b, Lp)  # noqa: E731
    if kv_type == "fp8":
        kv = synth.to_fp8(kv)
        arrays_of = lambda b: fp8_request_arrays(kv, b, Lp, Hkv)  # noqa: E731
    q = synth.layer_query(w, 0, DEV)
    states = [ostep.random_states(Hkv, N_att, N_att, max(t, 0), [0] * (Hkv * L), "streaming", sinks)
              for t in ts]
    pos = torch.tensor(ts, dtype=torch.int32, device=DEV)
    lay = B.kv_layout(kv.k, k_scale=kv.k_scale, v_scale=kv.v_scale)
    st0 = torch.zeros(B.state_bytes(p, s), dtype=torch.uint8, device=DEV)
    arrays = [arrays_of(b) for b in range(Bn)]
    outs = []
    for fused in (True, False):
        bufs, _ = run(p, s, q, kv, pos, st0, fused, lay)
        check_layer_vs_oracle(p, s, q, arrays, ts, states, bufs.plan, bufs.out, None,
                              bufs.logits if kv_type == "bf16" else None)
        outs.append(bufs.out)
    assert torch.equal(*outs)


@pytest.mark.parametrize("heads", [(4, 4), (8, 4)])
def test_long_skip_lists_report_bad_states(heads):
    """A state with too few entries, one with an offset outside the window and
    a repeated offset, each in a list of over 1024 entries: the fused step and
    plan flag the same (request, KV head) pairs and keep the same rows."""
    Hq, Hkv = heads
    Bn, N_r, N_att, grid, d, Lp = 17, 1500, 310, 40, 64, 20
    p = B.make_params(Lp, grid, grid, N_r, N_att)
    s = B.make_shape(Bn, Hq, Hkv, d)
    assert B.launch_info(p, s).kept_read == 0
    ts = [1599, 1400, -1, 5000, 0] + [700 + 50 * i for i in range(Bn - 5)]
    states, _ = c_replay_states(N_r, N_att, grid * grid, [min(t, 1599) for t in ts], Hkv,
                                random.Random(5))
    st0 = states_to_buffer(p, s, states, [min(t, 1599) for t in ts])
    cnt, _, off = B.state_views(p, s, st0)
    cnt[0] = 1100                    # request 0, head 0: 90 entries missing
    off[1, 1150] = -1                # request 0, head 1: offset 65535
    off[Hkv, 3] = off[Hkv, 4].clone()  # request 1, head 0: one offset twice
    w = synth.Workload("longflags", 1, Bn, Hq, Hkv, d, Lp, grid, grid, N_r)
    kv = synth.layer_kv(w, 0, DEV)
    q = synth.layer_query(w, 0, DEV)
    pos = torch.tensor(ts, dtype=torch.int32, device=DEV)
    views = []
    for fused in (True, False):
        bufs, _ = run(p, s, q, kv, pos, st0, fused)
        views.append(B.plan_views(p, s, bufs.plan))
    (cnt, flg, idx), (rcnt, rflg, ridx) = views
    assert torch.equal(cnt, rcnt) and torch.equal(flg, rflg)
    want = torch.zeros(Bn, Hkv, dtype=torch.int32)
    want[2], want[3] = B.FLAG_INACTIVE, B.FLAG_POS_CLAMPED
    want[0, 0], want[0, 1], want[1, 0] = B.FLAG_STATE_BEHIND, B.FLAG_BAD_OFFSET, B.FLAG_COUNT
    assert torch.equal(flg.cpu().view(Bn, Hkv), want)
    # the fused step attends the first N_att of a bad set's rows, as plan lists them
    assert torch.equal(idx, ridx)


@pytest.mark.parametrize("N_r,N_att,grid", [
    (1200, 90, 36),    # few words, each all kept, half kept, or nearly all skipped
    (3300, 2100, 60),  # over 64 words: full ones first, then a remainder
])
def test_long_skip_plans_from_dense_to_sparse_windows(N_r, N_att, grid):
    """plan where it ranks a long skip list's window by words, from the first
    position (nothing skipped) to the last, against the oracle's kept positions."""
    L = grid * grid
    ts = sorted({t for t in (0, 1, 31, 32, 33, 62, 63, 64, 65, 95, N_att // 2, N_att - 1, N_att,
                             N_att + 1, N_att + 40, (N_att + N_r) // 2, 2047, 2048, 2049,
                             N_r - 1, N_r, L - 1) if t < L})
    p, s = B.make_params(8, grid, grid, N_r, N_att), B.make_shape(len(ts), 2, 2, 64)
    states, kept = c_replay_states(N_r, N_att, L, ts, 2, random.Random(N_r))
    st = states_to_buffer(p, s, states, ts)
    buf = torch.zeros(B.plan_bytes(p, s), dtype=torch.uint8, device=DEV)
    B.plan(p, s, torch.tensor(ts, dtype=torch.int32, device=DEV), st, buf)
    cnt, flg, idx = (x.cpu() for x in B.plan_views(p, s, buf))
    assert not flg.any()
    for pair in range(2 * len(ts)):
        want = [int(x) for x in kept[pair // 2][pair % 2]]
        assert idx[pair, :int(cnt[pair])].tolist() == want, (ts[pair // 2], pair % 2)


def test_long_skip_plans_across_the_pair_rules():
    """The same requests planned 16, 528 (no loads ahead of the position) and 2064
    at a time (a wave per pair again for 1110 entries): the same plans."""
    N_r, N_att, grid = 1200, 90, 40
    ts = [-1, 0, 1, 88, 89, 90, 130, 640, 1198, 1199, 1200, 1599, 5000, 700, 900, 1100]
    p = B.make_params(8, grid, grid, N_r, N_att)
    states, _ = c_replay_states(N_r, N_att, grid * grid, [min(t, 1599) for t in ts], 1,
                                random.Random(3))
    ref, kernels = None, set()
    for times in (1, 33, 129):
        n = 16 * times
        s = B.make_shape(n, 1, 1, 64)
        one = states_to_buffer(p, B.make_shape(16, 1, 1, 64), states, [min(t, 1599) for t in ts])
        st = torch.zeros(B.state_bytes(p, s), dtype=torch.uint8, device=DEV)
        for dst, src in zip(B.state_views(p, s, st), B.state_views(p, B.make_shape(16, 1, 1, 64), one)):
            dst.copy_(src.repeat(*([times] + [1] * (src.dim() - 1))))
        pos = torch.tensor(ts * times, dtype=torch.int32, device=DEV)
        buf = torch.zeros(B.plan_bytes(p, s), dtype=torch.uint8, device=DEV)
        (got,) = launches(lambda: B.plan(p, s, pos, st, buf))
        kernels.add(got[3])
        torch.cuda.synchronize()
        views = [v.view(times, 16, *v.shape[1:]) for v in B.plan_views(p, s, buf)]
        if ref is None:
            ref = [v[0] for v in views]
            assert ref[0].tolist() == [0 if t < 0 else min(t + 1, N_att) for t in ts]
        for v, r in zip(views, ref):
            assert (v == r).all()
    assert len(kernels) == 3


@pytest.mark.parametrize("d,heads,most", [(64, (2, 2), 73), (128, (4, 2), 42)])
def test_dense_combine_of_many_splits(d, heads, most):
    """Requests of 1, 8, 9, at most 64 and the most splits in one launch, over
    a workspace of NaNs."""
    Hq, Hkv = heads
    grid, Lp, Bn = 96, 20, 6
    L = grid * grid
    pd = B.make_params(Lp, grid, grid, L, L, B.MODE_DENSE)
    s = B.make_shape(Bn, Hq, Hkv, d)
    info = B.launch_info(pd, s)
    c = info.rows_per_split
    assert info.max_splits == most
    ts = [c - Lp - 1, 8 * c - Lp - 1, 8 * c - Lp, min(64 * c - Lp, L) - 1, L - 1, -1]
    w = synth.Workload("splits", 1, Bn, Hq, Hkv, d, Lp, grid, grid, L, outlier_frac=0.01)
    kv = synth.layer_kv(w, 0, DEV)
    q = synth.layer_query(w, 0, DEV)
    pos = torch.tensor(ts, dtype=torch.int32, device=DEV)
    ws = torch.full((B.workspace_bytes(pd, s),), 0xFF, dtype=torch.uint8, device=DEV)  # NaN
    out = torch.full((Bn, Hq, d), 7.0, device=DEV)
    B.decode_attention(pd, s, q, kv.k, kv.v, B.kv_layout(kv.k), pos, None, d ** -0.5, out, None, ws)
    check_layer_vs_oracle(pd, s, q, [request_arrays(kv, b, Lp) for b in range(Bn)], ts, None, None,
                          out)
