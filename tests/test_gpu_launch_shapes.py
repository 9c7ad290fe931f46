"""Launch shapes the library chooses for calls whose launch information does not
say them (fp8 caches, the kernels after the split kernel), read from a captured
graph: (workgroups, threads, dynamic LDS, kernel)."""

import pytest
import torch

from paper_2609_19702_amd import binding as B
from paper_2609_19702_amd import synth
from tests.gpu_util import DEV, check_layer_vs_oracle, fp8_request_arrays, launches, say

pytestmark = pytest.mark.gpu


def shapes(batch, heads, d, Lp, grid, N_r, N_att, mode=B.MODE_DIAGONAL, kv_type="bf16", fused=True):
    """Launches of one decode step (or of ``decode_attention`` on its plan)."""
    Hq, Hkv = heads
    p, s = B.make_params(Lp, grid, grid, N_r, N_att, mode), B.make_shape(batch, Hq, Hkv, d)
    w = synth.Workload("shapes", 1, batch, Hq, Hkv, d, Lp, grid, grid, N_r)
    kv = synth.layer_kv(w, 0, DEV)
    if kv_type == "fp8":
        kv = synth.to_fp8(kv)
    q = synth.layer_query(w, 0, DEV)
    lay = B.kv_layout(kv.k, k_scale=kv.k_scale, v_scale=kv.v_scale)
    pos = torch.zeros(batch, dtype=torch.int32, device=DEV)
    bufs = B.alloc_buffers(p, s, DEV)
    B.state_reset(p, s, bufs.state)
    if fused:
        got = launches(lambda: B.decode_step(p, s, q, kv.k, kv.v, lay, pos, bufs.state, bufs.plan,
                                             0.1, bufs.out, bufs.logits, bufs.workspace))
    else:
        B.plan(p, s, pos, bufs.state, bufs.plan)
        got = launches(lambda: B.decode_attention(p, s, q, kv.k, kv.v, lay, pos, bufs.plan, 0.1,
                                                  bufs.out, bufs.logits, bufs.workspace))
    say("launches", batch, heads, d, Lp, N_r, N_att, mode, kv_type, got)
    return got


@pytest.mark.parametrize("mode,N_r,N_att,selecting,lds", [
    (B.MODE_WINDOW, 900, 600, 0, 0),              # nothing is ever selected
    (B.MODE_DIAGONAL, 900, 200, 1, 0),            # a short window: one wave
    (B.MODE_DIAGONAL, 900, 600, 4, 600 * 4 * 4),  # a long one: a wave per head, terms in LDS
])
def test_combine_has_the_waves_its_selection_needs(mode, N_r, N_att, selecting, lds):
    split, combine = shapes(8, (16, 4), 64, 480, 32, N_r, N_att, mode)
    assert split[0] > 8 * 4
    assert combine[:3] == (8 * 4, 64 * (4 + selecting), lds)


@pytest.mark.parametrize("d,rows", [(64, (150, 40)), (128, (120, 29))])
@pytest.mark.parametrize("fused", [True, False])
def test_fp8_launches_of_four_tiles_run_the_general_kernel(d, rows, fused):
    """One workgroup per pair either way; more than four tiles take the kernel of
    up to sixteen waves."""
    def split(batch, Lp, N_att):
        (got,) = shapes(batch, (4, 4), d, Lp, 24, 2 * N_att, N_att, kv_type="fp8", fused=fused)
        assert got[0] == batch * 4
        return got
    few, many = split(17, *rows), split(129, *rows)  # neither keeps lists
    assert few[1] == many[1] == 256 and few[3] == many[3]
    longer = split(17, rows[0] + 64, rows[1])
    assert longer[1] == 320 + 64 * (d == 128) and longer[3] != few[3]


@pytest.mark.parametrize("batch,lds", [(64, 8 * 2000 * 4), (65, 0)])
def test_select_of_many_pairs_keeps_its_lds_resident(batch, lds):
    """Eight heads' softmaxes of 2000 keys: 64000 bytes per workgroup, for up to
    512 pairs (two to a CU); past that one wave each, from memory."""
    p, s = B.make_params(0, 70, 70, 4000, 2000), B.make_shape(batch, 64, 8, 64)
    bufs = B.alloc_buffers(p, s, DEV)
    pos = torch.full((batch,), -1, dtype=torch.int32, device=DEV)
    (got,) = launches(lambda: B.select(p, s, pos, bufs.plan, bufs.logits, bufs.state))
    assert got[2] == lds and got[0] == (batch * 8 if lds else batch * 8 // 4)


def test_dense_fp8_builds_of_one_and_two_tiles_agree():
    """48 requests (1920 splits) run the build with one tile in flight per wave, 24
    of them (960) the one with two: the same outputs, bit for bit, and the oracle's."""
    Bn, Hq, Hkv, d, Lp, grid = 48, 16, 8, 128, 100, 32
    w = synth.Workload("dense_fp8", 1, Bn, Hq, Hkv, d, Lp, grid, grid, 64, outlier_frac=0.01)
    kv = synth.to_fp8(synth.layer_kv(w, 0, DEV))
    q = synth.layer_query(w, 0, DEV)
    L = grid * grid
    ts = [L - 1, 0, -1, 155, 156, 411] + [(37 * i) % L for i in range(Bn - 6)]
    p = B.make_params(Lp, grid, grid, L, L, B.MODE_DENSE)
    outs, kernels = [], []
    for n in (Bn, Bn // 2):
        s = B.make_shape(n, Hq, Hkv, d)
        pos = torch.tensor(ts[:n], dtype=torch.int32, device=DEV)
        bufs = B.alloc_buffers(p, s, DEV)
        lay = B.kv_layout(kv.k, k_scale=kv.k_scale, v_scale=kv.v_scale)
        split, _ = launches(lambda: B.decode_attention(
            p, s, q, kv.k, kv.v, lay, pos, None, d ** -0.5, bufs.out, None, bufs.workspace))
        torch.cuda.synchronize()
        outs.append(bufs.out)
        kernels.append(split)
    assert kernels[0][0] == 1920 and kernels[1][0] == 960 and kernels[0][3] != kernels[1][3]
    assert torch.equal(outs[0][:Bn // 2], outs[1])
    check_layer_vs_oracle(p, B.make_shape(6, Hq, Hkv, d), q,
                          [fp8_request_arrays(kv, b, Lp, Hkv) for b in range(6)], ts[:6], None,
                          None, outs[1][:6])
