"""Launch shapes the library chooses for calls whose launch information does not
say them (fp8 caches, the kernels after the split kernel), read from a captured
graph: (workgroups, threads, dynamic LDS, kernel)."""

import pytest
import torch

from paper_2609_19702_amd import binding as B
from paper_2609_19702_amd import synth
from tests.gpu_util import DEV, launches, say

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
