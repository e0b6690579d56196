"""The measurement hooks (losa_profile_enable / losa_profile_read): every launch form is bracketed, whether its events are
recorded on the stream around it or bound to its dispatch."""
import time

import pytest
import torch

from oracle import losa_oracle as orc
from paper_2604_12056_amd import binding as L
from paper_2604_12056_amd import synth
from paper_2604_12056_amd.device_inputs import config_of

from parity_util import Rig

pytestmark = pytest.mark.gpu


def rig(B, G, d, dtype, tuning=None):
    w = synth.config(0).replace(B=B, Hq=2 * G, Hkv=2, d=d, g=16, batch=2, seq_lens=(333, 1000), n_active=max(1, B // 2), topk_pages=6,
                                T=3, outliers="lognormal", dtype=dtype, name=f"profile-B{B}-G{G}-{dtype}")
    return Rig(w, tuning=tuning)


def stages_of(r, call):
    """Launches per stage of one call, whose times have to fit into the time it took on the host's clock.  The hooks are switched
    on for this call alone: events that already hold a time would give it for a launch that is not recorded."""
    L.losa_profile_enable(r.ctx, True)
    try:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        call()
        torch.cuda.synchronize()
        wall_ms = 1e3 * (time.perf_counter() - t0)
        ms, launches = L.losa_profile_read(r.ctx)
        assert all(0.0 < ms[s] <= wall_ms if launches[s] else ms[s] == 0.0 for s in L.STAGES), (ms, launches, wall_ms)
        empty, none = L.losa_profile_read(r.ctx)   # the record is cleared by the read
        assert not any(empty.values()) and not any(none.values())
        return {s: n for s, n in launches.items() if n}
    finally:
        L.losa_profile_enable(r.ctx, False)


@pytest.mark.parametrize("tuning", [{}, {L.LOSA_TUNE_UNION_IN_ATTENTION: 0}, {L.LOSA_TUNE_SHARED_TILES: 0}])
@pytest.mark.parametrize("B,G,d,dtype", [
    (8, 1, 64, "bf16"), (16, 4, 128, "bf16"),     # up to 64 query rows per KV head: row tiles by a count on the device
    (13, 5, 64, "bf16"), (64, 4, 128, "bf16"),    # 65 to 256: a launch for heads of up to 64 rows, one for those with more
    (37, 7, 64, "bf16"),                          # more: one launch for all
    (16, 4, 64, "f32")])
def test_every_launch_form_is_timed(B, G, d, dtype, tuning):
    r = rig(B, G, d, dtype, tuning)
    w, blk, kv = r.w, r.blk, r.layer.kv
    step = {"locality": 1, "score": 1, "topk": 1, "attn": 1, "merge": 1}

    def sparse(mode, param):
        L.losa_step(r.ctx, kv, 1, blk.h[1], blk.h[0], blk.q[1], mode, param, w.topk_pages, blk.o_p, blk.lse_p)

    def separate(sel_pages, sel_count, cap):
        L.losa_select_active(r.ctx, blk.h[1], blk.h[0], orc.SEL_TOPK, float(w.n_active), blk.delta, blk.mask, blk.active_idx, blk.active_count)
        L.losa_score_pages(r.ctx, kv, blk.q[1], blk.active_idx, blk.active_count, w.topk_pages, None, blk.sel_pages, blk.sel_count, blk.cap)
        L.losa_sparse_attn(r.ctx, kv, blk.q[1], blk.active_idx, blk.active_count, sel_pages, sel_count, cap, blk.o_p, blk.lse_p)

    try:
        assert stages_of(r, lambda: L.losa_page_bounds(r.ctx, kv)) == {"bounds": 1}
        assert stages_of(r, lambda: L.losa_step(r.ctx, kv, 0, None, None, blk.q[0], orc.SEL_TOPK, 1.0, w.topk_pages, blk.o_p,
                                                blk.lse_p)) == {"attn": 1, "merge": 1}
        for mode, param in ((orc.SEL_TOPK, float(w.n_active)), (orc.SEL_FRACTION, 1.0), (orc.SEL_THRESHOLD, 1e-3), (orc.SEL_MASS, 0.5)):
            assert stages_of(r, lambda: sparse(mode, param)) == step, (mode, param)
        assert stages_of(r, lambda: separate(blk.sel_pages, blk.sel_count, blk.cap)) == step
        assert stages_of(r, lambda: separate(None, None, 0)) == step
    finally:
        r.close()


def test_calls_between_two_reads_add_up():
    """Time and count of several calls add up; switching the hooks off and on again starts an empty record."""
    r = rig(16, 4, 64, "bf16")
    w, blk = r.w, r.blk
    try:
        L.losa_profile_enable(r.ctx, True)
        L.losa_page_bounds(r.ctx, r.layer.kv)
        for t in (1, 2, 1):
            L.losa_step(r.ctx, r.layer.kv, t, blk.h[t], blk.h[t - 1], blk.q[t], orc.SEL_MASS, 0.5, w.topk_pages, blk.o_p, blk.lse_p)
        ms, launches = L.losa_profile_read(r.ctx)
        assert launches["attn"] == 3 and launches["bounds"] == 1 and ms["attn"] > 0
        L.losa_page_bounds(r.ctx, r.layer.kv)
        L.losa_profile_enable(r.ctx, False)
        L.losa_profile_enable(r.ctx, True)
        assert not any(L.losa_profile_read(r.ctx)[1].values())
    finally:
        L.losa_profile_enable(r.ctx, False)
        r.close()
