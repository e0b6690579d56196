"""Stage-by-stage comparison of the HIP path (through the C ABI) with the CPU oracle.

Tolerances (from the benchmark spec, restated here):
  * active masks and page sets: bit-exact, except items within 1e-5 (relative to
    max(1, |v|)) of the deciding value v (the n-th locality score / the K-th page bound):
    both sides decide in float32 but sum in different orders, so only such near-ties may
    differ; each is checked against the oracle's float64 value and counted.
  * o_p, lse_p: max-abs 2e-2 with bfloat16 inputs, 1e-4 with float inputs.
"""
from __future__ import annotations

import numpy as np
import torch

from oracle import losa_oracle as orc
from paper_2604_12056_amd import binding as L
from paper_2604_12056_amd import synth
from paper_2604_12056_amd.device_inputs import DeviceBlock, DeviceLayer, config_of, to_host

NEAR_TIE = 1e-5


def tol(w: synth.Workload) -> float:
    return 2e-2 if w.dtype == "bf16" else 1e-4


class Rig:
    """A workload on the device next to its oracle state."""

    def __init__(self, w: synth.Workload, device="cuda:0", mutate=None, tuning=None):
        self.w = w
        self.inp = synth.make_inputs(w)
        if mutate is not None:      # edits the host inputs in place before either side sees them
            mutate(self.inp)
        self.layer = DeviceLayer(self.inp, device)
        self.blk = DeviceBlock(self.inp, device)
        self.ctx = L.losa_create(config_of(w, max_topk_pages=w.max_pages), device)
        for knob, value in (tuning or {}).items():      # launch-shape switches: same results, other code paths
            L.losa_set_tuning(self.ctx, knob, value)
        self.cache = orc.PrefixCache(self.inp.K, self.inp.V, w.g)
        rows = w.batch * w.B
        self.o_ref = np.zeros((rows, w.Hq, w.d))
        self.L_ref = np.zeros((rows, w.Hq))
        self.near_ties = 0

    def close(self):
        self.ctx.close()


def workspace_parts(ctx) -> dict:
    """{name: bytes of the workspace (a view)} as losa_create carves it: which buffers a call wrote tells which launches it made."""
    c = ctx.cfg
    G, heads, tokens = c.num_q_heads // c.num_kv_heads, c.max_batch * c.num_kv_heads, c.max_batch * c.block_size
    rows, pages = c.block_size * G, c.max_pages_per_seq
    part_rows = max(1024 * min(rows, 64), max(heads, 256) * ((rows + 31) // 32 * 32))
    copy_words = 16 if pages <= 512 else 32 if pages <= 1024 else ((pages + 31) // 32 + 3) // 4 * 4
    copies = 256 // copy_words if copy_words <= 32 else 1 if rows <= 64 else 2 if rows <= 128 else 4 if rows <= 256 else 8
    sizes = {"delta": tokens * 4, "mask": tokens, "active_idx": tokens * 4, "active_count": c.max_batch * 4, "scores": heads * rows * pages * 4,
             "rowmaps": heads * rows * ((pages + 31) // 32) * 4, "tickets": heads * 4, "sel_pages": heads * pages * 4, "sel_count": heads * 4,
             "partial_o": part_rows * c.head_dim * 4, "partial_m": part_rows * 4, "partial_l": part_rows * 4, "entries": heads * pages * 4,
             "q_act": heads * rows * c.head_dim * 2, "seq_tickets": c.max_batch * 4, "union_bits": heads * max(256, copy_words * copies) * 4}
    assert sum(-(-n // 256) * 256 for n in sizes.values()) == L.losa_workspace_bytes(c), "the library carves its workspace in another way"
    at, parts = (-ctx.workspace.data_ptr()) % 256, {}
    for name, n in sizes.items():
        parts[name] = ctx.workspace[at:at + n]
        at += -(-n // 256) * 256
    return parts


def check_near_tie_sets(got: set, want: set, value64, K_eff: int, what: str) -> int:
    """Two picked sets may differ only in items whose float64 value is within NEAR_TIE of the
    K-th largest.  Returns the number of differing items."""
    if got == want:
        return 0
    assert len(got) == len(want), f"{what}: sizes differ {len(got)} vs {len(want)}"
    vals = np.sort(np.asarray(value64))[::-1]
    vk = vals[K_eff - 1]
    lim = NEAR_TIE * max(1.0, abs(vk))
    for p in got ^ want:
        assert abs(value64[p] - vk) <= lim, f"{what}: item {p} value {value64[p]} vs k-th {vk} is not a near-tie"
    return len(got ^ want)


def check_page_bounds(rig: Rig):
    w = rig.w
    L.losa_page_bounds(rig.ctx, rig.layer.kv)
    torch.cuda.synchronize()
    meta = synth.load(to_host(rig.layer.meta)).astype(np.float64)          # [num_pages, Hkv, 2, d]
    for b in range(w.batch):
        kmin, kmax = rig.cache.bounds[b]
        phys = rig.inp.page_indices[rig.inp.page_indptr[b]: rig.inp.page_indptr[b + 1]]
        assert np.array_equal(meta[phys, :, 0, :], kmin), f"min keys differ (seq {b})"
        assert np.array_equal(meta[phys, :, 1, :], kmax), f"max keys differ (seq {b})"


def check_select_active(rig: Rig, t: int, mode: int, param: float):
    w, blk = rig.w, rig.blk
    L.losa_select_active(rig.ctx, blk.h[t], blk.h[t - 1], mode, param, blk.delta, blk.mask, blk.active_idx,
                         blk.active_count)
    torch.cuda.synchronize()
    delta = blk.delta.cpu().numpy()
    ref = orc.locality_score(rig.inp.h[t], rig.inp.h[t - 1])
    np.testing.assert_allclose(delta, ref, rtol=2e-6, atol=1e-30)
    mask = blk.mask.cpu().numpy()
    idx = blk.active_idx.cpu().numpy().reshape(w.batch, w.B)
    cnt = blk.active_count.cpu().numpy()
    active = []
    for b in range(w.batch):
        A_ref = orc.active_set(ref[b * w.B:(b + 1) * w.B], mode, param)
        A = idx[b, :cnt[b]]
        assert np.all(idx[b, cnt[b]:] == -1) and list(A) == sorted(A)
        assert np.array_equal(np.nonzero(mask[b * w.B:(b + 1) * w.B])[0], A)
        if mode == orc.SEL_THRESHOLD:
            for i in set(A) ^ set(A_ref):
                assert abs(ref[b * w.B + i] - param) <= NEAR_TIE * max(1.0, abs(param))
                rig.near_ties += 1
        elif mode == orc.SEL_MASS:
            # a different count is acceptable only if the running sum sits within the near-tie band of the target
            if len(A) != len(A_ref):
                srt = np.sort(ref[b * w.B:(b + 1) * w.B])[::-1]
                k = min(len(A), len(A_ref))
                assert abs(srt[:k].sum() - param * srt.sum()) <= NEAR_TIE * max(1.0, srt.sum())
                rig.near_ties += 1
            else:
                assert set(A.tolist()) == set(A_ref.tolist())
        else:
            rig.near_ties += check_near_tie_sets(set(A.tolist()), set(A_ref.tolist()), ref[b * w.B:(b + 1) * w.B],
                                                 len(A_ref), f"active set seq {b}")
        active.append(A_ref)
    return active


def upload_active(rig: Rig, active):
    w, blk = rig.w, rig.blk
    idx = np.full((w.batch, w.B), -1, dtype=np.int32)
    cnt = np.zeros(w.batch, dtype=np.int32)
    for b, A in enumerate(active):
        idx[b, :len(A)] = A
        cnt[b] = len(A)
    blk.active_idx.copy_(torch.from_numpy(idx.reshape(-1)))
    blk.active_count.copy_(torch.from_numpy(cnt))


def upload_union(rig: Rig, union):
    w, blk = rig.w, rig.blk
    sel = np.full((w.batch, w.Hkv, blk.cap), -1, dtype=np.int32)
    cnt = np.zeros((w.batch, w.Hkv), dtype=np.int32)
    for (b, j), I in union.items():
        sel[b, j, :len(I)] = I
        cnt[b, j] = len(I)
    blk.sel_pages.copy_(torch.from_numpy(sel))
    blk.sel_count.copy_(torch.from_numpy(cnt))


def oracle_selection(rig: Rig, t: int, active, topk: int):
    """Oracle page scores / picks / unions for given active sets (no attention)."""
    w = rig.w
    qf = orc.widen(rig.inp.q[t])
    scores, picks, union = {}, {}, {}
    for b in range(w.batch):
        kmin, kmax = rig.cache.bounds[b]
        for j in range(w.Hkv):
            sets = []
            for i in active[b]:
                for h in range(j * w.G, (j + 1) * w.G):
                    s = orc.page_upper_bound(qf[b * w.B + i, h], kmin[:, j], kmax[:, j])
                    scores[(b, int(i), h)] = s
                    picks[(b, int(i), h)] = orc.top_pages(s, topk)
                    sets.append(picks[(b, int(i), h)])
            union[(b, j)] = orc.union_pages(sets)
    return scores, picks, union


def check_score_pages(rig: Rig, t: int, active, topk: int):
    """Feeds the oracle's active sets; compares per-query picks and the unions."""
    w, blk = rig.w, rig.blk
    upload_active(rig, active)
    topk_out = torch.full((w.batch, w.B, w.Hq, topk), -7, dtype=torch.int32, device=blk.q.device)
    L.losa_score_pages(rig.ctx, rig.layer.kv, blk.q[t], blk.active_idx, blk.active_count, topk, topk_out,
                       blk.sel_pages, blk.sel_count, blk.cap)
    torch.cuda.synchronize()
    scores, picks, union = oracle_selection(rig, t, active, topk)
    tk = topk_out.cpu().numpy()
    sel = blk.sel_pages.cpu().numpy()
    cnt = blk.sel_count.cpu().numpy()
    for b in range(w.batch):
        P = w.pages_per_seq[b]
        Keff = min(topk, P)
        for j in range(w.Hkv):
            got_union = set()
            exact = True
            for a, i in enumerate(active[b]):
                for h in range(j * w.G, (j + 1) * w.G):
                    row = tk[b, a, h]
                    got = row[:Keff]
                    assert np.all(row[Keff:] == -1) and list(got) == sorted(got) and len(set(got)) == Keff
                    assert got.min() >= 0 and got.max() < P
                    d = check_near_tie_sets(set(got.tolist()), set(picks[(b, int(i), h)].tolist()),
                                            scores[(b, int(i), h)], Keff, f"top pages b{b} tok{i} h{h}")
                    rig.near_ties += d
                    exact &= d == 0
                    got_union |= set(got.tolist())
            U = sel[b, j, :cnt[b, j]]
            assert list(U) == sorted(got_union), f"union b{b} kv{j} is not the union of the emitted picks"
            if exact:
                assert np.array_equal(U, union[(b, j)])
    return union


def check_score_pages_shared(rig: Rig, t: int, active, topk: int):
    """The shared-budget variant: one page set per (sequence, KV head), against the oracle's
    shared_top_pages on the same active sets.  Returns the sets the device produced."""
    w, blk = rig.w, rig.blk
    upload_active(rig, active)
    blk.sel_pages.fill_(-7)
    L.losa_score_pages_shared(rig.ctx, rig.layer.kv, blk.q[t], blk.active_idx, blk.active_count, topk,
                              blk.sel_pages, blk.sel_count, blk.cap)
    torch.cuda.synchronize()
    scores, _, _ = oracle_selection(rig, t, active, topk)
    sel = blk.sel_pages.cpu().numpy()
    cnt = blk.sel_count.cpu().numpy()
    got_sets = {}
    for b in range(w.batch):
        P = w.pages_per_seq[b]
        Keff = min(topk, P) if len(active[b]) else 0
        for j in range(w.Hkv):
            assert cnt[b, j] == Keff, f"shared budget b{b} kv{j}: {cnt[b, j]} pages, expected {Keff}"
            got = sel[b, j, :Keff]
            got_sets[(b, j)] = got.astype(np.int32)
            if Keff == 0:
                continue
            assert list(got) == sorted(set(got.tolist())) and got.min() >= 0 and got.max() < P
            rows = np.stack([scores[(b, int(i), h)] for i in active[b] for h in range(j * w.G, (j + 1) * w.G)])
            want = orc.shared_top_pages(rows, topk)
            best64 = rows.max(axis=0)
            rig.near_ties += check_near_tie_sets(set(got.tolist()), set(want.tolist()), best64, Keff,
                                                 f"shared pages b{b} kv{j}")
    return got_sets


def check_sparse_attn(rig: Rig, t: int, active, union, dense: bool = False):
    """Feeds the oracle's active sets and unions; compares (o_p, lse_p) on active rows and
    requires every other row to be bit-identical to what it was."""
    w, blk = rig.w, rig.blk
    before_o, before_l = blk.o_p.clone(), blk.lse_p.clone()
    if dense:
        L.losa_sparse_attn(rig.ctx, rig.layer.kv, blk.q[t], None, None, None, None, 0, blk.o_p, blk.lse_p)
    else:
        upload_active(rig, active)
        upload_union(rig, union)
        L.losa_sparse_attn(rig.ctx, rig.layer.kv, blk.q[t], blk.active_idx, blk.active_count, blk.sel_pages,
                           blk.sel_count, blk.cap, blk.o_p, blk.lse_p)
    torch.cuda.synchronize()
    o_ref, L_ref = rig.o_ref, rig.L_ref
    orc.losa_step(rig.cache, 0 if dense else 1, None, None, rig.inp.q[t], 0, 0, 0, w.B, w.Hq, o_ref, L_ref,
                  forced_active=None if dense else active, forced_union=None if dense else union)
    compare_state(rig, active if not dense else [np.arange(w.B)] * w.batch, before_o, before_l)


def compare_state(rig: Rig, active, before_o=None, before_l=None):
    w, blk = rig.w, rig.blk
    o = blk.o_p.cpu().numpy().astype(np.float64)
    lse = blk.lse_p.cpu().numpy().astype(np.float64)
    rows = np.concatenate([b * w.B + np.asarray(A, dtype=np.int64) for b, A in enumerate(active)]) \
        if len(active) else np.zeros(0, dtype=np.int64)
    if len(rows):
        assert np.all(np.isfinite(o[rows])), "non-finite attention output"
        err_o = np.abs(o[rows] - rig.o_ref[rows]).max()
        # an empty key set gives lse = -inf on both sides (the neutral element of the merge)
        empty = np.isneginf(rig.L_ref[rows])
        assert np.array_equal(np.isneginf(lse[rows]), empty), "lse_p = -inf exactly where no key was attended to"
        err_l = np.abs(np.where(empty, 0.0, lse[rows]) - np.where(empty, 0.0, rig.L_ref[rows])).max()
        assert err_o <= tol(w), f"o_p max-abs error {err_o} > {tol(w)}"
        assert err_l <= tol(w), f"lse_p max-abs error {err_l} > {tol(w)}"
    if before_o is not None:
        stable = np.setdiff1d(np.arange(w.batch * w.B), rows)
        assert torch.equal(blk.o_p[stable], before_o[stable]), "a stable row of o_p was written"
        assert torch.equal(blk.lse_p[stable], before_l[stable]), "a stable row of lse_p was written"


def gpu_union_of(rig: Rig, t: int, gpu_active, topk: int, scores, picks):
    """The union the device builds for the given active sets, through losa_score_pages on the same
    inputs, with every per-query pick validated against the oracle's float64 scores (only
    near-ties of the K-th bound may differ).  Returns ({(b, j): pages}, differing picks)."""
    w, blk = rig.w, rig.blk
    upload_active(rig, gpu_active)
    topk_out = torch.full((w.batch, w.B, w.Hq, topk), -7, dtype=torch.int32, device=blk.q.device)
    L.losa_score_pages(rig.ctx, rig.layer.kv, blk.q[t], blk.active_idx, blk.active_count, topk, topk_out,
                       blk.sel_pages, blk.sel_count, blk.cap)
    torch.cuda.synchronize()
    tk = topk_out.cpu().numpy()
    sel = blk.sel_pages.cpu().numpy()
    cnt = blk.sel_count.cpu().numpy()
    union, differing = {}, 0
    for b in range(w.batch):
        Keff = min(topk, w.pages_per_seq[b])
        for j in range(w.Hkv):
            got_union = set()
            for a, i in enumerate(gpu_active[b]):
                for h in range(j * w.G, (j + 1) * w.G):
                    got = tk[b, a, h, :Keff]
                    differing += check_near_tie_sets(set(got.tolist()), set(picks[(b, int(i), h)].tolist()),
                                                     scores[(b, int(i), h)], Keff, f"top pages b{b} tok{i} h{h}")
                    got_union |= set(got.tolist())
            U = sel[b, j, :cnt[b, j]]
            assert list(U) == sorted(got_union), f"union b{b} kv{j} is not the union of the emitted picks"
            union[(b, j)] = U.astype(np.int32)
    return union, differing


def follow_step(rig: Rig, t: int, mode: int, param: float, topk: int, gpu_mask, gpu_cnt):
    """Advances the oracle state (rig.o_ref, rig.L_ref) by sparse step t.  The device's decisions
    (active mask and union sizes as losa_step reported them) must be the oracle's; where a
    near-tie made the device decide differently, the difference is validated item by item
    against the oracle's float64 values and the oracle then follows the device's (validated)
    active set and union, so the outputs of the step are compared in every case.
    Returns the active sets the step used."""
    w = rig.w
    o_save, L_save = rig.o_ref.copy(), rig.L_ref.copy()
    tr = orc.losa_step(rig.cache, t, rig.inp.h[t], rig.inp.h[t - 1], rig.inp.q[t], mode, param, topk, w.B, w.Hq,
                       rig.o_ref, rig.L_ref, keep_scores=True)
    mask = np.asarray(gpu_mask).reshape(w.batch, w.B)
    cnt = np.asarray(gpu_cnt).reshape(w.batch, w.Hkv)
    gpu_active = [np.nonzero(mask[b])[0].astype(np.int32) for b in range(w.batch)]
    same_active = all(np.array_equal(gpu_active[b], tr.active[b]) for b in range(w.batch))
    if not same_active:      # validate the device's active sets as near-ties of the n-th locality score
        for b in range(w.batch):
            if mode == orc.SEL_THRESHOLD:
                for i in set(gpu_active[b].tolist()) ^ set(tr.active[b].tolist()):
                    assert abs(tr.delta[b * w.B + i] - param) <= NEAR_TIE * max(1.0, abs(param))
                    rig.near_ties += 1
            elif mode == orc.SEL_MASS and len(gpu_active[b]) != len(tr.active[b]):
                srt = np.sort(tr.delta[b * w.B:(b + 1) * w.B])[::-1]
                k = min(len(gpu_active[b]), len(tr.active[b]))
                assert abs(srt[:k].sum() - param * srt.sum()) <= NEAR_TIE * max(1.0, srt.sum())
                rig.near_ties += 1
            else:
                rig.near_ties += check_near_tie_sets(set(gpu_active[b].tolist()), set(tr.active[b].tolist()),
                                                     tr.delta[b * w.B:(b + 1) * w.B], len(tr.active[b]), "active set")
        scores, picks, ref_union = oracle_selection(rig, t, gpu_active, topk)
    else:
        scores, picks, ref_union = tr.scores, tr.picks, tr.union
    # The device's own union for these active sets (losa_step keeps its list in the workspace, so it
    # is rebuilt through losa_score_pages on the same inputs): every pick validated, the sizes
    # required to be the ones losa_step reported, the contents required to be the oracle's unless a
    # validated near-tie changed a pick.
    union, differing = gpu_union_of(rig, t, gpu_active, topk, scores, picks)
    rig.near_ties += differing
    for (b, j), I in union.items():
        assert int(cnt[b, j]) == len(I), f"losa_step reported {cnt[b, j]} union pages for b{b} kv{j}, losa_score_pages {len(I)}"
        if differing == 0:
            assert np.array_equal(I, ref_union[(b, j)]), f"union b{b} kv{j} differs from the oracle's"
    if same_active and differing == 0:
        return gpu_active
    rig.o_ref[:], rig.L_ref[:] = o_save, L_save
    orc.losa_step(rig.cache, t, None, None, rig.inp.q[t], mode, param, topk, w.B, w.Hq, rig.o_ref, rig.L_ref,
                  forced_active=gpu_active, forced_union=union)
    return gpu_active


def run_steps_end_to_end(rig: Rig, steps, mode: int, param: float, topk: int):
    """losa_step over the given step indices, GPU state vs oracle state after every step."""
    w, blk = rig.w, rig.blk
    for t in steps:
        before_o, before_l = blk.o_p.clone(), blk.lse_p.clone()
        L.losa_step(rig.ctx, rig.layer.kv, t, blk.h[t] if t else None, blk.h[t - 1] if t else None, blk.q[t],
                    mode, param, topk, blk.o_p, blk.lse_p, blk.mask, blk.sel_count)
        torch.cuda.synchronize()
        if t == 0:
            orc.losa_step(rig.cache, 0, None, None, rig.inp.q[0], mode, param, topk, w.B, w.Hq, rig.o_ref, rig.L_ref)
            compare_state(rig, [np.arange(w.B)] * w.batch)
            continue
        gpu_active = follow_step(rig, t, mode, param, topk, blk.mask.cpu().numpy(), blk.sel_count.cpu().numpy())
        compare_state(rig, gpu_active, before_o, before_l)
