"""Kernels and dispatch branches at the sizes where they can go wrong - edges of tiles and of row groups,
remainders, the smallest and largest of a range - each against the CPU oracle.  Tolerances are those of
parity_util (2e-2 for bfloat16 inputs, 1e-4 for float inputs, sets exact up to verified near-ties)."""
import numpy as np
import pytest
import torch

from oracle import losa_oracle as orc
from paper_2604_12056_amd import binding as L
from paper_2604_12056_amd import synth
from paper_2604_12056_amd.device_inputs import config_of, to_host

from parity_util import (Rig, check_page_bounds, check_sparse_attn, compare_state, gpu_union_of, oracle_selection, run_steps_end_to_end,
                         workspace_parts)

pytestmark = pytest.mark.gpu


def workload(B, G, Hkv, d, g, lens, n, topk=6, dtype="bf16", T=3):
    return synth.config(0).replace(B=B, Hq=Hkv * G, Hkv=Hkv, d=d, g=g, batch=len(lens), seq_lens=tuple(lens), n_active=n,
                                   topk_pages=topk, T=T, outliers="lognormal", dtype=dtype,
                                   name=f"edge-B{B}-G{G}-d{d}-g{g}-{dtype}")


@pytest.mark.parametrize("half_values", [1, 0])
@pytest.mark.parametrize("B,G,d,g,n", [
    (13, 5, 128, 16, 13),     # 65 rows: the smallest count the many-row kernel serves, three row wavefronts of 32
    (32, 4, 128, 32, 32),     # 128 rows: the last count its two token groups serve
    (43, 3, 128, 16, 43),     # 129 rows: the first with one token group, a last row wavefront of one row
    (64, 4, 64, 32, 33),      # 132 of 256 rows active
    (64, 4, 128, 32, 64),     # 256 rows: a full row group
    (37, 7, 64, 16, 37)])     # 259 rows: a second row group of three rows
def test_many_row_kernel_at_the_edges_of_its_row_counts(B, G, d, g, n, half_values):
    """Stages of 64 tokens: prefixes one token around a stage, a page and a block of 32, one that leaves
    whole workgroups without a stage, and page lists that end inside a stage."""
    w = workload(B, G, 2, d, g, (63, 64, 65, 97, 64 * 9 + 1, 1500), n)
    r = Rig(w, tuning={L.LOSA_TUNE_HALF_PRECISION_VALUES: half_values})
    try:
        check_page_bounds(r)
        check_sparse_attn(r, 0, None, None, dense=True)
        rng = np.random.Generator(np.random.Philox(B * G))
        active = [np.sort(rng.permutation(B)[:n]).astype(np.int32) for _ in range(w.batch)]
        lists = {(b, j): np.sort(rng.permutation(P)[:max(1, P - 1 - j)]).astype(np.int32)
                 for b, P in enumerate(w.pages_per_seq) for j in range(w.Hkv)}
        check_sparse_attn(r, 1, active, lists)
        run_steps_end_to_end(r, range(2), orc.SEL_TOPK, float(n), w.topk_pages)
        run_steps_end_to_end(r, [2], orc.SEL_MASS, 1.0, w.topk_pages)      # the count stays on the device
    finally:
        r.close()


@pytest.mark.parametrize("n", [10, 36, 37, 64])     # 70, 252 | 259, 448 rows: one row group | two
def test_counted_rows_of_a_block_with_two_row_groups(n):
    """64 tokens x 7 heads: the grid has the row groups the count needs, not those of the whole block."""
    w = workload(64, 7, 1, 64, 16, (64 * 40 + 9, 700, 1), n)
    r = Rig(w)
    r.ctx.workspace.fill_(255)
    try:
        check_page_bounds(r)
        run_steps_end_to_end(r, range(2), orc.SEL_TOPK, float(n), w.topk_pages)
    finally:
        r.close()


@pytest.mark.parametrize("workgroups", [8, 9, 12, 64, 1024])
def test_merge_of_partials_laid_out_by_fragments(workgroups):
    """Chunk counts around the line between the merge's two forms (up to 8 chunks, more), and more chunks than
    one batch of a split workgroup's wavefronts holds."""
    w = workload(32, 7, 1, 128, 16, (64 * 70 + 5,), 32)
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: workgroups})
    try:
        check_sparse_attn(r, 0, None, None, dense=True)
    finally:
        r.close()


@pytest.mark.parametrize("chunks", [1, 2, 4, 5, 8, 9, 16, 17, 31, 64, 65, 100, 300])
def test_merge_by_fragments_at_the_edges_of_its_forms(chunks):
    """Chunk counts around the lines between the forms (4, 16, 64) and around what a form's wavefronts hold at a
    time, next to sequences that leave most chunks unwritten.  The workspace starts as NaN: a slot nobody wrote must
    not be looked at."""
    w = workload(19, 4, 1, 64, 16, (64 * 600 + 5, 64 * 3, 1), 19)
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: 3 * chunks})
    r.ctx.workspace.fill_(255)
    try:
        check_sparse_attn(r, 0, None, None, dense=True)
        check_page_bounds(r)
        run_steps_end_to_end(r, [1], orc.SEL_TOPK, 18.0, w.topk_pages)      # 72 rows: the counts come from the device
    finally:
        r.close()


@pytest.mark.parametrize("workgroups", [4, 20, 72, 1024])
@pytest.mark.parametrize("B,G,d,g", [(33, 4, 128, 16), (32, 8, 64, 32), (17, 5, 128, 32)])
def test_merge_of_heads_with_few_and_many_rows_in_one_launch(B, G, d, g, workgroups):
    """A count only the device knows: heads of up to 64 rows and of more in one launch, none active in one sequence."""
    w = workload(B, G, 1, d, g, (64 * 33 + 1, 700, 64 * 20, 1500), B)
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: workgroups})
    r.ctx.workspace.fill_(255)
    try:
        check_page_bounds(r)
        rng = np.random.Generator(np.random.Philox(B + workgroups))
        lists = {(b, 0): np.sort(rng.permutation(P)[:max(1, P - 2)]).astype(np.int32) for b, P in enumerate(w.pages_per_seq)}
        for counts in ((64 // G, 64 // G + 1, B, 0), (B, 1, 64 // G + 2, B - 1)):
            active = [np.sort(rng.permutation(B)[:n]).astype(np.int32) for n in counts]
            check_sparse_attn(r, 1, active, lists)
    finally:
        r.close()


@pytest.mark.parametrize("B,G,d,g,n,workgroups", [
    (8, 5, 128, 16, 3, 256),     # 15 rows: one short of a row block
    (8, 2, 64, 32, 8, 256),      # 16 rows, pages of two 16-token tiles
    (17, 1, 128, 32, 17, 7),     # 17 rows: a second row block of one row, a few shares
    (32, 7, 64, 16, 7, 1024),    # 49 rows, more shares than pages in the short prefixes
    (9, 13, 64, 16, 5, 256),     # 65 rows: the scoring kernel's second chunk of rows is one row
    (8, 4, 128, 16, 4, 1)])      # one share: more than 64 pages per wavefront, a second batch of page entries
def test_float_mode_at_the_edges_of_rows_pages_and_shares(B, G, d, g, n, workgroups):
    """Prefixes around a 16-token tile, a page, the scoring kernel's 8 pages and the share count."""
    w = workload(B, G, 1, d, g, (1, 15, 17, 33, 8 * g + 1, 4900), n, dtype="f32")
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: workgroups})
    try:
        check_page_bounds(r)
        run_steps_end_to_end(r, range(w.T), orc.SEL_TOPK, float(n), w.topk_pages)
        check_sparse_attn(r, 1, [r.inp.picked[1, b] for b in range(w.batch)],
                          {(b, 0): np.arange(0, P, 2, dtype=np.int32) for b, P in enumerate(w.pages_per_seq)})
    finally:
        r.close()


@pytest.mark.parametrize("Hq,Hkv,d,batch", [
    (6, 2, 128, 1), (6, 2, 64, 3),   # channels of a head spread over workgroups
    (64, 8, 128, 1),                 # the last head count they are spread for ...
    (65, 5, 128, 1), (43, 1, 64, 3)])   # ... and the first ones a workgroup takes all channels of
@pytest.mark.parametrize("B", [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64])
def test_block_merge_at_the_edges_of_row_and_key_tiles(B, Hq, Hkv, d, batch):
    """Row tiles of 16, key tiles of 32, tokens staged in pairs; one sequence has an empty prefix."""
    ctx = L.losa_create(L.make_config(max_batch=batch, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, hidden_size=Hq * d,
                                      page_size=16, block_size=B, max_pages_per_seq=4, max_topk_pages=1,
                                      dtype=L.LOSA_BF16), torch.device("cuda"))
    gen = torch.Generator().manual_seed(B * Hq + d)
    q, k, v = (torch.randn((batch * B, n, d), generator=gen).to(torch.bfloat16) for n in (Hq, Hkv, Hkv))
    o_p, lse_p = torch.randn((batch * B, Hq, d), generator=gen), torch.randn((batch * B, Hq), generator=gen) + 3
    o_p[-B:], lse_p[-B:] = float("nan"), float("-inf")
    dev = [x.cuda() for x in (q, k, v, o_p, lse_p)]
    out, o_b, lse_b = torch.empty_like(dev[3]), torch.empty_like(dev[3]), torch.empty_like(dev[4])
    try:
        L.losa_block_merge(ctx, *dev, out, o_b, lse_b)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    ref = orc.block_attention_and_merge(q.float().numpy(), k.float().numpy(), v.float().numpy(), np.nan_to_num(o_p.numpy()),
                                        lse_p.numpy(), B)
    for got, want in zip((out, o_b, lse_b), ref):
        assert np.abs(got.cpu().numpy() - want).max() <= 2e-2
    # Probabilities enter as a bfloat16 pair: high part truncated, remainder (below 2^-7 of it) rounded to 8 bits, so off
    # by at most 2^-16 each, and an output by 2^-16 of the largest value; exponentials and sums in float add less than 2e-5.
    for got, want in zip((out, o_b, lse_b), ref):
        assert np.abs(got.cpu().numpy() - want).max() <= 2.0 ** -16 * float(v.float().abs().max()) + 2e-5


@pytest.mark.parametrize("B", [16, 64])
def test_block_merge_in_place(B):
    """The result and the block's log-sum-exp written over the prefix statistics they are merged with, at a size whose
    channels are otherwise spread over workgroups (8 heads: 32 of them): bit for bit those of separate buffers."""
    Hq, Hkv, d = 8, 2, 128
    ctx = L.losa_create(L.make_config(max_batch=1, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, hidden_size=Hq * d,
                                      page_size=16, block_size=B, max_pages_per_seq=4, max_topk_pages=1,
                                      dtype=L.LOSA_BF16), torch.device("cuda"))
    gen = torch.Generator().manual_seed(B)
    q, k, v = (torch.randn((B, n, d), generator=gen).to(torch.bfloat16).cuda() for n in (Hq, Hkv, Hkv))
    o_p, lse_p = torch.randn((B, Hq, d), generator=gen).cuda(), torch.randn((B, Hq), generator=gen).cuda() + 3
    out, o_b, lse_b = torch.empty_like(o_p), torch.empty_like(o_p), torch.empty_like(lse_p)
    try:
        L.losa_block_merge(ctx, q, k, v, o_p, lse_p, out, o_b, lse_b)
        for _ in range(20):
            o_io, lse_io = o_p.clone(), lse_p.clone()
            L.losa_block_merge(ctx, q, k, v, o_io, lse_io, o_io, None, lse_io)
            torch.cuda.synchronize()
            assert torch.equal(o_io, out) and torch.equal(lse_io, lse_b)
    finally:
        ctx.close()


@pytest.mark.parametrize("B", [1, 2, 4, 5, 16, 63, 255, 256, 257, 1023, 1024])
def test_cumulative_mass_at_the_edges_of_its_prefix_sums(B):
    """Block sizes around the four scores per read and the 256 tokens the scoring kernel ranks for itself.  Scores
    are squares of small integers, so every sum is exact and the sets, full of ties, have to be equal."""
    rng, H, dev = np.random.Generator(np.random.Philox(B)), 64, "cuda:0"
    v = rng.integers(0, 8, size=(3, B)).astype(np.float32)
    v[2] = 0.0                                      # a sequence without any change
    h = torch.from_numpy(np.repeat(v.reshape(-1, 1), H, axis=1)).to(dev, torch.bfloat16)
    out = (torch.zeros(3 * B, device=dev), torch.zeros(3 * B, dtype=torch.uint8, device=dev),
           torch.zeros(3 * B, dtype=torch.int32, device=dev), torch.zeros(3, dtype=torch.int32, device=dev))
    for tau in (0.0, 2.0 ** -20, 0.25, 0.5, 0.75, 1.0):   # (products with the total are exact too)
        L.losa_select_active_static(L.LOSA_BF16, 3, B, H, h, torch.zeros_like(h), orc.SEL_MASS, tau, *out)
        mask, idx, count = (x.cpu().numpy() for x in out[1:])
        for b in range(3):
            A = orc.active_set(v[b] ** 2, orc.SEL_MASS, tau)
            assert np.array_equal(idx[b * B:b * B + count[b]], A) and np.all(idx[b * B + count[b]:(b + 1) * B] == -1)
            assert np.array_equal(np.nonzero(mask[b * B:(b + 1) * B])[0], A)
    if B <= 64:
        w = workload(B, 1, 1, 64, 16, (33, 300), max(1, B // 3))
        r = Rig(w)
        try:
            check_page_bounds(r)
            run_steps_end_to_end(r, range(2), orc.SEL_MASS, 0.5, w.topk_pages)
            run_steps_end_to_end(r, [2], orc.SEL_MASS, 1.0, w.topk_pages)
        finally:
            r.close()


@pytest.mark.parametrize("B,select_round", [(B, 0) for B in (1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 128, 255, 256)] +
                         [(B, 1 << 30) for B in (1, 2, 3, 4, 5, 31, 32, 33, 63, 64)])
def test_active_set_of_a_step_at_the_edges_of_its_ranking(B, select_round):
    """losa_step ranks the block where it scores: a lane per token up to 64 tokens, by the sixteen wavefronts of the launch that also
    selects or, with the selection's grid set, by the four of the scoring kernel; a thread per token beyond, in the scoring kernel.
    Scores are squares of small integers, full of ties, so the sets have to be equal; three query heads per KV head."""
    rng, d, dev = np.random.Generator(np.random.Philox(B)), 64, "cuda:0"
    v = rng.integers(0, 8, size=(3, B)).astype(np.float32)
    v[2] = 0.0                                      # a sequence without any change
    lens = torch.tensor([40, 200, 1], dtype=torch.int32, device=dev)
    pages, Hq, Hkv, g = [3, 13, 1], 6, 2, 16
    h = torch.from_numpy(np.repeat(v.reshape(-1, 1), Hq * d, axis=1)).to(dev, torch.bfloat16)
    gen = torch.Generator(device=dev)
    gen.manual_seed(B)
    draw = lambda *shape: torch.randn(shape, generator=gen, device=dev).to(torch.bfloat16)
    kv = L.PagedKV(draw(17, Hkv, g, d), draw(17, Hkv, d, g), draw(17, Hkv, 2, d),
                   torch.tensor([0, 3, 16, 17], dtype=torch.int32, device=dev),
                   torch.randperm(17, generator=gen, device=dev).to(torch.int32), lens, max_seq_pages=13)
    ctx = L.losa_create(L.make_config(max_batch=3, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, hidden_size=Hq * d,
                                      page_size=g, block_size=B, max_pages_per_seq=13, max_topk_pages=2), dev)
    L.losa_set_tuning(ctx, L.LOSA_TUNE_SELECT_ROUND, select_round)
    try:
        L.losa_page_bounds(ctx, kv)
        q = draw(3 * B, Hq, d)
        o_p, lse_p = torch.zeros((3 * B, Hq, d), device=dev), torch.zeros((3 * B, Hq), device=dev)
        mask = torch.zeros(3 * B, dtype=torch.uint8, device=dev)
        order = [kv.page_indices[a:a + n].long() for a, n in ((0, 3), (3, 13), (16, 1))]
        tokens = lambda x: [to_host(x[order[b]].transpose(1, 2).reshape(-1, Hkv, d)[:int(lens[b])]) for b in range(3)]
        cache = orc.PrefixCache(tokens(kv.k_pages), tokens(kv.v_pages.transpose(2, 3)), g)
        for mode, param in ((orc.SEL_TOPK, 0.0), (orc.SEL_TOPK, 1.0), (orc.SEL_TOPK, float(B // 2)), (orc.SEL_TOPK, float(B)),
                            (orc.SEL_FRACTION, 0.3), (orc.SEL_THRESHOLD, 8.0), (orc.SEL_THRESHOLD, -1.0),
                            (orc.SEL_MASS, 0.0), (orc.SEL_MASS, 0.25), (orc.SEL_MASS, 0.75), (orc.SEL_MASS, 1.0)):
            mask.fill_(9)
            o_p.fill_(7.0)
            lse_p.fill_(7.0)
            one = scored_in_one_launch(ctx, lambda: L.losa_step(ctx, kv, 1, h, torch.zeros_like(h), q, mode, param, 2, o_p, lse_p, mask))
            assert not mask.any() or one == (B <= 64 and not select_round)
            got = mask.cpu().numpy().reshape(3, B)
            want = [orc.active_set(v[b] ** 2, mode, param) for b in range(3)]
            for b in range(3):
                assert np.array_equal(got[b], np.isin(np.arange(B), want[b]).astype(np.uint8)), (b, mode, param)
            # the list, of which every wavefront that ranks holds a copy, is what the rest of the step goes by
            o, lse = np.full((3 * B, Hq, d), 7.0), np.full((3 * B, Hq), 7.0)
            orc.losa_step(cache, 1, None, None, to_host(q), mode, param, 2, B, Hq, o, lse, forced_active=want)
            active = np.concatenate([b * B + want[b] for b in range(3)])
            stable = np.setdiff1d(np.arange(3 * B), active)
            got_o, got_l = o_p.cpu().numpy(), lse_p.cpu().numpy()
            assert np.all(got_o[stable] == 7.0) and np.all(got_l[stable] == 7.0), (mode, param)
            assert np.all(np.abs(got_o[active] - o[active]) <= 2e-2) and np.all(np.abs(got_l[active] - lse[active]) <= 2e-2), (mode, param)
    finally:
        ctx.close()


@pytest.mark.parametrize("dtype,B,G,select_round", [("bf16", 9, 8, 0), ("bf16", 16, 7, 0), ("bf16", 33, 4, 0), ("bf16", 64, 4, 0), ("bf16", 65, 4, 0),
                                                    ("bf16", 256, 2, 0), ("f32", 24, 4, 0), ("bf16", 9, 8, 1 << 30), ("bf16", 33, 4, 1 << 30),
                                                    ("bf16", 64, 4, 1 << 30)])     # (set: ranked in the scoring kernel, see above)
def test_scores_that_are_no_number_rank_with_infinity(dtype, B, G, select_round):
    """Several tokens whose change is NaN and one whose change is infinite: top-n selections hold exactly n tokens (64 query
    rows per KV head at most, and fewer than there are such tokens), the steps attend for exactly those, over a
    workspace that holds no page table of an earlier step."""
    n = 64 // G if B * G > 64 else B // 2
    rng = np.random.Generator(np.random.Philox(B * G))
    odd = [np.sort(rng.permutation(B)[:min(B, n + 2)]), np.array([0, B - 1]), np.sort(rng.permutation(B)[:3])]

    def poison(inp):
        nan, inf = (0x7FC0, 0x7F80) if dtype == "bf16" else (np.nan, np.inf)
        for b in range(3):
            inp.h[1, b * B + odd[b], 5] = nan
            inp.h[1, b * B + odd[b][-1], 5] = inf
    w = workload(B, G, 1, 64, 16, (700, 33, 160), n, dtype=dtype)
    r = Rig(w, mutate=poison, tuning={L.LOSA_TUNE_SELECT_ROUND: select_round})
    blk = r.blk
    r.ctx.workspace.fill_(255)
    try:
        check_page_bounds(r)
        run_steps_end_to_end(r, [0], orc.SEL_TOPK, 1.0, w.topk_pages)
        delta = orc.locality_score(r.inp.h[1], r.inp.h[0]).reshape(3, B)
        assert all(np.isnan(delta[b, odd[b][:-1]]).all() and np.isposinf(delta[b, odd[b][-1]]) for b in range(3))
        for mode, param in ((orc.SEL_TOPK, 1.0), (orc.SEL_TOPK, float(n)), (orc.SEL_FRACTION, n / B), (orc.SEL_TOPK, float(B)),
                            (orc.SEL_THRESHOLD, 1e-3), (orc.SEL_MASS, 0.5)):
            want = [orc.active_set(delta[b], mode, param) for b in range(3)]
            before_o, before_l = blk.o_p.clone(), blk.lse_p.clone()
            L.losa_step(r.ctx, r.layer.kv, 1, blk.h[1], blk.h[0], blk.q[1], mode, param, w.topk_pages, blk.o_p, blk.lse_p, blk.mask,
                        blk.sel_count)
            torch.cuda.synchronize()
            mask, pages = blk.mask.cpu().numpy().reshape(3, B), blk.sel_count.cpu().numpy()
            assert all(np.array_equal(np.nonzero(mask[b])[0], want[b]) for b in range(3)), (mode, param)
            scores, picks, _ = oracle_selection(r, 1, want, w.topk_pages)
            union, _ = gpu_union_of(r, 1, want, w.topk_pages, scores, picks)
            assert all(pages[b, 0] == len(union[b, 0]) for b in range(3))
            orc.losa_step(r.cache, 1, None, None, r.inp.q[1], mode, param, w.topk_pages, w.B, w.Hq, r.o_ref, r.L_ref,
                          forced_active=want, forced_union=union)
            compare_state(r, want, before_o, before_l)
            for call in (lambda *out: L.losa_select_active(r.ctx, blk.h[1], blk.h[0], mode, param, *out),
                         lambda *out: L.losa_select_active_static(r.ctx.cfg.dtype, 3, B, w.H, blk.h[1], blk.h[0], mode, param, *out)):
                call(blk.delta, blk.mask, blk.active_idx, blk.active_count)
                idx, count = blk.active_idx.cpu().numpy().reshape(3, B), blk.active_count.cpu().numpy()
                assert all(np.array_equal(idx[b, :count[b]], want[b]) for b in range(3)), (mode, param)
    finally:
        r.close()


@pytest.mark.parametrize("P", [1, 7, 64, 255, 256, 2047, 2048, 2049, 4096, 4097, 8192, 8193, 16384])
def test_selection_at_the_edges_of_its_digits_buckets_and_threads(P):
    """Scores set one by one (a page's bounds are its value in one channel, the query is 1, -1 or 0 there): clusters that
    overflow the bucket ranked directly, ladders of neighbouring floats that need every digit, few values, one value,
    the whole float range, infinities.  Picks and unions have to be equal: larger score first, then smaller page."""
    rng, d, B, g, dev = np.random.Generator(np.random.Philox(P)), 64, 4, 16, "cuda:0"
    ladder = (np.float32(3.0).view(np.int32) + rng.integers(0, 3 * P, P)).astype(np.int32).view(np.float32)
    wide = (rng.choice([-1.0, 1.0], P) * 10.0 ** rng.uniform(-30, 30, P)).astype(np.float32)
    normal = (40 + 10 * rng.standard_normal(P)).astype(np.float32)
    kinds = {"normal": normal, "wide": wide, "ladder": ladder,
             "cluster": np.where(rng.random(P) < 0.3, 7 + 1e-4 * rng.random(P), 50 * rng.standard_normal(P)).astype(np.float32),
             "few": rng.integers(-2, 3, P).astype(np.float32), "one": np.full(P, -1.5, np.float32),
             "infinite": np.where(rng.random(P) < 0.1, rng.choice([-np.inf, np.inf], P), normal).astype(np.float32)}
    page_ids = torch.from_numpy(rng.permutation(P).astype(np.int32)).to(dev)
    one_page = torch.zeros((1, 1, g, d), device=dev)
    meta = torch.zeros((P, 1, 2, d), device=dev)
    kv = L.PagedKV(one_page.expand(P, 1, g, d), one_page.reshape(1, 1, d, g).expand(P, 1, d, g), meta,
                   torch.tensor([0, P], dtype=torch.int32, device=dev), page_ids,
                   torch.tensor([P * g - 3], dtype=torch.int32, device=dev), max_seq_pages=P)
    ctx = L.losa_create(L.make_config(max_batch=1, num_q_heads=1, num_kv_heads=1, head_dim=d, hidden_size=d, page_size=g,
                                      block_size=B, max_pages_per_seq=P, max_topk_pages=P, dtype=L.LOSA_F32), dev)
    active, count = torch.arange(B, dtype=torch.int32, device=dev), torch.tensor([B], dtype=torch.int32, device=dev)
    sel, cnt = torch.zeros((1, 1, P), dtype=torch.int32, device=dev), torch.zeros((1, 1), dtype=torch.int32, device=dev)
    try:
        for kind, value in kinds.items():
            meta[page_ids.long(), 0, :, 0] = torch.from_numpy(value).to(dev)[:, None]
            scale = np.array([1.0, -1.0, 2.0 if kind == "infinite" else 0.0, 1.0], np.float32)
            q = torch.zeros((B, 1, d), device=dev)
            q[:, 0, 0] = torch.from_numpy(scale).to(dev)
            for K in sorted({1, min(2, P), min(65, P), max(1, P // 16), max(1, P - 1), P}):
                tk = torch.full((1, B, 1, K), -7, dtype=torch.int32, device=dev)
                L.losa_score_pages(ctx, kv, q, active, count, K, tk, sel, cnt, P)
                torch.cuda.synchronize()
                got = tk.cpu().numpy().reshape(B, K)
                with np.errstate(over="ignore"):
                    want = [np.sort(np.argsort(-(s * value), kind="stable")[:K]) for s in scale]
                for r in range(B):
                    assert np.array_equal(got[r], want[r]), (kind, K, r)
                union = np.unique(np.concatenate(want))
                assert int(cnt.item()) == len(union) and np.array_equal(sel.cpu().numpy().reshape(-1)[:len(union)], union), (kind, K)
                L.losa_score_pages_shared(ctx, kv, q, active, torch.ones_like(count), K, sel, cnt, P)   # row 0 alone
                torch.cuda.synchronize()
                assert int(cnt.item()) == K and np.array_equal(sel.cpu().numpy().reshape(-1)[:K], want[0]), (kind, K, "shared")
    finally:
        ctx.close()


def rows_of_every_kind(rng, P, bf16):
    """Page values of rows that a selection treats in different ways: one histogram, several, every digit, ties cut, one value."""
    base, step, shift = (0x4040, 1, 16) if bf16 else (0x40400000, 3, 0)      # 3.0
    spread = 100 if bf16 else step * P                                      # neighbouring numbers of the type
    ladder = ((base + rng.integers(0, spread, P)) << shift).astype(np.uint32).view(np.float32)
    rows = [(40 + 10 * rng.standard_normal(P)), np.full(P, -1.5), ladder, rng.integers(-2, 3, P),
            np.where(rng.random(P) < 0.3, 7 + 1e-4 * rng.random(P), 50 * rng.standard_normal(P)),
            rng.choice([-1.0, 1.0], P) * 10.0 ** rng.uniform(-30, 30, P), rng.standard_normal(P)]
    return [torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16 if bf16 else torch.float32).float().numpy() for x in rows]


@pytest.mark.parametrize("P", [65, 2047, 2048, 2049, 4097, 8193, 16384])
def test_selection_of_several_rows_per_workgroup_with_the_list(P):
    """Rows of different kinds come one after the other in a workgroup, whose LDS state the next row starts from: up to eight
    rows each (61 rows: eight workgroups, the last ones with one row less).  A row reads its kind's channel."""
    rng, d, B, g, dev = np.random.Generator(np.random.Philox(P)), 64, 61, 16, "cuda:0"
    kinds = rows_of_every_kind(rng, P, bf16=False)
    kind_of = [(r // 8 + r) % len(kinds) for r in range(B)]       # changes along a workgroup's rows r, r + 8, r + 16, ...
    sign = np.where(np.arange(B) % 3 == 2, -1.0, 1.0).astype(np.float32)
    page_ids = torch.from_numpy(rng.permutation(P).astype(np.int32)).to(dev)
    meta, one_page = torch.zeros((P, 1, 2, d), device=dev), torch.zeros((1, 1, g, d), device=dev)
    for c, value in enumerate(kinds):
        meta[page_ids.long(), 0, :, c] = torch.from_numpy(value).to(dev)[:, None]
    q = torch.zeros((B, 1, d), device=dev)
    q[torch.arange(B), 0, torch.tensor(kind_of)] = torch.from_numpy(sign).to(dev)
    kv = L.PagedKV(one_page.expand(P, 1, g, d), one_page.reshape(1, 1, d, g).expand(P, 1, d, g), meta,
                   torch.tensor([0, P], dtype=torch.int32, device=dev), page_ids,
                   torch.tensor([P * g - 3], dtype=torch.int32, device=dev), max_seq_pages=P)
    ctx = L.losa_create(L.make_config(max_batch=1, num_q_heads=1, num_kv_heads=1, head_dim=d, hidden_size=d, page_size=g,
                                      block_size=B, max_pages_per_seq=P, max_topk_pages=P, dtype=L.LOSA_F32), dev)
    active, count = torch.arange(B, dtype=torch.int32, device=dev), torch.zeros(1, dtype=torch.int32, device=dev)
    sel, cnt = torch.zeros((1, 1, P), dtype=torch.int32, device=dev), torch.zeros((1, 1), dtype=torch.int32, device=dev)
    try:
        for rnd, n in ((1, B), (1, 9), (B // 2, B)):              # (the last: three rows each)
            L.losa_set_tuning(ctx, L.LOSA_TUNE_SELECT_ROUND, rnd)
            count.fill_(n)
            for K in sorted({1, max(1, P // 16), P // 2, P - 1, P}):
                tk = torch.full((1, B, 1, K), -7, dtype=torch.int32, device=dev)
                L.losa_score_pages(ctx, kv, q, active, count, K, tk, sel, cnt, P)
                torch.cuda.synchronize()
                want = [np.sort(np.argsort(-(sign[r] * kinds[kind_of[r]]), kind="stable")[:K]) for r in range(n)]
                got = tk.cpu().numpy().reshape(B, K)
                for r in range(n):
                    assert np.array_equal(got[r], want[r]), (rnd, n, K, r, kind_of[r])
                union = np.unique(np.concatenate(want))
                assert int(cnt.item()) == len(union) and np.array_equal(sel.cpu().numpy().reshape(-1)[:len(union)], union), (rnd, n, K)
    finally:
        ctx.close()


@pytest.mark.parametrize("P,B,G", [(65, 17, 1), (2048, 17, 1), (2049, 17, 1), (4097, 61, 1), (16384, 17, 1),
                                   (65, 61, 3), (2048, 61, 3), (4097, 61, 3), (8193, 61, 3)])
def test_selection_of_several_rows_per_workgroup_with_the_bitmap(P, B, G):
    """The same in losa_step, whose selection leaves a bitmap: up to four rows a workgroup, counts known to the host and to
    the device only.  All keys are zero, so that every token of the union has the same weight, and a page's values are its
    own signs in 64 channels: the sums, whole numbers, tell which pages the union holds."""
    rng, d, g, dev = np.random.Generator(np.random.Philox(P + B)), 64, 16, "cuda:0"
    kinds = rows_of_every_kind(rng, P, bf16=True)
    page_ids = rng.permutation(P).astype(np.int32)
    signs = rng.choice([-1.0, 1.0], (P, d)).astype(np.float32)              # by logical page
    meta, v_pages = torch.zeros((P, 1, 2, d)), torch.zeros((P, 1, d, g))
    for c, value in enumerate(kinds):
        meta[page_ids, 0, :, c] = torch.from_numpy(value)[:, None]
    v_pages[page_ids, 0] = torch.from_numpy(signs)[:, :, None]
    kind_of = (np.arange(B * G) // 4 + np.arange(B * G)) % len(kinds)
    q = torch.zeros((B * G, d))
    q[torch.arange(B * G), torch.from_numpy(kind_of)] = 1.0
    bf = lambda x: x.to(torch.bfloat16).to(dev)
    kv = L.PagedKV(bf(torch.zeros((P, 1, g, d))), bf(v_pages), bf(meta), torch.tensor([0, P], dtype=torch.int32, device=dev),
                   torch.from_numpy(page_ids).to(dev), torch.tensor([P * g], dtype=torch.int32, device=dev), max_seq_pages=P)
    ctx = L.losa_create(L.make_config(max_batch=1, num_q_heads=G, num_kv_heads=1, head_dim=d, hidden_size=G * d, page_size=g,
                                      block_size=B, max_pages_per_seq=P, max_topk_pages=P), dev)
    ctx.workspace.fill_(255)
    h = bf(torch.ones((B, G * d)))
    o_p, lse_p = torch.zeros((B, G, d), device=dev), torch.zeros((B, G), device=dev)
    mask, cnt = torch.zeros(B, dtype=torch.uint8, device=dev), torch.zeros((1, 1), dtype=torch.int32, device=dev)
    try:
        for rnd in (1, B * G // 2):
            L.losa_set_tuning(ctx, L.LOSA_TUNE_SELECT_ROUND, rnd)
            for mode, param, n in ((orc.SEL_TOPK, float(B), B), (orc.SEL_TOPK, 5.0, 5), (orc.SEL_THRESHOLD, 0.5, B)):
                for K in sorted({1, max(1, P // 64), max(1, P // 8)}):
                    L.losa_step(ctx, kv, 1, h, torch.zeros_like(h), bf(q).reshape(B, G, d), mode, param, K, o_p, lse_p, mask, cnt)
                    torch.cuda.synchronize()
                    union = np.unique(np.concatenate([np.argsort(-kinds[kind_of[r]], kind="stable")[:K] for r in range(n * G)]))
                    assert int(mask.sum()) == n and int(cnt.item()) == len(union), (rnd, mode, n, K)
                    total = signs[union].sum(axis=0)
                    got = o_p.cpu().numpy()[:n].reshape(-1, d).astype(np.float64) * len(union)
                    assert np.abs(got - total).max() <= 0.25, (rnd, mode, n, K)       # a page more, less or another: 1 or 2
                    assert np.abs(lse_p.cpu().numpy()[:n] - np.log(len(union) * g)).max() <= 1e-4
    finally:
        ctx.close()


@pytest.mark.parametrize("page", [16, 32])
@pytest.mark.parametrize("B,G,d", [
    (13, 5, 128),     # 65 rows: two token groups
    (32, 4, 64),      # 128 rows
    (43, 3, 64),      # 129 rows: one token group
    (64, 4, 128)])    # 256 rows
def test_many_row_kernel_normalises_with_the_weights_it_applies(B, G, d, page):
    """Half-precision numerators: what their roundings have in common has to cancel.  One token carries a row and
    arrives after the reference was taken, 4 to 7.5 log2 units above it, so that its numerator is rounded at every
    place of the half-precision grid; its value is 100 in half of the channels, and one channel is 3 in every token.
    With weights w_i (1 + e_i), |e_i| <= 2^-11, divided by their own sum, an output is off by at most
    2^-11 * sum w_i |v_i - o| to first order, plus float arithmetic (1e-4 at |v| = 100)."""
    n, Hkv, rows, unit = 200, 2, B * G, np.log(2.0) * np.sqrt(d)
    rng = np.random.Generator(np.random.Philox(B * G + page))
    bf = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16)
    q = np.zeros((B, Hkv * G, d))
    q[:, :, 0], q[:, :, 1] = 1.0, rng.random((B, Hkv * G))
    k = np.zeros((n, d))
    k[:, 0] = -20 * unit
    k[[0, 32], 0] = 0.0                             # the reference of either token group
    k[70, :2] = 4 * unit, 3.5 * unit
    v = rng.standard_normal((n, d))
    v[70, :d // 2], v[:, d - 1] = 100.0, 3.0
    q, k, v = bf(q), bf(k), bf(v)
    pages = -(-n // page)
    kp, vp = torch.zeros((pages * page, d), dtype=torch.bfloat16), torch.zeros((pages * page, d), dtype=torch.bfloat16)
    kp[:n], vp[:n] = k, v
    kp = kp.reshape(pages, 1, page, d).expand(-1, Hkv, -1, -1).contiguous().cuda()
    vp = vp.reshape(pages, 1, page, d).transpose(2, 3).expand(-1, Hkv, -1, -1).contiguous().cuda()
    ints = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
    kv = L.PagedKV(kp, vp, torch.zeros((pages, Hkv, 2, d), dtype=torch.bfloat16, device="cuda"), ints(0, pages),
                   torch.arange(pages, dtype=torch.int32, device="cuda"), ints(n))
    ctx = L.losa_create(L.make_config(max_batch=1, num_q_heads=Hkv * G, num_kv_heads=Hkv, head_dim=d, hidden_size=Hkv * G * d,
                                      page_size=page, block_size=B, max_pages_per_seq=pages, max_topk_pages=1), "cuda:0")
    o_p, lse_p = torch.zeros((B, Hkv * G, d), device="cuda"), torch.zeros((B, Hkv * G), device="cuda")
    try:
        L.losa_set_tuning(ctx, L.LOSA_TUNE_ATTN_WORKGROUPS, 1)      # one workgroup walks all of the tokens
        L.losa_sparse_attn(ctx, kv, q.cuda(), None, None, None, None, 0, o_p, lse_p)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    q64, k64, v64 = (x.double().numpy() for x in (q.reshape(-1, d), k, v))
    s = q64 @ k64.T / np.sqrt(d)
    top = s.max(axis=1, keepdims=True)
    lse = np.log(np.exp(s - top).sum(axis=1)) + top[:, 0]
    w = np.exp(s - lse[:, None])
    o = w @ v64
    bound = np.stack([2.0 ** -11 * (w[r][:, None] * np.abs(v64 - o[r])).sum(axis=0) for r in range(len(w))]) + 1e-4
    err = np.abs(o_p.cpu().double().numpy().reshape(-1, d) - o)
    assert len(w) == Hkv * rows and (err <= bound).all(), f"off by {(err / bound).max():.1f} times the bound, {err.max():.3g}"
    assert np.abs(lse_p.cpu().numpy().reshape(-1) - lse).max() <= 2e-5      # the unrounded sum


@pytest.mark.parametrize("d,page", [(64, 16), (128, 32)])
def test_float_mode_keeps_values_near_the_end_of_the_range(d, page):
    """Values of 1e33 under a token that scores 15 above the reference its wavefront took first: a weight of e^15
    times the value is past the range of a float, their quotient is not.  Relative bound 1e-4, the mode's."""
    B, heads, pages = 4, 2, 9
    n, unit = pages * page - 3, np.sqrt(d)
    rng = np.random.Generator(np.random.Philox(d))
    q, k = np.zeros((B, heads, d), np.float32), np.zeros((n, d), np.float32)
    q[:, :, 0] = 1.0
    k[:, 0] = -30 * unit
    k[::4 * page, 0] = (0, -unit, 15 * unit)        # pages 0 and 8 belong to one wavefront of the first workgroup
    v = (rng.standard_normal((n, d)) * 1e33).astype(np.float32)
    kp, vp = np.zeros((pages * page, d), np.float32), np.full((pages * page, d), np.nan, np.float32)
    kp[:n], vp[:n] = k, v
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    kv = L.PagedKV(dev(kp.reshape(pages, 1, page, d)), dev(vp.reshape(pages, 1, page, d).transpose(0, 1, 3, 2)),
                   torch.zeros((pages, 1, 2, d), device="cuda"), dev(np.array([0, pages], np.int32)),
                   dev(np.arange(pages, dtype=np.int32)), dev(np.array([n], np.int32)))
    ctx = L.losa_create(L.make_config(max_batch=1, num_q_heads=heads, num_kv_heads=1, head_dim=d, hidden_size=heads * d,
                                      page_size=page, block_size=B, max_pages_per_seq=pages, max_topk_pages=1,
                                      dtype=L.LOSA_F32), "cuda:0")
    o_p, lse_p = torch.zeros((B, heads, d), device="cuda"), torch.zeros((B, heads), device="cuda")
    try:
        for workgroups in (1, 256):
            L.losa_set_tuning(ctx, L.LOSA_TUNE_ATTN_WORKGROUPS, workgroups)
            L.losa_sparse_attn(ctx, kv, dev(q), None, None, None, None, 0, o_p, lse_p)
            torch.cuda.synchronize()
            s = (q.reshape(-1, d).astype(np.float64) @ k.T.astype(np.float64)) / unit
            w = np.exp(s - 15.0)
            o, lse = (w @ v.astype(np.float64)) / w.sum(axis=1, keepdims=True), 15.0 + np.log(w.sum(axis=1))
            assert np.abs(o_p.cpu().numpy().reshape(-1, d) - o).max() <= 1e-4 * 1e33
            assert np.abs(lse_p.cpu().numpy().reshape(-1) - lse).max() <= 1e-4
    finally:
        ctx.close()


@pytest.mark.parametrize("page,limit,reserved", [
    (16, 5, 5), (16, 512, 512),              # copies of 16 words, the last prefix for them ...
    (16, 513, 513), (32, 1024, 1024),        # ... of 32 ...
    (16, 1025, 1025), (16, 2048, 2048), (16, 2049, 2049),   # ... and one bitmap, no copies
    (16, 40, 3000), (16, 600, 600 + 4096)])  # a context reserved for more pages than the call says it uses
def test_union_at_the_edges_of_its_copies(page, limit, reserved):
    """Every number of rows per copy (the rows of 1, 7 and 16 tokens, 4 heads each, over 16, 8 or 1 copies), the
    count known to the host and to the device only; every word of the bitmap gets a pick (the budget is a third)."""
    w = workload(16, 4, 1, 64, page, (limit * page - 3, max(1, limit // 3) * page + 1, 1), 16, topk=max(1, limit // 3), T=5)
    r = Rig(w)
    r.ctx.close()
    cfg = config_of(w, max_topk_pages=w.max_pages)
    cfg.max_pages_per_seq = reserved
    r.ctx = L.losa_create(cfg, "cuda:0")
    r.ctx.workspace.fill_(255)
    try:
        check_page_bounds(r)
        run_steps_end_to_end(r, range(1), orc.SEL_TOPK, 1.0, w.topk_pages)
        for t, n in ((1, 1.0), (2, 7.0), (3, 16.0)):
            run_steps_end_to_end(r, [t], orc.SEL_TOPK, n, w.topk_pages)
        run_steps_end_to_end(r, [4], orc.SEL_MASS, 0.5, w.topk_pages)
    finally:
        r.close()


@pytest.mark.parametrize("page,limit,B,G,workgroups", [
    (16, 5, 17, 4, 256), (16, 512, 33, 8, 256),       # 68 and 264 rows over copies of 16 words
    (16, 1024, 40, 4, 256),                           # ... of 32
    (16, 1025, 33, 4, 256), (32, 1100, 64, 4, 64),    # one copy per 64 rows: two (68 .. 132 rows), four (256)
    (16, 2049, 64, 7, 256),                           # ... eight (448)
    (16, 4099, 17, 4, 1),                             # one workgroup owns every page of a head
    (16, 16384, 17, 4, 2)])                           # the longest list of own pages: two heads, one workgroup each
def test_union_of_more_than_64_rows_at_the_edges_of_its_copies(page, limit, B, G, workgroups):
    """The many-row kernel makes the list of its own pages from the bitmap's copies; counts known to the host (all
    rows, the fewest it serves) and to the device only, next to a prefix that leaves most workgroups without a stage."""
    few = -(-65 // G)
    w = workload(B, G, 1, 64, page, (limit * page - 3, min(limit, 7) * page + 1), B, topk=max(1, limit // 9), T=4)
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: workgroups})
    r.ctx.workspace.fill_(255)
    try:
        check_page_bounds(r)
        run_steps_end_to_end(r, range(1), orc.SEL_TOPK, 1.0, w.topk_pages)
        run_steps_end_to_end(r, [1], orc.SEL_TOPK, float(B), w.topk_pages)
        run_steps_end_to_end(r, [2], orc.SEL_TOPK, float(few), w.topk_pages)
        run_steps_end_to_end(r, [3], orc.SEL_MASS, 0.9, w.topk_pages)
    finally:
        r.close()


@pytest.mark.parametrize("B,G,d,page,n", [(8, 4, 64, 16, 3), (8, 7, 128, 32, 7), (8, 8, 64, 32, 8), (24, 4, 128, 16, 17), (40, 7, 64, 16, 40)])
def test_listed_pages_that_do_not_exist_count_for_nothing(B, G, d, page, n):
    """Page lists are resolved in the attention kernels: pages outside the sequence, in any place of a list, and lists of an
    empty sequence leave the result of the other pages (neutral statistics if there are none); a second batch of
    list entries per wavefront."""
    w = workload(B, G, 1, d, page, (page * 300 - 5, page * 3, 1), n)
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: 3})
    blk, kv = r.blk, r.layer.kv
    dev = blk.q.device
    rng = np.random.Generator(np.random.Philox(B + G))
    try:
        active = torch.full((3, B), -1, dtype=torch.int32, device=dev)
        active[:, :n] = torch.from_numpy(np.sort(np.stack([rng.permutation(B)[:n] for _ in range(3)]), axis=1).astype(np.int32)).to(dev)
        count = torch.full((3,), n, dtype=torch.int32, device=dev)
        lens = kv.seq_lens.clone()
        lens[2] = 0
        part = L.PagedKV(kv.k_pages, kv.v_pages, kv.meta, kv.page_indptr, kv.page_indices, lens, max_seq_pages=300)
        valid = [np.sort(rng.permutation(300)[:211]), np.array([0, 2]), np.array([], dtype=np.int64)]
        cap, results = 300, []
        for extra in (0, 1):
            lists, cnt = torch.full((3, 1, cap), -9, dtype=torch.int32, device=dev), torch.zeros((3, 1), dtype=torch.int32, device=dev)
            for b in range(3):
                pages = valid[b]
                if extra:
                    bad = np.array([-1, 2 ** 31 - 1, -2 ** 31, (300, 3, 0)[b], (300, 3, 0)[b] + 5])
                    pages = rng.permutation(np.concatenate([pages, bad]))
                lists[b, 0, :len(pages)] = torch.from_numpy(pages.astype(np.int32)).to(dev)
                cnt[b, 0] = len(pages)
            o_p, lse_p = torch.full_like(blk.o_p, 3.0), torch.full_like(blk.lse_p, 3.0)
            L.losa_sparse_attn(r.ctx, part, blk.q[1], active, count, lists, cnt, cap, o_p, lse_p)
            torch.cuda.synchronize()
            results.append((o_p.cpu().numpy(), lse_p.cpu().numpy()))
        (o0, l0), (o1, l1) = results
        orc.losa_step(r.cache, 1, None, None, r.inp.q[1], 0, 0, 0, B, w.Hq, r.o_ref, r.L_ref,
                      forced_active=[active[b, :n].cpu().numpy() for b in range(3)], forced_union={(b, 0): valid[b] for b in range(3)})
        for b in range(3):
            rows = b * B + active[b, :n].cpu().numpy()
            if b == 2:
                assert np.all(o0[rows] == 0) and np.all(o1[rows] == 0) and np.all(l0[rows] == -np.inf) and np.all(l1[rows] == -np.inf)
            else:   # other shares, other order of the sums: half the parity tolerance
                assert np.abs(o0[rows] - r.o_ref[rows]).max() <= 2e-2 and np.abs(l0[rows] - r.L_ref[rows]).max() <= 2e-2
                assert np.abs(o0[rows] - o1[rows]).max() <= 1e-2 and np.abs(l0[rows] - l1[rows]).max() <= 1e-2
        untouched = np.setdiff1d(np.arange(3 * B), np.concatenate([b * B + active[b, :n].cpu().numpy() for b in range(3)]))
        assert np.all(o1[untouched] == 3.0) and np.all(l1[untouched] == 3.0)
    finally:
        r.close()


@pytest.mark.parametrize("B,G,d,page", [(9, 7, 128, 16), (16, 4, 64, 32), (33, 7, 64, 16), (40, 4, 128, 32)])
@pytest.mark.parametrize("chunks", [1, 4, 5, 8, 9])
def test_merge_of_few_chunks(B, G, d, page, chunks):
    """Chunk counts at the edges of the merge's forms, next to a sequence with fewer chunks than the launch; counts known to
    the host and to the device only, the latter up to 64 rows per head and with heads above and below them in one launch."""
    few = 9 if G == 7 else 16   # the most tokens whose rows are at most 64
    w = workload(B, G, 1, d, page, (page * 70 - 5, page * 2 + 1, 1), few, topk=40, T=6)
    r = Rig(w, tuning={L.LOSA_TUNE_ATTN_WORKGROUPS: chunks * 3})
    r.ctx.workspace.fill_(255)
    try:
        check_page_bounds(r)
        run_steps_end_to_end(r, [0], orc.SEL_TOPK, 1.0, w.topk_pages)
        run_steps_end_to_end(r, [1], orc.SEL_TOPK, float(few), w.topk_pages)
        run_steps_end_to_end(r, [2], orc.SEL_TOPK, 1.0, w.topk_pages)
        run_steps_end_to_end(r, [3], orc.SEL_MASS, 0.02, w.topk_pages)
        run_steps_end_to_end(r, [4], orc.SEL_MASS, 0.5, w.topk_pages)
        run_steps_end_to_end(r, [5], orc.SEL_MASS, 1.0, w.topk_pages)
    finally:
        r.close()


def scored_in_one_launch(ctx, step):
    """Whether the step that `step` makes scores and selects in one launch, which keeps no score matrix in memory.  (The scores of
    pages that exist are no NaN of all ones.)"""
    ctx.workspace.fill_(255)
    step()
    torch.cuda.synchronize()
    return bool((workspace_parts(ctx)["scores"].view(torch.int32) == -1).all())


ONE_LAUNCH = [(P, 64, 1, 16, B, G, H) for P in (1, 15, 64, 65, 255, 256)        # hidden states are taken in the launch up to 512
              for B, G, H in ((1, 1, 64), (17, 1, 520), (33, 3, 512), (64, 4, 256))]
ONE_LAUNCH += [(P, d, 8, g, 64, 4, H) for P, d, g, H in (                       # two tiles of pages per wavefront: 256 and 144 workgroups
    (257, 64, 16, 512), (383, 64, 32, 520), (511, 64, 16, 256), (512, 64, 32, 1024), (257, 128, 32, 520), (258, 128, 16, 256), (383, 128, 16, 1024),
    (511, 128, 32, 520), (512, 128, 16, 512), (512, 128, 32, 64))]


@pytest.mark.parametrize("P,d,Hkv,g,B,G,H", ONE_LAUNCH)
def test_scoring_and_selection_in_one_launch(P, d, Hkv, g, B, G, H):
    """Short prefixes: a launch that scores and selects (and scores the tokens, where hidden states are short) against numpy's picks and,
    bit for bit, against the separate launches; that it was one launch is seen from the score matrix.  Rows, values and sums as in the
    test of the bitmap above; two sequences; a KV head's channels hold the kinds of row one further than those of the head before."""
    rng, dev = np.random.Generator(np.random.Philox(P + B)), "cuda:0"
    lens = [P * g - 5, max(1, P * g // 3)]
    pages = [(n + g - 1) // g for n in lens]
    total = sum(pages)
    kinds = [rows_of_every_kind(rng, p, bf16=True) for p in pages]
    nk = len(kinds[0])
    page_ids = rng.permutation(total).astype(np.int32)
    signs = rng.choice([-1.0, 1.0], (total, d)).astype(np.float32)              # by logical page, one sequence behind the other
    bf = lambda x: x.to(torch.bfloat16).to(dev)
    meta, v_pages = torch.zeros((total, Hkv, 2, d)), torch.zeros((total, Hkv, d, g), dtype=torch.bfloat16)
    for b, first in enumerate((0, pages[0])):
        for c, value in enumerate(kinds[b]):
            for j in range(Hkv):
                meta[page_ids[first:first + pages[b]], j, :, (c - j) % nk] = torch.from_numpy(value)[:, None]
    v_pages[page_ids] = torch.from_numpy(signs).to(torch.bfloat16)[:, None, :, None].expand(-1, Hkv, -1, g)
    kind_of = (np.arange(B * G) // 4 + np.arange(B * G)) % nk
    one_hot = torch.nn.functional.one_hot(torch.from_numpy(kind_of), d).float().reshape(1, B, 1, G, d)
    q = bf(one_hot.expand(2, B, Hkv, G, d).contiguous()).reshape(2 * B, Hkv * G, d)
    kv = L.PagedKV(torch.zeros((total, Hkv, g, d), dtype=torch.bfloat16, device=dev), v_pages.to(dev), bf(meta),
                   torch.tensor([0, pages[0], total], dtype=torch.int32, device=dev), torch.from_numpy(page_ids).to(dev),
                   torch.tensor(lens, dtype=torch.int32, device=dev), max_seq_pages=P)
    ctx = L.losa_create(L.make_config(max_batch=2, num_q_heads=Hkv * G, num_kv_heads=Hkv, head_dim=d, hidden_size=H, page_size=g,
                                      block_size=B, max_pages_per_seq=P, max_topk_pages=P), dev)
    h = bf(torch.from_numpy((1.0 + rng.permutation(2 * B).astype(np.float32) / 64)[:, None].repeat(H, 1)))    # Delta = its square: no ties
    order = np.argsort(-to_host(h.float()).reshape(2, B, H)[:, :, 0], axis=1, kind="stable")
    out = lambda: (torch.zeros((2 * B, Hkv * G, d), device=dev), torch.zeros((2 * B, Hkv * G), device=dev),
                   torch.zeros(2 * B, dtype=torch.uint8, device=dev), torch.zeros((2, Hkv), dtype=torch.int32, device=dev))
    some = (B + 2) // 3 if Hkv == 1 else 33
    modes = [(orc.SEL_TOPK, float(B), B), (orc.SEL_TOPK, float(some), some)]
    if P <= 128:      # counts that only the device knows: beyond, the separate launches
        modes += [(orc.SEL_THRESHOLD, 0.5, B), (orc.SEL_THRESHOLD, 1e9, 0), (orc.SEL_MASS, 0.4, None)]
    try:
        for mode, param, n in modes:
            for K in sorted({1, max(1, P // 8), max(1, P - 1), P}):
                got, separate = out(), out()
                for o, rnd, one in ((got, 0, True), (separate, 1 << 30, n == 0)):      # (no active token: no scores either way)
                    L.losa_set_tuning(ctx, L.LOSA_TUNE_SELECT_ROUND, rnd)
                    step = lambda: L.losa_step(ctx, kv, 1, h, torch.zeros_like(h), q, mode, float(param), K, *o)
                    assert scored_in_one_launch(ctx, step) == one, (mode, n, K, rnd)
                assert all(torch.equal(x, y) for x, y in zip(got, separate)), (mode, n, K)
                o_p, lse_p, mask, cnt = (x.cpu().numpy() for x in got)
                for b, first in enumerate((0, pages[0])):
                    active = np.flatnonzero(mask[b * B:(b + 1) * B])
                    assert n is None or set(active) == set(order[b, :n]), (mode, n, K)
                    if not len(active):
                        assert not cnt[b].any()
                        continue
                    used = {int(k) for a in active for k in kind_of[a * G:a * G + G]}     # of head 0
                    picks = [np.argsort(-value, kind="stable")[:K] for value in kinds[b]]
                    last = lens[b] - (pages[b] - 1) * g                                   # tokens of the last page
                    for j in range(Hkv):
                        union = np.unique(np.concatenate([picks[(k + j) % nk] for k in used]))
                        assert cnt[b, j] == len(union), (mode, n, K, b, j)
                        weight = np.where(union == pages[b] - 1, last, g).astype(np.float64)
                        want = (signs[first + union] * weight[:, None]).sum(axis=0) / weight.sum()
                        err = np.abs(o_p[b * B + active].reshape(len(active), Hkv, G, d)[:, j] - want).max()
                        assert err * weight.sum() <= 0.25 * min(last, g), (mode, n, K, b, j)
    finally:
        ctx.close()


class OnePagePrefix:
    """Sequences whose pages are all the same few, for launches over prefixes of any length: the values of a physical page are its
    number, so a dense step's output is known."""

    def __init__(self, tokens, B, G, Hkv, d, g, batch=1, hidden=64):
        ints, self.heads, self.rows = (lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")), Hkv, B * G
        P = -(-tokens // g)
        ids = torch.arange(P, dtype=torch.int32, device="cuda") % 7
        v = torch.arange(7, device="cuda", dtype=torch.bfloat16)[:, None, None, None].expand(7, Hkv, d, g).contiguous()
        zeros = lambda *shape: torch.zeros(shape, device="cuda", dtype=torch.bfloat16)
        self.kv = L.PagedKV(zeros(7, Hkv, g, d), v, zeros(7, Hkv, 2, d), ints(*range(0, (batch + 1) * P, P)), ids.repeat(batch), ints(*[tokens] * batch),
                            max_seq_pages=P)
        self.ctx = L.losa_create(L.make_config(max_batch=batch, num_q_heads=Hkv * G, num_kv_heads=Hkv, head_dim=d, hidden_size=hidden, page_size=g,
                                               block_size=B, max_pages_per_seq=P, max_topk_pages=P), "cuda:0")
        weights = torch.full((P,), float(g), dtype=torch.float64, device="cuda")
        weights[-1] = tokens - (P - 1) * g
        self.mean, self.tokens = float((ids.double() * weights).sum() / tokens), tokens
        self.q, self.o_p = zeros(batch * B, Hkv * G, d), torch.zeros((batch * B, Hkv * G, d), device="cuda")
        self.lse_p, self.h = torch.zeros((batch * B, Hkv * G), device="cuda"), (zeros(batch * B, hidden) + 1, zeros(batch * B, hidden))

    def dense_shares(self):
        """Shares that the dense step's page list was split into: work items whose partials were written."""
        self.ctx.workspace.fill_(255)
        L.losa_step(self.ctx, self.kv, 0, None, None, self.q, orc.SEL_TOPK, 1.0, 1, self.o_p, self.lse_p)
        torch.cuda.synchronize()
        assert float((self.o_p - self.mean).abs().max()) <= 1e-3 and float((self.lse_p - np.log(self.tokens)).abs().max()) <= 1e-4
        written = int((workspace_parts(self.ctx)["partial_m"].view(torch.int32) != -1).sum())
        assert written % (self.heads * self.rows) == 0
        return written // (self.heads * self.rows)


def test_attention_workgroups_can_be_set_back_to_their_default():
    """A context whose number of workgroups was changed and set back splits a prefix as one that was never touched."""
    r = OnePagePrefix(16384, 16, 4, 1, 128, 16)
    try:
        default = r.dense_shares()
        for value, shares in ((100, 100), (256, default), (1, 1), (1024, 512), (256, default)):     # 512 tiles of 32 tokens
            L.losa_set_tuning(r.ctx, L.LOSA_TUNE_ATTN_WORKGROUPS, value)
            assert r.dense_shares() == shares, value
    finally:
        r.ctx.close()


@pytest.mark.parametrize("tokens,Hkv,d,g,shares", [
    (32768, 1, 128, 16, 64), (32768, 1, 64, 16, 128),          # what the merge takes in one go
    (131072, 1, 128, 16, 128), (524288, 1, 128, 32, 256),      # 4096 and 16384 tiles: 2 * sqrt(tiles)
    (524288, 2, 128, 32, 128), (524288, 1, 64, 32, 256)])      # ... at most a workgroup per compute unit
def test_long_prefixes_of_few_heads_fill_the_chip(tokens, Hkv, d, g, shares):
    r = OnePagePrefix(tokens, 16, 4, Hkv, d, g)
    try:
        assert r.dense_shares() == shares
    finally:
        r.ctx.close()


@pytest.mark.parametrize("tokens,G,Hkv,d,shares", [
    (100, 1, 1, 128, 2), (1024, 1, 1, 128, 16), (1024, 1, 8, 128, 16), (1024, 4, 4, 128, 16),   # two tiles of 32 tokens a share ...
    (2048, 4, 4, 128, 16), (1024, 4, 8, 128, 8), (1024, 1, 1, 64, 8)])   # ... four where 4096 rows of partials are passed, and with 64 channels
def test_short_prefixes_are_split_into_shares_of_two_or_four_tiles(tokens, G, Hkv, d, shares):
    r = OnePagePrefix(tokens, 16, G, Hkv, d, 16)
    try:
        assert r.dense_shares() == shares
    finally:
        r.ctx.close()


@pytest.mark.parametrize("P,d,Hkv,batch,n,hidden,one", [   # 7 query heads per KV head
    (100, 128, 1, 1, 2, 520, True), (192, 128, 4, 1, 2, 520, True), (193, 128, 4, 1, 3, 520, False),
    (256, 128, 8, 4, 2, 520, False), (256, 128, 8, 5, 2, 520, True),                         # 32 and 40 workgroups
    (256, 64, 1, 1, 2, 520, True), (257, 64, 1, 1, 2, 520, False), (384, 64, 4, 1, 8, 520, False),   # 64 channels: up to 256 pages ...
    (257, 64, 1, 1, 2, 512, True), (384, 64, 4, 1, 8, 64, True), (385, 64, 4, 1, 8, 64, False),     # ... to 384 where it scores the tokens too
    (320, 64, 8, 8, 2, 520, True), (321, 64, 8, 8, 2, 520, False), (384, 64, 8, 16, 2, 520, True),  # ... with 64, and with 128 workgroups
    (320, 64, 1, 1, 16, 520, False), (320, 64, 1, 1, 17, 520, True), (384, 64, 1, 4, 17, 520, False),
    (384, 64, 1, 5, 17, 520, True),                                                                 # ... with eight tiles of rows
    (512, 128, 8, 3, 13, 520, True), (512, 128, 8, 6, 13, 520, False), (288, 128, 8, 6, 13, 520, True), (512, 128, 8, 16, 8, 520, True),
    (513, 128, 8, 16, 8, 520, False)])
def test_which_prefixes_are_scored_and_selected_in_one_launch(P, d, Hkv, batch, n, hidden, one):
    r = OnePagePrefix(16 * P - 5, 32, 7, Hkv, d, 16, batch, hidden)
    count, K = torch.zeros((batch, Hkv), dtype=torch.int32, device="cuda"), P // 3
    try:
        assert one == scored_in_one_launch(r.ctx, lambda: L.losa_step(r.ctx, r.kv, 1, *r.h, r.q, orc.SEL_TOPK, float(n), K, r.o_p, r.lse_p,
                                                                      None, count))
        assert bool((count == K).all())                      # every page scores the same: the first ones
        mean = float((torch.arange(K) % 7).double().mean())
        o_p = r.o_p.reshape(batch, 32, -1)
        assert float((o_p[:, :n] - mean).abs().max()) <= 1e-2 and float(o_p[:, n:].abs().max()) == 0.0
    finally:
        r.ctx.close()


def test_a_step_whose_grids_are_shaped_scores_and_selects_in_two_launches():
    """Each switch that shapes or names one of the two launches brings them back, and its default the one launch."""
    r = OnePagePrefix(64 * 16, 32, 7, 4, 128, 16)
    try:
        one = lambda: scored_in_one_launch(r.ctx, lambda: L.losa_step(r.ctx, r.kv, 1, *r.h, r.q, orc.SEL_TOPK, 6.0, 9, r.o_p, r.lse_p))
        assert one()
        for knob, value, default in ((L.LOSA_TUNE_SELECT_ROUND, 100, 0), (L.LOSA_TUNE_SCORE_ROUND, 1, 1280), (L.LOSA_TUNE_SCORE_ROUND, 1 << 30, 1280),
                                     (L.LOSA_TUNE_RANK_IN_SCORES, 0, 1), (L.LOSA_TUNE_UNION_IN_ATTENTION, 0, 1)):
            L.losa_set_tuning(r.ctx, knob, value)
            assert not one(), (knob, value)
            L.losa_set_tuning(r.ctx, knob, default)
            assert one(), (knob, default)
    finally:
        r.ctx.close()
