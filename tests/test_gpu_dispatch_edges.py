"""Branches of the kernels' dispatch at the sizes where they can go wrong: the edges of their tiles, remainders, the
smallest and largest of their range, and what must not depend on the branch."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_11822_amd as rs
import rs_synth as S
from oracle import lm, moe
from tests.gpu_util import END_TO_END, TOL, Rig, check_cache_against_oracle, check_tensor, gather_prompt_kv, to_dev
from tests.test_gpu_hybrid import _hybrid_case
from tests.test_gpu_moe import _check_routing, _moe_rig

pytestmark = pytest.mark.gpu
f32 = S.bf16_bits_to_f32


# rows and columns around the tiles of the head's passes: the weight-streaming one (up to 64 rows, 256 columns a
# workgroup), the tiles of 128, 192 and 256 rows; every column count leaves a partly empty last tile
@pytest.mark.parametrize("shape,vocab,n", [(S.WIDE, 4228, 1), (S.WIDE, 4228, 64), (S.MID, 1028, 33), (S.MID, 1028, 65),
                                           (S.MID, 1284, 128), (S.MID, 2052, 129), (S.MID, 1028, 192), (S.MID, 2052, 193), (S.MID, 2052, 256),
                                           (S.MID, 1028, 300), (S.MID, 1028, 385)])
def test_head_logits_and_choice(shape, vocab, n):
    rig = Rig(shape, n_blocks=4, max_prefill_tokens=16, max_decode_batch=n, max_context=64, with_oracle=False)
    try:
        hb = S.head_weights(shape.d_model, vocab)
        lm_head = hb["lm_head"].copy()
        lm_head[7] = lm_head[vocab - 3] = lm_head[vocab // 2]     # equal logits in three places: the lowest column wins
        hb["lm_head"] = lm_head
        hd = {k: to_dev(v) for k, v in hb.items()}
        rig.ctx.set_head(hd["embed"], hd["final_norm"], hd["lm_head"], vocab, -1)
        x_bits = S.hidden_states(n, shape.d_model, 9)
        row = n - 1                                               # ... and are this row's largest
        x_bits[row] = S.f32_to_bf16_bits(40.0 * f32(lm_head[7]))
        x = to_dev(x_bits)
        logits = torch.full((n, vocab), float("nan"), dtype=torch.float32, device="cuda")
        out, out2 = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        rig.ctx.lm_head_greedy(rs.RS_SIDE_DECODE, x, n, logits, out)
        rig.ctx.lm_head_greedy(rs.RS_SIDE_DECODE, x, n, None, out2)
        rig.ctx.sync(rs.RS_SIDE_DECODE)
        got, tok = logits.cpu().numpy(), out.cpu().numpy()
        check_tensor("logits", got, lm.head_logits(f32(x_bits), hb["final_norm"], lm_head, shape.rms_eps))
        assert np.array_equal(tok, np.argmax(got, axis=1)) and tok[row] == 7
        assert torch.equal(out, out2)
    finally:
        rig.close()


# the weight-streaming pass at the edges of its 32-row tiles (one to four of them), its largest pass and the first one
# beyond; prompt rows, decode rows and both
@pytest.mark.parametrize("shape", [S.WIDE, S.TINY])
@pytest.mark.parametrize("lens,starts,ctx", [([31], [0], []), ([1, 32], [0, 0], []), ([64], [16], [7]), ([40, 25], [0, 32], []),
                                             ([5], [0], [0, 15, 16] + list(range(1, 93))), ([128], [0], []), ([100], [48], list(range(3, 31))),
                                             ([], [], list(range(0, 128))), ([129], [0], [])])
def test_streamed_pass(shape, lens, starts, ctx):
    orc_sent = np.float32(-777.0)
    B, T = len(ctx), sum(lens)
    held = [s + n for s, n in zip(starts, lens)] + [c + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 4
    tabs = S.shuffled_block_tables(held, n_blocks, stream=9)
    ptab, dtab = tabs[:len(lens)], tabs[len(lens):]
    rig = Rig(shape, n_blocks, max(T + B, sum(starts), sum(ctx), 1), max(B, 1), max(max(held), 2))
    try:
        L = rig.olayers[0]
        Kc, Vc = L.new_cache(n_blocks, fill=orc_sent)
        for tab, before, stream in ((ptab, starts, 60), (dtab, ctx, 61)):     # what is cached before the pass
            keep = [i for i, n in enumerate(before) if n > 0]
            for at in range(0, len(keep), rs.RS_MAX_PREFILL_REQS):
                part = keep[at:at + rs.RS_MAX_PREFILL_REQS]
                cu = np.concatenate([[0], np.cumsum([before[i] for i in part])]).astype(np.int32)
                xb = S.hidden_states(int(cu[-1]), shape.d_model, stream=stream + 10 * at)
                rig.prefill(xb, cu, tab[part])
                L.prefill(f32(xb), cu, tab[part], Kc, Vc)
        xb = S.hidden_states(T + B, shape.d_model, stream=62)
        x, cu = f32(xb), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        if not lens:
            y_bits = rig.decode(xb, np.asarray(ctx, np.int32), dtab)
        elif not B and not any(starts):
            y_bits = rig.prefill(xb, cu, ptab)
        else:
            y_bits = rig.hybrid(xb, cu, starts, ptab, np.asarray(ctx, np.int32) if B else None, dtab if B else None)
        if lens:
            check_tensor("prompt rows", f32(y_bits)[:T], L.prefill_chunk(x[:T], cu, starts, ptab, Kc, Vc), x[:T], 2, elem_mult=END_TO_END)
        if B:
            check_tensor("decode rows", f32(y_bits)[T:], L.decode(x[T:], np.asarray(ctx, np.int32), dtab, Kc, Vc), x[T:], 2, elem_mult=END_TO_END)
        check_cache_against_oracle(rig, Kc, Vc, orc_sent)
    finally:
        rig.close()


# the sparse block's tiles: with two experts every row goes to both, so an expert has exactly `n` rows: each height of
# tile (128 to 256 rows in steps of 32) at its edges, one tile an expert and several, four and more of two heights, up to 512 rows
# with streamed weights; 32 rows a router workgroup
@pytest.mark.parametrize("n", [1, 32, 33, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257, 384, 385, 512, 513, 577, 672, 768, 769, 833, 1025])
def test_sparse_block_tiles(n):
    rig, mw, L = _moe_rig(S.WIDE, 2, S.blocks_for(n) + 2, n, 1, n + 1)
    try:
        tabs = S.shuffled_block_tables([n], S.blocks_for(n) + 2, stream=23)
        xb, cu = S.hidden_states(n, S.WIDE.d_model, stream=23), np.array([0, n], np.int32)
        y_bits = rig.prefill(xb, cu, tabs)
        Kc, Vc = L.new_cache(S.blocks_for(n) + 2)
        x = f32(xb)
        _, x1_ref, _, _ = L.prefill(x, cu, tabs, Kc, Vc)
        sel, wt_got = rig.ctx.debug_read_moe_routing(rs.RS_SIDE_PREFILL, n)
        lg = moe.router_logits(oracle.rmsnorm(x1_ref, L.g2, S.WIDE.rms_eps), mw["router"]).astype(np.float64)
        wt = (1.0 / (1.0 + np.exp(lg[:, ::-1] - lg)))[np.arange(n)[:, None], sel]
        assert np.all(np.sort(sel, axis=1) == [0, 1]) and np.abs(wt_got - wt).max() <= TOL
        y_ref, _, _, _ = L.prefill(x, cu, tabs, Kc, Vc, sel=sel, wt=wt.astype(np.float32))
        check_tensor("y", f32(y_bits), y_ref, x, 2, elem_mult=END_TO_END)
    finally:
        rig.close()


# uneven experts: tiles of 128 and 160 rows beside those of the large ones, in a pass that streams the expert weights (up to 256
# rows times the experts) and in one that does not
@pytest.mark.parametrize("n", [1024, 1025, 1600])
def test_sparse_block_uneven_experts(n):
    shape, E, few = S.WIDE, 4, [150, 100]
    n_blocks = S.blocks_for(n) + 2
    rig, mw, L = _moe_rig(shape, E, n_blocks, n, 1, n + 1)
    try:
        two = np.tile([0, 1], (n, 1))
        for e, rows in zip((2, 3), few):                          # experts 2 and 3 get these many rows, the others the rest
            two[np.arange(rows) * 4 + e, 1] = e
        tabs, cu = S.shuffled_block_tables([n], n_blocks, stream=37), np.array([0, n], np.int32)
        xb = S.f32_to_bf16_bits(f32(S.hidden_states(n, shape.d_model, stream=37)) + 1.5 * f32(mw["router"])[two].sum(1))
        y_bits = rig.prefill(xb, cu, tabs)
        Kc, Vc = L.new_cache(n_blocks)
        x = f32(xb)
        _, x1_ref, _, _ = L.prefill(x, cu, tabs, Kc, Vc)
        sel, wt = _check_routing(rs.RS_SIDE_PREFILL, rig, L, mw, x1_ref, n)
        # a row in some hundreds leans elsewhere after attention: what counts is that the two experts have a tile of 5 and of 4 row blocks
        rows = np.bincount(sel.ravel(), minlength=E)[2:]
        assert 128 < rows[0] <= 160 and 96 < rows[1] <= 128
        y_ref, _, _, _ = L.prefill(x, cu, tabs, Kc, Vc, sel=sel, wt=wt)
        check_tensor("y", f32(y_bits), y_ref, x, 2, elem_mult=END_TO_END)
    finally:
        rig.close()


# a decode row of a sparse layer is the same bits alone and in a batch of up to 64: the output projection's K slices follow from the
# layer's widths (3584x3840, and 6144x6144, where what the workspace holds for a row leaves fewer of them), not from the rows
@pytest.mark.parametrize("shape", [S.LayerShape("slices-3584", 3584, 30, 10, 128, 1024), S.LayerShape("slices-6144", 6144, 48, 12, 128, 1024)])
def test_decode_rows_do_not_depend_on_their_batch(shape):
    ctx = np.array([(7 * i) % 40 for i in range(64)], np.int32)
    held = [int(c) + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=36)
    rig, mw, L = _moe_rig(shape, 2, n_blocks, 16, 64, 40)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        rig.load_pools_from_logical(S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2))
        xb = S.hidden_states(64, shape.d_model, stream=36)
        whole = rig.decode(xb, ctx, tabs, max_ctx=40)
        for n in (1, 8, 9, 61, 62):
            print(shape.name, n, flush=True)
            assert np.array_equal(rig.decode(xb[:n], ctx[:n], tabs[:n], max_ctx=40), whole[:n]), f"a batch of {n}"
    finally:
        rig.close()


# the same of a dense layer: one to four rows take kernels of their own, whose sums are the streams' (K slices in order, sums of squares
# by their parts), so a row's hidden state and its cache entries are the same bits alone and in a batch
@pytest.mark.parametrize("shape", [S.LLAMA8B, S.LayerShape("rows-2048", 2048, 32, 8, 64, 4608), S.LayerShape("rows-2560", 2560, 20, 4, 128, 10240),
                                   S.LayerShape("rows-3584", 3584, 28, 4, 128, 18944), S.WIDE])
def test_dense_decode_rows_do_not_depend_on_their_batch(shape):
    B = 40
    ctx = np.array([(37 * i) % 300 for i in range(B)], np.int32)
    held = [int(c) + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=41)
    rig = Rig(shape, n_blocks, 16, B, 300, with_oracle=False)
    try:
        kb, vb = S.kv_cache_bits(n_blocks, shape.n_kv_heads, shape.head_dim)
        xb = S.hidden_states(B, shape.d_model, stream=41)
        own = lambda bits, n: [bits[tabs[i, ctx[i] // 16], ctx[i] % 16] for i in range(n)]   # the rows' own tokens
        for split in ((256, 256), (128, 128), (96, 160), (64, 192)):
            rig.ctx.set_cu_split(*split)
            rig.load_pools_from_logical(kb, vb)
            whole = rig.decode(xb, ctx, tabs, max_ctx=300)
            kv = own(rig.k_bits_logical(), B), own(rig.v_bits_logical(), B)
            for n in (1, 2, 3, 4, 5, 33):
                print(shape.name, split, n, flush=True)
                rig.load_pools_from_logical(kb, vb)
                assert np.array_equal(rig.decode(xb[:n], ctx[:n], tabs[:n], max_ctx=300), whole[:n]), f"a batch of {n}"
                assert np.array_equal(own(rig.k_bits_logical(), n), kv[0][:n]) and np.array_equal(own(rig.v_bits_logical(), n), kv[1][:n]), f"a batch of {n}"
    finally:
        rig.close()


# prompt attention: single 128-query tiles and pairs of them, one and two teams over the key tiles, at odd and even numbers
# of 64-key tiles; own operands (the kernel's q and cache, the oracle's attention).  A gain of 8 makes the scores large
# (tens of powers of two): the maximum moves far from tile to tile.
@pytest.mark.parametrize("gain", [1.0, 8.0])
@pytest.mark.parametrize("shape,lens", [(S.TINY, [64]), (S.MID, [65]), (S.MID, [129]), (S.TINY, [700]), (S.MID, [300, 1, 200]),
                                        (S.MID, [4100]), (S.MID, [4224]), (S.MID, [130] * 63 + [257]), (S.TINY, [130] * 64), (S.ODD, [200])])
def test_prompt_attention_units(shape, lens, gain):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, n_blocks = int(cu[-1]), sum(S.blocks_for(n) for n in lens) + 2
    tabs = S.shuffled_block_tables(lens, n_blocks, stream=24)
    rig = Rig(shape, n_blocks, T, 1, max(lens) + 1, with_oracle=False)
    try:
        w = rig.wdev[0]
        g1 = w["g1"] * gain
        rig.ctx.set_weights(0, g1, w["wqkv"], w["wo"], w["g2"], w["wg"], w["wu"], w["wd"])
        rig.prefill(S.hidden_states(T, shape.d_model, stream=24), cu, tabs)
        read = lambda which, width: f32(rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, which, (T, width)))
        q, got = read(1, shape.qkv_dim)[:, :shape.q_dim].reshape(T, shape.n_q_heads, shape.head_dim), read(2, shape.q_dim)
        k, v = gather_prompt_kv(rig, cu, tabs)
        rows = np.unique(np.concatenate([cu[1:] - 1, cu[:-1], np.arange(min(T, 256)), np.arange(max(T - 140, 0), T)]))
        ref = oracle.attn_causal(q, k, v, cu, rows=rows).reshape(T, shape.q_dim)
        check_tensor("attention", got[rows], ref[rows])
    finally:
        rig.close()


# a hybrid batch whose decode rows have one and several chunks of keys, with an even and an odd number of kv heads (the one
# launch takes them two at a time), and with as many prompt rows as one team of waves would take alone
@pytest.mark.parametrize("shape,lens,starts,ctx", [(S.ODD, [70], [32], [600, 5, 511, 512]), (S.MID, [200], [48], [1, 1025]), (S.TINY, [90, 300], [0, 16], [0, 700])])
def test_hybrid_attention_in_one_launch(shape, lens, starts, ctx):
    _hybrid_case(shape, lens, starts, ctx)


# the one launch in workgroups of two teams and, where the bound of the contexts says that the decode rows are the longer part, of one:
# the same bits, and against the oracle; head_dim 64 and 128, several prompt tiles with earlier keys, an odd number of kv heads
@pytest.mark.parametrize("shape,lens,starts,B", [(S.MID, [90], [16], 40), (S.ODD, [200, 31], [0, 48], 50), (S.TINY, [140, 1], [32, 0], 50)])
def test_hybrid_attention_in_small_workgroups(shape, lens, starts, B):
    ctx, longest = np.array([(37 * i) % 300 for i in range(B)], np.int32), 2600
    held, T = [s + n for s, n in zip(starts, lens)] + [longest] * B, sum(lens)
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=39)
    rig = Rig(shape, n_blocks, T + B, B, longest)
    try:
        kb, vb = S.kv_cache_bits(n_blocks, shape.n_kv_heads, shape.head_dim)
        cu, xb, got = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), S.hidden_states(T + B, shape.d_model, stream=39), []
        for bound in (301, longest):
            rig.load_pools_from_logical(kb, vb)
            got.append(rig.hybrid(xb, cu, starts, tabs[:len(lens)], ctx, tabs[len(lens):], max_ctx=bound))
        assert np.array_equal(got[0], got[1])
        x, Kc, Vc = f32(xb), f32(kb), f32(vb)
        check_tensor("prompt rows", f32(got[0])[:T], rig.olayers[0].prefill_chunk(x[:T], cu, starts, tabs[:len(lens)], Kc, Vc), x[:T], 2, elem_mult=END_TO_END)
        check_tensor("decode rows", f32(got[0])[T:], rig.olayers[0].decode(x[T:], ctx, tabs[len(lens):], Kc, Vc), x[T:], 2, elem_mult=END_TO_END)
    finally:
        rig.close()


# the same where the decode rows have one chunk each, which their workgroups finish, on the whole chip and on partitions (their
# time is judged by the units): the same bits on every one, and as a batch of two decode rows, which take the large workgroups
def test_small_workgroups_finish_contexts_of_one_chunk():
    shape, B, T = S.MID, 60, 16
    ctx = np.array([(37 * i) % 300 for i in range(B)], np.int32)
    held = [T] + [int(c) + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=42)
    rig = Rig(shape, n_blocks, T + B, B, 301)
    try:
        kb, vb = S.kv_cache_bits(n_blocks, shape.n_kv_heads, shape.head_dim)
        xb, cu, got = S.hidden_states(T + B, shape.d_model, stream=42), np.array([0, T], np.int32), []
        for n, split in ((B, (256, 256)), (B, (128, 128)), (B, (64, 192)), (2, (256, 256))):
            rig.ctx.set_cu_split(*split)
            rig.load_pools_from_logical(kb, vb)
            rig.hybrid(xb[:T + n], cu, [0], tabs[:1], ctx[:n], tabs[1:1 + n], max_ctx=301)
            got.append(rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, 2, (T + n, shape.q_dim)))
        assert all(np.array_equal(g, got[0][:len(g)]) for g in got)
        rig.load_pools_from_logical(kb, vb)
        y, x, Kc, Vc = rig.hybrid(xb, cu, [0], tabs[:1], ctx, tabs[1:], max_ctx=301), f32(xb), f32(kb), f32(vb)
        check_tensor("prompt rows", f32(y)[:T], rig.olayers[0].prefill_chunk(x[:T], cu, [0], tabs[:1], Kc, Vc), x[:T], 2, elem_mult=END_TO_END)
        check_tensor("decode rows", f32(y)[T:], rig.olayers[0].decode(x[T:], ctx, tabs[1:], Kc, Vc), x[T:], 2, elem_mult=END_TO_END)
    finally:
        rig.close()


# the forms that prompt attention takes as the side's compute units become few: two teams of waves, one that does both
# teams' work one after the other, tiles and pairs of tiles, decode rows in the same launch and in one of their own; with
# one key tile a row, and with chunks that have earlier keys.  The same bits in all of them.
@pytest.mark.parametrize("shape,lens,starts,ctx", [(S.MID, [4100], [0], []), (S.MID, [4000], [0], []), (S.MID, [2200], [0], []), (S.MID, [64] * 24, [0] * 24, []), (S.MID, [1100, 65], [0, 0], []),
                                                   (S.TINY, [130] * 40, [0] * 40, []), (S.TINY, [130] * 30, [0] * 30, []), (S.MID, [4100], [0], [3, 600]), (S.MID, [1500], [272], [5, 700, 1030]), (S.ODD, [900, 40], [0, 64], [300]),
                                                   (S.TINY, [2000, 700], [16, 48], [40, 512])])
def test_prompt_attention_same_bits_on_every_partition(shape, lens, starts, ctx):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(cu[-1]), len(ctx)
    held = [s + n for s, n in zip(starts, lens)] + [c + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=26)
    rig = Rig(shape, n_blocks, T + B, max(B, 1), max(held) + 1, with_oracle=False)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        rig.load_pools_from_logical(S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2))
        xb = S.hidden_states(T + B, shape.d_model, stream=26)
        want = None
        for split in ((256, 256), (192, 64), (128, 128), (96, 160), (64, 192)):
            print("split", split, flush=True)
            rig.ctx.set_cu_split(*split)
            y = rig.hybrid(xb, cu, starts, tabs[:len(lens)], np.asarray(ctx, np.int32) if B else None, tabs[len(lens):] if B else None)
            got = (rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, 2, (T + B, shape.q_dim)), y)
            want = want or got
            for name, a, b in zip(("attention", "y"), got, want):
                assert np.array_equal(a, b), f"{name} differs at split {split}"
    finally:
        rig.close()


# the sums of a prompt's rows are cut into even and odd key tiles by the prompts alone, whether decode rows are beside them or
# not: few prompt workgroups, as many as one launch takes, more than that, and more than are cut at all
@pytest.mark.parametrize("lens", [[1100], [2100], [4000], [4100], [130] * 33])
def test_prompt_attention_same_bits_beside_decode_rows(lens):
    shape, ctx = S.MID, [3, 600]
    cu, starts = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), [0] * len(lens)
    T, held = int(cu[-1]), lens + [c + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=27)
    rig = Rig(shape, n_blocks, T + len(ctx), len(ctx), max(held) + 1, with_oracle=False)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        rig.load_pools_from_logical(S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2))
        xb = S.hidden_states(T + len(ctx), shape.d_model, stream=27)
        read = lambda: rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, 2, (T, shape.q_dim))
        rig.hybrid(xb[:T], cu, starts, tabs[:len(lens)])
        alone = read()
        rig.hybrid(xb, cu, starts, tabs[:len(lens)], np.asarray(ctx, np.int32), tabs[len(lens):])
        assert np.array_equal(read(), alone)
    finally:
        rig.close()


# merging the chunks of a context: a launch for few chunks and one for any number, the same bits for a context that both take
# (the bound of the batch's contexts chooses); empty, one-chunk, edge and longest contexts, odd numbers of heads, more than 64 chunks
@pytest.mark.parametrize("shape", [S.TINY, S.MID, S.ODD])
def test_decode_chunk_merge(shape):
    ctx = np.array([0, 1, 510, 511, 512, 1023, 1024, 1535, 1536, 2047, 700], np.int32)
    B, far = len(ctx), 34000
    n_blocks = int(sum(S.blocks_for(int(c) + 1) for c in ctx)) + S.blocks_for(far + 1) + 2
    tabs = S.shuffled_block_tables([int(c) + 1 for c in ctx] + [far + 1], n_blocks, stream=28)
    rig = Rig(shape, n_blocks, 16, B + 1, far + 1)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        kb, vb = S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2)
        xb = S.hidden_states(B + 1, shape.d_model, stream=28)
        read = lambda n: rig.ctx.debug_read_workspace(rs.RS_SIDE_DECODE, 2, (n, shape.q_dim))
        got = []
        for max_ctx in (512, 1024, 2048, 2560, 20000):
            rows = np.flatnonzero(ctx < max_ctx)
            rig.load_pools_from_logical(kb, vb)
            rig.decode(xb[:B], np.minimum(ctx, max_ctx - 1), tabs[:B], max_ctx=max_ctx)
            got.append((rows, read(B)))
        for rows, bits in got:
            assert np.array_equal(bits[rows], got[-1][1][rows])
        # and against the oracle's attention on the kernel's own operands, with a context of 67 chunks among them
        ctx2 = np.concatenate([ctx, [far]]).astype(np.int32)
        rig.load_pools_from_logical(kb, vb)
        rig.decode(xb, ctx2, tabs)
        q = f32(rig.ctx.debug_read_workspace(rs.RS_SIDE_DECODE, 1, (B + 1, shape.qkv_dim)))[:, :shape.q_dim].reshape(B + 1, shape.n_q_heads, shape.head_dim)
        K, V = f32(rig.k_bits_logical()), f32(rig.v_bits_logical())
        ref = oracle.attn_paged(q, K, V, tabs, ctx2 + 1).reshape(B + 1, shape.q_dim)
        check_tensor("attention", f32(read(B + 1)), ref)
    finally:
        rig.close()


# a decode row whose position is outside the rotary table is reported; what comes out for it, and for the rows beside it, is a
# function of the inputs and not of what the buffers held before
@pytest.mark.parametrize("B", [3, 100, 130])
def test_row_without_a_position_depends_on_its_inputs_alone(B):
    shape, longest = S.WIDE, 48
    ctx = (np.arange(B) % longest).astype(np.int32)
    ctx[1] = longest                                              # the first position past the table
    held = [longest + 1] * B
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=30)
    rig = Rig(shape, n_blocks, 16, B, longest, max_pos=longest, with_oracle=False)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        cl, tab = torch.from_numpy(ctx).cuda(), torch.from_numpy(np.ascontiguousarray(tabs, np.int32)).cuda()
        got = []
        for other in (31, 32):
            rig.decode(S.hidden_states(B, shape.d_model, stream=other), ctx % longest, tabs, max_ctx=longest)
            rig.load_pools_from_logical(S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2))
            x = to_dev(S.hidden_states(B, shape.d_model, stream=30))
            y = torch.empty_like(x)
            torch.cuda.synchronize()
            rig.ctx.decode_layer(0, x, y, cl, tab, tab.shape[1], B, longest)
            with pytest.raises(rs.RapidServeError) as e:
                rig.ctx.sync(rs.RS_SIDE_DECODE)
            assert e.value.code == rs.RS_ERR_BAD_BLOCK
            got.append(y.clone())
        assert torch.equal(got[0].view(torch.int16), got[1].view(torch.int16))
    finally:
        rig.close()


# the experts' tiles: of every height (rows an expert 1 to about 600), blocks of padding left out, and the down projection's 128
# columns wide where all of them run at once (256 CUs here) or 256 (32, and 64 from two units an expert).  The same bits in both;
# the first of them against the oracle under the library's routing.
@pytest.mark.parametrize("T,E", [(1, 8), (97, 8), (330, 4), (420, 4), (480, 4), (620, 8), (1000, 8), (760, 3)])
def test_expert_tiles_of_either_width(T, E):
    shape, n_blocks, ref = S.WIDE, S.blocks_for(T) + 2, None
    tabs, xb = S.shuffled_block_tables([T], n_blocks, stream=36), S.hidden_states(T, S.WIDE.d_model, stream=36)
    rig, mw, L = _moe_rig(shape, E, n_blocks, T, 1, T + 1)
    try:
        for split in ((256, 256), (32, 224), (64, 192)):
            print(T, E, split, flush=True)
            rig.ctx.set_cu_split(*split)
            y = rig.prefill(xb, [0, T], tabs)
            if ref is None:
                ref, x = y, f32(xb)
                _, x1, _, _ = L.prefill(x, np.array([0, T], np.int32), tabs, *L.new_cache(n_blocks))
                sel, wt = _check_routing(rs.RS_SIDE_PREFILL, rig, L, mw, x1, T)
                want, _, _, _ = L.prefill(x, np.array([0, T], np.int32), tabs, *L.new_cache(n_blocks), sel=sel, wt=wt)
                check_tensor("y", f32(y), want, x, 2, elem_mult=END_TO_END)
            assert np.array_equal(y, ref), f"differs at split {split}"
    finally:
        rig.close()


# units of up to 320 rows by eight waves: experts of 257 to 320 rows in one, of 513 to 640 in two, fuller ones beside them in two lower ones, a last round
# in halves; experts that have as many units either way (256 CUs, which these widths do not fill: four waves, 32 and 64: eight).  The same bits on every partition, checked as above.
@pytest.mark.parametrize("T,E", [(450, 3), (420, 3), (900, 3), (1000, 7), (470, 3), (500, 3)])
def test_tall_expert_tiles(T, E):
    test_expert_tiles_of_either_width(T, E)


# the experts' down projection by eight waves in tiles of 128 columns: experts of more than 256 rows beside others, at widths and on partitions where
# the tiles of either kind, shared out by themselves, would be one more on an XCD than it has compute units.  Another prompt goes before each
# pass, so that a tile that is not computed holds something else.  The first pass against the oracle's sparse block on the library's own operands: x1, and the
# routing with its weights, which the check of the routing allows 2e-2 of (where two experts' columns of four sigma each cancel, 0.4 % of a weight is more than
# the 2e-2 of a row's rms that an element is allowed).  On the same operands that is the bound, where a whole layer is allowed three times as much for its softmax.
@pytest.mark.parametrize("d,heads,T,E,cus", [(1280, (10, 2), 380, 3, 32), (1280, (10, 2), 400, 3, 32), (1536, (12, 4), 1000, 8, 96), (1536, (12, 4), 1060, 8, 96),
                                             (3584, (28, 4), 1040, 8, 224)])
def test_tall_expert_tiles_of_128_columns(d, heads, T, E, cus):
    shape, n_blocks, ref = S.LayerShape(f"experts-{d}", d, *heads, 128, 1024), S.blocks_for(T) + 2, None
    tabs, xb, other = S.shuffled_block_tables([T], n_blocks, stream=36), S.hidden_states(T, d, stream=36), S.hidden_states(T, d, stream=39)
    rig, mw, L = _moe_rig(shape, E, n_blocks, T, 1, T + 1)
    try:
        for split in ((cus, 256 - cus), (256, 256), (128, 128)):
            print(d, T, E, split, flush=True)
            rig.ctx.set_cu_split(*split)
            rig.prefill(other, [0, T], tabs)
            y = rig.prefill(xb, [0, T], tabs)
            if ref is None:
                ref, x1 = y, f32(rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, 3, (T, d)))
                _check_routing(rs.RS_SIDE_PREFILL, rig, L, mw, x1, T)
                sel, wt = rig.ctx.debug_read_moe_routing(rs.RS_SIDE_PREFILL, T)
                rows = np.bincount(sel.ravel(), minlength=E)
                assert 0 < (rows > 256).sum() < E and rows.max() <= 320, "experts of both kinds, in one unit each"
                check_tensor("y", f32(y), L._ffn(x1, sel, wt)[0], x1, 1)
            assert np.array_equal(y, ref), f"differs at split {split}"
    finally:
        rig.close()


# tiles of an odd number of 32-row blocks, whose waves do not all bring as many loads of a K tile: what a wave waits for is counted by the
# waves with fewer; 1536 rows: output and down projection with waves that only load.  Every pass gives the same bits (with one load too few waited
# for, one in some ten of these passes did not)
@pytest.mark.parametrize("T,split", [(576, (256, 256)), (300, (256, 256)), (1120, (128, 128)), (650, (96, 160)), (1536, (256, 256))])
def test_large_tile_products_repeat(T, split):
    n_blocks = S.blocks_for(T) + 2
    rig = Rig(S.LLAMA8B, n_blocks, T, 1, T + 1, with_oracle=False)
    try:
        rig.ctx.set_cu_split(*split)
        cu, tabs = np.array([0, T], np.int32), S.shuffled_block_tables([T], n_blocks, stream=37)
        x, tab = to_dev(S.hidden_states(T, S.LLAMA8B.d_model, stream=37)), torch.from_numpy(np.ascontiguousarray(tabs, np.int32)).cuda()
        y, first = torch.empty_like(x), None
        for i in range(60):
            torch.cuda.synchronize()
            rig.ctx.prefill_layer(0, x, y, cu, tab, tab.shape[1])
            rig.ctx.sync(rs.RS_SIDE_PREFILL)
            first = y.clone() if first is None else first
            assert torch.equal(y.view(torch.int16), first.view(torch.int16)), f"pass {i} differs"
    finally:
        rig.close()


# the same of the experts' eight-wave tiles, of 288 and of 320 rows: in the down projection 256 columns wide (32 CUs) and 128 (64 CUs)
@pytest.mark.parametrize("split", [(64, 192), (32, 224)])
def test_tall_expert_tiles_repeat(split):
    shape, T, E = S.WIDE, 1000, 7
    n_blocks = S.blocks_for(T) + 2
    rig, _, _ = _moe_rig(shape, E, n_blocks, T, 1, T + 1)
    try:
        rig.ctx.set_cu_split(*split)
        cu, tabs = np.array([0, T], np.int32), S.shuffled_block_tables([T], n_blocks, stream=36)
        x, tab = to_dev(S.hidden_states(T, shape.d_model, stream=36)), torch.from_numpy(np.ascontiguousarray(tabs, np.int32)).cuda()
        y, first = torch.empty_like(x), None
        for i in range(60):
            torch.cuda.synchronize()
            rig.ctx.prefill_layer(0, x, y, cu, tab, tab.shape[1])
            rig.ctx.sync(rs.RS_SIDE_PREFILL)
            first = y.clone() if first is None else first
            assert torch.equal(y.view(torch.int16), first.view(torch.int16)), f"pass {i} differs"
        rows = np.bincount(rig.ctx.debug_read_moe_routing(rs.RS_SIDE_PREFILL, T)[0].ravel(), minlength=E)
        assert ((rows > 256) & (rows <= 288)).any() and ((rows > 288) & (rows <= 320)).any(), rows
    finally:
        rig.close()


# passes of one to four rows, whose projections are finished in one kernel (five rows and the next kernels beside them): prompt rows,
# decode rows and both, head_dim 128 and 64, workgroups of one, two and four 16-column tiles; widths whose streams have too few K slices for
# that kernel.  The same bits on every partition.
@pytest.mark.parametrize("shape", [S.LLAMA8B, S.LayerShape("few-64", 1024, 16, 4, 64, 2560, 1e-5, 10000.0), S.LayerShape("few-64-2048", 2048, 32, 8, 64, 4608, 1e-5, 10000.0)])
@pytest.mark.parametrize("lens,starts,ctx", [([], [], [0]), ([], [], [15, 16]), ([], [], [700, 3, 31, 512]), ([], [], [5, 6, 7, 8, 300]), ([1], [32], []), ([3], [0], []),
                                             ([1, 2], [16, 0], [40])])
def test_passes_of_a_few_rows(shape, lens, starts, ctx):
    B, T, ctx = len(ctx), sum(lens), np.asarray(ctx, np.int32)
    held = [s + n for s, n in zip(starts, lens)] + [int(c) + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    cu, tabs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), S.shuffled_block_tables(held, n_blocks, stream=38)
    ptab, dtab = tabs[:len(lens)], tabs[len(lens):]
    rig = Rig(shape, n_blocks, T + B, max(B, 1), max(held) + 1)
    try:
        kb, vb = S.kv_cache_bits(n_blocks, shape.n_kv_heads, shape.head_dim)
        xb, want = S.hidden_states(T + B, shape.d_model, stream=38), None
        for split in ((256, 256), (128, 128), (64, 192), (192, 64), (96, 160)):
            print(shape.name, lens, B, split, flush=True)
            rig.ctx.set_cu_split(*split)
            rig.load_pools_from_logical(kb, vb)
            y = rig.hybrid(xb, cu, starts, ptab, ctx if B else None, dtab if B else None) if T else rig.decode(xb, ctx, dtab)
            got = [y] + [p.view(torch.int16).cpu().numpy() for p in (rig.k_pool, rig.v_pool)]
            want = got if want is None else want
            assert all(np.array_equal(p, q) for p, q in zip(got, want)), f"differs at split {split}"
        x, Kc, Vc = f32(xb), f32(kb), f32(vb)
        if T:
            check_tensor("prompt rows", f32(want[0])[:T], rig.olayers[0].prefill_chunk(x[:T], cu, starts, ptab, Kc, Vc), x[:T], 2, elem_mult=END_TO_END)
        if B:
            check_tensor("decode rows", f32(want[0])[T:], rig.olayers[0].decode(x[T:], ctx, dtab, Kc, Vc), x[T:], 2, elem_mult=END_TO_END)
    finally:
        rig.close()


# contexts of one chunk are finished by their workgroup where the bound says that all are, and by the merge where it does not: the same
# bits, a row without a context (refused, its attention zero) among them
@pytest.mark.parametrize("shape", [S.MID, S.TINY, S.ODD])
@pytest.mark.parametrize("ctx", [[0, 15, 300, 77, 511], [31, -1, 200]])
def test_decode_contexts_of_one_chunk(shape, ctx):
    B, ctx, longest = len(ctx), np.asarray(ctx, np.int32), 1100
    n_blocks = B * S.blocks_for(longest) + 2
    tabs = S.shuffled_block_tables([longest] * B, n_blocks, stream=40)
    rig = Rig(shape, n_blocks, 16, B, longest, with_oracle=False)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        cl, tab, got = torch.from_numpy(ctx).cuda(), torch.from_numpy(np.ascontiguousarray(tabs, np.int32)).cuda(), []
        for bound in (512, 513, longest):
            rig.load_pools_from_logical(S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2))
            x = to_dev(S.hidden_states(B, shape.d_model, stream=40))
            y = torch.empty_like(x)
            torch.cuda.synchronize()
            rig.ctx.decode_layer(0, x, y, cl, tab, tab.shape[1], B, bound)
            if (ctx < 0).any():
                with pytest.raises(rs.RapidServeError):
                    rig.ctx.sync(rs.RS_SIDE_DECODE)
            else:
                rig.ctx.sync(rs.RS_SIDE_DECODE)
            got.append((y.clone().view(torch.int16), rig.ctx.debug_read_workspace(rs.RS_SIDE_DECODE, 2, (B, shape.q_dim))))
            if (ctx < 0).any():
                assert not got[-1][1][ctx < 0].any() and got[-1][1][ctx >= 0].any()
        assert all(torch.equal(g[0], got[0][0]) and np.array_equal(g[1], got[0][1]) for g in got)
    finally:
        rig.close()


# the normalised rows can be read back where the pass made some, as the header says; a pass that folds its norms has none
@pytest.mark.parametrize("T,B", [(40, 0), (128, 0), (129, 0), (30, 20), (100, 60), (0, 1), (0, 128), (0, 129)])
def test_normalised_rows_where_there_are_some(T, B):
    shape, M = S.WIDE, T + B
    ctx = np.arange(B, dtype=np.int32)
    held = ([T] if T else []) + [int(c) + 1 for c in ctx]
    n_blocks = sum(S.blocks_for(n) for n in held) + 2
    tabs = S.shuffled_block_tables(held, n_blocks, stream=29)
    rig = Rig(shape, n_blocks, max(M, 1), max(B, 1), max(held) + 1, with_oracle=False)
    try:
        shp = (n_blocks, 16, shape.n_kv_heads, shape.head_dim)
        rig.load_pools_from_logical(S.normal_bf16(shp, S.SEED_CACHE, 1), S.normal_bf16(shp, S.SEED_CACHE, 2))
        xb, side = S.hidden_states(M, shape.d_model, stream=29), rs.RS_SIDE_PREFILL if T else rs.RS_SIDE_DECODE
        if not T:
            rig.decode(xb, ctx, tabs)
        elif not B:
            rig.prefill(xb, [0, T], tabs)
        else:
            rig.hybrid(xb, [0, T], [0], tabs[:1], ctx, tabs[1:])
        read = lambda which: rig.ctx.debug_read_workspace(side, which, (M, shape.d_model))
        if M <= 128:
            with pytest.raises(rs.RapidServeError) as e:
                read(0)
            assert e.value.code == rs.RS_ERR_STATE
        else:
            check_tensor("normalised rows", f32(read(0)), oracle.rmsnorm(f32(read(3)), f32(rig.wbits[0]["g2"]), shape.rms_eps))
    finally:
        rig.close()


# prompt attention rounds two things to bf16: the weights, relative to the row's maximum (the largest is exactly 1, those next to
# it sit where bf16 is finest), and the output.  Its error is no larger than that of a float64 evaluation with these two roundings
# (2 % for the sample; weights relative to a lagging maximum, anywhere in their binades, showed 5 to 6 % more)
@pytest.mark.parametrize("shape,T", [(S.TINY, 1500), (S.MID, 2048), (S.MID, 4300), (S.MID, 8300)])
def test_prompt_attention_error(shape, T):
    n_blocks = S.blocks_for(T) + 2
    tabs, cu = S.shuffled_block_tables([T], n_blocks, stream=33), np.array([0, T], np.int32)
    rig = Rig(shape, n_blocks, T, 1, T + 1, with_oracle=False)
    try:
        w, gain = rig.wdev[0], (4096 / shape.d_model) ** 0.5        # scores as spread as those of a 4096-wide layer
        rig.ctx.set_weights(0, w["g1"] * gain, w["wqkv"], w["wo"], w["g2"], w["wg"], w["wu"], w["wd"])
        rig.prefill(S.hidden_states(T, shape.d_model, stream=33), cu, tabs)
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda().double()
        read = lambda which, width: dev(f32(rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, which, (T, width))))
        q, got = read(1, shape.qkv_dim)[:, :shape.q_dim].reshape(T, shape.n_q_heads, shape.head_dim), read(2, shape.q_dim).reshape(T, shape.n_q_heads, shape.head_dim)
        k, v = (dev(t) for t in gather_prompt_kv(rig, cu, tabs))
        later = torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)
        err = ideal = 0.0
        for h in range(shape.n_q_heads):
            kv = h * shape.n_kv_heads // shape.n_q_heads
            s = (q[:, h] @ k[:, kv].t().contiguous() / shape.head_dim ** 0.5).masked_fill(later, float("-inf"))
            p = (s - s.max(1, keepdim=True).values).exp()
            total = p.sum(1, keepdim=True)
            exact = p @ v[:, kv].contiguous() / total
            rounded = (p.bfloat16().double() @ v[:, kv].contiguous() / total).bfloat16().double()
            err += float((got[:, h] - exact).square().sum())
            ideal += float((rounded - exact).square().sum())
        print(f"error {(err / ideal) ** 0.5:.4f} of the two roundings'", flush=True)
        assert err <= 1.02 ** 2 * ideal
    finally:
        rig.close()


# passes of the large layer shapes at row counts and partitions that take every form of their streams and epilogues: three and
# four row tiles with full-height and half-height workgroups, the gain folded in while the rows are staged or by a launch in front,
# and above 128 rows the K-sliced projections with the output projection's residual and norm in one (widths up to 4096 and
# above).  The same bits on every partition; sampled rows against the oracle.
@pytest.mark.parametrize("shape,passes", [(S.LLAMA8B, [([96], 0), ([70, 58], 0), ([], 65), ([], 128), ([60], 68), ([129], 0), ([100], 60)]),
                                          (S.LLAMA70B, [([33], 0), ([128], 0), ([], 101), ([150, 50], 0), ([300], 0)])])
def test_large_layer_passes_same_bits_on_every_partition(shape, passes):
    B_max, T_max = max(B for _, B in passes), max(sum(lens) for lens, _ in passes)
    ctx_all = np.array([(37 * i + 5) % 600 for i in range(max(B_max, 1))], np.int32)
    n_blocks = sum(S.blocks_for(int(c) + 1) for c in ctx_all) + T_max // 16 + 8
    rig = Rig(shape, n_blocks, max(T + B for T, B in ((sum(l), b) for l, b in passes)), max(B_max, 1), 608)
    try:
        L = rig.olayers[0]
        kb, vb = S.kv_cache_bits(n_blocks, shape.n_kv_heads, shape.head_dim)
        for lens, B in passes:
            T, ctx = sum(lens), ctx_all[:B]
            cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
            tabs = S.shuffled_block_tables(list(lens) + [int(c) + 1 for c in ctx], n_blocks, stream=34)
            ptab, dtab = tabs[:len(lens)], tabs[len(lens):]
            xb = S.hidden_states(T + B, shape.d_model, stream=34)
            want = None
            for split in ((256, 256), (128, 128), (160, 96), (64, 192), (192, 64)):
                print(shape.name, lens, B, split, flush=True)
                rig.ctx.set_cu_split(*split)
                rig.load_pools_from_logical(kb, vb)
                if not T:
                    y = rig.decode(xb, ctx, dtab)
                elif not B:
                    y = rig.prefill(xb, cu, ptab)
                else:
                    y = rig.hybrid(xb, cu, [0] * len(lens), ptab, ctx, dtab)
                want = y if want is None else want
                assert np.array_equal(y, want), f"y differs at split {split}"
            x, Kc, Vc = f32(xb), f32(kb), f32(vb)
            if T:
                rows = np.unique(np.array([0, T // 2, T - 1], np.int32))
                check_tensor("prompt rows", f32(want)[rows], L.prefill(x[:T], cu, ptab, Kc, Vc, rows=rows), x[rows], 2, elem_mult=END_TO_END)
            if B:
                rows = np.unique(np.array([0, B // 2, B - 1]))
                check_tensor("decode rows", f32(want)[T + rows], L.decode(x[T + rows], ctx[rows], dtab[rows], Kc, Vc), x[T + rows], 2, elem_mult=END_TO_END)
    finally:
        rig.close()


# the large-tile products at row counts that take every form of their schedule on some partition: tiles of 128 to 256 rows
# and of 192 columns, whole rounds with a last one of halves along either side, one to eight slices; the last row tile nearly
# empty (129, 193, 385, 577) and full (576).  Each product against float32 products of its own bf16 operands: an output is one
# rounding of a float32 sum (2^-8 of its value; 2^-7 for gate/up, whose reciprocal and exponential are approximate) and the
# order of up to 14336 terms (1e-4 of the outputs' size).  q and k are rotated: one rounding of the result and, where the product
# was stored first, one of each of the two terms.  The same bits on every partition.
@pytest.mark.parametrize("shape,rows", [(S.LLAMA8B, [129, 193, 300, 385, 576, 577, 900, 1025, 1300]), (S.LLAMA70B, [160, 170, 333, 545, 577, 1000, 1153]), (S.ODD, [150, 700])])
def test_large_tile_products(shape, rows):
    n_blocks = S.blocks_for(max(rows)) + 4
    rig = Rig(shape, n_blocks, max(rows), 1, max(rows) + 1, with_oracle=False)
    w = rig.wdev[0]
    try:
        for T in rows:
            cu, tabs = np.array([0, T], np.int32), S.shuffled_block_tables([T], n_blocks, stream=35)
            xb, first = S.hidden_states(T, shape.d_model, stream=35), None
            for split in ((256, 256), (128, 128), (64, 192), (96, 160)):
                print(shape.name, T, split, flush=True)
                rig.ctx.set_cu_split(*split)
                y = rig.prefill(xb, cu, tabs)
                widths = {0: shape.d_model, 1: shape.qkv_dim, 2: shape.q_dim, 3: shape.d_model, 4: shape.ffn_dim}
                got = {k: rig.ctx.debug_read_workspace(rs.RS_SIDE_PREFILL, k, (T, n)) for k, n in widths.items()}
                got[5] = y
                first = got if first is None else first
                assert all(np.array_equal(got[k], first[k]) for k in got), f"differs at split {split}"
            t = {k: to_dev(v).float() for k, v in first.items()}
            x = to_dev(xb).float()
            norm = (x * torch.rsqrt((x * x).mean(1, keepdim=True) + shape.rms_eps) * w["g1"].float()).bfloat16().float()
            v0 = shape.q_dim + (shape.qkv_dim - shape.q_dim) // 2
            act = t[0] @ w["wg"].float().t()
            act = act * torch.sigmoid(act) * (t[0] @ w["wu"].float().t())
            qkv = norm @ w["wqkv"].float().t()
            half, n_rot = shape.head_dim // 2, v0 // shape.head_dim
            phi = torch.arange(T, device="cuda").double()[:, None] * shape.rope_base ** (-torch.arange(half, device="cuda").double() / half)
            cos, sin = phi.cos().float()[:, None], phi.sin().float()[:, None]
            lo, hi = qkv[:, :v0].reshape(T, n_rot, 2, half).unbind(2)
            rot = torch.stack((lo * cos - hi * sin, hi * cos + lo * sin), 2).reshape(T, v0)
            terms = torch.stack(((lo * cos).abs() + (hi * sin).abs(), (hi * cos).abs() + (lo * sin).abs()), 2).reshape(T, v0)
            k = torch.from_numpy(gather_prompt_kv(rig, cu, tabs)[0]).cuda().reshape(T, -1)
            for name, g, ref, two in (("q", t[1][:, :shape.q_dim], rot[:, :shape.q_dim], terms[:, :shape.q_dim]), ("k", k, rot[:, shape.q_dim:], terms[:, shape.q_dim:])):
                # the operand is formed again here, as v's below: its slack, for the two terms
                slack = 2 * 2 * 25 * 2 ** -8 * ref.square().mean().sqrt() / shape.d_model ** 0.5
                worst = ((g - ref).abs() / (2 ** -8 * (ref.abs() + two) + slack)).max().item()
                print(f"  {name}: {worst:.3f} of the allowed error", flush=True)
                assert worst <= 1.0, name
            for name, g, ref, ulp in (("v", t[1][:, v0:], qkv[:, v0:], 2 ** -8), ("x1", t[3], x + t[2] @ w["wo"].float().t(), 2 ** -8),
                                      ("act", t[4], act, 2 ** -7), ("y", t[5], t[3] + t[4] @ w["wd"].float().t(), 2 ** -8)):
                size = ref.square().mean().sqrt()
                # v's operand is formed again here, and one element in some 10^4 is so near the middle of two bf16 that it rounds
                # the other way: 2^-8 of a term of size / sqrt(d), whose two factors reach five sigma each (25 terms); two of those
                slack = 1e-4 * size if name != "v" else 2 * 25 * 2 ** -8 * size / shape.d_model ** 0.5
                worst = ((g - ref).abs() / (ulp * ref.abs() + slack)).max().item()
                print(f"  {name}: {worst:.3f} of the allowed error", flush=True)
                assert worst <= 1.0, name
    finally:
        rig.close()


# tiles of 288 and 320 rows by eight waves, on some partition each: the last tile full, partly empty and of one row; as gate/up, in K slices, stored
# and with the residual; weights streamed and not; an odd number of K tiles.  (The host check of the dispatch rules holds the forms.)
@pytest.mark.parametrize("shape,rows", [(S.LLAMA8B, [288, 320, 640, 832, 1280, 1600, 1800]), (S.LLAMA70B, [290, 1100]), (S.ODD, [310, 640, 2593, 2881, 3169, 3521])])
def test_tall_products(shape, rows):
    test_large_tile_products(shape, rows)


# whole products in tiles of 128 x 256 whose loads four more waves issue: fewer K tiles (4, 5) than the ring has stages, an odd number of them (5, 33, 35)
# and many (448); stored and with the residual; weights streamed and not; the last row tile full and of one row
@pytest.mark.parametrize("shape,rows", [(S.LayerShape("one-head", 1024, 1, 1, 128, 1056), [128, 129, 500, 641, 897]), (S.LayerShape("odd-k", 1056, 8, 1, 128, 1120), [897, 1300, 1500]),
                                        (S.LayerShape("narrow", 160, 8, 1, 128, 1024), [128, 129, 400, 641]), (S.LLAMA8B, [1537])])
def test_fed_products(shape, rows):
    test_large_tile_products(shape, rows)
