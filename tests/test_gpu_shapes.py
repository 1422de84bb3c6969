"""GPU parity at the sizes where the kernels' tiles, splits and dispatch
rules have edges: small models against the float64 oracle."""
import numpy as np
import pytest

import synth
from oracle import Oracle
from tests.gpu_util import TILED_CASES, check_readout, fill_cache, make_session, row_err, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2
F32_TOL = 1e-5    # fp32 bar of the parity tests (a 1024-term fp32 sum: ~32 x 6e-8 typical)


def prompts_and_steps(shape, lens, tol, steps=2):
    """Prompts, the boundary and a few greedy steps on the oracle's tokens."""
    W = synth.make_weights(shape, seed=0)
    prompts = [synth.make_tokens(1, 10 + i, (L,), shape.vocab) for i, L in enumerate(lens)]
    orc = Oracle(shape, W.values)
    obs = orc.prefill(prompts, run_boundary=True)
    sess = make_session(shape, W, max_batch=len(lens), max_pos=max(lens) + steps + 1, max_prompt=max(lens))
    sess.k_pages.fill_(0xFF)  # slots no position has written hold NaN
    sess.v_pages.fill_(0xFF)
    t = sess.prefill(prompts, run_boundary=True)
    check_readout(t, obs, tol, "boundary")
    toks = [o["next"] for o in obs]
    for step in range(steps):
        outs = orc.decode_step(tokens=toks)
        t = sess.decode(tokens=toks)
        check_readout(t, outs, tol, f"step {step}")
        for key, ref in (("h1_out", "h1"), ("h2_out", "h2")):
            assert row_err(to_np(t[key]), np.stack([o[ref] for o in outs])).max() <= tol, (step, key)
        toks = [o["next"] for o in outs]
    sess.close()


# widths around the fp32 projection's 32-element units and eight waves (a
# lone partial unit, one unit, a partial ninth), 16-column tiles with odd
# segment ends, and row blocks of 16, 32 and 64
@pytest.mark.parametrize("d,dh,f,vocab,lens", [
    (20, 4, 7, 17, [3]),
    (32, 8, 33, 31, [1, 17]),
    (260, 64, 95, 130, [33, 5, 16]),
    (288, 32, 1025, 4100, [65, 64]),
])
def test_f32_projection_edges(d, dh, f, vocab, lens):
    shape = synth.ModelShape(n_layers=2, d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=dh, d_ff=f, vocab=vocab,
                             dtype="f32", has_embeddings=True, std=0.1, coupling_std=0.5)
    prompts_and_steps(shape, lens, F32_TOL)


# head sizes that are and are not whole 16-dimension pieces, groups of one to
# four query heads, prompt tiles and pages around 16, more pages than waves
# (8 x 16 positions), and caches on both sides of one 64-page split in a batch
@pytest.mark.parametrize("dh,nq,nkv,lens", [
    (4, 3, 3, [1, 15, 16, 17]),
    (12, 6, 2, [2, 31]),
    (128, 4, 4, [129, 130]),
    (100, 8, 2, [127]),
    (16, 2, 1, [1022, 1040, 7]),
])
def test_f32_attention_edges(dh, nq, nkv, lens):
    shape = synth.ModelShape(n_layers=1, d_model=64, n_q_heads=nq, n_kv_heads=nkv, head_dim=dh, d_ff=96, vocab=64,
                             dtype="f32", has_embeddings=True, std=0.2, coupling_std=0.5)
    prompts_and_steps(shape, lens, F32_TOL, steps=4)


# fills that start and end inside pages, one position, whole pages, sources on
# and off 16-byte boundaries: every filled slot is the source's bits, every
# other slot keeps what it held
@pytest.mark.parametrize("dtype,dh,nkv,start,count,off", [
    ("bf16", 128, 2, 0, 48, 0),
    ("bf16", 128, 2, 5, 1, 0),
    ("bf16", 128, 1, 13, 40, 0),
    ("bf16", 128, 2, 3, 61, 1),
    ("f32", 64, 3, 16, 35, 0),
    ("f32", 12, 2, 1, 30, 0),
    ("f32", 12, 2, 1, 30, 1),
])
def test_kv_fill_edges(dtype, dh, nkv, start, count, off):
    from paper_2608_12385_amd import binding
    shape = synth.ModelShape(n_layers=2, d_model=128, n_q_heads=nkv, n_kv_heads=nkv, head_dim=dh, d_ff=128, vocab=0,
                             dtype=dtype, has_embeddings=False)
    sess = make_session(shape, synth.make_weights(shape), max_batch=2, max_pos=80)
    wt = torch.int16 if dtype == "bf16" else torch.int32
    binding.dbt_kv_reserve(sess.kv, 0, 17)
    pages = binding.dbt_kv_reserve(sess.kv, 1, 64)
    g = torch.Generator().manual_seed(1)
    src = [torch.randint(-30000, 30000, (off + count * nkv * dh,), generator=g).to(wt).cuda() for _ in range(2)]
    sess.k_pages.fill_(0x55)
    sess.v_pages.fill_(0x55)
    want = []
    for pool, s, kdim in ((sess.k_pages, src[0], True), (sess.v_pages, src[1], False)):
        w = pool.view(wt).view(2, -1, nkv, 16 * dh).clone()
        rows = s[off:].view(count, nkv, dh)
        for i in range(count):
            pos = start + i
            blk = w[1, pages[pos // 16]]
            (blk.view(nkv, 16, dh)[:, pos % 16] if kdim else blk.view(nkv, dh, 16)[:, :, pos % 16]).copy_(rows[i])
        want.append(w)
    binding.dbt_kv_fill(sess.kv, 1, 1, start, count, src[0][off:].data_ptr(), src[1][off:].data_ptr(), sess.stream)
    torch.cuda.synchronize()
    for pool, w in ((sess.k_pages, want[0]), (sess.v_pages, want[1])):
        assert torch.equal(pool.view(wt).view(w.shape), w)
    sess.close()


# packed prompt passes in bf16 on both sides of one and two 128-row blocks of
# the streaming projections and of the tiled ones' 256 rows, prompts shorter
# than a page, longer than an attention tile, tiles of unequal prompts
@pytest.mark.parametrize("lens", [[1], [100, 27], [100, 1, 28], [200, 54, 1], [200, 55, 1], [3, 300, 16, 65, 129]])
def test_bf16_packed_prompts(lens):
    shape = synth.ModelShape(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=1, head_dim=128, d_ff=384, vocab=512,
                             dtype="bf16", has_embeddings=True, std=0.05, coupling_std=0.5)
    prompts_and_steps(shape, lens, BF16_TOL)


# widths at both ends of the fused gate/up kernel's narrow tiles (128 to 256 of
# them, up to 64 stacked rows) and of its wide ones, prompts of 1 to 65 rows,
# steps of 32 and 64 stacked rows, and of 96 (the narrow tiles' limit passed)
@pytest.mark.parametrize("f", [4096, 8192, 12288])
@pytest.mark.parametrize("lens", [[1], [5, 40], [63], [32, 32], [65], [1 + i % 3 for i in range(17)], [1] * 33])
def test_bf16_fused_gate_up_edges(f, lens):
    shape = synth.ModelShape(n_layers=1, d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=f, vocab=448,
                             dtype="bf16", has_embeddings=True, std=0.05, coupling_std=0.5)
    prompts_and_steps(shape, lens, BF16_TOL, steps=1)


# more sequences than one pass takes (128), and more rows (8192)
@pytest.mark.parametrize("lens", [[1 + i % 3 for i in range(131)], [900 + 31 * i for i in range(9)]])
def test_f32_several_prompt_passes(lens):
    shape = synth.ModelShape(n_layers=1, d_model=32, n_q_heads=2, n_kv_heads=1, head_dim=16, d_ff=40, vocab=64,
                             dtype="f32", has_embeddings=True, std=0.2, coupling_std=0.5)
    prompts_and_steps(shape, lens, F32_TOL, steps=1)


# outputs in place and through the workspace (arrays off 16-byte boundaries,
# overlapping, absent) hold the same bits, and nothing past them is written
@pytest.mark.parametrize("dtype,vocab", [("bf16", 448), ("bf16", 65536 + 64), ("f32", 33)])
@pytest.mark.parametrize("grouped", [True, False])
def test_step_outputs_in_place_and_copied(dtype, vocab, grouped):
    from paper_2608_12385_amd import binding
    nb, B, d = 2, 3, 256
    shape = synth.ModelShape(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=256, vocab=vocab,
                             dtype=dtype, has_embeddings=False, n_branches=nb, std=0.05, coupling_std=0.5)
    sess = make_session(shape, synth.make_weights(shape), max_batch=5, max_pos=40)
    for b in range(B):
        sess.reserve_fill(b, *[[x[1] if x[1] is not None else x[0]] for x in synth.make_kv(shape, 0, b, 20 + b)])
    h = torch.from_numpy(np.ascontiguousarray(synth.make_hidden(shape, B, paths=1 + nb))).cuda()
    sizes = dict(logits1=B * vocab, logits2=nb * B * vocab, h1_out=B * d, h2_out=nb * B * d, alpha=B)

    def step(off, skip=(), inplace=False):
        buf = {n: torch.full((s + 64,), 7.0, device="cuda") for n, s in sizes.items() if n not in skip}
        ptr = {n: t.data_ptr() + 4 * off for n, t in buf.items()}
        h1, h2 = h[0].clone(), h[1:].clone()
        if inplace:
            ptr["h1_out"], ptr["h2_out"] = h1.data_ptr(), h2.data_ptr()
        tok = torch.zeros(B, dtype=torch.int32, device="cuda")
        out = binding.dbt_step_out(next_token=tok.data_ptr(), **ptr)
        sin = sess.step_in(B, None, h1, h2)
        if grouped:
            binding.dbt_decode_step(sess.model, sess.kv, sin, 1, out, sess.stream)
        else:
            binding.dbt_decode_step_ungrouped(sess.model, sess.kv, sin, out, sess.stream)
        torch.cuda.synchronize()
        for b in range(B):
            binding.dbt_kv_truncate(sess.kv, b, 20 + b)
        got = {n: t[off:off + sizes[n]].clone() for n, t in buf.items()}
        for n, t in buf.items():
            if not (inplace and n in ("h1_out", "h2_out")):
                assert (t[:off] == 7.0).all() and (t[off + sizes[n]:] == 7.0).all(), n
        if inplace:
            got["h1_out"], got["h2_out"] = h1.flatten(), h2.flatten()
        got["next"] = tok
        return got

    want = step(0)
    for other in (step(1), step(4), step(0, skip=("logits2", "h1_out")), step(3, skip=("logits1", "logits2")),
                  step(0, inplace=True)):
        for n, t in other.items():
            assert torch.equal(t, want[n]), n
    sess.close()


@pytest.mark.parametrize("d,nq,nkv,f,lens", TILED_CASES)
def test_bf16_tiled_projections(d, nq, nkv, f, lens):
    shape = synth.ModelShape(n_layers=1, d_model=d, n_q_heads=nq, n_kv_heads=nkv, head_dim=128, d_ff=f, vocab=512,
                             dtype="bf16", has_embeddings=True, std=0.03, coupling_std=0.5)
    prompts_and_steps(shape, lens, BF16_TOL, steps=1)


# caches on both sides of the shortest split (24 pages, 384 positions): the
# boundary of the longest prompt launches a merge with nothing to merge, the
# steps cross into a second split
def test_bf16_attention_around_the_shortest_split():
    shape = synth.ModelShape(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=1, head_dim=128, d_ff=384, vocab=512,
                             dtype="bf16", has_embeddings=True, std=0.05, coupling_std=0.5)
    prompts_and_steps(shape, [384, 383, 17], BF16_TOL, steps=3)


# a model made for more and longer sequences than the call has: splits of 24,
# 86 (batch x KV heads >= 256) and 128 pages of an 8192-position window, caches
# of one position to several splits
@pytest.mark.parametrize("max_batch,nkv", [(4, 2), (64, 4), (8, 8)])
def test_bf16_short_caches_of_a_large_model(max_batch, nkv):
    shape = synth.ModelShape(n_layers=1, d_model=256, n_q_heads=nkv, n_kv_heads=nkv, head_dim=128, d_ff=256, vocab=0,
                             dtype="bf16", has_embeddings=False, std=0.05, coupling_std=0.5)
    W, lens = synth.make_weights(shape), [1, 383, 2049, 130]
    sess, orc = make_session(shape, W, max_batch=max_batch, max_pos=8192, num_pages=200), Oracle(shape, W.values)
    sess.k_pages.fill_(0xFF)
    sess.v_pages.fill_(0xFF)
    fill_cache(sess, orc, shape, lens)
    for step in range(2):
        h = synth.make_hidden(shape, len(lens), step=step)
        outs, t = orc.decode_step(h1=h[0], h2=h[1]), sess.decode(h1=h[0], h2=h[1])
        for key, ref in (("h1_out", "h1"), ("h2_out", "h2")):
            assert row_err(to_np(t[key]), np.stack([o[ref] for o in outs])).max() <= BF16_TOL, (step, key)
    sess.close()


# expert counts around the router's 16-expert blocks and 64-lane rows, batches
# around its 8- and 16-row workgroups, fan-outs up to all experts; prompts whose
# experts take streamed passes, one tile and several tiles of rows
@pytest.mark.parametrize("E,k1,k2,replay,lens", [
    (1, 1, 1, False, [5]),
    (17, 2, 8, False, [1] * 9),
    (64, 2, 2, True, [3] * 17),
    (100, 8, 3, False, [2, 7]),
    (256, 4, 4, True, [6]),
    (8, 2, 2, False, [90, 33]),
    (3, 2, 1, False, [300, 111]),
])
def test_moe_router_and_expert_tiles(E, k1, k2, replay, lens):
    shape = synth.ModelShape(n_layers=1, d_model=512, n_q_heads=4, n_kv_heads=1, head_dim=128, d_ff=0, vocab=448,
                             dtype="bf16", has_embeddings=True, n_experts=E, d_ff_expert=128, n_shared_experts=1,
                             d_ff_shared=256, top_k1=k1, top_k2=k2, replay=replay, std=0.05, coupling_std=0.5)
    prompts_and_steps(shape, lens, BF16_TOL, steps=1)


# routers of more than 128 experts: groups of 64 experts (one of a single
# expert, a partial one, four whole), the selection as a kernel of its own;
# steps, prompts and the boundary, fan-outs up to eight, a replayed branch.
# (Fan-outs at which the oracle's last chosen logit leads the next one by at
# least 0.2 % of the largest, about what the rounding of the states to bf16
# moves it by: with k2 = 8, 129 experts leave a lead of 0.02 % in one row.)
@pytest.mark.parametrize("E,k1,k2,replay,lens", [
    (129, 3, 4, False, [1] * 9),
    (200, 8, 3, False, [2, 40]),
    (256, 3, 3, True, [3] * 17),
])
def test_moe_router_groups(E, k1, k2, replay, lens):
    test_moe_router_and_expert_tiles(E, k1, k2, replay, lens)
