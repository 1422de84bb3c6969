"""Prompts prefilled alone and with others in one packed pass.  fp32 results are
the same bits.  In bf16 the rows of a pass choose how its projections sum
(streaming or tiled, splits of the reduction), so a prompt's results can differ
by rounding from batch to batch, and by no more; the same batch repeats its
bits."""
import numpy as np
import pytest

import synth
from tests.gpu_util import make_session, row_err, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def one_hot(W, name, rng, scale):
    """One entry of +-scale per row: sums of one product, the same in any order."""
    x = np.zeros_like(W.values[name])
    flat = x.reshape(-1, x.shape[-1])
    n = flat.shape[0]
    # every column is taken before one is taken twice
    col = np.concatenate([rng.permutation(flat.shape[1]) for _ in range(-(-n // flat.shape[1]))])[:n]
    flat[np.arange(n), col] = scale * rng.choice([-1.0, 1.0], n)
    W.values[name], W.bits[name] = x, synth.bf16_bits(x)


def alone_and_packed(shape, W, prompts, caches=False):
    """Outputs of each prompt prefilled alone, and of all in one call (twice: the
    same bits); with caches also each prompt's keys and values, layer by layer."""
    from paper_2608_12385_amd import binding
    sess = make_session(shape, W, max_batch=len(prompts), max_pos=max(map(len, prompts)) + 1,
                        max_prompt=max(map(len, prompts)))
    wt, g, dh = torch.bfloat16 if shape.dtype == "bf16" else torch.float32, shape.n_kv_heads, shape.head_dim

    def call(batch):
        for b in range(len(prompts)):
            binding.dbt_kv_truncate(sess.kv, b, 0)
        r = {k: to_np(v).copy() for k, v in sess.prefill(batch).items()}
        for b, p in enumerate(batch if caches else []):
            pages = torch.tensor(binding.dbt_kv_pages(sess.kv, b), device="cuda")
            k = sess.k_pages.view(wt).view(shape.n_layers, -1, g, 16, dh)[:, pages].transpose(2, 3)
            v = sess.v_pages.view(wt).view(shape.n_layers, -1, g, dh, 16)[:, pages].permute(0, 1, 4, 2, 3)
            for n, x in (("k", k), ("v", v)):
                r.setdefault(n, []).append(to_np(x.reshape(shape.n_layers, -1, g, dh)[:, :len(p)].float()))
        return r

    alone = [call([p]) for p in prompts]
    packed, again = call(prompts), call(prompts)
    for k in packed:
        for x, y in zip(packed[k], again[k]):
            np.testing.assert_array_equal(x, y, err_msg=k)
    sess.close()
    return {k: [a[k][0] for a in alone] for k in packed}, packed


# projections whose sums hold one product each (no rounding depends on their
# order), so that the intermediate's SwiGLU is all that could differ between
# the kernels: fewer than 256 rows alone, more together; experts of few rows
# alone, of enough rows for tiles together
@pytest.mark.parametrize("moe", [False, True])
def test_swiglu_is_the_same_function_in_every_pass(moe):
    kw = dict(n_layers=1, n_q_heads=4, n_kv_heads=1, head_dim=128, vocab=448, dtype="bf16", has_embeddings=True,
              coupling_std=0.5)
    if moe:
        shape = synth.ModelShape(d_model=512, d_ff=0, n_experts=2, d_ff_expert=512, n_shared_experts=1, d_ff_shared=512,
                                 top_k1=2, top_k2=2, **kw)
        names, down = ["X_gate", "X_up", "S_gate", "S_up"], ["X_down", "S_down"]
    else:
        shape = synth.ModelShape(d_model=2048, d_ff=2048, **kw)
        names, down = ["W_gate", "W_up"], ["W_down"]
    W, rng = synth.make_weights(shape, seed=4), np.random.default_rng(5)
    for n in names:
        one_hot(W, "L0." + n, rng, 8.0 if n.endswith("gate") else 1.0)
    for n in down:
        one_hot(W, "L0." + n, rng, 1.0)
    W.values["L0.W_O"][:] = 0.0
    W.bits["L0.W_O"][:] = 0
    prompts = [synth.make_tokens(1, 500 + i, (5 + i % 9,), shape.vocab) for i in range(60)]
    alone, packed = alone_and_packed(shape, W, prompts)
    for key in ("h1_out", "h2_out"):
        assert np.isfinite(np.stack(alone[key])).all()
        np.testing.assert_array_equal(packed[key], np.stack(alone[key]), err_msg=key)


@pytest.mark.parametrize("d,dh,f,lens", [(64, 16, 96, [3, 40, 17, 130, 1]), (260, 20, 683, [70, 300, 64, 2])])
def test_f32_prompts_do_not_depend_on_their_companions(d, dh, f, lens):
    shape = synth.ModelShape(n_layers=2, d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=dh, d_ff=f, vocab=130,
                             dtype="f32", has_embeddings=True, std=0.1, coupling_std=0.5)
    prompts = [synth.make_tokens(1, 10 + i, (L,), shape.vocab) for i, L in enumerate(lens)]
    alone, packed = alone_and_packed(shape, synth.make_weights(shape), prompts, caches=True)
    for key in packed:
        for b in range(len(lens)):
            np.testing.assert_array_equal(packed[key][b], alone[key][b], err_msg=key)


# passes below 256 rows alone and together, below alone and above together,
# above both ways (one with tiled and one with streamed experts), a companion
# that is one row past a tile
@pytest.mark.parametrize("E,lens", [(0, [40, 100, 7]), (0, [200, 150, 7]), (0, [300, 257]), (0, [255, 1, 1, 700]),
                                    (8, [40, 100, 7]), (8, [300, 90])])
def test_bf16_prompts_differ_by_rounding_from_batch_to_batch(E, lens):
    d = 512
    moe = dict(n_experts=E, d_ff_expert=128, n_shared_experts=1, d_ff_shared=256, top_k1=2, top_k2=2) if E else {}
    shape = synth.ModelShape(n_layers=2, d_model=d, n_q_heads=4, n_kv_heads=1, head_dim=128, d_ff=0 if E else 2048,
                             vocab=448, dtype="bf16", has_embeddings=True, std=0.05, coupling_std=0.5, **moe)
    prompts = [synth.make_tokens(1, 10 + i, (L,), shape.vocab) for i, L in enumerate(lens)]
    alone, packed = alone_and_packed(shape, synth.make_weights(shape), prompts, caches=True)
    # first layer: the same bf16 inputs, fp32 sums of d products of size 0.05 in
    # another order (at most d 2^-24 times the sum of their sizes each way),
    # then one rounding to bf16 (neighbours are 2^-7 apart at most)
    add = 2 * d * 2.0 ** -24 * d * 0.05
    for key in ("k", "v"):
        for x, y in zip(packed[key], alone[key]):
            assert bool((np.abs(x[0] - y[0]) <= 2.0 ** -7 * np.abs(y[0]) + add).all()), key
    # everything behind it: the bar that both sides keep against the oracle
    for key in ("logits1", "logits2", "h1_out", "h2_out"):
        assert row_err(packed[key], np.stack(alone[key])).max() <= 2e-2, key
    for key in ("k", "v"):
        for x, y in zip(packed[key], alone[key]):
            assert row_err(x[1], y[1]).max() <= (1.0 if E else 2e-2), key  # (MoE: a row can route another way at a tie)
