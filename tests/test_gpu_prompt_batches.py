"""Prompts prefilled alone and with others in one packed pass: which kernels run
a pass (streaming or tiled projections, streamed or tiled experts) follows from
its rows, and what they compute per element does not."""
import numpy as np
import pytest

import synth
from tests.gpu_util import make_session, to_np

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


def alone_and_packed(shape, W, prompts):
    """Outputs of each prompt prefilled alone, and of all in one call."""
    sess = make_session(shape, W, max_batch=len(prompts), max_pos=max(map(len, prompts)) + 1,
                        max_prompt=max(map(len, prompts)))
    from paper_2608_12385_amd import binding
    alone = []
    for p in prompts:
        alone.append({k: to_np(v).copy() for k, v in sess.prefill([p]).items()})
        binding.dbt_kv_truncate(sess.kv, 0, 0)
    packed = {k: to_np(v) for k, v in sess.prefill(prompts).items()}
    sess.close()
    return {k: np.concatenate([a[k] for a in alone]) for k in packed}, packed


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
        assert np.isfinite(alone[key]).all()
        np.testing.assert_array_equal(packed[key], alone[key], err_msg=key)
