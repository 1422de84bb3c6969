"""Output arrays that share memory with each other or with an input that is
still read: what they hold after the call is what copies at its end leave, in
the order alpha and tokens, logits1, logits2, h1_out, h2_out."""
import numpy as np
import pytest

import synth
from tests.gpu_util import make_session, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ORDER = ("alpha", "next_token", "logits1", "logits2", "h1_out", "h2_out")


# word offsets of the outputs in one buffer: final states over logits, the
# readout's outputs inside logits, branch outputs over the primary's
@pytest.mark.parametrize("at", [
    dict(logits1=0, h1_out=64, logits2=4096, h2_out=8192),
    dict(logits1=0, logits2=2048, h2_out=2048 + 512, h1_out=12288),
    dict(logits1=16, alpha=20, next_token=400, logits2=4096, h1_out=8192, h2_out=9216),
    dict(logits1=0, logits2=1500, h1_out=8192, h2_out=8196),
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("grouped", [True, False])
def test_step_outputs_that_overlap(dtype, at, grouped):
    from paper_2608_12385_amd import binding
    B, d, V = 3, 256, 512
    shape = synth.ModelShape(n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=256, vocab=V,
                             dtype=dtype, has_embeddings=False, std=0.05, coupling_std=0.5)
    sess = make_session(shape, synth.make_weights(shape), max_batch=B, max_pos=40)
    for b in range(B):
        sess.reserve_fill(b, *[[x[1] if x[1] is not None else x[0] for x in kv] for kv in
                               zip(*[synth.make_kv(shape, l, b, 20 + b) for l in range(2)])])
    h = torch.from_numpy(np.ascontiguousarray(synth.make_hidden(shape, B))).cuda()
    words = dict(alpha=B, next_token=B, logits1=B * V, logits2=B * V, h1_out=B * d, h2_out=B * d)

    def step(ptr):
        out, sin = binding.dbt_step_out(**ptr), sess.step_in(B, None, h[0], h[1])
        if grouped:
            binding.dbt_decode_step(sess.model, sess.kv, sin, 1, out, sess.stream)
        else:
            binding.dbt_decode_step_ungrouped(sess.model, sess.kv, sin, out, sess.stream)
        torch.cuda.synchronize()
        for b in range(B):
            binding.dbt_kv_truncate(sess.kv, b, 20 + b)

    buf = torch.full((16384,), 7, dtype=torch.int32, device="cuda")
    apart = {n: torch.zeros(s, dtype=torch.int32, device="cuda") for n, s in words.items()}
    step({n: t.data_ptr() for n, t in apart.items()})
    want = buf.clone()
    for n in ORDER:
        if n in at:
            want[at[n]:at[n] + words[n]] = apart[n]
    step({n: buf.data_ptr() + 4 * o for n, o in at.items()})
    assert torch.equal(buf, want)
    sess.close()


def test_prefill_states_over_the_tokens():
    """Final states over tokens that later passes still read: nine prompts
    take two passes of 8192 rows."""
    from paper_2608_12385_amd import binding
    shape = synth.ModelShape(n_layers=1, d_model=32, n_q_heads=2, n_kv_heads=1, head_dim=16, d_ff=40, vocab=64,
                             dtype="f32", has_embeddings=True, std=0.2, coupling_std=0.5)
    lens = [1000 + i for i in range(9)]
    prompts = [synth.make_tokens(1, 10 + i, (L,), shape.vocab) for i, L in enumerate(lens)]
    sess = make_session(shape, synth.make_weights(shape), max_batch=9, max_pos=1010, max_prompt=1008)
    want = {k: to_np(v).copy() for k, v in sess.prefill(prompts).items()}
    for b in range(9):
        binding.dbt_kv_truncate(sess.kv, b, 0)
    tok = torch.from_numpy(np.concatenate(prompts).astype(np.int32)).cuda()
    out, t = sess.outputs(9)
    first = (sum(lens) - 9 * 32) // 4 * 4
    out.h1_out = tok.data_ptr() + 4 * first
    binding.dbt_prefill(sess.model, sess.kv, tok.data_ptr(), lens, 9, 1, out, sess.stream)
    torch.cuda.synchronize()
    got = {k: to_np(v) for k, v in t.items()}
    got["h1_out"] = to_np(tok[first:first + 9 * 32].view(torch.float32)).reshape(9, 32)
    for k, v in want.items():
        np.testing.assert_array_equal(got[k], v, err_msg=k)
    sess.close()
