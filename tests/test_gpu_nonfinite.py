"""Keys and values that are not finite, on the GPU: a NaN key reaches the
result of every row that sees it, however the pages are dealt to waves and
splits; a score of -inf is a probability of zero; rows before a position never
see it."""
import numpy as np
import pytest

import synth
from oracle import Oracle
from tests.gpu_util import fill_cache, make_session, row_err, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def layer_shape(dtype, nq, nkv, dh):
    return synth.ModelShape(n_layers=1, d_model=128, n_q_heads=nq, n_kv_heads=nkv, head_dim=dh, d_ff=128, vocab=0,
                            dtype=dtype, has_embeddings=False, std=0.1, coupling_std=0.5)


# one or two pages of NaN keys: the wave that reads them reads no other page
# (fp32: a page per wave and turn; bf16: a pair of pages), reads them after or
# before others, or in another split; half a pair; and (last) the workgroup of
# a whole sequence
@pytest.mark.parametrize("dtype,nkv,batch,length,bad", [
    ("f32", 2, 3, 100, [2]),
    ("f32", 2, 3, 300, [0]),
    ("f32", 2, 3, 300, [15]),
    ("f32", 2, 3, 1200, [70]),
    ("f32", 2, 3, 112, [6]),
    ("bf16", 2, 3, 100, [3]),
    ("bf16", 2, 3, 100, [2, 3]),
    ("bf16", 2, 3, 383, [8, 9]),
    ("bf16", 2, 3, 700, [30, 31]),
    ("bf16", 2, 3, 273, [17]),
    ("bf16", 64, 4, 200, [4, 5]),
])
def test_nan_keys_reach_the_result(dtype, nkv, batch, length, bad):
    shape = layer_shape(dtype, nkv, nkv, 128 if dtype == "bf16" else 32)
    sess = make_session(shape, synth.make_weights(shape), max_batch=batch, max_pos=length + 4)
    fill_cache(sess, None, shape, [length] * batch)
    wt = torch.bfloat16 if dtype == "bf16" else torch.float32
    h = synth.make_hidden(shape, batch)
    clean = {k: to_np(v).copy() for k, v in sess.decode(h1=h[0], h2=h[1]).items()}
    from paper_2608_12385_amd import binding
    for b in range(batch):
        binding.dbt_kv_truncate(sess.kv, b, length)
    pool = sess.k_pages.view(wt).view(1, -1, nkv, 16 * shape.head_dim)
    for page in bad:
        pool[0, binding.dbt_kv_pages(sess.kv, 1)[page]] = float("nan")
    got = {k: to_np(v) for k, v in sess.decode(h1=h[0], h2=h[1]).items()}
    for key in ("h1_out", "h2_out"):
        assert bool(np.isnan(got[key][1]).all()), key
        for b in range(batch):
            if b != 1:
                np.testing.assert_array_equal(got[key][b], clean[key][b], err_msg=key)
    sess.close()


# a page of keys with an infinite first dimension: scores of +inf (not a
# number after the softmax) or of -inf (no weight), as the sign of the query's
# first dimension says; head sizes that are and are not whole 16-dimension
# pieces, a wave that reads this page alone
@pytest.mark.parametrize("dtype,dh,length", [("f32", 12, 100), ("f32", 16, 100), ("f32", 20, 300), ("f32", 100, 70),
                                             ("bf16", 128, 150)])
def test_infinite_keys(dtype, dh, length):
    shape, B = layer_shape(dtype, 1, 1, dh), 12
    W = synth.make_weights(shape)
    sess, orc = make_session(shape, W, max_batch=B, max_pos=length + 4), Oracle(shape, W.values)
    wt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for b in range(B):
        (k, kb), (v, vb) = synth.make_kv(shape, 0, b, length)
        k = k.copy()
        k[32:64, 0, 0] = np.inf  # pages 2 and 3
        orc.kv_fill(b, length, [k], [v])
        sess.reserve_fill(b, [kb if kb is not None else k], [vb if vb is not None else v])
        from paper_2608_12385_amd import binding
        pages = binding.dbt_kv_pages(sess.kv, b)
        pool = sess.k_pages.view(wt).view(1, -1, 1, 16, dh)
        pool[0, pages[2], 0, :, 0] = pool[0, pages[3], 0, :, 0] = float("inf")
    h = synth.make_hidden(shape, B)
    with np.errstate(all="ignore"):
        outs = orc.decode_step(h1=h[0], h2=h[1])
    t = sess.decode(h1=h[0], h2=h[1])
    seen = set()
    for key, ref in (("h1_out", "h1"), ("h2_out", "h2")):
        want, got = np.stack([o[ref] for o in outs]), to_np(t[key])
        for b in range(B):
            finite = bool(np.isfinite(want[b]).all())
            seen.add(finite)
            if finite:
                assert row_err(got[b:b + 1], want[b:b + 1]).max() <= (2e-2 if dtype == "bf16" else 1e-5), (key, b)
            else:
                assert bool(np.isnan(want[b]).any()) and bool(np.isnan(got[b]).all()), (key, b)
    assert seen == {True, False}
    sess.close()


def test_prompt_rows_before_an_infinite_value():
    """fp32 prompt whose token at position 5 has infinite values in layer 0:
    the rows before it in the same page are those of the prompt without it."""
    dh, d, L = 32, 64, 40
    shape = synth.ModelShape(n_layers=2, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=dh, d_ff=96, vocab=32,
                             dtype="f32", has_embeddings=True, std=0.2, coupling_std=0.5)
    W = synth.make_weights(shape)
    mark = 31
    W.values["E1"][:, 0] = 0.0
    W.values["E1"][mark, 0] = 4.0
    W.values["L0.W_V"][:, 0] = 3e38  # times 4 / rms: infinite for the marked token, zero for every other
    prompt = np.arange(L, dtype=np.int32) % 30
    marked = prompt.copy()
    marked[5] = mark
    pages = []
    for p in (prompt, marked):
        sess = make_session(shape, W, max_batch=1, max_pos=L + 4, max_prompt=L)
        sess.prefill([p], run_boundary=False)
        from paper_2608_12385_amd import binding
        first = binding.dbt_kv_pages(sess.kv, 0)[0]
        k = sess.k_pages.view(torch.float32).view(2, -1, 16, dh)[1, first]
        v = sess.v_pages.view(torch.float32).view(2, -1, dh, 16)[1, first].t()
        pages.append((to_np(k).copy(), to_np(v).copy()))
        sess.close()
    for clean, got in zip(*pages):
        assert bool(np.isfinite(clean).all()) and not bool(np.isfinite(got[5:]).any())
        np.testing.assert_array_equal(got[:5], clean[:5])
