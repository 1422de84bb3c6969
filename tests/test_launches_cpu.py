"""The library's launches, on the CPU: it runs in a child process on a stand-in
for the HIP runtime (fake_hip.c) that names and counts launches and fails the
one it is told to.  What a failing call leaves behind must not be used, and a
prompt's length alone chooses its attention kernel."""
import ctypes
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "fake_hip.c")],
                   check=True)
    return so


def run_child(fake, name):
    pre = " ".join(x for x in (fake, os.environ.get("LD_PRELOAD", "")) if x)
    r = subprocess.run([sys.executable, __file__, name, fake], capture_output=True, text=True, cwd=ROOT, timeout=300,
                       env=dict(os.environ, LD_PRELOAD=pre, PYTHONPATH=ROOT))
    assert r.returncode == 0 and "done" in r.stdout, (r.stdout + r.stderr)[-3000:]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_no_boundary_after_a_failed_prefill(fake, dtype):
    run_child(fake, "boundary_" + dtype)


def test_page_table_after_failed_launches(fake):
    run_child(fake, "pages")


def test_prompt_attention_by_the_prompts_own_length(fake):
    run_child(fake, "attention")


def test_large_routers_are_read_by_several_workgroups(fake):
    run_child(fake, "router")


def test_workspace_holds_every_pass_and_nothing_else(fake):
    run_child(fake, "workspace")


def test_tiled_projection_cases_reach_every_form(fake):
    run_child(fake, "tiles")


@pytest.mark.parametrize("form", ["tokens", "states"])
def test_steps_after_failed_launches(fake, form):
    run_child(fake, "steps_" + form)


# ---------------------------------------------------------------------------
# in the child
# ---------------------------------------------------------------------------

FAKE = 1 << 40  # placeholder device address, never dereferenced


class Program:
    def __init__(self, dtype="f32", max_batch=4, **kw):
        from paper_2608_12385_amd import binding as B
        self.B = B
        size = dict(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=256, vocab=512)
        if dtype == "f32":
            size = dict(d_model=48, n_q_heads=4, n_kv_heads=2, head_dim=16, d_ff=96, vocab=64)
        cfg = B.dbt_config(dtype=B.DBT_BF16 if dtype == "bf16" else B.DBT_F32, max_batch=max_batch, rms_eps=1e-5,
                           rope_theta=1e4,
                           **dict(dict(size, n_layers=2, has_embeddings=1, max_pos=256, max_prompt=64), **kw))
        self.layers = (B.dbt_layer_weights * cfg.n_layers)()
        for l in range(cfg.n_layers):
            for f, _ in B.dbt_layer_weights._fields_:
                setattr(self.layers[l], f, FAKE)
        self.bytes = B.dbt_workspace_bytes(cfg)
        w = B.dbt_weights(emb1=FAKE, emb2=FAKE, emb_norm=FAKE, final_norm=FAKE, lm_head=FAKE, h_layers=self.layers)
        self.model = B.dbt_create(cfg, w, FAKE)
        self.out = B.dbt_step_out(logits1=FAKE, logits2=FAKE, alpha=FAKE, next_token=FAKE, h1_out=FAKE, h2_out=FAKE)
        self.mpps = (cfg.max_pos + 15) // 16

    def cache(self, pages=64, nseq=4):
        """A cache and its page table (host memory: the stand-in writes it)."""
        table = (ctypes.c_int * (nseq * self.mpps))(*([-1] * (nseq * self.mpps)))
        return self.B.dbt_kv_create(self.model, FAKE, FAKE, pages, ctypes.addressof(table), self.mpps), table

    def status(self, fn, *a):
        try:
            fn(*a)
        except self.B.DbtError as e:
            return e.status
        return 0


def boundary(fk, dtype):
    """A boundary is valid directly after a prefill without one that succeeded,
    and never after one that failed: its logits, final states and kept rows
    are not those of the prompts."""
    p = Program(dtype)
    B, lens = p.B, [5, 20, 3]

    def prefill(kv, run):
        return p.status(B.dbt_prefill, p.model, kv, FAKE, lens, 3, run, p.out, 0)

    def fresh(kv):
        for b in range(3):
            B.dbt_kv_truncate(kv, b, 0)

    (one, _t1), (two, _t2) = p.cache(), p.cache()
    assert prefill(one, 0) == 0 and p.status(B.dbt_boundary, p.model, one, 3, p.out, 0) == 0
    assert p.status(B.dbt_boundary, p.model, one, 3, p.out, 0) == 4
    for run in (1, 0):
        fresh(one)
        fk.fake_reset(-1)
        assert prefill(one, run) == 0
        n = fk.fake_launches()
        assert n > 10
        for at in range(n):
            fresh(one)
            fresh(two)
            fk.fake_reset(-1)
            assert prefill(two, 0) == 0  # a boundary of the other cache is due, and lost with its rows
            fk.fake_reset(at)
            assert prefill(one, run) == 6, (run, at)
            fk.fake_reset(-1)
            for kv in (one, two):
                assert p.status(B.dbt_boundary, p.model, kv, 3, p.out, 0) == 4, (run, at, kv == one)


def pages(fk):
    """Page-table entries that a failing launch kept back are written by the
    next call: runs of consecutive pages and single entries, more of both than
    one launch takes."""
    nseq, mpps = 400, 16
    for at in range(12):
        p = Program("f32", max_batch=nseq)
        B = p.B
        kv, table = p.cache(nseq * 4, nseq)
        for b in range(nseq):  # one, two and three pages
            B.dbt_kv_reserve(kv, b, 16 * (1 + b % 3))
        for b in range(0, nseq, 5):  # freed pages: later rows are runs and singles mixed
            B.dbt_kv_truncate(kv, b, 0)
        for b in range(0, nseq, 10):
            B.dbt_kv_reserve(kv, b, 64)
        fk.fake_reset(at)
        first = p.status(B.dbt_kv_fill, kv, 0, 0, 0, 1, FAKE, FAKE, 0)
        failed = at < fk.fake_launches()
        assert first == (6 if failed else 0)
        fk.fake_reset(-1)
        if failed:
            assert p.status(B.dbt_kv_fill, kv, 0, 0, 0, 1, FAKE, FAKE, 0) == 0
        for b in range(nseq):
            want = B.dbt_kv_pages(kv, b)
            assert list(table[b * mpps:b * mpps + len(want)]) == want, (at, b)
        if not failed:
            assert at > 4, at  # several launches of each kind were tried
            return
    raise AssertionError("the flush never went through")


def steps(fk, form):
    """A step that fails at any launch leaves its sequences as they were, its
    new pages' table entries are still sent, and the step that follows it takes
    those pages and no more."""
    p = Program("bf16", n_layers=1, **(dict() if form == "tokens" else dict(has_embeddings=0, max_prompt=0)))
    B, lens = p.B, [16, 5, 32, 48]
    sin = B.dbt_step_in(batch=4, **(dict(tokens=FAKE) if form == "tokens" else dict(h1_in=FAKE, h2_in=FAKE)))
    calls = [lambda kv: p.status(B.dbt_decode_step, p.model, kv, sin, 1, p.out, 0),
             lambda kv: p.status(B.dbt_decode_step_ungrouped, p.model, kv, sin, p.out, 0)]
    for call in calls:
        at, n = 0, 1
        while at < n:
            kv, table = p.cache(16)
            for b, length in enumerate(lens):
                B.dbt_kv_reserve(kv, b, length)
            assert p.status(B.dbt_kv_fill, kv, 0, 0, 0, 1, FAKE, FAKE, 0) == 0  # the entries so far are written
            fk.fake_reset(at)
            assert call(kv) == 6, at
            assert [B.dbt_kv_length(kv, b) for b in range(4)] == lens, at
            fk.fake_reset(-1)
            assert p.status(B.dbt_kv_fill, kv, 0, 0, 0, 1, FAKE, FAKE, 0) == 0
            for b in range(4):
                want = B.dbt_kv_pages(kv, b)
                assert list(table[b * p.mpps:b * p.mpps + len(want)]) == want, (at, b)
            fk.fake_reset(-1)
            assert call(kv) == 0
            n = fk.fake_launches()
            assert [B.dbt_kv_length(kv, b) for b in range(4)] == [x + 1 for x in lens]
            assert [len(B.dbt_kv_pages(kv, b)) for b in range(4)] == [x // 16 + 1 for x in lens], at
            B.dbt_kv_destroy(kv)
            at += 1
        assert at > 6


def attention(fk):
    """Prompts of more pages than the page-sharing kernel holds ids for (1024)
    among shorter ones: each runs the kernel it runs alone."""
    for heads, short_kernel in ((4, "wide"), (3, "bf16")):  # (3 heads per KV head never share pages)
        p = Program("bf16", n_q_heads=heads, n_kv_heads=1, n_layers=1, max_pos=20000, max_prompt=20000)
        kv, _table = p.cache(8000)
        for lens, want in (([50, 7], [short_kernel]), ([16384], [short_kernel]), ([16385], ["bf16"]),
                           ([50, 16385, 60, 70], [short_kernel, "bf16", short_kernel])):
            if short_kernel == "bf16":
                want = ["bf16"] * (1 if sum(lens) <= 20000 else 2)
            for b in range(4):
                p.B.dbt_kv_truncate(kv, b, 0)
            fk.fake_reset(-1)
            p.B.dbt_prefill(p.model, kv, FAKE, lens, len(lens), 0, p.out, 0)
            names = [fk.fake_kernel(i).decode() for i in range(fk.fake_launches())]
            got = ["wide" if "prefill_wide" in n else "bf16" for n in names if "k_attn_prefill" in n]
            assert got == want, (heads, lens, got)


def router(fk):
    """One sequence and 256 experts: the router matrix is 1 MB at width 2048,
    and one workgroup reads 0.25 MB of it at most, as with 64 experts."""
    for E, groups in ((64, 1), (128, 1), (129, 3), (256, 4)):
        p = Program("bf16", n_layers=1, d_model=2048, d_ff=0, n_experts=E, d_ff_expert=128, d_ff_shared=128, top_k1=2,
                    top_k2=4)
        kv, _table = p.cache()
        fk.fake_reset(-1)
        p.B.dbt_decode_step(p.model, kv, p.B.dbt_step_in(tokens=FAKE, batch=1), 1, p.out, 0)
        names = [fk.fake_kernel(i).decode() for i in range(fk.fake_launches())]
        got = [fk.fake_groups(i) for i, n in enumerate(names) if "k_moe_route" in n]
        assert got == [groups], (E, got)
        assert sum("k_moe_select" in n for n in names) == (E > 128), E


def tiles(fk):
    """The GPU test's prompts of 256 rows and more run every tile shape of every
    epilogue, and plain projections in one to four splits."""
    import re
    from tests.gpu_util import TILED_CASES
    seen, splits = set(), set()
    for d, nq, nkv, f, lens in TILED_CASES:
        p = Program("bf16", max_batch=2, n_layers=1, d_model=d, n_q_heads=nq, n_kv_heads=nkv, d_ff=f,
                    max_pos=max(lens) + 1, max_prompt=max(lens))
        kv, _table = p.cache(200, 2)
        fk.fake_reset(-1)
        p.B.dbt_prefill(p.model, kv, FAKE, lens, len(lens), 0, p.out, 0)
        T = sum(lens)
        plain = [d, d]  # columns of W_O, down
        for i in range(fk.fake_launches()):
            m = re.search(r"k_gemm_tileILi(\d+)ELi(\d+)ELi(\d+)ELi(\d)ELb0", fk.fake_kernel(i).decode())
            if m:
                bm, bn, _bk, epi = map(int, m.groups())
                seen.add((bm, bn, epi))
                if epi == 0:
                    n = plain.pop()
                    splits.add(fk.fake_groups(i) // (-(-T // bm) * -(-n // bn)))
    assert seen == {(bm, bn, e) for bm, bn in ((256, 256), (128, 256), (128, 128)) for e in (0, 1, 2)}, seen
    assert splits == {1, 2, 3, 4}, splits


def workspace(fk):
    """Every prompt pass finds room for its slabs (each projection checks the
    room before its launch), the allocation-free step asks for the step's
    buffers alone, and nothing is reserved that no launch uses."""
    MB = 1 << 20
    for d, nq, nkv, f in ((256, 2, 1, 384), (2048, 16, 4, 5632), (4096, 32, 8, 14336), (1024, 8, 8, 4096),
                          (4224, 33, 11, 3200)):
        for longest, batch in ((100, 1), (127, 2), (128, 2), (255, 1), (256, 1), (300, 3), (1100, 2), (3000, 3)):
            p = Program("bf16", max_batch=batch, d_model=d, n_q_heads=nq, n_kv_heads=nkv, d_ff=f, n_layers=1,
                        max_pos=longest, max_prompt=longest)
            kv, _table = p.cache(1000, batch)
            for n in sorted({1, 17, 128, 129, 255, 256, 257, 600, longest} & set(range(1, longest + 1))):
                for b in range(batch):
                    p.B.dbt_kv_truncate(kv, b, 0)
                lens = [n] + [max(1, longest // 2)] * (batch - 1)
                assert p.status(p.B.dbt_prefill, p.model, kv, FAKE, lens, batch, 1, p.out, 0) == 0, (d, longest, lens)
            p.B.dbt_kv_destroy(kv)
            p.B.dbt_destroy(p.model)
    for longest in (256, 20000):  # a step does not use a prompt's buffers
        p = Program("bf16", max_batch=2, d_model=2048, n_q_heads=16, n_kv_heads=4, d_ff=5632, n_layers=1,
                    max_pos=20000, max_prompt=longest)
        kv, _table = p.cache(1000, 2)
        sin = p.B.dbt_step_in(tokens=FAKE, batch=1)
        assert p.status(p.B.dbt_decode_step_noalloc, p.model, kv, sin, 1, p.out, 0) == 0, longest

    def size(**kw):
        return Program("bf16", **kw).bytes

    # plain projections of short reductions or short prompts write one slab per row
    for kw in (dict(max_prompt=100, max_batch=2), dict(max_prompt=256, max_batch=4)):
        assert size(**kw) < 32 * MB, kw
    # router logits in memory for routers of several workgroups alone
    moe = dict(max_batch=512, max_prompt=0, n_layers=1, d_model=512, d_ff=0, d_ff_expert=128, d_ff_shared=128, top_k1=2,
               top_k2=4)
    few, many, more = (size(n_experts=E, **moe) for E in (127, 128, 129))
    assert many - few < 4096 and more - many >= 2 * 512 * 1024


if __name__ == "__main__":
    fk = ctypes.CDLL(sys.argv[2])
    fk.fake_kernel.restype = ctypes.c_char_p
    fk.fake_groups.restype = ctypes.c_uint
    what, _, arg = sys.argv[1].partition("_")
    dict(boundary=boundary, pages=pages, steps=steps, attention=attention, router=router, tiles=tiles,
         workspace=workspace)[what](*([fk, arg] if arg else [fk]))
    print("done")
