"""GPU parity of the two-phase chunk kernel, the one long work items run at head
dim 128, for every GQA group size, and of the other chunk kernel over the same
lengths at head dim 64: a few query rows over a long cached prefix, so that
each work item takes many key tiles, beside decodes in the same launch.  Prefix and chunk end inside a page and inside a 64-key tile, the last
query tile is ragged, a run of keys crosses query tiles, and every KV slot that
no token owns holds NaN (values past the range end are cleared in LDS).

Sampled rows against the float64 oracle at the parity bar.
"""
import numpy as np
import pytest

from paper_2609_07883_amd import api, synth
from paper_2609_07883_amd.synth import ModelShape
from tests.parity import TOL, Mirror, check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (q heads, kv heads, head dim, chunk, prefix)
CASES = [
    (16, 16, 64, 300, 16390),
    (16, 16, 128, 257, 32010),
    (32, 16, 128, 140, 20020),
    (32, 8, 128, 200, 16390),
    (64, 8, 128, 100, 16401),
    (128, 8, 128, 50, 16383),
    (64, 8, 64, 100, 16401),
    (128, 8, 64, 50, 16383),
]


@pytest.mark.parametrize("case", CASES, ids=[f"hq{c[0]}_hkv{c[1]}_hd{c[2]}" for c in CASES])
def test_long_prefix(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session
    hq, hkv, hd, C, P = case
    shape = ModelShape(n_layers=1, d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=256,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=32768)
    dec, ctx = [21, 22], [5, 700]
    plan = api.attention_plan(shape, ctx, [(P, C)])
    assert plan["chunk_two_phase"] == (hd == 128)
    qk_std = 0.16 * (64 / hd) ** 0.25
    sess = Session(shape, num_blocks=(P + C) // 16 + 60, max_c=C, max_b=2, qk_std=qk_std)
    sess.k_pool.fill_(float("nan"))
    sess.v_pool.fill_(float("nan"))
    torch.cuda.synchronize()
    mir = Mirror(sess, seed=5)
    for sid, n in [(3, P)] + list(zip(dec, ctx)):
        mir.create(sid)
        mir.install_context(sid, n)
    b = api.Batch(C, 3, P, dec, ctx)
    x = synth.embeddings(b.rows, shape.d_model, seed=1, stream=C)
    pw = 256 // (hq // hkv)  # positions of a query tile
    rows = sorted({r for r in (0, 1, 15, 16, 31, 32, pw - 1, pw, C - 2, C - 1, C, C + 1) if r < b.rows})
    y, yr, sg, sr = mir.step(b, x, rows=rows)
    assert sg == sr
    assert np.isfinite(np.asarray(y, dtype=np.float64)).all()
    check(y[rows], yr[rows], f"{case}")
    assert mir.kv_error(b, rows=rows) <= TOL


# (q heads, kv heads, head dim, chunk, prefix, chunk row with non-finite values)
NON_FINITE = [
    (16, 16, 128, 257, 32000, 215),  # a query tile of 256 positions, split over work-groups
    (8, 8, 128, 4096, 8192, 1215),
    (32, 8, 128, 4096, 3000, 1172),  # query tiles of 64 positions across two key tiles, whole
    (32, 8, 128, 200, 28682, 60),    # the same, split
]


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("case", NON_FINITE, ids=[f"hq{c[0]}_hkv{c[1]}_c{c[3]}" for c in NON_FINITE])
def test_non_finite_row_reaches_no_earlier_key_tile(case, bad):
    """A non-finite input row makes that token's K and V non-finite.  Rows of
    waves (32 / group positions each) that end before its 64-key tile never
    read its values, though later waves of their query tile do: they come out
    as if the row were finite, bit for bit, and so do the other sequences'."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session
    hq, hkv, hd, C, P, r = case
    shape = ModelShape(n_layers=1, d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=256,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=32768)
    dec, ctx = [21, 22], [5, 700]
    pw, tile = 32 * hkv // hq, 256 * hkv // hq
    first_bad = (P + r) // 64 * 64 - P               # first chunk row whose key tile holds row r
    safe = r // tile * tile + max(0, first_bad - r // tile * tile) // pw * pw
    assert safe > r // tile * tile                   # rows of r's own query tile among them
    assert api.attention_plan(shape, ctx, [(P, C)])["chunk_two_phase"]
    sess = Session(shape, num_blocks=(P + C) // 16 + 60, max_c=C, max_b=2, qk_std=0.16 * (64 / hd) ** 0.25)
    gen = torch.Generator(device=sess.dev).manual_seed(3)
    sess.k_pool.normal_(0.0, 1.0, generator=gen)
    sess.v_pool.normal_(0.0, 1.0, generator=gen)
    for sid, n in [(3, P)] + list(zip(dec, ctx)):
        sess.ctx.seq_create(sid)
        sess.ctx.seq_reserve(sid, n)
    b = api.Batch(C, 3, P, dec, ctx)
    x = synth.embeddings(b.rows, shape.d_model, seed=1, stream=C)
    sess.run(b, x)
    ref = sess.output(b.rows)
    sess.x_in[: b.rows].copy_(torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).to(sess.dev)
                              .view(torch.bfloat16))
    sess.x_in[r] = bad
    sess.run(b)
    got = sess.output(b.rows)
    rows = list(range(safe)) + [C, C + 1]
    assert np.isfinite(got[rows]).all()
    np.testing.assert_array_equal(got[rows], ref[rows])
    assert not np.isfinite(got[r]).all()
