"""GPU parity of the projections at the edges of the tile kernel: k ranges of
one, two, three and five 64-deep steps (its software pipeline starts and ends
inside them), rows on both sides of a 32-row block and of a tile, and widths of
one 128-column tile.  Every row of each stage against the float64 oracle at the
parity bar.

Weights are drawn at std 0.09 (about 1 / sqrt(d_model)), so that each
projection's share of the residual stream is of the stream's own size and an
error in it is not hidden behind the residual.
"""
import pytest

from paper_2609_07883_amd import api, synth
from paper_2609_07883_amd.synth import ModelShape
from tests.parity import TOL, Mirror, check, stage_errors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# ffn 64, 192, 320: the down projection's k is one, three, five steps; d_model
# 128 gives the others two
@pytest.mark.parametrize("rows", [33, 64, 65, 129])
@pytest.mark.parametrize("ffn", [64, 192, 320])
def test_short_k_ranges(ffn, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session
    shape = ModelShape(n_layers=1, d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=ffn,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=1024)
    sess = Session(shape, num_blocks=64, max_c=256, max_b=2, layers=[synth.layer_weights(shape, std=0.09)])
    mir = Mirror(sess)
    for sid, n in ((1, 20), (2, 33)):
        mir.create(sid)
        mir.install_context(sid, n)
    b = api.Batch(rows - 1, 1, 20, [2], [33])
    x = synth.embeddings(rows, shape.d_model, seed=1, stream=rows)
    y, yr, sg, sr = mir.step(b, x)
    assert sg == sr
    for name, e in stage_errors(mir, b, x).items():
        assert e["rel"] <= TOL, (name, e)
    check(y, yr, f"ffn {ffn}, {rows} rows")
    assert mir.kv_error(b) <= TOL


@pytest.mark.parametrize("rows", [24, 25, 32, 33])
def test_narrow_widths_at_the_narrow_kernels_last_rows(rows):
    """Projections of at most 3072 columns stay with the narrow kernel up to 32
    rows (two 16-row groups, the second one ragged at 25): decode-only
    iterations on both sides of the limit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session
    shape = ModelShape(n_layers=1, d_model=1024, n_q_heads=16, n_kv_heads=16, head_dim=64, ffn_dim=1536,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=1024)
    for n, k in ((3072, 1024), (1024, 1024), (1024, 1536)):
        assert (api.gemm_plan(rows, n, k)["cfg"] == api.GEMM_NARROW) == (rows <= 32)
    sess = Session(shape, num_blocks=64, max_c=0, max_b=rows, layers=[synth.layer_weights(shape, std=0.03)])
    mir = Mirror(sess)
    ids, ctx = list(range(1, rows + 1)), [i % 19 for i in range(rows)]
    for sid, n in zip(ids, ctx):
        mir.create(sid)
        mir.install_context(sid, n)
    b = api.Batch(0, 0, 0, ids, ctx)
    x = synth.embeddings(rows, shape.d_model, seed=1, stream=rows)
    y, yr, sg, sr = mir.step(b, x)
    assert sg == sr
    for name, e in stage_errors(mir, b, x).items():
        assert e["rel"] <= TOL, (name, e)
    check(y, yr, f"{rows} rows")
    assert mir.kv_error(b) <= TOL


@pytest.mark.parametrize("rows", [3, 8])
def test_few_rows_of_a_qkv_projection_as_wide_as_gate_up(rows):
    """160 heads of 128: 20480 qkv columns at row counts where a gate/up
    projection of that width streams its weights."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session
    shape = ModelShape(n_layers=1, d_model=1024, n_q_heads=128, n_kv_heads=16, head_dim=128, ffn_dim=128,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=1024)
    p = api.gemm_plan(rows, 20480, 1024)
    assert p["cfg"] == api.GEMM_STREAM and p["other_cfg"] != api.GEMM_STREAM
    sess = Session(shape, num_blocks=16, max_c=0, max_b=rows)
    mir = Mirror(sess)
    ids, ctx = list(range(1, rows + 1)), [i % 19 for i in range(rows)]
    for sid, n in zip(ids, ctx):
        mir.create(sid)
        mir.install_context(sid, n)
    b = api.Batch(0, 0, 0, ids, ctx)
    x = synth.embeddings(rows, shape.d_model, seed=1, stream=rows)
    y, yr, sg, sr = mir.step(b, x)
    assert sg == sr
    for name, e in stage_errors(mir, b, x).items():
        assert e["rel"] <= TOL, (name, e)
    check(y, yr, f"{rows} rows")
    assert mir.kv_error(b) <= TOL
