"""GPU parity of the weight-streaming gate/up kernel with its folded RMSNorm:
row counts at both ends of its range, hidden sizes that take different register
rings (8, 6 and 10 slices), and an FFN width whose 1032 units of eight outputs
do not divide evenly over the work-groups.  Every stage of decode-only
iterations against the float64 oracle at the parity bar.
"""
import pytest

from paper_2609_07883_amd import api, synth
from paper_2609_07883_amd.synth import ModelShape
from tests.parity import TOL, Mirror, check, stage_errors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d_model", [2048, 3072, 5120])
def test_few_rows(d_model):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session
    shape = ModelShape(n_layers=1, d_model=d_model, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn_dim=8256,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=1024)
    sess = Session(shape, num_blocks=128, max_c=0, max_b=9)
    mir = Mirror(sess)
    ids, ctx = list(range(1, 10)), [0, 5, 16, 33, 64, 7, 100, 31, 130]
    for sid, n in zip(ids, ctx):
        mir.create(sid)
        mir.install_context(sid, n)
    for step, rows in enumerate([1, 7, 8, 9]):  # 9: RMSNorm and the tile kernel
        assert (api.gemm_plan(rows, 2 * shape.ffn_dim, d_model)["cfg"] == api.GEMM_SKINNY) == (rows <= 8)
        lens = [n + sum(1 for r in [1, 7, 8, 9][:step] if i < r) for i, n in enumerate(ctx[:rows])]
        b = api.Batch(0, 0, 0, ids[:rows], lens)
        x = synth.embeddings(rows, d_model, seed=1, stream=rows)
        y, yr, sg, sr = mir.step(b, x)
        assert sg == sr
        for name, e in stage_errors(mir, b, x).items():
            assert e["rel"] <= TOL, (rows, name, e)
        check(y, yr, f"d_model {d_model}, {rows} rows")
