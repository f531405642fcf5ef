"""GPU parity of the weight-streaming gate/up kernel with its folded RMSNorm:
row counts at both ends of its range, hidden sizes that take different register
rings (8, 6 and 10 slices), and an FFN width whose 1032 units of eight outputs
do not divide evenly over the work-groups.  Every stage of decode-only
iterations against the float64 oracle at the parity bar.  Then every hidden
size the kernel is built for, its outputs against a float64 product of the
residual rows the same iteration left.
"""
import numpy as np
import pytest

from paper_2609_07883_amd import api, synth
from paper_2609_07883_amd.synth import ModelShape
from tests.parity import RMS_TOL, TOL, Mirror, check, rel_err, rms_err, stage_errors

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
        assert (api.gemm_plan(rows, 2 * shape.ffn_dim, d_model)["cfg"] == api.GEMM_STREAM) == (rows <= 8)
        lens = [n + sum(1 for r in [1, 7, 8, 9][:step] if i < r) for i, n in enumerate(ctx[:rows])]
        b = api.Batch(0, 0, 0, ids[:rows], lens)
        x = synth.embeddings(rows, d_model, seed=1, stream=rows)
        y, yr, sg, sr = mir.step(b, x)
        assert sg == sr
        for name, e in stage_errors(mir, b, x).items():
            assert e["rel"] <= TOL, (rows, name, e)
        check(y, yr, f"d_model {d_model}, {rows} rows")


# multiples of 1024 from 2048 to 6144 stream at any width from 16384 on; the
# others where 128-column tiles are 257 to 384 (n = 2 ffn), below 2048 also
# fewer.  A hidden size for every number of slices a wave takes: the multiples
# of 512, where all waves take as many, and others, where the last slices are
# missing from all waves or from four of the eight.
SIZES = [(1024, 8256), (1536, 8256), (2048, 8256), (2560, 16448), (3072, 8256), (3584, 18944), (4096, 8256),
         (4608, 16448), (5120, 8256), (5632, 16448), (6144, 8256), (6656, 17920), (7168, 16448), (7680, 16448),
         (8192, 16448), (1152, 8256), (1920, 8256), (2176, 16448), (2816, 19200), (3328, 18944), (3840, 19200),
         (4224, 17920), (4864, 16448), (5376, 16448), (5888, 16448), (6272, 16448), (6912, 16448), (7296, 16448),
         (7936, 16448), (1408, 8256), (3584, 24576)]


@pytest.mark.parametrize("d_model,ffn", SIZES)
def test_every_hidden_size(d_model, ffn):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_07883_amd.runtime import Session, tensor_to_f64
    shape = ModelShape(n_layers=1, d_model=d_model, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn_dim=ffn,
                       rms_eps=1e-5, rope_theta=10000.0, max_pos=1024)
    assert api.gemm_plan(8, 2 * ffn, d_model)["cfg"] == api.GEMM_STREAM
    assert api.gemm_plan(9, 2 * ffn, d_model)["cfg"] != api.GEMM_STREAM
    sess = Session(shape, num_blocks=16, max_c=0, max_b=8, device_weights=True)
    for sid in range(8):
        sess.ctx.seq_create(sid)
    w = sess.weights[0]
    g2, wgu = w["g2"].double(), w["wgu"].double()
    for rows in (1, 3, 8):
        b = api.Batch(0, 0, 0, list(range(rows)), [0] * rows)
        x = synth.embeddings(rows, d_model, seed=1, stream=rows)
        sess.run(b, x)
        h = torch.from_numpy(sess.view(api.VIEW_H, 0, rows, d_model, fp32=True)).to(sess.dev)
        act = sess.view(api.VIEW_ACT, 0, rows, ffn)
        n = h / torch.sqrt((h * h).mean(1, keepdim=True) + shape.rms_eps) * g2
        gate, up = (n @ wgu.T).split(ffn, 1)
        ref = tensor_to_f64(gate / (1 + torch.exp(-gate)) * up)
        assert np.isfinite(act).all()
        assert rel_err(act, ref) <= TOL and rms_err(act, ref) <= RMS_TOL, (rows, rel_err(act, ref))
