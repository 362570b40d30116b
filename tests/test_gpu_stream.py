"""Non-RoPE attention in one pass (stream_kernel, csrc/pv.hip) against the float64 oracle: both sides unquantized or quantized to the same
number of bits, units of one and of several groups, narrow ones, up to 16 heads, partial sets and splits, row limits, large logits; and which
calls take it (three kernels instead of four)."""

import numpy as np
import pytest

from oracle import palu_oracle as O
from workloads import synth

pytestmark = pytest.mark.gpu

CASES = [
    (4, 4, 256, 256, 1, "f16", 16, [1]), (8, 4, 256, 128, 1, "f16", 16, [33, 700]), (4, 1, 64, 64, 1, "bf16", 16, [97]),
    (6, 3, 96, 160, 1, "f16", 16, [64, 0, 513]), (4, 4, 32, 256, 4, "f16", 16, [290]), (2, 2, 256, 96, 8, "bf16", 16, [31, 129]),
    (8, 4, 256, 256, 1, "f16", 4, [1, 2047]), (4, 4, 128, 128, 1, "f16", 4, [95]), (5, 1, 128, 128, 1, "f16", 4, [161, 0, 32]),
    (4, 4, 128, 256, 4, "f16", 4, [300]), (4, 4, 256, 128, 1, "f16", 3, [130, 77]), (4, 2, 128, 128, 2, "f16", 2, [222]),
    (4, 4, 256, 256, 1, "f16", 4, [2047]), (8, 4, 128, 256, 1, "f16", 3, [1500, 1111]), (4, 1, 128, 128, 1, "f16", 2, [3000]), (4, 4, 256, 128, 1, "bf16", 16, [3000, 2500]),
]


@pytest.mark.parametrize("scale", [1.0, 8.0])
@pytest.mark.parametrize("heads,group,rk,rv,qpk,dtype,bits,lens", CASES)
def test_one_pass(heads, group, rk, rv, qpk, dtype, bits, lens, scale):
    from gpu_util import TOL_FP, TOL_I4, rel_err, run_hip, run_oracle, say
    layer = synth.uniform_layer(heads, group, rk, rv, rope_theta=0.0, q_per_kv=qpk)
    case = synth.make_case_orthonormal(layer, len(lens), max(lens), seed=heads + rk + rv + qpk, dtype=dtype)
    case.q = synth.round_to(case.q * scale, dtype)
    case.seq_lens = np.array(lens, np.int32) if len(lens) > 1 else None
    case.q_pos = np.maximum(np.array(lens, np.int32) - 1, 0)
    n = []
    if bits == 16:
        got, ref, tol = run_hip(case, n_launches=n), run_oracle(case), TOL_FP
    else:
        quant = {"k": O.quant_latent(case.Hk, bits=bits), "v": O.quant_latent(case.Hv, bits=bits)}
        got, ref, tol = run_hip(case, True, True, quant, bits=bits, n_launches=n), run_oracle(case, quant, True, True, bits=bits), TOL_I4
    some = np.array(lens) > 0
    err = max(rel_err(got[some], ref[some]))               # of every sequence and head by itself
    say(f"[one pass] {heads}/{group} heads rank {rk}/{rv} x{qpk} {dtype} {bits} bits {lens} q x{scale:g}: {err:.2e}")
    assert err <= tol and not got[~some].any()
    assert n == [4 if bits < 16 and group * qpk > 4 else 3]      # units of more than 4 heads over codes keep two launches


@pytest.mark.parametrize("heads,group,qpk,rk,rv,batch,seq,n_launches", [
    (32, 4, 1, 64, 64, 25, 400, 3), (32, 4, 1, 64, 64, 33, 400, 4), (8, 1, 4, 64, 64, 77, 653, 4), (32, 4, 1, 64, 64, 30, 2500, 3)])
def test_rounds_of_workgroups(heads, group, qpk, rk, rv, batch, seq, n_launches):
    """More workgroups than compute units: one launch for many and long splits, else two (sizes for 256 compute units)."""
    from gpu_util import rel_err, run_hip
    case = synth.make_case_orthonormal(synth.uniform_layer(heads, group, rk, rv, rope_theta=0.0, q_per_kv=qpk), batch, seq, seed=batch)
    n = []
    got, apart = run_hip(case, n_launches=n), run_hip(case, staged=True)
    assert n == [n_launches]
    assert rel_err(got, apart.astype(np.float64))[0] <= 1e-5      # the same splits, scores to the order of their float32 sums


@pytest.mark.parametrize("bits", [16, 4])
def test_row_limits(bits):
    import torch
    import paper_2407_21118_amd as P
    from gpu_util import TOL_FP, TOL_I4, make_desc, rel_err, to_dev
    layer = synth.uniform_layer(4, 4, 128, 256, rope_theta=0.0)
    batch, n_q, seq = 2, 4, 290
    case = synth.make_case_orthonormal(layer, batch, seq, seed=23 + bits)
    q = synth.round_to(np.random.default_rng(bits).standard_normal((batch, n_q, 4, 128)), "f16")
    q_len = np.array([[0, 5, 32, 290], [64, 128, 289, 1]], np.int32)
    q_pos = np.maximum(q_len - 1, 0).astype(np.int32)
    dv = lambda x: torch.from_numpy(x).cuda()
    half = lambda x: torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16)
    Hk, Hv, kw, hk, hv = case.Hk, case.Hv, {}, to_dev(case.Hk, "f16"), to_dev(case.Hv, "f16")
    if bits == 4:
        qk, qv = O.quant_latent(case.Hk), O.quant_latent(case.Hv)
        Hk, Hv, hk, hv = O.dequant_latent(*qk), O.dequant_latent(*qv), dv(qk[0]), dv(qv[0])
        kw = dict(hk_scale=half(qk[1]), hk_zero=half(qk[2]), hv_scale=half(qv[1]), hv_zero=half(qv[2]))
    got = P.palu_attn_decode_multi(make_desc(layer, "f16", bits == 4, bits == 4), batch, n_q, seq, seq, to_dev(q, "f16"), dv(q_pos), hk, hv,
                                   to_dev(case.Bk, "f16"), to_dev(case.Bv, "f16"), P.palu_rope_table_init(0.0, 128, seq), seq, q_len=dv(q_len), **kw)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    ref = np.asarray(O.attn_decode_multi(q, q_pos, q_len, Hk, Hv, case.Bk, case.Bv, layer.group_head_off, layer.k_rank_off, layer.v_rank_off,
                                         128, 0.0))
    some = q_len > 0
    assert rel_err(got[some], ref[some])[0] <= (TOL_FP if bits == 16 else TOL_I4) and not got[~some].any()
