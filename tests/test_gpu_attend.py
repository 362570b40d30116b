"""Scores and values of a run of tiles in one workgroup (csrc/attend16.hip) against the float64 oracle: runs shorter and longer than
the ring of tiles, shares of a run that are empty for some wavefronts, value ranks of part of a 128-column block, of one, two and
several, units over several groups, every number of query rows, row limits inside a run and before it; and which calls take it (two
kernels instead of three)."""

import numpy as np
import pytest

from oracle import palu_oracle as O
from workloads import synth

pytestmark = pytest.mark.gpu


def _layer(n_kv, group, rk, rv, q_per_kv=1):
    return synth.uniform_layer(n_kv, group, rk, rv, rope_theta=10000.0, q_per_kv=q_per_kv)


# heads, group, key rank, value rank, queries per key/value head, dtype, lengths, workgroups per unit and sequence (0: the library's choice)
CASES = [
    (4, 4, 256, 256, 1, "f16", [1], 0), (4, 4, 128, 128, 1, "f16", [33], 1), (8, 4, 256, 160, 1, "bf16", [97], 1),
    (4, 4, 224, 256, 1, "f16", [161], 1), (8, 4, 256, 384, 1, "f16", [257, 1], 1), (4, 4, 160, 32, 1, "f16", [2047], 1),
    (4, 1, 64, 64, 1, "f16", [130, 65], 1), (4, 1, 64, 96, 1, "bf16", [200], 2), (4, 2, 128, 128, 1, "f16", [129], 1),
    (4, 2, 96, 192, 1, "f16", [300, 40], 2), (6, 3, 192, 256, 1, "f16", [70], 1), (4, 4, 256, 256, 1, "f16", [511, 0, 96], 2),
    (4, 4, 256, 256, 4, "f16", [161, 33], 1), (4, 4, 128, 384, 2, "f16", [129], 1), (4, 4, 64, 128, 8, "f16", [200, 64], 2),
    (4, 2, 256, 160, 8, "bf16", [97], 1), (3, 3, 96, 96, 3, "f16", [333], 3), (4, 4, 160, 256, 5, "f16", [64, 0], 0),
    # at most four query rows to a unit
    (2, 1, 128, 96, 4, "f16", [300, 33], 1), (3, 1, 64, 64, 3, "bf16", [2047], 1), (2, 2, 256, 160, 2, "f16", [97, 0, 513], 2), (2, 1, 96, 128, 2, "f16", [161], 1),
    (4, 2, 224, 256, 2, "bf16", [700], 3), (2, 1, 128, 128, 1, "f16", [640, 31], 1),
]


# ... in runs through all sequences (chunks: workgroups per unit and sequence): runs that begin and end inside a sequence, empty sequences
# between others, several sequences to a run, runs longer than the values of one go (64 tiles)
FLAT_CASES = [
    (4, 4, 256, 256, 1, "f16", [511, 0, 96, 33, 0, 0, 1], 1), (8, 4, 128, 384, 1, "bf16", [200, 333, 64], 2), (4, 1, 64, 64, 1, "f16", [700, 650, 32], 3),
    (4, 2, 96, 160, 1, "f16", [65, 40, 0, 97, 31], 1), (4, 4, 256, 160, 1, "f16", [4200, 300], 1), (4, 1, 64, 96, 1, "f16", [300, 6500], 1),
    (4, 4, 160, 256, 1, "f16", [31] * 70, 1),
]


@pytest.mark.parametrize("heads,group,rk,rv,qpk,dtype,lens,chunks,flat", [c + (False,) for c in CASES] + [c + (True,) for c in FLAT_CASES])
def test_run_of_tiles(heads, group, rk, rv, qpk, dtype, lens, chunks, flat):
    import paper_2407_21118_amd as P
    from gpu_util import TOL_FP, rel_err, run_hip, run_oracle, say
    case = synth.make_case_orthonormal(_layer(heads, group, rk, rv, qpk), len(lens), max(lens), seed=heads + rk + rv + qpk, dtype=dtype)
    case.seq_lens = np.array(lens, np.int32) if len(lens) > 1 else None
    case.q_pos = np.maximum(np.array(lens, np.int32) - 1, 0)
    n = []
    P.palu_set_option("score_chunks", chunks if flat or case.seq_lens is None else 0)     # (with lengths the option means runs through all sequences)
    try:
        got = run_hip(case, n_launches=n)
    finally:
        P.palu_set_option("score_chunks", 0)
    ref = run_oracle(case)
    some = np.array(lens) > 0
    err = max(rel_err(got[some], ref[some]))               # of every sequence and head by itself
    say(f"[attend] {heads}/{group} heads rank {rk}/{rv} x{qpk} {dtype} {lens[:8]} chunks {chunks}: {err:.2e}")
    assert err <= TOL_FP and not got[~some].any()
    spans = next((g for g in (4, 2) if qpk == 1 and g * group <= 4 and g * rk <= 256 and g * group <= heads), 1)     # groups to a unit
    chosen = flat or case.seq_lens is None                 # the runs, by the option
    assert n == [2 if chosen or spans * rv <= 256 else 3]  # (these short runs)


RANKS = ([256, 64, 128, 224, 96, 160, 192, 256], [256, 160, 64, 128, 384, 32, 256, 192])


@pytest.mark.parametrize("kr,vr,dtype,lens,n_launches", [
    ([64, 256, 96], [256, 32, 160], "f16", [1], 2), ([256, 128, 224, 160], [96, 256, 128, 192], "bf16", [333, 0], 2),
    # more tiles than the compute units have workgroups: runs of several tiles, of other lengths from unit to unit
    (*RANKS, "f16", [9000], 2), (*RANKS, "bf16", [5000, 1700], 2), ([64, 256, 128, 192], [256, 256, 64, 128], "f16", [15000], 2),
    ([96, 64], [256, 128], "bf16", [16383, 7001], 2),
    # through all sequences, or more than 256 columns behind a run of one or two tiles: two launches
    ([64, 256, 96], [384, 32, 160], "f16", [1], 3), ([256, 128, 224, 160], [96, 256, 128, 416], "bf16", [333, 0], 3),
    ([192, 64, 256], [256, 160, 64], "f16", [129, 700, 0, 31, 65], 3), ([128, 96], [160, 512], "f16", [6000, 64, 5000], 3)])
def test_units_of_several_ranks(kr, vr, dtype, lens, n_launches):
    """Groups of different key and value ranks: for one and two sequences one launch, each unit with a number of workgroups of its own (sizes
    for 256 compute units)."""
    from gpu_util import TOL_FP, rel_err, run_hip, run_oracle, say
    layer = synth.ragged_layer(4 * len(kr), 4, kr, vr)
    case = synth.make_case_orthonormal(layer, len(lens), max(lens), seed=sum(kr) + len(lens), dtype=dtype)
    case.seq_lens = np.array(lens, np.int32) if len(lens) > 1 else None
    case.q_pos = np.maximum(np.array(lens, np.int32) - 1, 0)
    n = []
    got, ref = run_hip(case, n_launches=n), run_oracle(case)
    some = np.array(lens) > 0
    err = max(rel_err(got[some], ref[some]))
    say(f"[attend] ranks {kr} / {vr} {dtype} {lens}: {err:.2e}")
    assert err <= TOL_FP and not got[~some].any()
    assert n == [n_launches]


@pytest.mark.parametrize("heads,group,rk,rv,qpk,lens,n_launches", [
    (8, 4, 64, 64, 1, [4000] * 80, 3), (8, 4, 64, 256, 1, [1000] * 130, 2), (32, 4, 64, 192, 1, [500 - 5 * i for i in range(48)], 3),
    (32, 4, 64, 256, 1, [2043 - 20 * i for i in range(48)], 2), (32, 4, 64, 384, 1, [300 - i for i in range(100)], 3), (32, 4, 64, 384, 1, [600 - i for i in range(100)], 2),
    (8, 4, 128, 320, 1, [2500 - 9 * i for i in range(34)], 3), (8, 1, 128, 32, 1, [30000], 3), (8, 1, 96, 64, 1, [16384], 2),
    (8, 4, 64, 256, 6, [4000], 2), (8, 4, 64, 384, 6, [4000], 3), (4, 4, 64, 256, 6, [90000], 3), (4, 4, 64, 256, 5, [90000], 2), (4, 4, 64, 384, 5, [8000], 4),
    (8, 4, 128, 384, 1, [4000], 3), (8, 4, 128, 384, 1, [16000], 2), (32, 4, 64, 256, 1, [700] * 7, 3), (32, 4, 64, 256, 1, [1200] * 9, 2),
    (8, 4, 64, 384, 8, [4000], 3), (8, 4, 128, 384, 4, [16000], 2), (4, 1, 64, 64, 8, [90000], 3), (4, 1, 64, 64, 8, [20000], 2)])
def test_which_calls_take_one_launch(heads, group, rk, rv, qpk, lens, n_launches):
    """The rules' both sides, with the other way's result: runs through all sequences by their segments and value columns, one sequence
    whose runs would be longer than the value kernel's splits, blocks of rows and columns (sizes for 256 compute units)."""
    from gpu_util import TOL_FP, rel_err, run_hip
    case = synth.make_case_orthonormal(_layer(heads, group, rk, rv, qpk), len(lens), max(lens), seed=len(lens) + rv)
    case.seq_lens = np.array(lens, np.int32) if len(set(lens)) > 1 else None
    case.q_pos = np.array(lens, np.int32) - 1
    n = []
    got, apart = run_hip(case, n_launches=n), run_hip(case, staged=True).astype(np.float64)
    assert n == [n_launches]
    assert max(rel_err(got, apart)) <= TOL_FP


@pytest.mark.parametrize("n_q,qpk,rk,rv", [(1, 1, 256, 256), (2, 1, 128, 384), (4, 1, 256, 256), (3, 2, 64, 128), (8, 1, 160, 256)])
def test_row_limits_inside_a_run(n_q, qpk, rk, rv):
    """Row limits per query: none attended, inside the first set, at a set's edge, in the last rows."""
    import torch
    import paper_2407_21118_amd as P
    from gpu_util import TOL_FP, make_desc, rel_err, say, to_dev
    layer = _layer(4, 4, rk, rv, qpk)
    batch, seq = 2, 290
    case = synth.make_case_orthonormal(layer, batch, seq, seed=17 + n_q + rk)
    rng = np.random.default_rng(n_q * 100 + rk)
    q = synth.round_to(rng.standard_normal((batch, n_q, layer.n_q_heads, 128)), "f16")
    q_len = np.array([[0, 5, 32, 64, 128, 200, 289, 290][(j + b) % 8] if n_q > 1 else 37 + 200 * b for b in range(batch) for j in range(n_q)],
                     np.int32).reshape(batch, n_q)
    q_pos = np.maximum(q_len - 1, 0).astype(np.int32)
    dv = lambda x: torch.from_numpy(x).cuda()
    P.palu_set_option("score_chunks", 2)
    try:
        got = P.palu_attn_decode_multi(make_desc(layer, "f16"), batch, n_q, seq, seq, to_dev(q, "f16"), dv(q_pos), to_dev(case.Hk, "f16"),
                                       to_dev(case.Hv, "f16"), to_dev(case.Bk, "f16"), to_dev(case.Bv, "f16"),
                                       P.palu_rope_table_init(layer.rope_theta, 128, seq), seq, q_len=dv(q_len))
        torch.cuda.synchronize()
    finally:
        P.palu_set_option("score_chunks", 0)
    got = got.cpu().numpy()
    ref = O.attn_decode_multi(q, q_pos, q_len, case.Hk, case.Hv, case.Bk, case.Bv, layer.group_head_off, layer.k_rank_off, layer.v_rank_off,
                              128, layer.rope_theta, q_per_kv=qpk)
    some = q_len > 0
    err = max(rel_err(got[some], np.asarray(ref)[some]))
    say(f"[attend] {n_q} queries x{qpk} rank {rk}/{rv}: {err:.2e}")
    assert err <= TOL_FP
    assert not got[~some].any()


@pytest.mark.parametrize("rk,rv,lens,q_len,chunks", [(256, 256, [511, 0, 96, 33, 700], [37, 0, 96, 500, 512], 2), (64, 384, [300, 290, 64, 1, 150], [0, 289, 32, 1, 151], 1),
                                                     (128, 192, [4200, 300, 1000], [2100, 300, 999], 1)])
def test_row_limits_in_runs_through_all_sequences(rk, rv, lens, q_len, chunks):
    """Row limits beside sequence lengths: none attended, in a run's first segment and before its others, past the sequence's end."""
    import torch
    import paper_2407_21118_amd as P
    from gpu_util import TOL_FP, launches, make_desc, rel_err, to_dev
    layer, batch, seq = _layer(4, 4, rk, rv), len(lens), max(lens)
    case = synth.make_case_orthonormal(layer, batch, seq, seed=rk + rv)
    limits = np.minimum(lens, q_len).astype(np.int32)
    dv = lambda x: torch.from_numpy(np.asarray(x, np.int32)).cuda()
    out = torch.empty((batch, 1, 4, 128), dtype=torch.float32, device="cuda")
    args = (make_desc(layer, "f16"), batch, 1, seq, seq, to_dev(case.q[:, None], "f16"), dv(np.maximum(limits - 1, 0)[:, None]), to_dev(case.Hk, "f16"),
            to_dev(case.Hv, "f16"), to_dev(case.Bk, "f16"), to_dev(case.Bv, "f16"), P.palu_rope_table_init(layer.rope_theta, 128, seq), seq)
    kw = dict(q_len=dv(np.array(q_len)[:, None]), seq_lens=dv(lens), out=out)
    P.palu_set_option("score_chunks", chunks)
    try:
        P.palu_attn_decode_multi(*args, **kw)
        torch.cuda.synchronize()
        got = out.cpu().numpy()[:, 0]
        assert launches(lambda: P.palu_attn_decode_multi(*args, **kw)) == 2
    finally:
        P.palu_set_option("score_chunks", 0)
    ref = O.attn_decode(case.q, np.maximum(limits - 1, 0), case.Hk, case.Hv, case.Bk, case.Bv, layer.group_head_off, layer.k_rank_off, layer.v_rank_off, 128,
                        layer.rope_theta, None, limits)
    some = limits > 0
    assert max(rel_err(got[some], ref[some])) <= TOL_FP and not got[~some].any()


def test_more_runs_than_value_splits():
    """Many sequences of one unit: more partial results per sequence, and in all, than the value kernel's splits would make."""
    from gpu_util import TOL_FP, rel_err, run_hip, run_oracle
    lens = [(37 * i) % 301 for i in range(140)] + [2500]
    case = synth.make_case_orthonormal(_layer(4, 4, 64, 256), len(lens), max(lens), seed=5)
    case.seq_lens = np.array(lens, np.int32)
    case.q_pos = np.maximum(case.seq_lens - 1, 0)
    some = case.seq_lens > 0
    got, ref = run_hip(case), run_oracle(case)
    assert max(rel_err(got[some], ref[some])) <= TOL_FP and not got[~some].any()


@pytest.mark.parametrize("layer,dtype,seq,scale", [
    (_layer(8, 1, 128, 32), "f16", 40000, 4.0), (_layer(8, 2, 256, 64), "bf16", 30000, 4.0), (_layer(8, 2, 192, 64), "f16", 30000, 4.0),
    (synth.ragged_layer(32, 4, [256, 64, 128, 224, 96, 160, 192, 256], [256] * 8), "f16", 30000, 4.0),
    (_layer(8, 4, 256, 256), "f16", 16384, 4.0), (_layer(8, 4, 128, 128), "f16", 16384, 1.0)])
def test_as_precise_as_scores_and_values_apart(layer, dtype, seq, scale):
    """Probabilities are rounded to 16 bits against the running maximum of a wavefront's share of the sequence: whichever way a call
    takes, its shares are no longer than the splits of the value kernel, which the same call takes with events between its stages.
    Root mean square errors against float64 then differ by what other roundings of the same kind do: by less than 10 % over the
    at least 1024 outputs of eight independent heads or more (shares of two to four splits: 1.2 .. 1.8 at these queries)."""
    from gpu_util import run_hip, run_oracle, say
    case = synth.make_case_orthonormal(layer, 1, seq, seed=seq + layer.R_k, dtype=dtype)
    case.q = synth.round_to(case.q * scale, dtype)
    ref = run_oracle(case)
    one, apart = (np.sqrt(np.mean((run_hip(case, staged=s).astype(np.float64) - ref) ** 2)) for s in (False, True))
    say(f"[attend] {layer.R_k} / {layer.R_v} {dtype} {seq} q x{scale:g}: rms error {one:.3e}, stages apart {apart:.3e}")
    assert one <= 1.1 * apart


def test_units_of_fewer_heads_keep_the_exact_maximum():
    """Two heads to a unit, shares and splits of 64 tokens both: the value kernel, four heads to a unit, lets them all catch up with
    their running maxima where one of them rises, and a unit of two must not round more for catching up less often (errors
    of six draws together: its exact maximum can only be closer)."""
    from gpu_util import run_hip, run_oracle, say
    sums = np.zeros(2)
    for seed in range(6):
        case = synth.make_case_orthonormal(_layer(8, 1, 96, 64), 1, 16384, seed=seed)
        case.q = synth.round_to(case.q * 4.0, "f16")
        ref = run_oracle(case)
        sums += [np.sum((run_hip(case, staged=s).astype(np.float64) - ref) ** 2) for s in (False, True)]
    one, apart = np.sqrt(sums)
    say(f"[attend] two heads to a unit: error {one:.3e}, stages apart {apart:.3e}")
    assert one <= apart
