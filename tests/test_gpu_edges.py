"""Kernels at the sizes where their tiling can go wrong: edges of tiles, remainders, the smallest and largest of a
form's range, against the CPU oracle."""

import numpy as np
import pytest
import torch

import paper_2407_21118_amd as P
from oracle import palu_oracle as O
from workloads import synth

pytestmark = pytest.mark.gpu

from gpu_util import TOL_FP, TOL_I4, make_desc, rel_err, run_hip, run_oracle, say, to_dev  # noqa: E402


@pytest.mark.parametrize("heads,group,rk,rv,dtype", [(1, 1, 32, 96, "f16"), (3, 1, 32, 64, "bf16"), (5, 1, 96, 32, "f16"),
                                                      (32, 4, 256, 256, "bf16")])
def test_encode_token_tiles(heads, group, rk, rv, dtype):
    """The split-K projection at token counts around its tiles of 16 and depths (128 .. 4096) that leave wavefronts of the
    last workgroup without rows; column counts that end inside a workgroup's 128."""
    layer = synth.uniform_layer(heads, group, rk, rv)
    rng = np.random.default_rng(31)
    d = heads * 128
    Ak = synth.round_to(rng.standard_normal((d, layer.R_k)) / np.sqrt(d), dtype)
    Av = synth.round_to(rng.standard_normal((d, layer.R_v)) / np.sqrt(d), dtype)
    desc = make_desc(layer, dtype)
    dev_k, dev_v = to_dev(Ak, dtype), to_dev(Av, dtype)
    # one rounding to the cache dtype (half a unit in the last place, relative to the value) plus float32 sums of d
    # products: d eps / 2 of the sum of magnitudes, itself about sqrt(d) / d ... 1 of the result's size: 1e-5 is ample
    eps = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8
    for n_tok in (1, 2, 15, 16, 17, 32, 33, 48, 49, 63):
        x = synth.round_to(rng.standard_normal((n_tok, d)), dtype)
        hk = torch.full((n_tok + 1, layer.R_k), 7.0, dtype=dev_k.dtype, device="cuda")
        hv = torch.full((n_tok + 1, layer.R_v), 7.0, dtype=dev_v.dtype, device="cuda")
        P.palu_encode_kv(desc, to_dev(x, dtype), dev_k, dev_v, hk, layer.R_k, hv, layer.R_v)
        torch.cuda.synchronize()
        for got, A in ((hk, Ak), (hv, Av)):
            g, ref = got.float().cpu().numpy(), O.encode(x, A)
            err = np.abs(g[:n_tok] - ref) - eps * np.abs(ref)
            assert err.max() <= 1e-5 * np.abs(ref).max(), (n_tok, err.max())
            assert (g[n_tok] == 7.0).all()
    say(f"[edges] encode heads={heads} R={layer.R_k}/{layer.R_v} {dtype}")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("heads", [1, 3, 2])
def test_encode_infinities(heads, dtype):
    """The split-K projection of infinite inputs and weights in its first rows: infinities of the right sign where the sum has
    them and NaN only where it has both, also at depths (128, 384) whose last workgroup has wavefronts without rows."""
    layer = synth.uniform_layer(heads, 1, 64, 32)
    rng = np.random.default_rng(35)
    d = heads * 128
    sides = [synth.round_to(1.0 + rng.random((d, R)), dtype) * np.where(np.arange(R) % 2, -1.0, 1.0) for R in (layer.R_k, layer.R_v)]
    sides[0][3, 1], sides[1][63, 0] = np.inf, -np.inf
    desc = make_desc(layer, dtype)
    for n_tok in (1, 2, 17, 63):
        x = synth.round_to(1.0 + rng.random((n_tok, d)), dtype)
        x[n_tok - 1, 5] = np.inf
        hk, hv = (torch.full((n_tok, A.shape[1]), 7.0, dtype=to_dev(x, dtype).dtype, device="cuda") for A in sides)
        P.palu_encode_kv(desc, to_dev(x, dtype), *(to_dev(A, dtype) for A in sides), hk, layer.R_k, hv, layer.R_v)
        torch.cuda.synchronize()
        for got, A in ((hk, sides[0]), (hv, sides[1])):
            with np.errstate(invalid="ignore"):
                g, ref = got.float().cpu().numpy(), x.astype(np.float64) @ A.astype(np.float64)
            finite = np.isfinite(ref)
            assert np.array_equal(g[~finite], ref[~finite].astype(np.float32), equal_nan=True), (heads, n_tok)
            # one rounding to the cache dtype, sums of at most 384 products of one sign in float32
            assert (np.abs(g[finite] / ref[finite] - 1) <= (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) + 1e-5).all()
    say(f"[edges] encode infinities heads={heads} {dtype}")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("heads,rk,rv", [(1, 32, 160), (3, 64, 96), (8, 256, 32)])
def test_encode_gemm_tiles(heads, rk, rv, dtype):
    """The prompt-sized projection with every tile that the option names and the one it takes by itself, at token counts around the tiles' rows, column counts that end inside
    a tile (32 .. 2048) and depths shorter than the ring of stages (128 rows: two stages of six)."""
    layer = synth.uniform_layer(heads, 1, rk, rv)
    rng = np.random.default_rng(33)
    d = heads * 128
    Ak = synth.round_to(rng.standard_normal((d, layer.R_k)) / np.sqrt(d), dtype)
    Av = synth.round_to(rng.standard_normal((d, layer.R_v)) / np.sqrt(d), dtype)
    desc = make_desc(layer, dtype)
    dev_k, dev_v = to_dev(Ak, dtype), to_dev(Av, dtype)
    eps = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8                # the bound of test_encode_token_tiles
    for n_tok in (64, 65, 127, 129, 257):
        x = synth.round_to(rng.standard_normal((n_tok, d)), dtype)
        refs = O.encode(x, Ak), O.encode(x, Av)
        for tile in (0, 32, 64, 128, 256):
            hk = torch.full((n_tok + 1, layer.R_k), 7.0, dtype=dev_k.dtype, device="cuda")
            hv = torch.full((n_tok + 1, layer.R_v), 7.0, dtype=dev_v.dtype, device="cuda")
            P.palu_set_option("encode_tile_rows", tile)
            try:
                P.palu_encode_kv(desc, to_dev(x, dtype), dev_k, dev_v, hk, layer.R_k, hv, layer.R_v)
            finally:
                P.palu_set_option("encode_tile_rows", 0)
            torch.cuda.synchronize()
            for got, ref in zip((hk, hv), refs):
                g = got.float().cpu().numpy()
                err = np.abs(g[:n_tok] - ref) - eps * np.abs(ref)
                assert err.max() <= 1e-5 * np.abs(ref).max(), (n_tok, tile, err.max())
                assert (g[n_tok] == 7.0).all()
    say(f"[edges] encode GEMM heads={heads} R={layer.R_k}/{layer.R_v} {dtype}")


def odd_zero_rows(case, quant, b, rows):
    """Gives 128-channel block blk of row t of sequence b, for every (t, blk) of rows, a zero-point of n + 1/2 and codes n and
    n + 1 that fit the query of its group's first head: logits of 12, so that these rows share that head's softmax and a
    zero-point rounded to an integer, half a step in every channel, shows."""
    layer, (codes, scale, zero) = case.layer, quant["k"]
    for i, (t, blk) in enumerate(rows):
        blk %= layer.R_k // 128
        j = int(np.searchsorted(layer.k_rank_off, 128 * blk, side="right")) - 1
        r, size = layer.k_rank_off[j + 1] - layer.k_rank_off[j], layer.group_size(j)
        at = int(sum((layer.k_rank_off[g + 1] - layer.k_rank_off[g]) * layer.group_size(g) for g in range(j))) * 128
        B = case.Bk[at:at + r * size * 128].reshape(r, size * 128)[128 * blk - layer.k_rank_off[j]:][:128, :128]
        q = O.rope_rotate(case.q[b, layer.group_head_off[j] * layer.q_per_kv].astype(np.float64), case.q_pos[b], layer.rope_theta)
        w = B @ O.rope_rotate(q, -t, layer.rope_theta) / 128 ** 0.5
        n = (0, 7, 14)[i % 3]
        scale[b, t, blk], zero[b, t, blk] = 24.0 / np.abs(w).sum(), n + 0.5
        codes[b, t, 64 * blk:64 * blk + 64] = O.pack_codes((n + (w > 0)).astype(np.uint8), 4)


@pytest.mark.parametrize("odd_zero", [False, True])
@pytest.mark.parametrize("heads,group,rk,q_per_kv", [(4, 1, 128, 1), (3, 1, 128, 1), (2, 1, 256, 1), (4, 2, 256, 1), (8, 4, 128, 1),
                                                     (5, 5, 256, 1), (4, 4, 384, 1), (4, 4, 512, 2), (8, 8, 1024, 1), (2, 2, 128, 5)])
def test_quantized_keys_whole_head(heads, group, rk, q_per_kv, odd_zero):
    """4-bit keys on the whole-head score kernel: one, two and four groups to a workgroup, ranks in one slice and in several,
    lengths around its 32-token tiles; zero-points that the packed dequantization does not hold for (a fraction, a large one)
    in some tokens of some blocks."""
    layer = synth.uniform_layer(heads, group, rk, 128, q_per_kv=q_per_kv)
    rng = np.random.default_rng(5)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    lens = np.array([161, 1, 33, 96], np.int32)
    case = synth.Case("edges", layer, "f16", 4, 161, draw(4, layer.n_q_heads, 128), lens - 1, draw(4, 161, layer.R_k),
                      draw(4, 161, layer.R_v), draw(layer.b_elems("k"), by=rk ** -0.5), draw(layer.b_elems("v"), by=128 ** -0.5))
    case.seq_lens = lens
    quant = {"k": O.quant_latent(case.Hk)}
    if odd_zero:
        odd_zero_rows(case, quant, 0, [(70, 0), (160, 0), (70, -1), (160, -1)])
        odd_zero_rows(case, quant, 2, [(31, 0), (32, 0), (31, -1), (32, -1)])
        quant["k"][2][3, 50, 0] = 2001.0
    got, ref = run_hip(case, True, False, quant), run_oracle(case, quant, True, False)
    err = max(rel_err(got, ref))
    say(f"[edges] 4-bit keys heads={heads} group={group} rank={rk} q_per_kv={q_per_kv} odd={odd_zero} rel err {err:.3e}")
    assert err <= TOL_I4


@pytest.mark.parametrize("odd_zero", ["none", "some", "all"])
@pytest.mark.parametrize("lens", [None, [2245], [700, 0, 2245, 33, 96]])
@pytest.mark.parametrize("group,ranks,q_per_kv", [(1, [128, 128], 1), (2, [256, 256], 1), (3, [384, 256], 1), (2, [256], 3), (2, [256], 8),
                                                  (2, [128] * 4, 1), (4, [512], 2), (2, [128, 384], 4)])
def test_quantized_keys_long_runs(group, ranks, q_per_kv, lens, odd_zero):
    """4-bit keys in runs of many tiles, one workgroup to a sequence and head block (option score_chunks): 71 tiles of one
    sequence (more than the 64 that are looked through at a time), and runs that begin and end inside sequences; zero-points
    that the packed dequantization does not hold for in no tile, in single ones (early, late, neighbours, three apart, the
    last; a sequence without any between two with) and in all."""
    layer = synth.ragged_layer(group * len(ranks), group, ranks, [128] * len(ranks), q_per_kv=q_per_kv)
    rng = np.random.default_rng(9)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    n = np.array(lens or [2245], np.int32)
    batch, seq = len(n), 2245
    case = synth.Case("edges", layer, "f16", batch, seq, draw(batch, layer.n_q_heads, 128), np.maximum(n - 1, 0), draw(batch, seq, layer.R_k),
                      draw(batch, seq, layer.R_v), draw(layer.b_elems("k"), by=max(ranks) ** -0.5), draw(layer.b_elems("v"), by=128 ** -0.5))
    if lens:
        case.seq_lens = n
    quant = {"k": O.quant_latent(case.Hk)}
    if odd_zero == "some":
        odd_zero_rows(case, quant, int(np.argmax(n)), [(40, 0), (64, -1), (165, 0), (261, -1), (2079, 0), (2080, -1), (2244, 0)])
        if batch > 1:
            odd_zero_rows(case, quant, batch - 1, [(32, 0), (95, 0), (32, -1), (95, -1)])
    elif odd_zero == "all":
        quant["k"][2][:] += np.float16(0.5)
    P.palu_set_option("score_chunks", 1)
    try:
        got = run_hip(case, True, False, quant)
    finally:
        P.palu_set_option("score_chunks", 0)
    ref = run_oracle(case, quant, True, False)
    some = n > 0
    err = max(rel_err(got[some], ref[some]))
    say(f"[edges] 4-bit keys, long runs group={group} ranks={ranks} q_per_kv={q_per_kv} lens={lens} odd={odd_zero} rel err {err:.3e}")
    assert err <= TOL_I4 and not got[~some].any()


@pytest.mark.parametrize("lens", [False, True])
@pytest.mark.parametrize("group,ranks,q_per_kv", [(1, [384, 384], 1), (1, [512, 128, 512], 2), (2, [384, 256, 384], 1), (2, [512, 1024], 1), (4, [384], 1),
                                                  (4, [384, 128], 2), (3, [512, 384, 1024], 2), (1, [384], 4), (5, [384, 256], 1)])
def test_quantized_keys_of_ranks_above_256(group, ranks, q_per_kv, lens):
    """4-bit keys of ranks 384 and 512 on either side of the rule that slices them for the whole-head kernel (few heads per
    group; rank 384 alone or beside ranks that share its launches), beside ranks on the other kernel, shared and not."""
    layer = synth.ragged_layer(group * len(ranks), group, ranks, [64] * len(ranks), q_per_kv=q_per_kv)
    rng = np.random.default_rng(10)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    n = np.array([300, 65, 1], np.int32)
    case = synth.Case("edges", layer, "f16", 3, 300, draw(3, layer.n_q_heads, 128), n - 1, draw(3, 300, layer.R_k), draw(3, 300, layer.R_v),
                      draw(layer.b_elems("k"), by=max(ranks) ** -0.5), draw(layer.b_elems("v"), by=64 ** -0.5))
    if lens:
        case.seq_lens = n
    quant = {"k": O.quant_latent(case.Hk)}
    err = max(rel_err(run_hip(case, True, False, quant), run_oracle(case, quant, True, False)))
    say(f"[edges] 4-bit keys group={group} ranks={ranks} q_per_kv={q_per_kv} lens={lens} rel err {err:.3e}")
    assert err <= TOL_I4


@pytest.mark.parametrize("ranks,q_per_kv,dtype", [([64], 1, "f16"), ([256], 1, "bf16"), ([128], 3, "f16"), ([64, 96, 256], 1, "f16"), ([320], 1, "f16")])
@pytest.mark.parametrize("lens", ["mixed", "mixed, long runs", "many", "equal", "two", "one, equal"])
def test_runs_through_sequences(ranks, q_per_kv, dtype, lens):
    """Score workgroups over sequences of different lengths, empty ones and ones of one tile among them: runs inside a sequence
    (nine of up to 193 rows, two, one), runs that go through several (the same with as many workgroups as sequences, option score_chunks;
    more sequences than lanes, a few tiles to a run), and one length but more sequences than compute units."""
    n = len(ranks)
    layer = synth.Layer(4 * n, 128, list(range(0, 4 * n + 1, 4)), list(np.cumsum([0] + ranks)), list(np.cumsum([0] + [64] * n)), q_per_kv=q_per_kv)
    seq = {"mixed": 193, "mixed, long runs": 193, "many": 300, "equal": 65, "two": 193, "one, equal": 193}[lens]
    sl = {"many": [(37 * i) % 301 for i in range(150)], "equal": [65] * 300, "two": [70, 193], "one, equal": [193]}.get(lens, [193, 0, 1, 64, 0, 0, 32, 33, 160])
    batch = len(sl)
    rng = np.random.default_rng(6)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, dtype)  # noqa: E731
    case = synth.Case("edges", layer, dtype, batch, seq, draw(batch, layer.n_q_heads, 128), np.maximum(np.array(sl, np.int32) - 1, 0),
                      draw(batch, seq, layer.R_k), draw(batch, seq, layer.R_v), draw(layer.b_elems("k"), by=0.1), draw(layer.b_elems("v"), by=0.1))
    if "equal" not in lens:
        case.seq_lens = np.array(sl, np.int32)
    P.palu_set_option("score_chunks", 1 if "long" in lens else 0)
    try:
        got = run_hip(case)
    finally:
        P.palu_set_option("score_chunks", 0)
    ref = run_oracle(case)
    some = np.array(sl) > 0
    err = max(rel_err(got[some], ref[some]))
    say(f"[edges] runs ranks={ranks} q_per_kv={q_per_kv} {dtype} {lens} rel err {err:.3e}")
    assert err <= TOL_FP and not got[~some].any()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n_tok", [77, 290, 600, 1030, 2055, 4099])
def test_encode_gemm_tiles_by_cost(n_tok, dtype):
    """The prompt-sized projection with the tile it takes by itself, 2048 columns a side on 256 compute units, so that every tile
    is taken: both sides of 77 .. 2055 tokens 64 x 64, 64 x 128, 128 x 128, 128 x 256, 256 x 256; one side quantized of 77, 600,
    1030, 2055 and 4099 32 x 128, 64 x 128, 128 x 128, 128 x 256, 256 x 256.  Quantized: the bytes that the quantizer makes of
    the latents."""
    layer = synth.uniform_layer(2, 1, 1024)
    rng = np.random.default_rng(34)
    d, R = 256, 2048
    A = [synth.round_to(rng.standard_normal((d, R)) / np.sqrt(d), dtype) for _ in range(2)]
    x = synth.round_to(rng.standard_normal((n_tok, d)), dtype)
    xd, Ad = to_dev(x, dtype), [to_dev(a, dtype) for a in A]
    h = [torch.full((n_tok + 1, R), 7.0, dtype=xd.dtype, device="cuda") for _ in range(2)]
    P.palu_encode_kv(make_desc(layer, dtype), xd, *Ad, h[0], R, h[1], R)
    torch.cuda.synchronize()
    eps = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8                # the bound of test_encode_token_tiles
    for got, a in zip(h, A):
        g, ref = got.float().cpu().numpy(), x.astype(np.float32) @ a.astype(np.float32)
        assert (np.abs(g[:n_tok] - ref) - eps * np.abs(ref)).max() <= 1e-5 * np.abs(ref).max() and (g[n_tok] == 7.0).all()
    if n_tok != 290:
        q = [torch.full((n_tok + 1, R // 2), 0xA5, dtype=torch.uint8, device="cuda")] + [torch.full((n_tok + 1, R // 128), 7.0, dtype=torch.float16, device="cuda") for _ in range(2)]
        desc = P.LayerDesc(2, 128, layer.group_head_off, layer.k_rank_off, layer.v_rank_off, P.PALU_F16 if dtype == "f16" else P.PALU_BF16, quant_block=128)
        P.palu_encode_quant(desc, 0, xd, n_tok, Ad[0], *q)
        torch.cuda.synchronize()
        for got, ref in zip(q, O.quant_latent(h[0][:n_tok].float().cpu().numpy())):
            assert np.array_equal(got[:n_tok].cpu().numpy(), ref)
        assert (q[0][n_tok] == 0xA5).all() and (q[1][n_tok] == 7.0).all() and (q[2][n_tok] == 7.0).all()
    say(f"[edges] encode GEMM, tile by cost n_tok={n_tok} {dtype}")


@pytest.mark.parametrize("theta", [10000.0, 0.0])
@pytest.mark.parametrize("heads,group,rk,batch", [(4, 1, 64, 1), (16, 4, 64, 5), (20, 4, 128, 2), (28, 4, 256, 1), (3, 1, 96, 17), (2, 2, 512, 63)])
def test_step_with_few_columns(heads, group, rk, batch, theta):
    """A decode step whose query folds outnumber the projection's workgroups, in one launch with it or beside it: rows and
    outputs equal to the projection's and the attention's own calls."""
    layer = synth.uniform_layer(heads, group, rk, 64, rope_theta=theta)
    rng = np.random.default_rng(21)
    seq, d = 40, heads * 128
    draw = lambda *shape, by=1.0: to_dev(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    desc, x, q = make_desc(layer, "f16"), draw(batch, d), draw(batch, heads, 128)
    A = [draw(d, R, by=d ** -0.5) for R in (layer.R_k, layer.R_v)]
    caches = [draw(batch, seq, R) for R in (layer.R_k, layer.R_v)]
    B = [draw(layer.b_elems("k"), by=rk ** -0.5), draw(layer.b_elems("v"), by=64 ** -0.5)]
    rows = torch.arange(batch, dtype=torch.int32, device="cuda") * seq + seq - 1
    q_pos = torch.full((batch,), seq - 1, dtype=torch.int32, device="cuda")
    table = P.palu_rope_table_init(theta, 128, seq)
    step = [c.clone() for c in caches]
    got = P.palu_decode_step(desc, batch, seq, seq, x, *A, rows, q, q_pos, *step, *B, table, seq)
    P.palu_encode_kv(desc, x, *A, caches[0], layer.R_k, caches[1], layer.R_v, rows)
    ref = P.palu_attn_decode(desc, batch, seq, seq, q, q_pos, *caches, *B, table, seq)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(step, caches)) and torch.equal(got, ref)
    assert ref.abs().max() > 0
    say(f"[edges] step heads={heads} group={group} rank={rk} batch={batch} theta={theta}")


@pytest.mark.parametrize("batch,heads,group,rv,q_per_kv", [(31, 4, 4, 64, 1), (32, 4, 4, 96, 1), (33, 3, 1, 32, 2), (256, 4, 2, 64, 1), (257, 2, 2, 288, 3), (1, 256, 4, 32, 1)])
def test_merge_of_many_rows(batch, heads, group, rv, q_per_kv):
    """The merge kernels around their row counts (128 and 1024 rows; rows that do not fill a workgroup): outputs against the
    oracle, and the latent output times B_v against them."""
    layer = synth.uniform_layer(heads, group, 64, rv, q_per_kv=q_per_kv)
    rng = np.random.default_rng(8)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    seq = 130
    lens = np.array([(61 * i) % (seq + 1) for i in range(batch)], np.int32)
    lens[0] = seq
    case = synth.Case("edges", layer, "f16", batch, seq, draw(batch, layer.n_q_heads, 128), np.maximum(lens - 1, 0), draw(batch, seq, layer.R_k),
                      draw(batch, seq, layer.R_v), draw(layer.b_elems("k"), by=0.1), draw(layer.b_elems("v"), by=0.1))
    case.seq_lens = lens
    got, ref = run_hip(case), run_oracle(case)
    some = lens > 0
    err = max(rel_err(got[some], ref[some]))
    assert err <= TOL_FP and not got[~some].any()
    desc = make_desc(layer, "f16")
    table = P.palu_rope_table_init(layer.rope_theta, 128, seq)
    lat = P.palu_attn_decode_latent(desc, batch, seq, seq, to_dev(case.q, "f16"), torch.from_numpy(case.q_pos).cuda(), to_dev(case.Hk, "f16"),
                                    to_dev(case.Hv, "f16"), to_dev(case.Bk, "f16"), table, seq, seq_lens=torch.from_numpy(lens).cuda())
    torch.cuda.synchronize()
    z = lat.cpu().numpy().astype(np.float64).reshape(batch, layer.n_q_heads, rv)
    B = np.asarray(case.Bv, np.float64)
    out = np.empty((batch, layer.n_q_heads, 128))
    for h in range(layer.n_q_heads):
        kv = h // q_per_kv
        j, u = kv // group, kv % group
        Bj = B[j * rv * group * 128:(j + 1) * rv * group * 128].reshape(rv, group * 128)
        out[:, h] = z[:, h] @ Bj[:, u * 128:(u + 1) * 128]
    # float32 sums of at most 288 products on either side
    assert np.abs(out - got).max() <= 1e-5 * np.abs(out).max()
    say(f"[edges] merge rows={batch * layer.n_q_heads} rv={rv} q_per_kv={q_per_kv} rel err {err:.3e}")


@pytest.mark.parametrize("group,ranks,q_per_kv,dtype", [(4, [64, 32, 256, 320, 512, 1024], 1, "f16"), (1, [96, 32, 512, 2048, 64], 3, "bf16"), (5, [288, 64, 128, 224], 1, "f16"),
                                                        (3, [160, 512, 768], 2, "f16"), (2, [64, 64, 64, 128, 128, 96, 96], 1, "bf16"), (1, [64] * 7 + [32], 1, "f16")])
def test_score_weights_straight_from_b(group, ranks, q_per_kv, dtype):
    """Key weights that score workgroups transpose from B_k themselves: units of one, two and four groups, heads that do not fill
    a workgroup, ranks in one slice and in several, beside a rank of 32, which alone is laid out by the launch before."""
    layer = synth.ragged_layer(group * len(ranks), group, ranks, [64] * len(ranks), q_per_kv=q_per_kv)
    rng = np.random.default_rng(12)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, dtype)  # noqa: E731
    n = np.array([70, 1, 33], np.int32)
    Bk = np.concatenate([draw(r * group * 128, by=r ** -0.5) for r in ranks])
    case = synth.Case("edges", layer, dtype, 3, 70, draw(3, layer.n_q_heads, 128), n - 1, draw(3, 70, layer.R_k), draw(3, 70, layer.R_v), Bk,
                      draw(layer.b_elems("v"), by=64 ** -0.5))
    case.seq_lens = n
    err = max(rel_err(run_hip(case), run_oracle(case)))
    say(f"[edges] weights from B group={group} ranks={ranks} q_per_kv={q_per_kv} {dtype} rel err {err:.3e}")
    assert err <= TOL_FP


@pytest.mark.parametrize("rk,q_per_kv,dtype,bits", [(64, 4, "f16", 16), (96, 7, "bf16", 16), (64, 8, "f16", 16), (128, 5, "f16", 16), (160, 8, "bf16", 16), (256, 9, "f16", 16),
                                                    (128, 8, "f16", 4), (256, 8, "f16", 4)])
@pytest.mark.parametrize("flat", [False, True])
def test_query_products_on_matrix_cores(rk, q_per_kv, dtype, bits, flat):
    """Four queries and more of one key: every rank class with few matrix instructions to deal work out between, blocks of four
    queries with idle ones, a pass of one row behind one of eight; one run per sequence, and runs over the tiles of all
    sequences (FLAT); 4-bit keys with and without zero-points that need the float32 form."""
    layer = synth.uniform_layer(2, 2, rk, 128, q_per_kv=q_per_kv)
    rng = np.random.default_rng(3)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, dtype)  # noqa: E731
    seq = 330
    n = np.array([seq, 1, 16, 33, 177], np.int32)
    batch = len(n)
    case = synth.Case("edges", layer, dtype, batch, seq, draw(batch, layer.n_q_heads, 128), n + 5, draw(batch, seq, layer.R_k), draw(batch, seq, layer.R_v),
                      draw(layer.b_elems("k"), by=rk ** -0.5), draw(layer.b_elems("v"), by=128 ** -0.5))
    case.seq_lens = n
    quant = {}
    if bits == 4:
        quant = {"k": O.quant_latent(case.Hk), "v": O.quant_latent(case.Hv)}
        odd_zero_rows(case, quant, batch - 1, [(32, 0), (95, -1)])
    args = (bits == 4, bits == 4, quant)
    ref = run_oracle(case, args[2], *args[:2])
    P.palu_set_option("score_chunks", 3 if flat else 0)           # forced runs go through all sequences
    try:
        got = run_hip(case, *args)
    finally:
        P.palu_set_option("score_chunks", 0)
    err = max(rel_err(got, ref))
    say(f"[edges] query products rank={rk} q_per_kv={q_per_kv} {dtype} bits={bits} flat={flat} rel err {err:.3e}")
    assert err <= (TOL_I4 if bits == 4 else TOL_FP)


@pytest.mark.parametrize("group,ranks", [(1, [96] * 4), (1, [128] * 5), (1, [128, 128, 96, 96, 96, 32, 32]), (1, [256, 256, 160]), (2, [128] * 3), (2, [160] * 2),
                                         (2, [192] * 3), (2, [256, 256, 224, 224, 64, 64])])
@pytest.mark.parametrize("option", ["", "bf16", "score_waves 4", "score_waves 8", "score_fp8"])
def test_score_units_over_small_groups(group, ranks, option):
    """Groups of one and two heads, of which a workgroup takes two or four where their ranks fit the columns of its tile row
    (256 in the whole-head kernels, 512 in the general one), around those limits: equal neighbours that fit, fit in pairs only, or not at all."""
    layer = synth.ragged_layer(group * len(ranks), group, ranks, [64] * len(ranks))
    dtype = "bf16" if option == "bf16" else "f16"
    rng = np.random.default_rng(14)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, dtype)  # noqa: E731
    n = np.array([101, 17], np.int32)
    Bk = np.concatenate([draw(r * group * 128, by=r ** -0.5) for r in ranks])
    case = synth.Case("edges", layer, dtype, 2, 101, draw(2, layer.n_q_heads, 128), n - 1, draw(2, 101, layer.R_k), draw(2, 101, layer.R_v), Bk,
                      draw(layer.b_elems("v"), by=64 ** -0.5))
    case.seq_lens = n
    ref = run_oracle(case)
    if option == "score_fp8":                                     # ranks 64 .. 256 only
        ref8 = O.attn_decode_fp8_keys(case.q, case.q_pos, case.Hk, case.Hv, case.Bk, case.Bv, layer.group_head_off, layer.k_rank_off,
                                      layer.v_rank_off, layer.d_head, layer.rope_theta, case.k_pos, case.seq_lens, layer.q_per_kv)
        ref = np.where(np.repeat(np.array(ranks) >= 64, group)[None, :, None], ref8, ref)
    name, value = (option.split() + ["1"])[:2] if option.startswith("score") else ("score_waves", "0")
    P.palu_set_option(name, int(value))
    try:
        got = run_hip(case)
    finally:
        P.palu_set_option(name, 0)
    err = max(rel_err(got, ref))
    say(f"[edges] small groups group={group} ranks={ranks} {option} rel err {err:.3e}")
    assert err <= TOL_FP


def test_quantized_values_beside_one_dominant_token():
    """One cached row that outweighs each other one by exp(13.3), with a value of zero, over 65536 rows of one value: what the others add up to, a
    tenth of the weight, is the whole output.  Probability times scale is a 16-bit float against the running maximum of its split, so the rows that share
    the dominant one's split are below half its smallest step and lost: one split's share of the output, and the reason why
    splits of quantized values are kept short.  Eight units of four heads on 256 compute units: 288 rows or 0.44 % with eight
    wavefronts per compute unit (rows that share nothing with it are in one of the other splits)."""
    layer = synth.uniform_layer(32, 4, 128, 128, rope_theta=0.0)
    rng = np.random.default_rng(15)
    n, gap, scale, code = 65536, 13.3, 2.0 ** -6, 8
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    q, Bk, Bv = draw(1, 32, 128), draw(layer.b_elems("k"), by=128 ** -0.5), draw(layer.b_elems("v"), by=128 ** -0.5)
    Hk = np.zeros((1, n, layer.R_k))
    logits = np.empty(32)
    for j in range(8):
        fold = np.einsum("ruc,uc->ur", Bk[j * 65536:(j + 1) * 65536].reshape(128, 4, 128), q[0, 4 * j:4 * j + 4]) / np.sqrt(128)
        h = synth.round_to(np.linalg.lstsq(fold, np.full(4, gap), rcond=None)[0], "f16")
        Hk[0, 0, 128 * j:128 * j + 128] = h
        logits[4 * j:4 * j + 4] = fold @ h
    codes = torch.full((1, n, layer.R_v // 2), code * 17, dtype=torch.uint8, device="cuda")
    codes[0, 0] = 0
    hv_scale = torch.full((1, n, layer.R_v // 128), scale, dtype=torch.float16, device="cuda")
    table = P.palu_rope_table_init(0.0, 128, n)
    got = P.palu_attn_decode(make_desc(layer, "f16", v_i4=True), 1, n, n, to_dev(q, "f16"), torch.zeros(1, dtype=torch.int32, device="cuda"), to_dev(Hk, "f16"),
                             codes, to_dev(Bk, "f16"), to_dev(Bv, "f16"), table, n, hv_scale=hv_scale, hv_zero=torch.zeros_like(hv_scale))
    value = np.concatenate([Bv[j * 65536:(j + 1) * 65536].reshape(128, 4, 128).sum(0) for j in range(8)]) * code * scale
    ref = value * ((n - 1) / (n - 1 + np.exp(logits)))[:, None]
    err = max(rel_err(got.cpu().numpy(), ref[None]))
    say(f"[edges] dominant token: logits {logits.min():.3f} .. {logits.max():.3f}, rel err {err:.3e}")
    assert err <= TOL_I4


@pytest.mark.parametrize("waves", [0, 4, 8])
@pytest.mark.parametrize("ranks,bits", [([768, 1024], 16), ([512, 1024, 320], 16), ([1024], 4), ([2048, 128], 3)])
def test_rank_slices_with_every_schedule(ranks, bits, waves):
    """Ranks above 512, contracted in slices of 256 rows, under each schedule that option score_waves selects: as many score planes are
    summed as the slices write (one each where a wavefront has a whole head, two where it has half of one)."""
    layer = synth.ragged_layer(6 * len(ranks), 6, ranks, [128] * len(ranks))
    rng = np.random.default_rng(16)
    draw = lambda *shape, by=1.0: synth.round_to(rng.standard_normal(shape) * by, "f16")  # noqa: E731
    n = np.array([77, 32], np.int32)
    Bk = np.concatenate([draw(r * 6 * 128, by=r ** -0.5) for r in ranks])
    case = synth.Case("edges", layer, "f16", 2, 77, draw(2, layer.n_q_heads, 128), n - 1, draw(2, 77, layer.R_k), draw(2, 77, layer.R_v), Bk,
                      draw(layer.b_elems("v"), by=128 ** -0.5))
    case.seq_lens = n
    quant = {} if bits == 16 else {"k": O.quant_latent(case.Hk, bits=bits), "v": O.quant_latent(case.Hv, bits=bits)}
    ref = run_oracle(case, quant, bits != 16, bits != 16, bits=min(bits, 4))
    P.palu_set_option("score_waves", waves)
    try:
        got = run_hip(case, bits != 16, bits != 16, quant, bits=min(bits, 4))
    finally:
        P.palu_set_option("score_waves", 0)
    err = max(rel_err(got, ref))
    say(f"[edges] rank slices ranks={ranks} bits={bits} score_waves={waves} rel err {err:.3e}")
    assert err <= (TOL_FP if bits == 16 else TOL_I4)
