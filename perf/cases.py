"""The work a serving program gives this library, as a list of timed cases.

A case is one pass through the public entry points on one compressed attention layer:

  step     one decode step of `batch` sequences: append the new token to both latent caches, then attend
           (one call where the caches are unquantized; encode, quantize, attend where they are not)
  multi    several query tokens per sequence over rows that are already cached (a speculative-decoding check,
           a chunk of a prompt): palu_attn_decode_multi with a causal block
  prompt   the projection of a prompt, or of a chunk of one, into both caches (palu_encode_kv), quantized as it
           is stored where the caches are (palu_encode_quant per side)

Layers are those of the benchmark and the tests: groups of 1, 4 or 32 heads, ranks of 64 .. 2048 per group, equal or
different from group to group, multi-head and grouped-query, with and without RoPE, fp16, bf16 and 4 / 3 / 2-bit
latents.  Inputs follow the decomposition's statistics: activations and queries N(0, 1), A and B scaled so that latents
and rebuilt keys are of order one with the channels of a group falling off in size like the singular values they carry.
"""

import torch

import paper_2407_21118_amd as P
from workloads import synth

D_HEAD = 128


def _case(name, kind, heads=32, group=4, rk=256, rv=256, q_per_kv=1, theta=10000.0, dtype="f16", k_bits=16, v_bits=16,
          batch=1, seq=1, n_q=1, ragged=False, rank_seed=-1):
    """One case as plain values.  heads: key/value heads; group: of them per group; rk, rv: rank per group (with
    rank_seed >= 0: mean rank, the groups' ranks drawn like a rank search's); seq: rows attended (prompt: tokens);
    ragged: the sequences of the batch have different lengths, seq being the longest."""
    c = dict(kind=kind, heads=heads, group=group, rk=rk, rv=rv, q_per_kv=q_per_kv, theta=theta, dtype=dtype,
             k_bits=k_bits, v_bits=v_bits, batch=batch, seq=seq, n_q=n_q, ragged=ragged, rank_seed=rank_seed)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one short chat turn on a small layer; launches and host time are what it costs
        _case("step-small-1x1k", "step", heads=8, rk=128, rv=128, seq=1024),
        # the ordinary case: one sequence, 7B shape, half the cache size
        _case("step-1x16k", "step", seq=16384),
        # one long document, bfloat16
        _case("step-1x64k-bf16", "step", dtype="bf16", seq=65536),
        # a serving batch of many short sequences of different lengths
        _case("step-48x2k-ragged", "step", batch=48, seq=2043, ragged=True),
        # ranks found by a search: every group has its own
        _case("step-4x16k-ranks", "step", batch=4, seq=16384, rank_seed=0),
        # grouped-query model: four query heads share each key/value head
        _case("step-gqa-4x16k", "step", heads=8, q_per_kv=4, theta=500000.0, batch=4, seq=16384),
        # the quantized cache of a serving batch
        _case("step-q4-16x8k", "step", k_bits=4, v_bits=4, batch=16, seq=8192),
        # attention without rotation over a long quantized cache: pure latent streaming
        _case("step-norope-q4-1x64k", "step", theta=0.0, k_bits=4, v_bits=4, seq=65536),
        # one latent per head (no grouping), low rank
        _case("step-per-head-8x16k", "step", group=1, rk=64, rv=64, batch=8, seq=16384, ragged=True),
        # a speculative-decoding check of four tokens on the 75 % / 25 % allocation of keys and values
        _case("multi4-2x8k", "multi", rk=128, rv=384, batch=2, seq=8190, n_q=4),
        # filling the caches from a prompt
        _case("prompt-4096-bf16", "prompt", dtype="bf16", seq=4096),
        # a chunk of a prompt into a quantized cache
        _case("prompt-q4-500", "prompt", k_bits=4, v_bits=4, seq=500),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi], odd ones among them."""
    return int(round(lo * (hi / lo) ** rng.random()))


# what one drawn case may ask for: no more than the largest listed one (step-q4-16x8k and its reconstruction)
_MAX_FLOPS = 2.7e11
_MAX_BYTES = 7.0e8


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "multi", "prompt", "prompt"])
    quant = rng.random() < 0.35
    bits = rng.choice([4, 4, 4, 3, 2]) if kind != "prompt" else 4
    k_bits, v_bits = (rng.choice([(bits, bits), (bits, bits), (16, bits)]) if quant else (16, 16))
    if kind == "prompt" and quant:
        k_bits = v_bits = 4
    q_per_kv = rng.choice([1, 1, 1, 4])
    heads = {1: rng.choice([8, 32, 32]), 4: 8}[q_per_kv]
    group = rng.choice([1, 2, 4, 4, 4, 8, 32])
    group = min(group, heads)
    per_head = rng.choice([32, 64, 64, 96])                         # rank per head and side, i.e. 25 %, 50 % or 75 % kept
    unit = 128 if quant else 32
    rk = max(unit, min(2048, per_head * group) // unit * unit, 64)
    rv = max(unit, min(2048, rng.choice([32, 64, 96]) * group) // unit * unit, 64)
    if max(rk, rv) > 512:                                           # whole slices
        rk, rv = max(256, rk // 256 * 256), max(256, rv // 256 * 256)
    rank_seed = rng.randrange(8) if (not quant and q_per_kv == 1 and heads == 32 and group == 4 and rng.random() < 0.3) else -1
    if rank_seed >= 0:
        rk = rv = 256
    theta = rng.choice([10000.0, 10000.0, 10000.0, 500000.0, 0.0])
    dtype = rng.choice(["f16", "f16", "bf16"]) if not quant else "f16"
    n_q = rng.choice([2, 3, 4, 5, 8]) if kind == "multi" else 1
    while heads * q_per_kv * n_q > 256:
        n_q -= 1
    if kind == "prompt":
        batch, seq = 1, _log_int(rng, 64, 8192)
    else:
        batch, seq = _log_int(rng, 1, 48), _log_int(rng, 512, 65536)
    c = _case("", kind, heads, group, rk, rv, q_per_kv, theta, dtype, k_bits, v_bits, batch, seq, n_q,
              batch > 1 and rng.random() < 0.5, rank_seed)
    while True:
        w = work(c)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES:
            return c
        if c["batch"] > 4:
            c["batch"] = c["batch"] * 3 // 4
        else:
            c["seq"] = c["seq"] * 3 // 4


# ------------------------------------------------------------------ shapes

def _layer(c):
    if c["rank_seed"] >= 0:
        n_groups = c["heads"] // c["group"]
        return synth.ragged_layer(c["heads"], c["group"], synth.draw_ranks(c["rank_seed"], 0, n_groups, c["rk"] * n_groups),
                                  synth.draw_ranks(c["rank_seed"], 1, n_groups, c["rv"] * n_groups), rope_theta=c["theta"],
                                  q_per_kv=c["q_per_kv"])
    return synth.uniform_layer(c["heads"], c["group"], c["rk"], c["rv"], rope_theta=c["theta"], q_per_kv=c["q_per_kv"])


def _lens(c):
    """Rows attended per sequence: all of seq, or between half of it and all of it in no particular order."""
    if not c["ragged"]:
        return [c["seq"]] * c["batch"]
    return [c["seq"] - (977 * i) % max(1, c["seq"] // 2) for i in range(c["batch"])]


def _groups(layer):
    """(heads, key rank, value rank) of every group."""
    return [(layer.group_size(j), int(layer.k_rank_off[j + 1] - layer.k_rank_off[j]), int(layer.v_rank_off[j + 1] - layer.v_rank_off[j]))
            for j in range(layer.n_groups)]


def work(c):
    layer = _layer(c)
    d = layer.n_q_heads * D_HEAD
    Rk, Rv = int(layer.R_k), int(layer.R_v)

    def row_bytes(R, bits):
        return R * 2 if bits == 16 else R * bits // 8 + R // 128 * 4

    weights = 2 * d * (Rk + Rv)
    if c["kind"] == "prompt":
        n = c["seq"]
        return {"bytes": 2 * n * d + weights + n * (row_bytes(Rk, c["k_bits"]) + row_bytes(Rv, c["v_bits"])),
                "flops": 2.0 * n * d * (Rk + Rv)}
    T, nq, qpk = sum(_lens(c)), c["n_q"], c["q_per_kv"]
    rows = c["batch"] * nq
    by = T * (row_bytes(Rk, c["k_bits"]) + row_bytes(Rv, c["v_bits"])) + 2 * int(layer.b_elems("k") + layer.b_elems("v"))
    by += rows * d * (2 + 4)                                        # queries in, outputs out
    fl = 0.0
    for s, rk, rv in _groups(layer):
        if c["theta"] > 0:
            fl += 2.0 * T * s * D_HEAD * (rk + qpk * nq)            # keys rebuilt once, each multiplied by its queries
        else:
            fl += 2.0 * s * qpk * nq * rk * (T + c["batch"] * D_HEAD)
        fl += 2.0 * s * qpk * nq * rv * (T + c["batch"] * D_HEAD)
    if c["kind"] == "step":
        by += weights + c["batch"] * 2 * d + c["batch"] * (row_bytes(Rk, c["k_bits"]) + row_bytes(Rv, c["v_bits"]))
        fl += 2.0 * c["batch"] * d * (Rk + Rv)
    return {"bytes": by, "flops": fl}


def tolerance(c):
    """About four times the largest error seen against the same passes in 64-bit arithmetic (2-norm, listed cases):
    2.1e-4 for fp16 rows and for attention over unquantized latents (probabilities and new rows are rounded to fp16),
    1.75e-3 for bf16 rows, 4.6e-4 for attention over 4-bit latents.  Quantized prompts: 4e-6 of the code bytes and no
    zero-point differed; but a latent whose rounding flips at a tie can move the zero-point of its block by one, i.e.
    1 / 8 of it and all of the block's codes, so one such block is allowed for."""
    if c["kind"] == "prompt":
        if c["k_bits"] != 16:
            layer = _layer(c)
            blocks = c["seq"] * (int(min(layer.R_k, layer.R_v)) // 128)
            return {"rel": max(1e-4, 0.2 / blocks ** 0.5), "max": 0.2, "differ": max(2e-5, 1.5 / blocks)}
        return {"rel": 8e-4 if c["dtype"] == "f16" else 7e-3}
    if c["k_bits"] != 16 or c["v_bits"] != 16:
        return {"rel": 2e-3, "max": 0.15, "differ": 1e-4}
    return {"rel": 8e-4 if c["dtype"] == "f16" else 7e-3}


# ------------------------------------------------------------------ inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + stream)
    return g


def _randn(shape, g, dtype, scale=1.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale).to(dtype)


def _channel_scale(ranks):
    """Sizes of the latent channels of every group, largest first (mean square 1)."""
    out = []
    for r in ranks:
        s = torch.linspace(1.4, 0.6, r, device="cuda")
        out.append(s / s.square().mean().sqrt())
    return torch.cat(out)


def _quantized(layer, desc, side, H, bits):
    """A quantized cache side from unquantized latents, by the library's own quantizer."""
    batch, seq, R = H.shape
    codes = torch.empty((batch, seq, R * bits // 8), dtype=torch.uint8, device="cuda")
    scale = torch.empty((batch, seq, R // 128), dtype=torch.float16, device="cuda")
    zero = torch.empty_like(scale)
    P.palu_quant_latent(desc, side, H, R, batch * seq, codes, scale, zero)
    return codes, scale, zero


def prepare(c, seed):
    layer = _layer(c)
    td = torch.float16 if c["dtype"] == "f16" else torch.bfloat16
    act = P.PALU_F16 if c["dtype"] == "f16" else P.PALU_BF16
    lat = {16: act, 4: P.PALU_I4, 3: P.PALU_I3, 2: P.PALU_I2}
    desc = P.LayerDesc(layer.n_heads, D_HEAD, layer.group_head_off, layer.k_rank_off, layer.v_rank_off, act,
                       lat[c["k_bits"]], lat[c["v_bits"]], 128, layer.rope_theta, layer.q_per_kv)
    d, batch, seq, kind = layer.n_q_heads * D_HEAD, c["batch"], c["seq"], c["kind"]
    groups = _groups(layer)
    sk, sv = _channel_scale([g[1] for g in groups]), _channel_scale([g[2] for g in groups])
    s = dict(case=c, layer=layer, desc=desc)

    # projections: latents of N(0, 1) activations have the channel scales
    Ak = _randn((d, layer.R_k), _gen(seed, 1), torch.float32, d ** -0.5).mul_(sk).to(td)
    Av = _randn((d, layer.R_v), _gen(seed, 2), torch.float32, d ** -0.5).mul_(sv).to(td)
    if kind == "prompt":
        s.update(Ak=Ak, Av=Av, x=_randn((seq, d), _gen(seed, 3), td))
        if c["k_bits"] == 16:
            s.update(hk=torch.zeros((seq, layer.R_k), dtype=td, device="cuda"),
                     hv=torch.zeros((seq, layer.R_v), dtype=td, device="cuda"),
                     ws_e=torch.empty(P.palu_encode_workspace_bytes(desc, 2, seq), dtype=torch.uint8, device="cuda"))
        else:
            for side, R in (("k", layer.R_k), ("v", layer.R_v)):
                s["q" + side] = (torch.zeros((seq, R // 2), dtype=torch.uint8, device="cuda"),
                                 torch.zeros((seq, R // 128), dtype=torch.float16, device="cuda"),
                                 torch.zeros((seq, R // 128), dtype=torch.float16, device="cuda"))
        return s

    # reconstruction matrices, rows in the order of the channels (rebuilt keys and values of order one)
    def recon(which, stream, scales):
        parts, at = [], 0
        for size, rk, rv in groups:
            r = rk if which == "k" else rv
            parts.append(_randn((r, size * D_HEAD), _gen(seed, stream + at), torch.float32, r ** -0.5)
                         .mul_(scales[at:at + r, None]).to(td).reshape(-1))
            at += r
        return torch.cat(parts)

    s.update(Bk=recon("k", 10000, sk), Bv=recon("v", 20000, sv))
    Hk = _randn((batch, seq, layer.R_k), _gen(seed, 4), td).mul_(sk.to(td))
    Hv = _randn((batch, seq, layer.R_v), _gen(seed, 5), td).mul_(sv.to(td))
    s["quant"] = {}
    if c["k_bits"] != 16:
        Hk, s["quant"]["hk_scale"], s["quant"]["hk_zero"] = _quantized(layer, desc, 0, Hk, c["k_bits"])
    if c["v_bits"] != 16:
        Hv, s["quant"]["hv_scale"], s["quant"]["hv_zero"] = _quantized(layer, desc, 1, Hv, c["v_bits"])
    lens = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
    n_q = c["n_q"]
    s.update(hk=Hk, hv=Hv, seq_lens=lens if c["ragged"] else None,
             table=P.palu_rope_table_init(layer.rope_theta, D_HEAD, seq))
    if kind == "multi":
        # the n_q query tokens are the last rows of the cache: a causal block
        q_len = (lens[:, None] - n_q + 1 + torch.arange(n_q, dtype=torch.int32, device="cuda")[None]).contiguous()
        s.update(q=_randn((batch, n_q, layer.n_q_heads, D_HEAD), _gen(seed, 6), td), q_len=q_len,
                 q_pos=(q_len - 1).contiguous(),
                 out=torch.empty((batch, n_q, layer.n_q_heads, D_HEAD), dtype=torch.float32, device="cuda"))
        return s
    s.update(q=_randn((batch, layer.n_q_heads, D_HEAD), _gen(seed, 6), td), q_pos=lens - 1,
             x=_randn((batch, d), _gen(seed, 7), td),
             dst_row=(torch.arange(batch, dtype=torch.int32, device="cuda") * seq + lens - 1).contiguous(),
             out=torch.empty((batch, layer.n_q_heads, D_HEAD), dtype=torch.float32, device="cuda"),
             ws=torch.empty(P.palu_attn_decode_workspace_bytes(desc, batch, seq), dtype=torch.uint8, device="cuda"))
    if not s["quant"] and batch <= 2:
        s.update(Akt=Ak.t().contiguous(), Avt=Av.t().contiguous())
    else:
        s.update(Ak=Ak, Av=Av, ws_e=torch.empty(P.palu_encode_workspace_bytes(desc, 2, batch), dtype=torch.uint8, device="cuda"),
                 new_k=torch.empty((batch, layer.R_k), dtype=td, device="cuda"),
                 new_v=torch.empty((batch, layer.R_v), dtype=td, device="cuda"))
    return s


def run(s):
    c, desc, layer = s["case"], s["desc"], s["layer"]
    if c["kind"] == "prompt":
        if c["k_bits"] == 16:
            P.palu_encode_kv(desc, s["x"], s["Ak"], s["Av"], s["hk"], layer.R_k, s["hv"], layer.R_v, None, s["ws_e"])
            return [s["hk"], s["hv"]]
        P.palu_encode_quant(desc, 0, s["x"], c["seq"], s["Ak"], *s["qk"])
        P.palu_encode_quant(desc, 1, s["x"], c["seq"], s["Av"], *s["qv"])
        return [*s["qk"], *s["qv"]]
    batch, seq = c["batch"], c["seq"]
    if c["kind"] == "multi":
        P.palu_attn_decode_multi(desc, batch, c["n_q"], seq, seq, s["q"], s["q_pos"], s["hk"], s["hv"], s["Bk"], s["Bv"],
                                 s["table"], seq, q_len=s["q_len"], out=s["out"], seq_lens=s["seq_lens"], **s["quant"])
        return s["out"]
    if "Akt" in s:
        P.palu_decode_step_t(desc, batch, seq, seq, s["x"], s["Akt"], s["Avt"], s["dst_row"], s["q"], s["q_pos"], s["hk"],
                             s["hv"], s["Bk"], s["Bv"], s["table"], seq, out=s["out"], workspace=s["ws"],
                             seq_lens=s["seq_lens"])
    elif not s["quant"]:
        P.palu_decode_step(desc, batch, seq, seq, s["x"], s["Ak"], s["Av"], s["dst_row"], s["q"], s["q_pos"], s["hk"],
                           s["hv"], s["Bk"], s["Bv"], s["table"], seq, out=s["out"], workspace=s["ws"],
                           encode_workspace=s["ws_e"], seq_lens=s["seq_lens"])
    else:
        # quantized caches: project, quantize the new rows into place, attend
        if c["k_bits"] != 16:
            P.palu_encode_kv(desc, s["x"], s["Ak"], s["Av"], s["new_k"], layer.R_k, s["new_v"], layer.R_v, None, s["ws_e"])
            P.palu_quant_latent(desc, 0, s["new_k"], layer.R_k, batch, s["hk"], s["quant"]["hk_scale"],
                                s["quant"]["hk_zero"], s["dst_row"])
        else:
            P.palu_encode(desc, 0, s["x"], s["Ak"], s["hk"], layer.R_k, s["dst_row"], s["ws_e"])
            P.palu_encode(desc, 1, s["x"], s["Av"], s["new_v"], layer.R_v, None, s["ws_e"])
        P.palu_quant_latent(desc, 1, s["new_v"], layer.R_v, batch, s["hv"], s["quant"]["hv_scale"],
                            s["quant"]["hv_zero"], s["dst_row"])
        P.palu_attn_decode(desc, batch, seq, seq, s["q"], s["q_pos"], s["hk"], s["hv"], s["Bk"], s["Bv"], s["table"], seq,
                           out=s["out"], workspace=s["ws"], seq_lens=s["seq_lens"], **s["quant"])
    return [s["out"], s["hk"], s["hv"], *s["quant"].values()]
