"""Performance cases of the THC hot path: what a program that uses this library has it do, over the sizes, data types
and options it is used with, through the public entry points of `paper_2302_08545_amd.api`.

Four kinds of use:
  round    all n workers' buffers on one GPU: thc_compress_all, thc_aggregate, thc_decompress
  worker   one worker's share of a round: its own norms (thc_prepare_range over its one gradient), thc_compress with
           the agreed range, thc_decompress of the sums that come back
  server   the parameter server's share: thc_aggregate of n packed streams
  uniform  a round of the paper's simplified variant (Alg. 1), with or without the rotation

A case is a dict of plain values; `blocks` RHT blocks of 2^log2_block coordinates make a vector, of which the first
`real` carry data and the rest is the caller's zero padding.
"""
from __future__ import annotations

import math

import torch

from paper_2302_08545_amd import api

DEV = "cuda:0"
RHT_SEED = 0x5448435F53454544
ASCENDING, SPLIT = api.THC_ORDER_ASCENDING, api.THC_ORDER_SPLIT


def _case(kind, blocks, log2_block, n, b=4, g=30, agg_bits=8, dtype="f32", ef=False, order=SPLIT, values="gauss",
          p=1.0 / 32, rotate=False, real=0):
    d = blocks << log2_block
    return {"kind": kind, "blocks": blocks, "log2_block": log2_block, "n": n, "b": b, "g": g, "agg_bits": agg_bits,
            "dtype": dtype, "ef": ef, "order": order, "values": values, "p": p, "rotate": rotate,
            "real": min(real, d) if real else d}


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)

    return [
        # a small bucket with the binding's default stage order: a handful of microsecond-sized launches
        named("bucket_2p15", "round", 2, 14, 4, order=ASCENDING),
        # one 4 MB partition, the paper's unit of compression, four workers
        named("partition_2p20", "round", 1, 20, 4),
        # ResNet-50-shaped gradient as one 2^25-point transform, error feedback: more passes than any other block size
        named("resnet50_ef", "round", 1, 25, 8, ef=True, values="laplace", real=25_557_032),
        # VGG16-shaped gradient, eight workers: the headline configuration
        named("vgg16", "round", 256, 20, 8, values="two_scales", real=138_357_544),
        # BERT-large-shaped gradient, sixteen workers, outliers, 16-bit sums: the largest call
        named("bert_large_b4", "round", 321, 20, 16, agg_bits=16, values="outliers", real=336_000_000),
        # 2-bit indices on a part of the same vector (an odd number of blocks)
        named("bert_b2_41_blocks", "round", 41, 20, 16, b=2, g=8, values="outliers"),
        # GPT-2-XL-shaped prefix: bf16 gradients, blocks of 2^22, 32 workers, error feedback
        named("gpt2_xl_16_blocks_ef", "round", 16, 22, 32, agg_bits=16, dtype="bf16", ef=True, values="student_t"),
        # what one of eight workers does in a round, bf16 gradient padded to whole partitions, error feedback
        named("worker_bf16_ef", "worker", 25, 20, 8, dtype="bf16", ef=True, values="laplace", real=25_557_032),
        # parameter server, sixteen streams, sums at their exact width of 9 bits
        named("server_n16_w9", "server", 33, 20, 16, agg_bits=9),
        # Alg. 1 without rotation, error feedback
        named("uniform_ef", "uniform", 25, 20, 8, g=15, ef=True, values="laplace", real=25_557_032),
        # Alg. 1 on the rotated vectors (the ablation's "with rotation" arm)
        named("uniform_rotated", "uniform", 25, 20, 4, g=15, rotate=True),
        # one point of the NMSE-against-granularity sweep: 3-bit indices, ten workers, exact-width sums
        named("sweep_b3_g31", "round", 1, 20, 10, b=3, g=31, agg_bits=9, order=ASCENDING, values="lognormal",
              p=1.0 / 1024),
    ]


def draw(rng):
    kind = rng.choices(("round", "worker", "server", "uniform"), (5, 2, 1, 2))[0]
    n = rng.choice((1, 2, 3, 4, 5, 7, 8, 8, 8, 10, 12, 16, 16, 24, 32))
    b = rng.choice((1, 2, 2, 3, 4, 4, 4, 4, 4, 4, 8)) if kind != "uniform" else rng.choice((2, 3, 4, 4, 4))
    g = (1 << b) - 1
    if kind != "uniform" and b < 8:
        g = rng.choice((g, {1: 1, 2: 8, 3: 21, 4: 30}[b], {1: 1, 2: 8, 3: 31, 4: 30}[b], rng.randint(g, 51)))
    exact = max(1, (g * n).bit_length())
    agg_bits = exact if rng.random() < 0.25 else (8 if exact <= 8 else 16)
    log2_block = rng.choice((10, 12, 13, 14, 15, 16, 17, 18, 19, 20, 20, 20, 20, 20, 21, 22, 23, 25))
    ef = kind != "server" and rng.random() < 0.35
    # worker-coordinates of the call, spread over their logarithm from one small bucket to a large model's gradient
    vectors = 1 if kind == "worker" else n
    hi = {"round": 30.5, "worker": 28.5, "server": 31.0, "uniform": 29.5}[kind] - (1.5 if ef else 0.0)
    total = 2.0 ** rng.uniform(15.0, hi)
    blocks = min(int(total / vectors) >> log2_block, 1 << 15)
    while blocks == 0 and log2_block > 10 and vectors << log2_block > 2.0 ** hi:
        log2_block -= 1
    blocks = max(1, blocks)
    d = blocks << log2_block
    real = d if rng.random() < 0.5 else d - rng.randrange(1 << log2_block)
    return _case(kind, blocks, log2_block, n, b, g, agg_bits, rng.choice(("f32", "f32", "bf16")), ef,
                 rng.choice((ASCENDING, SPLIT, SPLIT)),
                 rng.choice(("gauss", "laplace", "two_scales", "outliers", "student_t", "lognormal")),
                 rng.choice((1.0 / 32, 1.0 / 32, 1.0 / 512)), kind == "uniform" and rng.random() < 0.5, real)


def _fill(x, kind, gen):
    """One worker's data into x (binary32), in pieces so that temporaries stay small."""
    for pos in range(0, x.numel(), 1 << 26):
        v = x[pos:pos + (1 << 26)]
        v.normal_(generator=gen)
        if kind == "gauss":
            v.mul_(1e-3)
        elif kind == "two_scales":           # most coordinates in one layer of a tenth of the scale
            v.mul_(1e-3)
            v[v.numel() // 10:v.numel() * 8 // 10].mul_(0.1)
        elif kind == "outliers":             # 0.1 % of the coordinates at fifty times the scale
            v.mul_(1e-3)
            at = torch.randint(0, v.numel(), (max(1, v.numel() // 1000),), generator=gen, device=v.device)
            v[at] *= 50.0
        elif kind == "student_t":            # three degrees of freedom
            chi = torch.zeros_like(v)
            for _ in range(3):
                chi += torch.empty_like(v).normal_(generator=gen).square_()
            v.div_(chi.div_(3.0).sqrt_()).mul_(1e-3)
        elif kind == "lognormal":
            v.exp_()
        elif kind == "laplace":              # product of a normal and a Rayleigh draw; layers of different scales
            r = torch.empty_like(v).exponential_(generator=gen)
            v.mul_(r.mul_(2.0).sqrt_()).mul_(1e-3)
            for k in range(8):
                v[v.numel() * k // 8:v.numel() * (k + 1) // 8].mul_(10.0 ** (-1.5 + 3.0 * ((5 * k) % 8) / 7.0))
        else:
            raise ValueError(kind)


def prepare(case, seed):
    kind, n, b, agg_bits = case["kind"], case["n"], case["b"], case["agg_bits"]
    d = case["blocks"] << case["log2_block"]
    gen = torch.Generator(device=DEV).manual_seed(seed)
    if kind == "uniform":
        table, t_p = list(range(1 << b)), 1.0
    else:
        table = list(range(1 << b)) if case["g"] == (1 << b) - 1 else api.thc_solve_table(b, case["g"], case["p"])[0]
        t_p = api.thc_threshold(case["p"])
    dtype = api.THC_DTYPE_BF16 if case["dtype"] == "bf16" else api.THC_DTYPE_F32

    def params(workers, bits):
        return api.make_params(d, 1 << case["log2_block"], workers, b, case["g"], t_p, RHT_SEED, table, bits, dtype,
                               case["order"])

    P = params(n, agg_bits)
    s = {"case": case, "P": P, "round": seed & 0xFFFF}
    W = 1 if kind == "worker" else n
    packed = torch.empty((W, d * b // 8), dtype=torch.uint8, device=DEV)
    agg = torch.empty(d * agg_bits // 8, dtype=torch.uint8, device=DEV)
    s.update(packed=packed, packed_list=list(packed.unbind(0)), agg=agg)
    if kind == "server":
        packed.random_(0, 256, generator=gen)
        return s

    grads = []
    x = torch.zeros(d, dtype=torch.float32, device=DEV)
    for i in range(W):
        _fill(x[:case["real"]], case["values"], gen)
        if case["values"] == "lognormal" and i:
            grads.append(grads[0])           # the sweep gives every worker the same gradient
        else:
            grads.append(x.to(torch.bfloat16) if case["dtype"] == "bf16" else x.clone())
    del x
    ef = torch.zeros((W, d), dtype=torch.float32, device=DEV) if case["ef"] else None
    s.update(grads=grads, ef=ef, ef_list=list(ef.unbind(0)) if ef is not None else None)
    s["range_M"] = torch.empty(case["blocks"], dtype=torch.float32, device=DEV)
    s["out"] = torch.empty(d, dtype=torch.float32, device=DEV)
    if kind == "uniform":
        s["range_m"] = torch.empty(case["blocks"], dtype=torch.float32, device=DEV)
        need = api.thc_uniform_workspace_bytes(P, case["rotate"])
    else:
        need = api.thc_workspace_bytes(P, case["ef"])
    if kind == "worker":
        # the worker's own norm, from a call that knows of one worker, and the sums the server sent back
        s["P1"] = params(1, 8 if case["g"] < 256 else 16)
        need = max(need, api.thc_workspace_bytes(s["P1"], case["ef"]))
        if agg_bits in (8, 16):
            agg.view(torch.uint8 if agg_bits == 8 else torch.int16).random_(
                0, min(case["g"] * n + 1, 1 << (8 if agg_bits == 8 else 15)), generator=gen)
        else:
            agg.random_(0, 256, generator=gen)
    s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    return s


def run(s):
    case, P, kind = s["case"], s["P"], s["case"]["kind"]
    if kind == "server":
        api.thc_aggregate(P, s["packed_list"], s["agg"])
        return {"agg": s["agg"]}
    s["round"] += 1                          # every round has its own diagonal and rounding draws
    rnd, ef, M, ws = s["round"], s["ef_list"], s["range_M"], s["ws"]
    if kind == "round":
        api.thc_compress_all(P, rnd, s["grads"], ef, M, s["packed_list"], ws)
        api.thc_aggregate(P, s["packed_list"], s["agg"])
        api.thc_decompress(P, rnd, s["agg"], M, s["out"], ws)
    elif kind == "worker":
        api.thc_prepare_range(s["P1"], s["grads"], ef, M, ws)
        api.thc_compress(P, 0, rnd, s["grads"][0], ef[0] if ef else None, M, s["packed_list"][0], ws)
        api.thc_decompress(P, rnd, s["agg"], M, s["out"], ws)
    else:
        m, rot = s["range_m"], case["rotate"]
        api.thc_uniform_prepare_range(P, rnd, s["grads"], ef, rot, m, M, ws)
        for i in range(case["n"]):
            api.thc_uniform_compress(P, i, rnd, s["grads"][i], ef[i] if ef else None, rot, m, M, s["packed_list"][i], ws)
        api.thc_aggregate(P, s["packed_list"], s["agg"])
        api.thc_uniform_decompress(P, rnd, s["agg"], rot, m, M, s["out"], ws)
    outs = {"packed": s["packed"], "range_M": M, "out": s["out"]}
    if kind != "worker":
        outs["agg"] = s["agg"]
    if kind == "uniform":
        outs["range_m"] = s["range_m"]
    if ef:
        outs["ef"] = s["ef"]
    return outs


def work(case):
    """Every datum once: gradients (and error-feedback buffers) in, packed streams out and in, sums out and in, the
    estimate out; one addition per coordinate and butterfly stage of every transform."""
    d = case["blocks"] << case["log2_block"]
    b, w, L = case["b"], case["agg_bits"], case["log2_block"]
    in_b = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "server":
        return {"bytes": d * (case["n"] * b + w) / 8, "flops": d * case["n"]}
    W = 1 if case["kind"] == "worker" else case["n"]
    per_worker = in_b + (8 if case["ef"] else 0) + b / 8
    per_coord = W * per_worker + w / 8 + 4
    if case["kind"] != "worker":
        per_coord += (W * b + w) / 8
    transforms = (W * (2 if case["ef"] else 1) + 1) if case["kind"] != "uniform" or case["rotate"] else 0
    return {"bytes": d * per_coord, "flops": d * (transforms * L + 2 * W)}


def tolerance(case):
    """Indices and sums are reproducible (draws, stage order and rounding are fixed): at most one in a million may sit
    within an ulp of a threshold.  Floats are binary32 sums of up to 2^25 terms in a fixed order."""
    return {"rel": 1e-5, "differ": 1e-6}
