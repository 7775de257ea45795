"""Kernel variants and dispatch branches at the sizes where they can go wrong, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import thc_oracle as o
from paper_2302_08545_amd import api

from .test_gpu_parity import DEV, GpuRound, assert_indices_match, both_params, make_grads, rel_l2, to_np32

pytestmark = pytest.mark.gpu


def _round_against_oracle(P, L, R, grads, rnd, efs=None):
    """compress_all, aggregate, decompress; the oracle works from the range the GPU computed."""
    n, b = L.n, L.b
    dg = [x.to(DEV) for x in grads]
    gn = [to_np32(x) for x in grads]
    R.compress_all(rnd, dg)
    R.aggregate()
    R.decompress(rnd)
    M_ref, M = o.prepare_range(P, gn, efs), R.range_M.cpu().numpy()
    assert np.all(np.abs(M - M_ref) <= np.abs(M_ref) * 2.0 ** -23)
    pks = []
    for i in range(n):
        pk, ne = o.compress(P, i, rnd, gn[i], None if efs is None else efs[i], M)
        assert_indices_match(R.packed[i].cpu().numpy(), pk, b, f"worker {i}")
        if efs is not None:
            assert rel_l2(R.efs[i].cpu().numpy(), ne) <= 1e-5, f"worker {i}"
        pks.append(R.packed[i].cpu().numpy())
    Y = o.aggregate(P, pks)
    assert np.array_equal(R.agg_numpy(), Y)
    assert rel_l2(R.out.cpu().numpy(), o.decompress(P, rnd, Y, M)) <= 1e-5


@pytest.mark.parametrize("b,g", [(1, 1), (1, 255), (2, 8), (4, 30), (4, 100), (4, 128), (7, 200), (8, 255)])
@pytest.mark.parametrize("log2_block", [10, 13])
def test_clamped_coordinates_end_in_the_outer_indices(b, g, log2_block):
    """Ranges far inside the data: a third of the coordinates lie outside.  The fast form of the quantizer has no clamp
    and is taken per block only where the top index is certain for whatever lies above the range."""
    block, K = 1 << log2_block, 24
    T = o.solve_table(b, g, 1 / 32) if g < 100 else [round(i * g / ((1 << b) - 1)) for i in range(1 << b)]
    P, L = both_params(block * K, block, 1, b=b, g=g, agg_bits=8, table=T)
    x = make_grads(block * K, 1, seed=b * 256 + g)
    M = (np.random.default_rng(g).uniform(0.5, 1.5, K) * 1e-3).astype(np.float32)
    R = GpuRound(L)
    R.compress_each(5, [x[0].to(DEV)], range_M=torch.from_numpy(M).to(DEV))
    assert_indices_match(R.packed[0].cpu().numpy(), o.compress(P, 0, 5, to_np32(x[0]), None, M)[0], b)


@pytest.mark.parametrize("log2_block,K,n,b,g,agg_bits,bf16,ef,order", [
    (22, 64, 1, 4, 30, 8, False, False, 1),      # just enough tiles for the large ones
    (22, 64, 1, 4, 30, 8, False, False, 0), (22, 64, 1, 4, 30, 16, False, True, 0), (22, 64, 1, 4, 30, 8, True, True, 1),
    (23, 1, 2, 4, 30, 8, True, True, 0), (23, 1, 1, 3, 21, 5, False, False, 1),
    (24, 1, 2, 4, 30, 16, False, True, 1), (24, 1, 1, 8, 255, 8, False, False, 0), (25, 1, 1, 2, 8, 9, True, True, 0)])
def test_tiles_of_2_to_the_15(log2_block, K, n, b, g, agg_bits, bf16, ef, order):
    block = 1 << log2_block
    T = list(range(256)) if b == 8 else None
    P, L = both_params(block * K, block, n, b=b, g=g, agg_bits=agg_bits, bf16=bf16, order=order, table=T)
    if K > 1:                                    # long: blocks 0 and K - 1 are compared
        gen = torch.Generator(device=DEV).manual_seed(22)
        x = torch.randn(block * K, device=DEV, generator=gen) * 1e-3
        x = x.to(torch.bfloat16) if bf16 else x
        R = GpuRound(L, ef=ef)
        e = {}
        if ef:
            R.efs[0].copy_(torch.randn(block * K, device=DEV, generator=gen) * 2e-4)
            e = {k: R.efs[0][k * block:(k + 1) * block].cpu().numpy() for k in (0, K - 1)}
        R.compress_all(3, [x])
        R.aggregate()
        R.decompress(3)
        M, pk, agg, out = R.range_M.cpu().numpy(), R.packed[0].cpu().numpy(), R.agg_numpy(), R.out.cpu().numpy()
        for k in (0, K - 1):
            Pk = o.Params(d=block, block=block, n=1, b=b, g=g, t_p=P.t_p, seed=P.seed, table=P.table,
                          agg_bits=agg_bits, order=order)
            gk = to_np32(x[k * block:(k + 1) * block])
            assert abs(M[k] - o.prepare_range(Pk, [gk], [e[k]] if ef else None)[0]) <= M[k] * 2.0 ** -23
            ref, ne = o.compress(Pk, 0, 3, gk, e.get(k), M[k:k + 1], j0=k * block)
            if ef:
                assert rel_l2(R.efs[0][k * block:(k + 1) * block].cpu().numpy(), ne) <= 1e-5
            assert_indices_match(pk[k * block // 2:(k + 1) * block // 2], ref, b)
            Y = o.aggregate(Pk, [pk[k * block // 2:(k + 1) * block // 2]])
            assert np.array_equal(agg[k * block:(k + 1) * block], Y)
            assert rel_l2(out[k * block:(k + 1) * block], o.decompress(Pk, 3, Y, M[k:k + 1], j0=k * block)) <= 1e-5
        return
    R = GpuRound(L, ef=ef)
    efs = None
    if ef:
        for i, e in enumerate(R.efs):
            e.copy_(make_grads(block, 1, 2e-4, seed=90 + i)[0])
        efs = [e.cpu().numpy() for e in R.efs]
    _round_against_oracle(P, L, R, make_grads(block, n, seed=log2_block, bf16=bf16), 3, efs)


@pytest.mark.parametrize("log2_block,K,n,b,g,order", [
    (10, 1, 1, 3, 21, 0), (10, 13, 3, 4, 30, 0), (12, 7, 10, 3, 21, 0), (13, 5, 64, 2, 3, 0), (14, 3, 4, 4, 30, 0),
    (15, 1, 5, 3, 31, 1), (16, 2, 33, 2, 3, 1), (17, 3, 2, 3, 21, 1), (19, 1, 7, 1, 1, 0), (20, 1, 10, 3, 21, 1),
    (21, 1, 3, 4, 30, 0), (22, 1, 2, 3, 21, 1), (16, 16, 32, 4, 30, 1), (16, 17, 32, 4, 30, 1), (10, 16384, 1, 4, 30, 0),
    (10, 16385, 1, 4, 30, 0), (13, 1024, 3, 4, 30, 0), (13, 1025, 3, 4, 30, 0), (14, 7, 9, 8, 255, 0), (17, 8, 8, 4, 30, 1),
    (17, 9, 8, 4, 30, 1), (17, 20, 4, 4, 30, 0), (17, 21, 4, 4, 30, 0), (18, 1, 17, 4, 30, 1), (20, 1, 33, 2, 3, 1),
    (15, 512, 1, 4, 30, 0), (15, 513, 1, 4, 30, 0), (16, 128, 3, 4, 30, 1), (16, 129, 3, 4, 30, 1), (13, 63, 5, 4, 30, 0)])
def test_range_found_by_the_last_pass(log2_block, K, n, b, g, order):
    """Small calls of blocks of up to 2^20: the quantizer adds the norms up itself.  The range is that of thc_prepare_range
    and the streams are those of thc_compress, bit for bit, and both are the oracle's.  Pairs of rows of 2^15 to 2^17 that
    differ in one block lie on either side of a limit of the rule (2^16 x 32 workers: 4096 workgroups; x 3: 3072; 2^15 x 1:
    2048; 2^17: 1024 and 1280); 2^21 and 2^22 take the range kernel.  Blocks of up to 2^14 come to the quantizer here only
    with more than four workers; the rows with fewer go block by block, as all of thc_compress does at these sizes."""
    block = 1 << log2_block
    table = list(range(256)) if b == 8 else None
    agg_bits = 8 if g * n < 256 else 16
    P, L = both_params(block * K, block, n, b=b, g=g, agg_bits=agg_bits, order=order, table=table)
    x = make_grads(block * K, n, seed=log2_block + K)
    dg = [v.to(DEV) for v in x]
    A, B = GpuRound(L), GpuRound(L)
    A.compress_all(9, dg)
    B.prepare(dg)
    B.compress_each(9, dg)
    assert torch.equal(A.range_M, B.range_M)
    for p, q in zip(A.packed, B.packed):
        assert torch.equal(p, q)
    M, gn = A.range_M.cpu().numpy(), [to_np32(v) for v in x]
    M_ref = o.prepare_range(P, gn)
    assert np.all(np.abs(M - M_ref) <= np.abs(M_ref) * 2.0 ** -23)
    assert_indices_match(A.packed[n - 1].cpu().numpy(), o.compress(P, n - 1, 9, gn[n - 1], None, M)[0], b)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 13])
@pytest.mark.parametrize("b,g", [(1, 1), (1, 100), (2, 8), (2, 255), (3, 21), (3, 255), (4, 17), (5, 40), (6, 63),
                                 (7, 127), (8, 255)])
def test_sums_of_any_width(b, g, n):
    """Exact width, 8 bits where they fit, and 16; 33 * 1024 coordinates leave the last workgroup mostly empty."""
    block, K = 1 << 10, 33
    T = [round(i * g / ((1 << b) - 1)) for i in range(1 << b)]
    exact = (g * n).bit_length()
    pk = np.random.default_rng(n * 256 + g).integers(0, 256, (n, block * K * b // 8), dtype=np.uint8)
    pk[:, :64] = 255                              # sums of g * n
    for agg_bits in sorted({exact, max(exact, 8), 16}):
        P, L = both_params(block * K, block, n, b=b, g=g, agg_bits=agg_bits, table=T)
        R = GpuRound(L)
        for i in range(n):
            R.packed[i].copy_(torch.from_numpy(pk[i]))
        R.aggregate()
        assert np.array_equal(R.agg_numpy(), o.aggregate(P, list(pk)))


@pytest.mark.parametrize("b,g,agg_bits,n", [(4, 30, 8, 8), (4, 15, 7, 8), (4, 30, 9, 9), (4, 100, 16, 8), (2, 8, 8, 16),
                                            (2, 8, 16, 16), (3, 31, 9, 11), (1, 1, 6, 32), (5, 36, 8, 7), (8, 255, 16, 4),
                                            (4, 30, 16, 32), (4, 15, 9, 31), (3, 7, 3, 1)])
def test_sums_of_streams_beyond_the_cache(b, g, agg_bits, n):
    """Streams of 80 MB and more together go past the caches: the whole against slices of it, which do not, bit for bit; the
    last workgroup is mostly empty.  Of 31 and 32 workers with four loads in flight; a single stream of 3-bit indices is kept."""
    block, K = 1 << 10, ((5 << 12) if n < 30 or b != 4 else 9 << 10) * (12 if n == 1 else 1) + 1
    T = [round(i * g / ((1 << b) - 1)) for i in range(1 << b)]
    assert n * block * K * b // 8 >= 80 << 20
    _, L = both_params(block * K, block, n, b=b, g=g, agg_bits=agg_bits, table=T)
    gen = torch.Generator(device=DEV).manual_seed(b * 64 + n)
    packed = [torch.randint(0, 256, (block * K * b // 8,), dtype=torch.uint8, device=DEV, generator=gen) for _ in range(n)]
    agg = torch.zeros(block * K * agg_bits // 8, dtype=torch.uint8, device=DEV)
    api.thc_aggregate(L, packed, agg)
    step = 1 << 12
    for k in range(0, K, step):
        m = min(step, K - k)
        _, S = both_params(block * m, block, n, b=b, g=g, agg_bits=agg_bits, table=T)
        part = torch.zeros(block * m * agg_bits // 8, dtype=torch.uint8, device=DEV)
        api.thc_aggregate(S, [p[k * block * b // 8:(k + m) * block * b // 8].clone() for p in packed], part)
        assert torch.equal(part, agg[k * block * agg_bits // 8:(k + m) * block * agg_bits // 8])


@pytest.mark.parametrize("log2_block,K,n,b,g,agg_bits,bf16,ef", [
    (10, 1, 1, 4, 30, 8, False, True), (10, 19, 2, 3, 21, 6, True, True), (11, 5, 2, 4, 30, 16, False, True),
    (12, 3, 3, 8, 255, 10, True, True), (13, 2, 2, 4, 30, 8, True, True), (14, 1, 1, 4, 30, 5, False, True),
    (14, 2, 2, 3, 21, 16, True, True), (14, 5, 2, 4, 30, 8, True, True), (15, 1, 2, 2, 8, 5, False, True),
    (15, 3, 1, 4, 30, 16, True, True), (15, 2, 2, 4, 30, 8, False, False)])
def test_whole_inverse_in_one_launch(log2_block, K, n, b, g, agg_bits, bf16, ef):
    """Rounds on blocks of up to 2^15, whose decompression is one launch; odd numbers of blocks leave the last tile partly
    empty.  Error feedback takes the inverse in one launch here at 2^15; up to 2^14 it is part of the worker side's own
    launch (the uniform variant takes the inverse at every size)."""
    block = 1 << log2_block
    P, L = both_params(block * K, block, n, b=b, g=g, agg_bits=agg_bits, bf16=bf16,
                       table=list(range(256)) if b == 8 else None)
    R = GpuRound(L, ef=ef)
    efs = None
    if ef:
        for i, e in enumerate(R.efs):
            e.copy_(make_grads(block * K, 1, 2e-4, seed=70 + i)[0])
        efs = [e.cpu().numpy() for e in R.efs]
    _round_against_oracle(P, L, R, make_grads(block * K, n, seed=log2_block, bf16=bf16), 6, efs)


@pytest.mark.parametrize("order", [0, 1], ids=["ascending", "split"])
@pytest.mark.parametrize("log2_block,K,n,bf16,ef,single_launch", [
    (20, 1, 1, False, False, 0), (22, 1, 1, False, False, 0), (22, 1, 63, True, False, 0), (22, 1, 64, False, False, 0),
    (22, 4, 16, True, False, 0), (22, 4, 16, False, False, 1), (22, 64, 1, False, True, 0), (24, 1, 1, False, True, 0),
    (24, 1, 3, True, False, 0), (24, 1, 1, True, True, 0)])
def test_norms_are_added_up_in_one_order_whatever_the_tile(log2_block, K, n, bf16, ef, single_launch, order):
    """M must not depend on the call that forms it: n workers or one, a shard or the whole, tiles of 2^13 or 2^15 (from 64
    blocks of 2^22 on), one launch or several.  The squares of the last block add up to 1 + 2^-23 + 2^-48, the square of
    a tie between two binary32 numbers, and twelve times 2^-54.  Those are lost when added one by one to a sum of 1 or
    more, and 3 * 2^-52, which settles the tie, when added up four to a thread first, as every call has to do."""
    block = 1 << log2_block
    x = torch.zeros(block * K, dtype=torch.bfloat16 if bf16 else torch.float32, device=DEV)
    last = x[block * (K - 1):]
    last[0] = 1.0
    last[4:16] = 2.0 ** -27
    last[torch.tensor([5, 9, 14], device=DEV) << 16] = torch.tensor([2.0 ** -12, 2.0 ** -12, 2.0 ** -24], device=DEV).to(x.dtype)
    want = (1 + 2.0 ** -23) / 2.0 ** (log2_block // 2)
    _, L = both_params(block * K, block, n, agg_bits=16, bf16=bf16, order=order, single_launch=single_launch)
    L.t_p = 1.0
    R = GpuRound(L, ef=ef)
    if ef:                                       # half of every coordinate in the buffer
        x = x * 0.5
        for e in R.efs:
            e.copy_(x.to(torch.float32))
    R.prepare([x] * n)
    assert R.range_M[K - 1].item() == want
    R.range_M.zero_()
    R.compress_all(2, [x] * n)
    assert R.range_M[K - 1].item() == want
    if single_launch:
        assert R.status() == 0


@pytest.mark.parametrize("log2_block,K,n,b,g,bf16,ef", [
    (10, 1, 1, 4, 30, False, True), (10, 19, 2, 3, 21, True, True), (10, 9, 4, 4, 30, True, False),
    (11, 5, 3, 1, 1, False, True), (11, 7, 4, 2, 8, False, False), (12, 3, 4, 8, 255, False, True),
    (12, 7, 2, 2, 8, True, False), (13, 3, 2, 4, 30, False, True), (13, 1, 33, 4, 30, True, True),
    (14, 1, 4, 4, 30, False, False), (14, 2, 4, 5, 40, True, False), (14, 3, 2, 4, 30, True, True), (14, 1, 1, 8, 128, False, True),
    # either side of the limits of the rule, in workgroups of 8192 coordinates: found by every workgroup up to 512 (2^14 with
    # one worker 1024), norms first from 512, 640 or where 2^14 fills the chip evenly, with error feedback in 2^14 up to 512
    (13, 128, 4, 4, 30, False, False), (13, 129, 4, 4, 30, False, False), (13, 64, 8, 4, 30, False, False),
    (13, 63, 8, 4, 30, False, False), (13, 40, 16, 2, 8, False, False), (13, 39, 16, 2, 8, False, False),
    (10, 4097, 1, 4, 30, False, False), (14, 64, 4, 4, 30, False, False), (14, 65, 4, 4, 30, False, False),
    (14, 32, 8, 4, 30, False, False), (14, 28, 8, 4, 30, False, False), (14, 64, 8, 2, 3, True, False),
    (14, 512, 1, 4, 30, False, False), (14, 513, 1, 4, 30, False, False), (14, 64, 4, 4, 30, False, True),
    (14, 65, 4, 4, 30, False, True), (14, 65, 4, 3, 21, True, True), (14, 512, 4, 4, 30, False, False),
    (14, 512, 4, 4, 30, True, True),
    # two workgroups to a block: the fewest, 64 of them before the split, one more
    (14, 1, 1, 4, 30, False, False), (14, 16, 4, 3, 21, True, False), (14, 17, 4, 4, 30, False, False),
    (14, 21, 3, 8, 255, False, False), (14, 64, 1, 2, 8, False, False), (14, 65, 1, 4, 30, True, False)])
def test_worker_side_block_by_block(log2_block, K, n, b, g, bf16, ef):
    """Blocks of up to 2^14, whose worker side is one launch once the range is known: thc_compress_all gives what
    thc_prepare_range and thc_compress give, bit for bit, whichever way its range comes about, and both are the oracle's.
    Without error feedback its first and its last blocks are also what the passes make of them, which a call of five and more
    workers on a few blocks still takes; with it, 2^14 with 513 to 4095 workgroups takes the passes."""
    block = 1 << log2_block
    agg_bits = 8 if g * n < 256 else 16
    table = list(range(256)) if (b, g) == (8, 255) else [round(i * g / 255) for i in range(256)] if b == 8 else None
    if b == 8 and g < 255:
        b, table = 7, [round(i * g / 127) for i in range(128)]
    P, L = both_params(block * K, block, n, b=b, g=g, agg_bits=agg_bits, bf16=bf16, table=table)
    x = make_grads(block * K, n, seed=log2_block + K, bf16=bf16)
    dg = [v.to(DEV) for v in x]
    A, B = GpuRound(L, ef=ef), GpuRound(L, ef=ef)
    e = make_grads(block * K, n, 3e-4, seed=7 * K) if ef else None
    for R in (A, B):
        for i in range(n if ef else 0):
            R.efs[i].copy_(e[i])
    for rnd in (3, 4):                           # the second round starts from the first one's buffers
        before = [v.cpu().numpy() for v in A.efs] if ef else None
        A.compress_all(rnd, dg)
        B.prepare(dg)
        B.compress_each(rnd, dg)
        assert torch.equal(A.range_M, B.range_M)
        for p, q in zip(A.packed, B.packed):
            assert torch.equal(p, q)
        for p, q in zip(A.efs or [], B.efs or []):
            assert torch.equal(p, q)
    M, gn = A.range_M.cpu().numpy(), [to_np32(v) for v in x]
    M_ref = o.prepare_range(P, gn, before)
    assert np.all(np.abs(M - M_ref) <= np.abs(M_ref) * 2.0 ** -23)
    for i in range(n) if block * K * n <= 1 << 19 else (n - 1,):
        pk, ne = o.compress(P, i, 4, gn[i], before[i] if ef else None, M)
        assert_indices_match(A.packed[i].cpu().numpy(), pk, b)
        if ef:
            assert rel_l2(A.efs[i].cpu().numpy(), ne) <= 1e-5
    if ef:
        return
    N, k = max(n, 5), min(K, 3)                  # the workers that are added repeat the first one: the range stays
    for first in {0, K - k}:
        at = slice(first * block, (first + k) * block)
        _, S = both_params(block * k, block, N, b=b, g=g, agg_bits=16, bf16=bf16, table=table, first_block=first)
        Q = GpuRound(S)
        Q.compress_all(4, [v[at].clone() for v in dg] + [dg[0][at].clone()] * (N - n))
        assert torch.equal(Q.range_M, A.range_M[first:first + k])
        for p, q in zip(A.packed, Q.packed):
            assert torch.equal(p[at.start // 8 * b:at.stop // 8 * b], q)


@pytest.mark.parametrize("every_call", [False, True], ids=["compress", "compress_all"])
def test_worker_side_of_more_than_2_to_the_36_coordinates(every_call):
    """A launch takes fewer than 2^32 threads, so the longest vectors go in several: blocks on either side of a seam and
    the last one against the oracle, each at a scale of its own.  128 GB of bf16."""
    block, K = 1 << 14, (1 << 22) + 1
    P, L = both_params(block * K, block, 1, b=1, g=1, agg_bits=1, bf16=True, table=[0, 1])
    v = make_grads(block, 1, seed=36, bf16=True)[0]
    x = torch.empty(block * K, dtype=torch.bfloat16, device=DEV)
    scale = 2.0 ** (torch.arange(K, device=DEV) % 5).to(torch.bfloat16)
    torch.mul(v.to(DEV).expand(K, block), scale[:, None], out=x.view(K, block))
    packed = torch.zeros(block * K // 8, dtype=torch.uint8, device=DEV)
    ws = torch.empty(api.thc_workspace_bytes(L, False), dtype=torch.uint8, device=DEV)
    M = torch.rand(K, device=DEV, generator=torch.Generator(device=DEV).manual_seed(36)) * 1e-3 + 1e-3
    given = M.clone()
    if every_call:
        api.thc_compress_all(L, 8, [x], None, M, [packed], ws)
    else:
        api.thc_compress(L, 0, 8, x, None, M, packed, ws)
    Pk = o.Params(d=block, block=block, n=1, b=1, g=1, t_p=P.t_p, seed=P.seed, table=P.table, agg_bits=1)
    for k in (0, (1 << 20) - 1, 1 << 20, (1 << 22) - 1, 1 << 22):
        gk, Mk = to_np32(x[k * block:(k + 1) * block]), M[k:k + 1].cpu().numpy()
        if every_call:
            want = o.prepare_range(Pk, [gk])
            assert abs(Mk[0] - want[0]) <= want[0] * 2.0 ** -23
        else:
            assert Mk[0] == given[k].item()
        ref = o.compress(Pk, 0, 8, gk, None, Mk, j0=k * block)[0]
        assert_indices_match(packed[k * block // 8:(k + 1) * block // 8].cpu().numpy(), ref, 1, f"block {k}")


@pytest.mark.parametrize("K,agg_bits", [(1, 8), (3, 9), (704, 8), (705, 8), (705, 9), (705, 16), (1024, 9), (1025, 8), (640, 5),
                                        (641, 5), (1280, 9), (1281, 9), (1537, 9), (1792, 4), (1793, 4), (2978, 12), (2979, 12), (7169, 8),
                                        (512, 9), (513, 9), (640, 8), (641, 8), (2560, 5), (2561, 8)])
def test_inverse_of_2_to_the_14_by_one_block_or_two_a_workgroup(K, agg_bits):
    """Both kernels give the same bits: the whole vector against its slices of at most eight blocks, which take one block a
    workgroup, on either side of the rule's limits; block 0 and the last one against the oracle."""
    block, g = 1 << 14, 15 if agg_bits < 5 else 30
    P, L = both_params(block * K, block, 1, g=g, agg_bits=agg_bits)
    R = GpuRound(L)
    gen = torch.Generator(device=DEV).manual_seed(K)
    R.agg.copy_(torch.randint(0, 256, R.agg.shape, generator=gen, device=DEV, dtype=torch.uint8))
    R.range_M.copy_(torch.rand(K, generator=gen, device=DEV) + 0.5)
    R.decompress(11)
    for k in range(0, K, max(8, K // 5)):
        n = min(8, K - k)
        _, S = both_params(block * n, block, 1, g=g, agg_bits=agg_bits)
        S.first_block = k
        Q = GpuRound(S)
        Q.agg.copy_(R.agg[k * block // 8 * agg_bits:(k + n) * block // 8 * agg_bits])
        Q.range_M.copy_(R.range_M[k:k + n])
        Q.decompress(11)
        assert torch.equal(Q.out, R.out[k * block:(k + n) * block])
    Y, M, out = R.agg_numpy(), R.range_M.cpu().numpy(), R.out.cpu().numpy()
    Pk = o.Params(d=block, block=block, n=1, b=P.b, g=P.g, t_p=P.t_p, seed=P.seed, table=P.table, agg_bits=agg_bits)
    for k in {0, K - 1}:
        ref = o.decompress(Pk, 11, Y[k * block:(k + 1) * block], M[k:k + 1], j0=k * block)
        assert rel_l2(out[k * block:(k + 1) * block], ref) <= 1e-5


@pytest.mark.parametrize("log2_block,K,n,ef,order", [(16, 512, 2, False, 1), (16, 513, 2, False, 0), (16, 1025, 1, False, 1),
                                                     (18, 65, 2, True, 1), (20, 33, 1, True, 0), (25, 2, 1, True, 1)])
def test_walk_from_the_last_tile(log2_block, K, n, ef, order):
    """Launches above 2^26 worker-coordinates, 2^25 with error feedback, walk their tiles last one first: the whole against
    its single blocks, which do not, bit for bit, at the first block, the last one and one between."""
    block = 1 << log2_block
    _, L = both_params(block * K, block, n, order=order)
    R = GpuRound(L, ef=ef)
    gen = torch.Generator(device=DEV).manual_seed(K)
    x = [torch.randn(block * K, device=DEV, generator=gen) * 1e-3 for _ in range(n)]
    old = []
    for e in R.efs or []:
        e.copy_(torch.randn(block * K, device=DEV, generator=gen) * 2e-4)
        old.append(e.clone())
    R.compress_all(4, x)
    for k in {0, K // 2, K - 1}:
        _, S = both_params(block, block, n, order=order, first_block=k)
        Q = GpuRound(S, ef=ef)
        at = slice(k * block, (k + 1) * block)
        for q, e in zip(Q.efs or [], old):
            q.copy_(e[at])
        Q.compress_all(4, [v[at].clone() for v in x])
        assert Q.range_M[0] == R.range_M[k]
        for q, p in zip(Q.packed, R.packed):
            assert torch.equal(q, p[k * block // 2:(k + 1) * block // 2])
        for q, e in zip(Q.efs or [], R.efs or []):
            assert torch.equal(q, e[at])


@pytest.mark.parametrize("log2_block,K,step,n,bf16,ef,order", [
    # 2^26 coordinates and more of all vectors: the error-feedback inverse's first pass; bf16 gradients of more than 160 MB with
    # their buffers on tiles of 2^15
    (18, 132, 40, 2, False, True, 0), (18, 132, 40, 2, True, True, 1), (23, 5, 2, 1, True, True, 0), (23, 5, 2, 1, True, True, 1),
    # more than 64 MB of gradients and buffers in blocks of up to 2^13: the norms and the blocks
    (10, 9001, 4000, 2, False, False, 0), (11, 4500, 2000, 2, False, True, 0), (12, 1400, 600, 2, True, True, 0),
    (13, 1201, 500, 1, False, True, 0),
    # estimates of 40 to 192 MB by way of every kernel that writes them
    (10, 10241, 4096, 1, False, False, 0), (13, 1281, 512, 1, False, False, 0), (14, 641, 256, 1, False, False, 0),
    (14, 2560, 256, 1, False, False, 0), (15, 323, 128, 1, False, False, 0), (16, 160, 64, 1, False, False, 1),
    (20, 11, 4, 1, False, False, 0), (22, 3, 1, 1, False, False, 1), (23, 6, 2, 1, False, False, 0), (24, 3, 1, 1, False, False, 1)])
def test_a_large_call_gives_what_its_slices_give(log2_block, K, step, n, bf16, ef, order):
    """Rules that look at the size of a launch choose how memory is read and written, never what is computed: a whole round on
    large vectors, every output bit for bit that of rounds on slices which lie on the other side of those rules."""
    B, rnd = 1 << log2_block, 5
    gen = torch.Generator(device=DEV).manual_seed(log2_block * K)
    dt = torch.bfloat16 if bf16 else torch.float32
    grads = [(torch.randn(B * K, device=DEV, generator=gen) * 1e-3).to(dt) for _ in range(n)]
    efs = [torch.randn(B * K, device=DEV, generator=gen) * 1e-4 for _ in range(n)] if ef else None

    def run(k, m):
        _, L = both_params(B * m, B, n, bf16=bf16, order=order, first_block=k)
        R = GpuRound(L, ef)
        if ef:
            for i in range(n):
                R.efs[i].copy_(efs[i][k * B:(k + m) * B])
        R.compress_all(rnd, [g[k * B:(k + m) * B].clone() for g in grads])
        R.aggregate()
        R.decompress(rnd)
        return R

    whole = run(0, K)
    for k in range(0, K, step):
        m = min(step, K - k)
        part, at = run(k, m), slice(k * B, (k + m) * B)
        assert torch.equal(part.range_M, whole.range_M[k:k + m])
        assert torch.equal(part.out, whole.out[at])
        for i in range(n):
            assert torch.equal(part.packed[i], whole.packed[i][k * B // 2:(k + m) * B // 2])
            if ef:
                assert torch.equal(part.efs[i], whole.efs[i][at])
