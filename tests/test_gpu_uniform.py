"""Uniform THC (Alg. 1) on the GPU library against the oracle: global min/max ranges, uniform stochastic
quantization with and without the rotation, error feedback, the estimate of the mean."""
import numpy as np
import pytest
import torch

from oracle import thc_oracle as o
from paper_2302_08545_amd import api
from tests.test_gpu_parity import DEV, SEED, assert_indices_match, make_grads, rel_l2, to_np32

pytestmark = pytest.mark.gpu
F32 = np.float32


def uparams(d, block, n, b, agg_bits, bf16=False, first_block=0, order=0):
    T = list(range(2 ** b))
    P = o.Params(d=d, block=block, n=n, b=b, g=2 ** b - 1, t_p=1.0, seed=SEED, table=T, agg_bits=agg_bits, order=order)
    L = api.make_params(d, block, n, b, 2 ** b - 1, 1.0, SEED, T, agg_bits,
                        api.THC_DTYPE_BF16 if bf16 else api.THC_DTYPE_F32, stage_order=order, first_block=first_block)
    return P, L


@pytest.mark.parametrize("rotate", [False, True], ids=["plain", "rotated"])
@pytest.mark.parametrize("block,K,n,b,agg_bits,ef,first_block", [
    (1 << 10, 5, 3, 4, 8, False, 0), (1 << 12, 2, 4, 2, 4, True, 0), (1 << 14, 2, 8, 4, 7, False, 0),
    (1 << 16, 1, 2, 8, 9, True, 0), (1 << 20, 1, 3, 1, 2, False, 0), (1 << 21, 1, 2, 3, 4, True, 0),
    (1 << 12, 3, 2, 4, 8, True, (1 << 22) + 3)])
def test_uniform_round(block, K, n, b, agg_bits, ef, first_block, rotate):
    _uniform_round(block, K, n, b, agg_bits, ef, first_block, rotate)


@pytest.mark.parametrize("log2_block,K,n,b,agg_bits,ef,order", [
    (17, 3, 2, 4, 8, True, 1), (20, 2, 3, 4, 6, False, 1), (22, 1, 2, 4, 8, True, 1),
    (23, 1, 2, 4, 8, True, 0), (23, 2, 2, 3, 4, True, 1), (24, 1, 1, 4, 16, True, 1), (25, 1, 1, 2, 2, True, 0),
    (25, 1, 1, 8, 8, False, 1)])
def test_uniform_round_on_large_rotated_blocks(log2_block, K, n, b, agg_bits, ef, order):
    """Blocks of 2^23 to 2^25: a forward transform with a middle pass, an inverse one on tiles of 2^15 coordinates whose
    range is not symmetric."""
    _uniform_round(1 << log2_block, K, n, b, agg_bits, ef, 0, True, order)


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("b", [4, 3])
@pytest.mark.parametrize("log2_block", [10, 11, 12, 13, 14, 15])
def test_uniform_round_with_error_feedback_on_small_rotated_blocks(log2_block, b, bf16):
    """The error-feedback inverse in one launch at every block size that takes it, from 4-bit and from other indices; the last
    tile is partly empty where a tile holds several blocks."""
    _uniform_round(1 << log2_block, 5 if log2_block < 14 else 3, 2, b, 8, True, 0, True, bf16=bf16)


@pytest.mark.parametrize("block,K,b,bf16", [(1 << 10, 1, 4, True), (1 << 10, 5, 3, True), (1 << 11, 3, 4, False),
                                            (1 << 13, 3, 4, True), (1 << 16, 2, 8, True)])
def test_uniform_round_with_error_feedback_without_rotation(block, K, b, bf16):
    """Small vectors: tiles of 4096 coordinates, the last one partly empty in the first three rows."""
    _uniform_round(block, K, 2, b, 16, True, 3, False, bf16=bf16)


@pytest.mark.parametrize("agg_bits", [8, 16, 7])
def test_estimate_without_rotation_by_its_size(agg_bits):
    """An estimate of more than 4 MB is stored otherwise than its slices: the same values."""
    block, K = 1 << 10, 1025
    _, L = uparams(K * block, block, 3, 4, agg_bits)
    gen = torch.Generator(device=DEV).manual_seed(agg_bits)
    agg = torch.randint(0, 256, (K * block * agg_bits // 8,), dtype=torch.uint8, device=DEV, generator=gen)
    m, M = -torch.rand(K, device=DEV, generator=gen), torch.rand(K, device=DEV, generator=gen)
    out = torch.zeros(K * block, device=DEV)
    api.thc_uniform_decompress(L, 0, agg, False, m, M, out, None)
    for k in range(0, K, 400):
        n = min(400, K - k)
        _, S = uparams(n * block, block, 3, 4, agg_bits)
        part, cut = torch.zeros(n * block, device=DEV), agg[k * block * agg_bits // 8:(k + n) * block * agg_bits // 8].clone()
        api.thc_uniform_decompress(S, 0, cut, False, m[k:k + n].clone(), M[k:k + n].clone(), part, None)
        assert torch.equal(part, out[k * block:(k + n) * block])


@pytest.mark.parametrize("bf16,ef", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("n", [1, 3])
def test_range_of_vectors_beyond_the_cache(n, bf16, ef):
    """Inputs this large together are read past the caches: minimum and maximum of every block, exactly; the last tile
    holds one block of eight."""
    block = 1 << 10
    per = (2 if bf16 else 4) + (4 if ef else 0)
    K = ((256 << 20) // per // n // block) // 8 * 8 + 9
    assert n * K * block * per >= 256 << 20
    _, L = uparams(K * block, block, n, 4, 8, bf16=bf16)
    gen = torch.Generator(device=DEV).manual_seed(n)
    grads = [torch.randn(K * block, device=DEV, generator=gen).to(torch.bfloat16 if bf16 else torch.float32) for _ in range(n)]
    efs = [torch.randn(K * block, device=DEV, generator=gen) for _ in range(n)] if ef else None
    m, M = torch.zeros(K, device=DEV), torch.zeros(K, device=DEV)
    ws = torch.empty(api.thc_uniform_workspace_bytes(L, False), dtype=torch.uint8, device=DEV)
    api.thc_uniform_prepare_range(L, 0, grads, efs, False, m, M, ws)
    lo, hi = torch.full((K,), float("inf"), device=DEV), torch.full((K,), float("-inf"), device=DEV)
    for i in range(n):
        x = grads[i].float() + (efs[i] if ef else 0.0)
        lo, hi = torch.minimum(lo, x.view(K, block).amin(1)), torch.maximum(hi, x.view(K, block).amax(1))
    assert torch.equal(m, lo) and torch.equal(M, hi)


@pytest.mark.parametrize("log2_block,K,step,order", [(16, 530, 130, 1), (17, 260, 130, 0), (20, 33, 16, 1), (21, 17, 8, 0)])
def test_range_of_rotated_vectors_beyond_the_cache(log2_block, K, step, order):
    """Half-rotated vectors of more than 256 MB together are read past the caches: the range of each block, and the indices, are
    those of slices that are not."""
    B, n, rnd = 1 << log2_block, 2, 3
    assert n * B * K * 4 > 256 << 20 and n * B * step * 4 <= 256 << 20
    gen = torch.Generator(device=DEV).manual_seed(log2_block)
    grads = [torch.randn(B * K, device=DEV, generator=gen) for _ in range(n)]

    def run(k, c):
        _, L = uparams(B * c, B, n, 4, 8, first_block=k, order=order)
        g = [x[k * B:(k + c) * B].clone() for x in grads]
        m, M = torch.zeros(c, device=DEV), torch.zeros(c, device=DEV)
        ws = torch.empty(api.thc_uniform_workspace_bytes(L, True), dtype=torch.uint8, device=DEV)
        packed = torch.zeros(B * c // 2, dtype=torch.uint8, device=DEV)
        api.thc_uniform_prepare_range(L, rnd, g, None, True, m, M, ws)
        api.thc_uniform_compress(L, 1, rnd, g[1], None, True, m, M, packed, ws)
        return m, M, packed

    m, M, packed = run(0, K)
    for k in range(0, K, step):
        c = min(step, K - k)
        pm, pM, pp = run(k, c)
        assert torch.equal(pm, m[k:k + c]) and torch.equal(pM, M[k:k + c])
        assert torch.equal(pp, packed[k * B // 2:(k + c) * B // 2])


@pytest.mark.parametrize("K,bf16,ef", [(1024, False, True), (1025, False, True), (1025, True, True), (4096, False, False),
                                       (4097, False, False), (16384, False, False), (16385, False, False)])
def test_quantizer_of_one_group_of_coordinates_a_thread_or_two(K, bf16, ef):
    """Either side of the limits of uniform_one_group: the whole vector against its slices of at most 21 blocks, which take
    one group, bit for bit; both leave the last tile partly empty."""
    block, b = 1 << 10, 3
    gen = torch.Generator(device=DEV).manual_seed(K)
    x = torch.randn(K * block, device=DEV, generator=gen) * 1e-3
    x = x.to(torch.bfloat16) if bf16 else x
    e0 = torch.randn(K * block, device=DEV, generator=gen) * 2e-4 if ef else None
    rm = torch.rand(K, generator=gen, device=DEV) * -2e-3 - 1e-3
    rM = torch.rand(K, generator=gen, device=DEV) * 2e-3 + 1e-3

    def compress(first, k):
        at = slice(first * block, (first + k) * block)
        packed = torch.zeros(k * block * b // 8, dtype=torch.uint8, device=DEV)
        e = e0[at].clone() if ef else None
        _, L = uparams(k * block, block, 2, b, 8, bf16=bf16, first_block=first)
        api.thc_uniform_compress(L, 1, 5, x[at].clone(), e, False, rm[first:first + k].clone(), rM[first:first + k].clone(), packed,
                                 None)
        return packed, e

    packed, e = compress(0, K)
    for first, k in ((0, 16), (K // 2, 21), (K - 21, 21), (K - 1, 1)):
        p, q = compress(first, k)
        assert torch.equal(p, packed[first * block * b // 8:(first + k) * block * b // 8])
        assert not ef or torch.equal(q, e[first * block:(first + k) * block])


def _uniform_round(block, K, n, b, agg_bits, ef, first_block, rotate, order=0, bf16=False):
    d = block * K
    j0 = first_block * block            # the buffers hold a slice of a longer vector
    P, L = uparams(d, block, n, b, agg_bits, bf16=bf16, first_block=first_block, order=order)
    grads = make_grads(d, n, seed=block % 97 + b, bf16=bf16)
    for i, g in enumerate(grads):
        g += 0.002 * (i - 1)                                      # asymmetric ranges: m != -M
    dg = [g.to(DEV) for g in grads]
    gn = [to_np32(g) for g in grads]
    gen = torch.Generator().manual_seed(5)
    efs0 = [(torch.randn(d, generator=gen) * 2e-4).numpy() for _ in range(n)] if ef else None
    defs = [torch.from_numpy(e).to(DEV) for e in efs0] if ef else None
    ws = torch.empty(api.thc_uniform_workspace_bytes(L, rotate), dtype=torch.uint8, device=DEV)
    rm = torch.zeros(K, dtype=torch.float32, device=DEV)
    rM = torch.zeros(K, dtype=torch.float32, device=DEV)
    packed = [torch.zeros(d * b // 8, dtype=torch.uint8, device=DEV) for _ in range(n)]
    agg = torch.zeros(d * agg_bits // 8, dtype=torch.uint8, device=DEV)
    out = torch.zeros(d, dtype=torch.float32, device=DEV)
    rnd = 3
    api.thc_uniform_prepare_range(L, rnd, dg, defs, rotate, rm, rM, ws)
    m_ref, M_ref = o.uniform_range(P, rnd, gn, efs0, rotate, j0)
    # minima and maxima are order-independent: the range is bit-exact, rotated or not
    assert np.array_equal(rm.cpu().numpy(), m_ref) and np.array_equal(rM.cpu().numpy(), M_ref)
    packed_ref = []
    for i in range(n):
        api.thc_uniform_compress(L, i, rnd, dg[i], None if defs is None else defs[i], rotate, rm, rM, packed[i], ws)
        pk, ne = o.uniform_compress(P, i, rnd, gn[i], None if efs0 is None else efs0[i], m_ref, M_ref, rotate, j0)
        assert_indices_match(packed[i].cpu().numpy(), pk, b, f"worker {i}")
        packed_ref.append(pk)
        if ef:
            assert rel_l2(defs[i].cpu().numpy(), ne) <= 1e-5
    api.thc_aggregate(L, packed, agg)
    Y = o.aggregate(P, packed_ref)
    assert np.array_equal(agg.cpu().numpy(), o.aggregate_stream(P, Y))
    api.thc_uniform_decompress(L, rnd, agg, rotate, rm, rM, out, ws)
    ref = o.uniform_decompress(P, rnd, Y, m_ref, M_ref, rotate, j0)
    assert rel_l2(out.cpu().numpy(), ref) <= 1e-5


@pytest.mark.parametrize("log2_block,K,n", [(20, 33, 2), (14, 2049, 2), (12, 16385, 1)])
def test_range_pass_of_the_rotated_variant_from_the_last_tile(log2_block, K, n):
    """Above 2^26 worker-coordinates the range pass walks its tiles last one first: the range and the streams of the whole
    against those of its single blocks, which do not."""
    block, b = 1 << log2_block, 4

    def compress(L, x):
        k = L.d // block
        ws = torch.empty(api.thc_uniform_workspace_bytes(L, True), dtype=torch.uint8, device=DEV)
        rm, rM = torch.zeros(k, device=DEV), torch.zeros(k, device=DEV)
        api.thc_uniform_prepare_range(L, 6, x, None, True, rm, rM, ws)
        packed = [torch.zeros(L.d * b // 8, dtype=torch.uint8, device=DEV) for _ in x]
        for i in range(n):
            api.thc_uniform_compress(L, i, 6, x[i], None, True, rm, rM, packed[i], ws)
        return rm, rM, packed

    gen = torch.Generator(device=DEV).manual_seed(K)
    x = [torch.randn(block * K, device=DEV, generator=gen) * 1e-3 + 1e-3 * i for i in range(n)]
    rm, rM, packed = compress(uparams(block * K, block, n, b, 16, order=1)[1], x)
    for k in (0, K // 2, K - 1):
        at = slice(k * block, (k + 1) * block)
        m, M, one = compress(uparams(block, block, n, b, 16, order=1, first_block=k)[1], [v[at].clone() for v in x])
        assert m[0] == rm[k] and M[0] == rM[k]
        for p, q in zip(packed, one):
            assert torch.equal(p[k * block // 2:(k + 1) * block // 2], q)


def test_uniform_needs_the_identity_table():
    L = api.make_params(1 << 12, 1 << 12, 2, 2, 8, 1.0, SEED, [0, 3, 5, 8], 8)
    z = torch.zeros(16, dtype=torch.float32, device=DEV)
    with pytest.raises(api.ThcError) as e:
        api.thc_uniform_decompress(L, 0, z, False, z, z, z, z)
    assert e.value.status == -2


def test_bf16_uniform_plain():
    d, block, n, b = 1 << 13, 1 << 12, 2, 4
    P, L = uparams(d, block, n, b, 8, bf16=True)
    grads = make_grads(d, n, seed=4, bf16=True)
    dg = [g.to(DEV) for g in grads]
    gn = [to_np32(g) for g in grads]
    ws = torch.empty(api.thc_uniform_workspace_bytes(L, False), dtype=torch.uint8, device=DEV)
    rm = torch.zeros(2, dtype=torch.float32, device=DEV)
    rM = torch.zeros(2, dtype=torch.float32, device=DEV)
    api.thc_uniform_prepare_range(L, 0, dg, None, False, rm, rM, ws)
    m_ref, M_ref = o.uniform_range(P, 0, gn, None, False)
    assert np.array_equal(rm.cpu().numpy(), m_ref) and np.array_equal(rM.cpu().numpy(), M_ref)
    pk = torch.zeros(d * b // 8, dtype=torch.uint8, device=DEV)
    api.thc_uniform_compress(L, 1, 0, dg[1], None, False, rm, rM, pk, None)
    ref, _ = o.uniform_compress(P, 1, 0, gn[1], None, m_ref, M_ref, False)
    assert_indices_match(pk.cpu().numpy(), ref, b)


def test_uniform_compress_of_more_than_2_to_the_35_coordinates():
    """A launch takes fewer than 2^32 threads, so the longest vectors go in several: blocks on either side of every seam
    and the last one, each with a range of its own, against the oracle.  64 GB of bf16."""
    block, K, b = 1 << 14, (1 << 21) + 1, 1
    _, L = uparams(K * block, block, 2, b, 2, bf16=True)
    v = make_grads(block, 1, seed=35, bf16=True)[0]
    x = torch.empty(K * block, dtype=torch.bfloat16, device=DEV)
    x.view(K, block).copy_(v.to(DEV).expand(K, block))
    gen = torch.Generator(device=DEV).manual_seed(35)
    rm = torch.rand(K, generator=gen, device=DEV) * -2e-3 - 1e-3
    rM = torch.rand(K, generator=gen, device=DEV) * 2e-3 + 1e-3
    packed = torch.zeros(K * block * b // 8, dtype=torch.uint8, device=DEV)
    api.thc_uniform_compress(L, 1, 8, x, None, False, rm, rM, packed, None)
    P, _ = uparams(block, block, 2, b, 2)
    for k in (0, (1 << 20) - 1, 1 << 20, (1 << 21) - 1, 1 << 21):
        ref, _ = o.uniform_compress(P, 1, 8, to_np32(v), None, rm[k:k + 1].cpu().numpy(), rM[k:k + 1].cpu().numpy(), False,
                                    k * block)
        assert_indices_match(packed[k * block * b // 8:(k + 1) * block * b // 8].cpu().numpy(), ref, b, f"block {k}")
