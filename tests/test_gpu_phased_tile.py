"""Every epilogue of the phased 256 x 256 tile (plan tile 17), called directly
with the tile and split fixed: rows at, one past and between multiples of the
tile and of the 64 rows a wave skips, one and several bands of row tiles, one to
several K slabs, and K splits with a short last part (gate and up split too).

Against float64 products of the same operands; rows and columns past the
product must stay as they were.  Bounds: a 16-bit result is one rounding of a
sum that fp32 additions leave within 2^-22 of the sum of its terms' magnitudes
(K <= 1088 in 32-term matrix ops, the partial sums of a random sum growing as
their root); 32-bit results that alone.  The 16-wave tile adds and rounds in
the same order, so what it stores are the same bits: a plan that moves a product
from one tile to the other changes no output."""

import pytest
import torch

import paper_2608_01821_amd as dv
from internal import EPI_ADD_F32, EPI_STORE, EPI_SWIGLU, launch_gemm16

pytestmark = pytest.mark.gpu

DT = {"f16": (torch.float16, dv.DAVET_F16, 2.0 ** -11),
      "bf16": (torch.bfloat16, dv.DAVET_BF16, 2.0 ** -8)}
PHASED, SIXTEEN_WAVES = 17, 16
ROWS = [1, 64, 65, 192, 255, 256, 257, 321, 512, 4353]
SENTINEL = 77.0


def _operands(M, N, K, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn((M, K), generator=g, device="cuda").to(dtype)
    B = (torch.randn((N, K), generator=g, device="cuda") * 0.05).to(dtype)
    a, b = A.double(), B.double()
    return A, B, a @ b.T, a.abs() @ b.abs().T


def _within(got, ref, bound):
    assert bool(((got.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("dtype", list(DT))
@pytest.mark.parametrize("K", [64, 128, 192, 1024])
@pytest.mark.parametrize("M", ROWS)
def test_epilogues(M, K, dtype):
    t, code, ulp = DT[dtype]
    N = 768
    A, B, ref, mag = _operands(M, N, K, t, M + K)

    def run(epi, tile, out, n_out, **kw):
        half = N // 2
        B2 = B[half:] if epi == EPI_SWIGLU else None
        assert launch_gemm16(code, epi, tile, 1, A, B, B2, out, M, N, K, n_out,
                             **kw) == 0
        torch.cuda.synchronize()
        assert bool((out[M:] == SENTINEL).all())
        return out[:M]

    def fresh(n, kind=t):
        return torch.full((M + 3, n), SENTINEL, device="cuda", dtype=kind)

    err = 2.0 ** -22 * mag
    # residual: the sum is added to a row of values as large
    base = torch.randn((M, N), device="cuda")
    outs = []
    for tile in (PHASED, SIXTEEN_WAVES):
        out = fresh(N, torch.float32)
        out[:M] = base
        outs.append(run(EPI_ADD_F32, tile, out, N))
    full = base.double() + ref
    _within(outs[0], full, err + 2.0 ** -23 * (full.abs() + ref.abs()))
    assert torch.equal(*outs)
    # plain store
    outs = [run(EPI_STORE, tile, fresh(N), N) for tile in (PHASED, SIXTEEN_WAVES)]
    _within(outs[0], ref, err + ulp * ref.abs() + 2.0 ** -24)
    assert torch.equal(*outs)
    stored = outs[0]
    # gate and up
    outs = [run(EPI_SWIGLU, tile, fresh(N // 2), N // 2)
            for tile in (PHASED, SIXTEEN_WAVES)]
    g, u = ref[:, :N // 2], ref[:, N // 2:]
    eg, eu = err[:, :N // 2], err[:, N // 2:]
    h = g / (1 + torch.exp(-g)) * u
    # |silu'| <= 1.1; __expf and the quotient a few roundings
    _within(outs[0], h, (ulp + 2.0 ** -20) * h.abs() + 1.1 * eg * u.abs() +
            g.abs() * eu + 2.0 ** -24)
    assert torch.equal(*outs)
    # rotary store: two heads' queries and two heads' keys, then values
    pos = torch.arange(M, device="cuda", dtype=torch.int32) % 50 + 3
    ang = torch.arange(60, device="cuda").double()[:, None] * \
        10000.0 ** (-torch.arange(64, device="cuda").double() / 64)
    cs = torch.stack([ang.cos(), ang.sin()], -1).float()
    outs = [run(EPI_STORE, tile, fresh(N), N, pos=pos, cs=cs, rope_cols=512)
            for tile in (PHASED, SIXTEEN_WAVES)]
    x = ref[:, :512].reshape(M, 4, 2, 64)
    e = err[:, :512].reshape(M, 4, 2, 64).sum(2, keepdim=True)
    c = cs[pos.long()].double()[:, None]
    rot = torch.stack([x[:, :, 0] * c[..., 0] - x[:, :, 1] * c[..., 1],
                       x[:, :, 1] * c[..., 0] + x[:, :, 0] * c[..., 1]], 2)
    _within(outs[0][:, :512].reshape(M, 4, 2, 64), rot, ulp * rot.abs() + e +
            2.0 ** -22 * x.abs().sum(2, keepdim=True) + 2.0 ** -24)
    assert torch.equal(*outs)
    assert torch.equal(outs[0][:, 512:], stored[:, 512:])


@pytest.mark.parametrize("epi", [EPI_ADD_F32, EPI_SWIGLU])
@pytest.mark.parametrize("ksplit,K", [(2, 448), (3, 448), (5, 1088), (8, 1024)])
@pytest.mark.parametrize("M", [1, 65, 256, 321, 4353])
def test_split_partials(M, ksplit, K, epi):
    N = 512
    A, B, ref, mag = _operands(M, N, K, torch.float16, M + ksplit)
    slabs = -(-(K // 64) // ksplit) * 64
    parts = []
    for tile in (PHASED, SIXTEEN_WAVES):
        part = torch.full((ksplit * M * N + 64,), SENTINEL, device="cuda")
        assert launch_gemm16(dv.DAVET_F16, epi, tile, ksplit, A, B,
                             B[N // 2:] if epi == EPI_SWIGLU else None, None, M,
                             N, K, N, part=part) == 0
        torch.cuda.synchronize()
        assert bool((part[ksplit * M * N:] == SENTINEL).all())
        parts.append(part[:ksplit * M * N].reshape(ksplit, M, N))
    for k in range(ksplit):
        a = A[:, k * slabs:(k + 1) * slabs].double()
        b = B[:, k * slabs:(k + 1) * slabs].double()
        _within(parts[0][k], a @ b.T, 2.0 ** -22 * (a.abs() @ b.abs().T))
    assert torch.equal(*parts)


def test_split_without_work_is_refused():
    # 6 parts of 7 slabs: two each leave the last two parts none
    A = torch.zeros((1, 448), device="cuda", dtype=torch.float16)
    B = torch.zeros((256, 448), device="cuda", dtype=torch.float16)
    part = torch.zeros(6 * 256, device="cuda")
    assert launch_gemm16(dv.DAVET_F16, EPI_ADD_F32, PHASED, 6, A, B, None, None,
                         1, 256, 448, 256, part=part) != 0
