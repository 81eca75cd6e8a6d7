"""Token counts that are not a multiple of 16, through the automatic choice: the tiled
kernel with a partial last token tile, against the float64 oracle and, for its error and
for values that are not finite, the generic kernel that ran such shapes before.  Covers
one to four landmark-tile counts per residue of N mod 32 (a missing second tile, a
partial one), single tokens, m = N and both landmark modes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_08520_amd import binding as B
from paper_2506_08520_amd import workloads as W
from helpers import check, to_dev, to_host

pytestmark = pytest.mark.gpu

# (n_windows, heads, N, d, m, mode)
SHAPES = [
    (1, 1, 1, 8, 1, 0),       # one token
    (3, 2, 4, 12, 4, 0),      # m = N, one partial tile
    (5, 2, 9, 16, 9, 0),
    (2, 3, 17, 32, 17, 1),    # one token past a tile, two landmark tiles
    (2, 2, 31, 24, 1, 1),     # one token short of a pair of tiles
    (2, 2, 33, 30, 11, 1),    # a third tile of one token
    (3, 2, 36, 30, 9, 0),     # 6 x 6 windows
    (3, 2, 49, 32, 7, 0),     # 7 x 7: a fourth tile of one token
    (2, 2, 81, 20, 9, 0),
    (2, 2, 100, 16, 25, 0),   # 10 x 10: two landmark tiles
    (1, 2, 196, 28, 49, 0),   # 14 x 14: four landmark tiles
    (1, 2, 126, 8, 63, 1),
    (1, 2, 42, 32, 42, 1),    # three landmark tiles, m = N
    (1, 1, 2025, 30, 25, 0),  # 45 x 45
    (1, 1, 9999, 16, 33, 1),  # long segments
    (1, 1, 9604, 32, 49, 0),  # 98 x 98
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_ragged(shape, dtype):
    nw, h, N, d, m, mode = shape
    q, k, v = W.iid((nw, h, N, d), seed=N * 17 + d + m, dtype=dtype)
    ref = oracle.forward(q, k, v, m, iters=6, mode=mode)
    t = [to_dev(x, dtype) for x in (q, k, v)]
    got = to_host(B.nystra_attn_forward_ex(*t, m, opts=B.make_opts(landmark_mode=mode)))
    check(got, ref, dtype, f"ragged {shape} {dtype}")


@pytest.mark.parametrize("shape", [(40, 2, 49, 30, 7, 0), (20, 2, 100, 16, 25, 0),
                                   (8, 2, 196, 32, 49, 0), (20, 1, 126, 24, 9, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_bf16_is_computed_in_fp32(shape):
    """bf16 inputs, fp32 arithmetic: past the rounding of the stored result, the
    error is that of fp32 sums (at most 1e-5 of RMS over these shapes: a few
    hundred roundings of 6e-8), where 16-bit operands measure 4e-5 and more."""
    nw, h, N, d, m, mode = shape
    q, k, v = W.iid((nw, h, N, d), seed=N * 17 + d + m, dtype="bf16")
    ref = oracle.forward(q, k, v, m, iters=6, mode=mode)
    t = [to_dev(x, "bf16") for x in (q, k, v)]
    got = to_host(B.nystra_attn_forward_ex(*t, m, opts=B.make_opts(landmark_mode=mode)))
    check(got, ref, "bf16", f"ragged {shape} bf16", beyond_bar=1e-5)


@pytest.mark.parametrize("N,d,m", [(36, 24, 1), (36, 20, 6), (49, 24, 7), (100, 24, 1),
                                   (100, 16, 25), (225, 30, 9), (900, 30, 1), (900, 30, 2)])
def test_error_is_the_generic_kernels(N, d, m):
    """fp32: the median over 512 units of a unit's error against 64 bits, beside that
    of the generic kernel.  Both are a few roundings of 6e-8; 15% is what the median
    moves with another draw (3%) and what shapes differ by either way (10%), where
    one chain of roundings over the keys measures 1.4 to 1.7."""
    side = int(round(N ** 0.5))
    g = torch.Generator().manual_seed(N + d + m)
    q, k, v = (torch.randn(512, 1, N, d, generator=g) for _ in range(3))
    rows = [n for n in range(1, m + 1) if m % n == 0 and side % n == 0 and side % (m // n) == 0]
    gc = max(n for n in rows if n * n <= m)
    gr = m // gc

    def pool(x):
        x = x.view(512, gr, side // gr, gc, side // gc, d)
        return x.mean((2, 4)).reshape(512, m, d)

    q6, k6, v6 = (t.double()[:, 0] for t in (q, k, v))
    s, qb, kb = d ** -0.5, pool(q6), pool(k6)
    su = s * (qb @ k6.transpose(1, 2))
    mu = su.amax(2, keepdim=True)
    gu, a = torch.exp(su - mu), torch.exp(s * (qb @ kb.transpose(1, 2)) - mu)
    z = a.transpose(1, 2) / (a.sum(1).amax(1) * a.sum(2).amax(1)).view(-1, 1, 1)
    eye = torch.eye(m, dtype=a.dtype)
    for _ in range(6):
        x = a @ z
        z = 0.25 * (z @ (13 * eye - x @ (15 * eye - x @ (7 * eye - x))))
    gl = torch.softmax(s * (q6 @ kb.transpose(1, 2)), 2)
    ref = (gl @ (z @ (gu @ v6))) / (gl @ (z @ gu.sum(2, keepdim=True)))
    err = {}
    for variant in (B.VARIANT_GENERIC, B.VARIANT_AUTO):
        o = B.nystra_attn_forward_ex(q.cuda(), k.cuda(), v.cuda(), m,
                                     opts=B.make_opts(variant=variant)).cpu().double()[:, 0]
        e = (o - ref).square().sum((1, 2)) / ref.square().sum((1, 2))
        err[variant] = e.sqrt().median().item()
    ratio = err[B.VARIANT_AUTO] / err[B.VARIANT_GENERIC]
    print(f"ragged N={N} d={d} m={m}: {err[B.VARIANT_AUTO]:.2e}, {ratio:.2f} of the generic kernel's")
    assert ratio <= 1.15


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_neighbours_untouched(dtype):
    """Rows past a unit's last token are the next unit's: outputs of every unit
    equal those of the unit computed alone, and the bytes after O stay."""
    q, k, v = (to_dev(x, dtype) for x in W.iid((7, 1, 49, 30), seed=3, dtype=dtype))
    pad = 64
    buf = torch.full((q.numel() + pad,), 7.0, dtype=q.dtype, device="cuda")
    out = buf[:q.numel()].view(q.shape)
    B.nystra_attn_forward_ex(q, k, v, 7, out=out)
    assert (buf[q.numel():] == 7.0).all()
    for u in (0, 3, 6):
        alone = B.nystra_attn_forward_ex(q[u:u + 1].contiguous(), k[u:u + 1].contiguous(),
                                         v[u:u + 1].contiguous(), 7)
        assert torch.equal(alone[0], out[u])
    for t in (q, k, v):                 # nothing of a neighbour's rows reaches a unit
        t[3] = float("nan")
    again = B.nystra_attn_forward_ex(q, k, v, 7)
    assert torch.isnan(again[3]).all()
    assert all(torch.equal(again[u], out[u]) for u in (0, 1, 2, 4, 5, 6))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,d,m,mode", [(36, 12, 1, 0), (49, 30, 7, 0), (49, 16, 7, 0),
                                        (100, 16, 25, 0), (100, 20, 25, 0), (196, 32, 49, 0),
                                        (105, 24, 35, 1)])
def test_values_that_are_not_finite(N, d, m, mode, dtype):
    """-inf keys mask, as do keys of the type's lowest value: the first tokens (whole
    pairs of tiles of a wave), the last ones, single ones.  Infinities and NaN in V reach their
    column and nothing else.  Everything as the generic kernel gives it."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(N + d + m)
    q, k, v = (torch.randn(8, 1, N, d, generator=g) for _ in range(3))
    q = q.abs() + 0.5
    side = int(round(N ** 0.5))
    low = torch.finfo(tdt).min
    third = (N // 3 // side) * side if mode == 0 else N // 3
    # every feature, the first only, the last only: each slot of a chunk of eight
    k[0, :, :third], k[1, :, :third, 0], k[2, :, N - 1, d - 1] = -np.inf, -np.inf, -np.inf
    k[3, :, min(40, N // 2):], k[4, :, 5] = -np.inf, low
    v[5, :, N - 2, 3], v[6, :, 1, d - 1] = np.inf, np.nan
    t = [x.to(tdt).cuda() for x in (q, k, v)]
    got, ref = (B.nystra_attn_forward_ex(*t, m, opts=B.make_opts(landmark_mode=mode, variant=var))
                .float().cpu() for var in (B.VARIANT_AUTO, B.VARIANT_GENERIC))
    assert torch.isfinite(ref[7]).all() and (m == 1 or torch.isfinite(ref[0]).all())
    for u in range(8):
        same = torch.equal(torch.isnan(got[u]), torch.isnan(ref[u])) and \
            torch.equal(got[u][torch.isinf(ref[u])], ref[u][torch.isinf(ref[u])])
        ok = torch.isfinite(ref[u])
        near = same and torch.allclose(got[u][ok], ref[u][ok], rtol=2e-2, atol=2e-2)
        assert near, f"unit {u}: {int(torch.isnan(got[u]).sum())} NaN, {int(torch.isnan(ref[u]).sum())} expected"


def test_automatic_choice_is_the_tiled_kernel():
    """The two kernels add in other orders, so their bits tell them apart; a head width
    without a tiled form stays with the generic one."""
    for d, tiled in ((16, True), (22, False)):
        t = [to_dev(x, "f32") for x in W.iid((4, 2, 100, d), seed=11, dtype="f32")]
        auto = B.nystra_attn_forward_ex(*t, 25)
        generic = B.nystra_attn_forward_ex(*t, 25, opts=B.make_opts(variant=B.VARIANT_GENERIC))
        assert torch.equal(auto, generic) != tiled
        assert (auto - generic).abs().max() <= 1e-4


def test_named_variants_unchanged():
    """By name such shapes stay GENERIC only."""
    assert B.nystra_select_variant(100, 16, 25) == B.VARIANT_GENERIC
    q = torch.zeros((1, 1, 100, 16), device="cuda")
    with pytest.raises(B.NystraError):
        B.nystra_attn_forward_ex(q, q, q, 25, opts=B.make_opts(variant=B.VARIANT_TILED))


def test_unaligned_bf16_takes_the_generic_kernel():
    """bf16 tensors on odd halfwords (not 4-byte aligned) stay accepted."""
    q, k, v = W.iid((2, 1, 49, 30), seed=9, dtype="bf16")
    t = []
    for x in (q, k, v):
        b = torch.empty(x.size + 1, dtype=torch.bfloat16, device="cuda")
        b[1:] = to_dev(x, "bf16").view(-1)
        t.append(b[1:].view(x.shape))
    got = to_host(B.nystra_attn_forward_ex(*t, 7))
    check(got, oracle.forward(q, k, v, 7, iters=6, mode=0), "bf16", "ragged, odd halfwords")
