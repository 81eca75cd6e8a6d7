"""The fused bf16 transformer layer against the composition of torch layers it
stands for, both measured against float64: LayerNorm, block, residual,
LayerNorm, MLP, residual.  The fused path keeps the residual stream and the
MLP's sums in fp32 where the composition rounds them to bf16, so its error must
not be larger than the composition's (with 10% for the other draw of
roundings), besides a bound of its own."""
import numpy as np
import pytest
import torch
from scipy.special import erf
from torch import nn

from oracle import block as OB
from paper_2506_08520_amd.module import SwinTransformerBlock

pytestmark = pytest.mark.gpu


def make(C, heads, w, s, m, attention, ratio=2.0, seed=0):
    torch.manual_seed(seed)
    blk = SwinTransformerBlock(C, heads, w, s, m=m, mlp_ratio=ratio, attention=attention,
                               dtype=torch.bfloat16)
    with torch.no_grad():
        blk.attn.w_qkv.copy_(torch.randn(C, 3 * C) / C ** 0.5)
        blk.attn.b_qkv.copy_(0.02 * torch.randn(3 * C))
        blk.attn.w_proj.copy_(torch.randn(C, C) / C ** 0.5)
        blk.attn.b_proj.copy_(0.02 * torch.randn(C))
        for ln in (blk.norm1, blk.norm2):
            ln.weight.copy_(1 + 0.1 * torch.randn(C))
            ln.bias.copy_(0.1 * torch.randn(C))
        blk.mlp[0].weight.mul_(1.7)
        blk.mlp[2].weight.mul_(1.7)
    return blk.eval()


def composed(blk, x):
    """The layer as separate torch layers around the attention module."""
    x = x + blk.attn(blk.norm1(x))
    return x + blk.mlp(blk.norm2(x))


def n64(t):
    return t.detach().double().cpu().numpy()


def layer_norm(x, ln):
    mu = x.mean(-1, keepdims=True)
    var = ((x - mu) ** 2).mean(-1, keepdims=True)
    return (x - mu) / np.sqrt(var + ln.eps) * n64(ln.weight) + n64(ln.bias)


def exact(blk, x):
    a, (l1, _, l2) = blk.attn, blk.mlp
    xn = n64(x)
    h = xn + OB.block_forward(layer_norm(xn, blk.norm1), n64(a.w_qkv), n64(a.b_qkv),
                              n64(a.w_proj), n64(a.b_proj), heads=a.heads, window=a.window,
                              shift=a.shift, m=max(a.m, 1), attention=a.attention)
    b1 = 0 if l1.bias is None else n64(l1.bias)
    b2 = 0 if l2.bias is None else n64(l2.bias)
    u = layer_norm(h, blk.norm2) @ n64(l1.weight).T + b1
    return h + (0.5 * u * (1 + erf(u / np.sqrt(2)))) @ n64(l2.weight).T + b2


# Channels at and beside each padded width (32, 64, 128, 192, 256), rows that
# leave a partial row tile (4 x 12 = 48, 15 x 20 = 300), hidden widths with a
# partial last step (4, 36, 360), and both attentions.
CASES = [
    (1, 4, 12, 4, 2, 4, 2, 4, "nystrom", 1.0),
    (1, 15, 20, 28, 1, 5, 2, 1, "nystrom", 9 / 7),
    (2, 8, 16, 32, 1, 8, 4, 8, "nystrom", 2.0),
    (1, 16, 24, 36, 1, 8, 0, 16, "exact", 1.0),
    (1, 16, 16, 64, 2, 16, 8, 32, "nystrom", 4.0),
    (1, 20, 30, 96, 6, 10, 5, 25, "nystrom", 2.0),
    (1, 16, 16, 128, 4, 8, 4, 16, "nystrom", 2.0),
    (2, 24, 16, 180, 6, 8, 4, 16, "nystrom", 2.0),
    (1, 8, 8, 192, 6, 8, 0, 16, "exact", 0.0625),
    (1, 7, 21, 240, 8, 7, 3, 7, "nystrom", 2.0),
    (1, 16, 32, 256, 8, 8, 4, 16, "nystrom", 2.0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_fused_layer(case):
    Bn, H, Wd, C, heads, w, s, m, attention, ratio = case
    blk = make(C, heads, w, s, m, attention, ratio)
    x = torch.randn(Bn, H, Wd, C, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    assert blk._fusable(x)
    ref = exact(blk, x)
    y, z = blk(x), composed(blk, x)
    rms = np.sqrt((ref ** 2).mean())
    e = {k: np.sqrt(((n64(t) - ref) ** 2).mean()) / rms for k, t in (("fused", y), ("composed", z))}
    print(f"layer {case}: rel {e}")
    # bf16 roundings of the normalised rows, Q/K/V, O, the hidden units and Y:
    # about six of 2^-9 / sqrt(3) each, amplified by the pseudo-inverse.
    assert e["fused"] <= 1.3e-2
    assert e["fused"] <= 1.1 * e["composed"]
    assert np.abs(n64(y) - ref).max() <= 0.15 * rms


# Maps whose QKV product runs on the row-resident kernel (128 row blocks of 128 and
# more) at each padded width, and on the weight-resident one with two row tiles a wave.
LARGE = [
    (1, 128, 136, 28, 2, 8, 4, 16), (1, 130, 130, 32, 1, 10, 5, 25), (1, 128, 136, 60, 2, 8, 0, 16),
    (1, 133, 126, 96, 6, 7, 3, 7), (2, 72, 128, 128, 4, 8, 4, 16), (1, 128, 136, 180, 6, 8, 4, 16),
    (1, 130, 130, 240, 8, 10, 5, 25), (1, 128, 128, 256, 8, 8, 4, 32),
    (1, 80, 160, 240, 8, 8, 4, 16), (1, 100, 130, 256, 8, 10, 0, 25),
]


@pytest.mark.parametrize("case", LARGE, ids=lambda c: "x".join(map(str, c)))
def test_fused_layer_large_maps(case):
    """As test_fused_layer, on six windows of the map (the last rows among them)."""
    Bn, H, Wd, C, heads, w, s, m = case
    blk = make(C, heads, w, s, m, "nystrom")
    x = torch.randn(Bn, H, Wd, C, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    assert blk._fusable(x)
    idx = OB.window_tokens_roll(Bn, H, Wd, w, s)
    pick = idx[np.unique(np.linspace(0, idx.shape[0] - 1, 6).round().astype(int))]
    rows = torch.from_numpy(pick).cuda()
    y, z = blk(x), composed(blk, x)
    assert torch.isfinite(y).all()
    blk.attn.shift = 0
    ref = exact(blk, x.view(-1, C)[rows].view(-1, w, w, C))
    rms = np.sqrt((ref ** 2).mean())
    e = {k: np.sqrt(((n64(t.view(-1, C)[rows]).reshape(ref.shape) - ref) ** 2).mean()) / rms
         for k, t in (("fused", y), ("composed", z))}
    print(f"layer {case}: rel {e}")
    assert e["fused"] <= 1.3e-2
    assert e["fused"] <= 1.1 * e["composed"]


def test_no_biases():
    blk = make(64, 2, 8, 4, 16, "nystrom")
    blk.mlp[0].bias = blk.mlp[2].bias = None
    x = torch.randn(1, 16, 16, 64, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    assert blk._fusable(x)
    ref = exact(blk, x)
    assert np.sqrt(((n64(blk(x)) - ref) ** 2).mean() / (ref ** 2).mean()) <= 1.3e-2


@pytest.mark.parametrize("affine,biases", [(False, False), (False, True), (True, False)])
def test_norms_without_parameters(affine, biases):
    """LayerNorm without weight and bias, or without bias alone, is composed,
    whatever biases the MLP has."""
    blk = make(64, 2, 8, 4, 16, "nystrom")
    kw = dict(dtype=torch.bfloat16, device="cuda")
    blk.norm1 = nn.LayerNorm(64, elementwise_affine=affine, bias=False, **kw)
    if not biases:
        blk.mlp[0].bias = blk.mlp[2].bias = None
    x = torch.randn(1, 16, 16, 64, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    assert not blk._fusable(x) and torch.equal(blk(x), composed(blk, x))


@pytest.mark.parametrize("eps", [float("inf"), float("nan")])
def test_eps_that_is_not_finite(eps):
    """Refused by the C entry, so composed."""
    blk = make(64, 2, 8, 4, 16, "nystrom")
    blk.norm2.eps = eps
    x = torch.randn(1, 16, 16, 64, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    y, z = blk(x), composed(blk, x)
    assert not blk._fusable(x) and torch.equal(torch.isnan(y), torch.isnan(z))
    assert torch.equal(y.nan_to_num(), z.nan_to_num())


@pytest.mark.parametrize("layout", ["channels first", "transposed", "slice", "rows", "expanded"])
def test_layout_of_the_result(layout):
    """The result lies in memory as the composition's does."""
    blk = make(64, 2, 8, 4, 16, "nystrom")
    g = torch.Generator().manual_seed(7)
    x = torch.randn(2, 64, 16, 24, generator=g).bfloat16().cuda()
    x = {"channels first": lambda: x.permute(0, 2, 3, 1),
         "transposed": lambda: x.permute(0, 2, 3, 1).contiguous().transpose(1, 2),
         "slice": lambda: torch.cat([x, x], 1).permute(0, 2, 3, 1).contiguous()[..., 64:],
         "rows": lambda: x.permute(0, 3, 2, 1).contiguous()[:, ::3],
         "expanded": lambda: x[:1].permute(0, 2, 3, 1).contiguous().expand(3, 16, 24, 64)}[layout]()
    assert not x.is_contiguous() and blk._fusable(x)
    y = blk(x)
    assert y.stride() == composed(blk, x).stride()
    assert torch.equal(y, blk(x.contiguous()))


def test_weights_are_read_every_call():
    """Writes through .data (no version bump) to the norms and the MLP count."""
    blk = make(64, 2, 8, 4, 16, "nystrom")
    x = torch.randn(1, 16, 16, 64, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    blk(x)
    for p in (blk.norm1.weight, blk.norm2.bias, blk.mlp[0].weight, blk.mlp[2].weight,
              blk.mlp[2].bias):
        p.data.mul_(1.5)
    ref = exact(blk, x)
    assert np.sqrt(((n64(blk(x)) - ref) ** 2).mean() / (ref ** 2).mean()) <= 1.3e-2


def test_large_values_and_gelu_tails():
    """Hidden units far into both tails of the GELU, rows with a large mean."""
    blk = make(64, 2, 8, 0, 16, "exact", 4.0)
    with torch.no_grad():
        blk.mlp[0].weight.mul_(10)
    x = torch.randn(1, 16, 16, 64, generator=torch.Generator().manual_seed(9)) * 3 + 40
    x = x.bfloat16().cuda()
    ref, y, z = exact(blk, x), blk(x), composed(blk, x)
    rms = np.sqrt((ref ** 2).mean())
    assert np.sqrt(((n64(y) - ref) ** 2).mean()) <= 1.1 * np.sqrt(((n64(z) - ref) ** 2).mean())
    assert np.isfinite(n64(y)).all() and rms > 0


def test_values_that_are_not_finite():
    """NaN and infinities stay in the windows of their tokens, and in a token's own
    row where they arise after the attention, as in the composition."""
    blk = make(64, 2, 8, 4, 16, "exact")
    x = torch.randn(1, 32, 32, 64, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    x[0, 5, 6, 7], x[0, 21, 30, 0] = float("nan"), float("inf")
    y, z = blk(x), composed(blk, x)
    assert torch.equal(torch.isfinite(y), torch.isfinite(z))
    assert (~torch.isfinite(y)).sum() == 2 * 64 * 64
    ok = torch.isfinite(z)
    assert (y[ok].float() - z[ok].float()).abs().max() <= 0.15 * z[ok].float().std()
    x = x.nan_to_num(nan=0.5, posinf=0.5)
    blk.mlp[0].bias.data[5] = float("inf")       # GELU(inf) = inf: every value of Y
    y, z = blk(x), composed(blk, x)
    assert torch.equal(torch.isnan(y), torch.isnan(z)) and torch.equal(y[torch.isinf(z)], z[torch.isinf(z)])
    assert torch.isinf(z).any()


@pytest.mark.parametrize("C,H", [(64, 16), (180, 128), (320, 16)])
def test_graph_replays(C, H):
    """The layer captured in a graph: replays after changes of the input, with the
    program's own work between them, equal the eager call."""
    blk = make(C, C // 30 if C == 180 else C // 32, 8, 4, 16, "nystrom")
    gen = torch.Generator().manual_seed(7)
    x = torch.randn(1, H, H, C, generator=gen).bfloat16().cuda()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        blk(x)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = blk(x)
    for _ in range(3):
        x.copy_(torch.randn(1, H, H, C, generator=gen).bfloat16())
        want = blk(x).clone()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


class _Twice(nn.Linear):
    def forward(self, x):
        return 2 * super().forward(x)


def test_observed_or_altered_layers_are_composed():
    x = torch.randn(1, 16, 16, 64, generator=torch.Generator().manual_seed(7)).bfloat16().cuda()
    seen = []
    blk = make(64, 2, 8, 4, 16, "nystrom")
    h = blk.mlp[1].register_forward_hook(lambda *a: seen.append(1))
    assert not blk._fusable(x) and torch.equal(blk(x), composed(blk, x)) and seen
    h.remove()
    assert blk._fusable(x)
    blk.mlp[1] = nn.GELU(approximate="tanh")
    assert not blk._fusable(x)
    blk = make(64, 2, 8, 4, 16, "nystrom")
    lin = _Twice(64, 128, dtype=torch.bfloat16, device="cuda")
    lin.load_state_dict(blk.mlp[0].state_dict())
    blk.mlp[0] = lin
    assert not blk._fusable(x) and torch.equal(blk(x), composed(blk, x))
    blk = make(64, 2, 8, 4, 16, "nystrom")
    assert not blk._fusable(x.float())
    with torch.autocast("cuda", dtype=torch.bfloat16):
        assert not blk._fusable(x)
    with torch.autograd.forward_ad.dual_level():
        assert not blk._fusable(x)
    assert blk._fusable(x.transpose(1, 2))   # other strides: made contiguous
    assert torch.equal(blk(x.transpose(1, 2)), blk(x.transpose(1, 2).contiguous()))
