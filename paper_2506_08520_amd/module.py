"""PyTorch-ROCm modules around the window-attention block of libnystra.

``NystraWindowAttention`` is a drop-in replacement for the (shifted-)window
multi-head self-attention of SwinIR / Uformer-style restoration models (the
W-MSA / SW-MSA module of Sec. 1): feature map in, feature map out, with the
QKV projection, window partition, attention, head merge, output projection
and window reverse all in HIP kernels (``nystra_block_forward``).  PnP-Nystra
is training-free, so the modules are inference-only: their outputs carry no
autograd history.

``SwinTransformerBlock`` is the transformer block those models stack
(LayerNorm, window attention, residual, LayerNorm, MLP, residual), with the
window attention replaced; LayerNorm and the MLP are plain torch layers, run
as such or, where nothing observes or alters them, by the fused bf16 kernels of
nystra_layer_forward with the same weights.
Relative-position bias and the shifted-window mask are not applied: Eqs.
(1)-(8) have neither.
"""
import math

import torch
from torch import nn

from . import binding as B


class NystraWindowAttention(nn.Module):
    """Window attention on x [B, H, W, C] (channels last, contiguous).

    Weights follow the ``y = x W`` convention of the C ABI: ``w_qkv`` [C, 3C]
    (Q, K, V column blocks, head j taking columns j d_h .. (j+1) d_h - 1 of
    each), ``w_proj`` [C, C].  ``attention`` is "nystrom" (PnP-Nystra with
    ``m`` landmarks and ``iters`` pseudo-inverse iterations) or "exact"."""

    def __init__(self, dim, heads, window, shift=0, m=16, iters=6, attention="nystrom",
                 landmark_mode=B.LM_POOL2D, dtype=torch.float32, device="cuda"):
        super().__init__()
        if dim % heads != 0:
            raise ValueError("heads must divide dim")
        if attention not in ("nystrom", "exact"):
            raise ValueError(attention)
        self.dim, self.heads, self.window, self.shift = dim, heads, window, shift
        self.m, self.iters, self.attention = m, iters, attention
        self.opts = B.make_opts(pinv_iters=iters, landmark_mode=landmark_mode)
        kw = dict(dtype=dtype, device=device)
        self.w_qkv = nn.Parameter(torch.empty(dim, 3 * dim, **kw), requires_grad=False)
        self.b_qkv = nn.Parameter(torch.zeros(3 * dim, **kw), requires_grad=False)
        self.w_proj = nn.Parameter(torch.empty(dim, dim, **kw), requires_grad=False)
        self.b_proj = nn.Parameter(torch.zeros(dim, **kw), requires_grad=False)
        self._ws = None
        self._packed, self._packed_key = None, None

    @classmethod
    def from_linear(cls, qkv, proj, heads, window, shift=0, **kw):
        """From the nn.Linear layers of an existing model (weight [out, in])."""
        dim = proj.in_features
        mod = cls(dim, heads, window, shift, dtype=qkv.weight.dtype,
                  device=qkv.weight.device, **kw)
        with torch.no_grad():
            mod.w_qkv.copy_(qkv.weight.t())
            mod.w_proj.copy_(proj.weight.t())
            if qkv.bias is not None:
                mod.b_qkv.copy_(qkv.bias)
            if proj.bias is not None:
                mod.b_proj.copy_(proj.bias)
        return mod

    def _workspace(self, x):
        shape = B.BlockShape(*x.shape[:3], self.dim, self.heads, self.window, self.shift)
        att = B.BLOCK_NYSTROM if self.attention == "nystrom" else B.BLOCK_EXACT
        code = B.F32 if x.dtype == torch.float32 else B.BF16
        need = B.nystra_block_workspace_size(shape, self.m, code, self.opts, att)
        if self._ws is None or self._ws.numel() < need or self._ws.device != x.device:
            self._ws = torch.empty(max(need, 1), dtype=torch.uint8, device=x.device)
        return self._ws, att

    def _packed_weights(self):
        """The GEMMs' packed image of w_qkv and w_proj, packed again only when
        either weight changed (new storage, or an in-place update, which
        advances the tensor's version counter)."""
        key = tuple((t.data_ptr(), t._version, t.dtype) for t in (self.w_qkv, self.w_proj))
        if key != self._packed_key:
            self._packed = B.nystra_block_pack_weights(self.w_qkv, self.w_proj)
            self._packed_key = key
        return self._packed

    @torch.no_grad()
    def forward(self, x):
        if x.dim() != 4 or x.shape[-1] != self.dim:
            raise ValueError(f"expected [B, H, W, {self.dim}]")
        x = x.contiguous()
        ws, att = self._workspace(x)
        return B.nystra_block_forward(x, self.w_qkv, self.b_qkv, self.w_proj, self.b_proj,
                                      self.heads, self.window, shift=self.shift, m=self.m,
                                      opts=self.opts, attention=att, workspace=ws,
                                      packed=self._packed_weights())


class SwinTransformerBlock(nn.Module):
    """x + attn(norm1(x)), then + mlp(norm2(.)), on x [B, H, W, C]."""

    def __init__(self, dim, heads, window, shift=0, mlp_ratio=2.0, m=16, iters=6,
                 attention="nystrom", dtype=torch.float32, device="cuda"):
        super().__init__()
        kw = dict(dtype=dtype, device=device)
        self.norm1 = nn.LayerNorm(dim, **kw)
        self.attn = NystraWindowAttention(dim, heads, window, shift, m, iters, attention,
                                          dtype=dtype, device=device)
        self.norm2 = nn.LayerNorm(dim, **kw)
        hidden = int(dim * mlp_ratio)
        self.mlp = nn.Sequential(nn.Linear(dim, hidden, **kw), nn.GELU(),
                                 nn.Linear(hidden, dim, **kw))

    def _fusable(self, x):
        """Whether nystra_layer_forward computes what the composition of the
        layers does: plain layers of their exact types with bf16 weights on x's
        device, no hook on any of them, no autocast, tracing, compilation, transform,
        forward-mode level or torch mode that would see the torch calls.

        fp32, and more than 256 channels, keep the composition (there is no fused
        kernel for them)."""
        # What has no fused kernel leaves before the submodules are looked up: 4 us
        # of a 110 us call at C = 320, 1024 rows.
        if (type(x) is not torch.Tensor or x.dtype != torch.bfloat16 or not x.is_cuda or
                x.dim() != 4 or x.numel() == 0):
            return False
        C = x.shape[-1]
        if C > 256 or C % 4 != 0:
            return False
        n1, n2, attn, mlp = self.norm1, self.norm2, self.attn, self.mlp
        if (type(attn) is not NystraWindowAttention or type(n1) is not nn.LayerNorm or
                type(n2) is not nn.LayerNorm or type(mlp) is not nn.Sequential or len(mlp) != 3):
            return False
        fc1, act, fc2 = mlp
        if (type(fc1) is not nn.Linear or type(act) is not nn.GELU or type(fc2) is not nn.Linear or
                act.approximate != "none" or attn.dim != C or attn.heads < 1 or
                (C // attn.heads) % 2 != 0 or
                n1.normalized_shape != (C,) or n2.normalized_shape != (C,) or
                not (math.isfinite(n1.eps) and math.isfinite(n2.eps))):
            return False
        hidden = fc1.weight.shape[0]
        # The biases of the MLP may be absent; the norms' weights and biases may not.
        want = [(n1.weight, (C,)), (n1.bias, (C,)), (n2.weight, (C,)), (n2.bias, (C,)),
                (fc1.weight, (hidden, C)), (fc2.weight, (C, hidden)),
                (attn.w_qkv, (C, 3 * C)), (attn.b_qkv, (3 * C,)),
                (attn.w_proj, (C, C)), (attn.b_proj, (C,))]
        if fc1.bias is not None:
            want.append((fc1.bias, (hidden,)))
        if fc2.bias is not None:
            want.append((fc2.bias, (C,)))
        for t, shape in want:
            if (type(t) not in (nn.Parameter, torch.Tensor) or t.dtype != x.dtype or
                    t.device != x.device or tuple(t.shape) != shape or not t.is_contiguous()):
                return False
        if hidden % 4 != 0 or hidden < 4 or any(
                t.data_ptr() % 4 != 0 for t in (x, fc1.weight, fc2.weight)):
            return False
        if any(p.data_ptr() % 4 != 0 for p in (attn.w_qkv, attn.w_proj)):
            return False
        if 3 * (x.numel() + 128) >= 1 << 32 or x.numel() >= 1 << 31:
            return False
        mod = nn.modules.module
        if (mod._global_forward_hooks or mod._global_forward_pre_hooks or
                any(s._forward_hooks or s._forward_pre_hooks or "forward" in s.__dict__
                    for s in (n1, n2, attn, mlp, fc1, act, fc2))):
            return False
        return not (torch.is_autocast_enabled("cuda") or torch.jit.is_tracing() or
                    torch.compiler.is_compiling() or torch._C._len_torch_function_stack() or
                    torch._C._len_torch_dispatch_stack() or
                    torch._C._functorch.peek_interpreter_stack() is not None or
                    torch.autograd.forward_ad._current_level >= 0)

    def _forward_fused(self, x):
        attn, (fc1, _, fc2) = self.attn, self.mlp
        xc = x.contiguous()
        ws, att = attn._workspace(xc)
        y = B.nystra_layer_forward(
            xc, attn.w_qkv, attn.b_qkv, attn.w_proj, attn.b_proj, attn._packed_weights(),
            (self.norm1.weight, self.norm1.bias, self.norm1.eps),
            (self.norm2.weight, self.norm2.bias, self.norm2.eps), fc1.weight, fc1.bias,
            fc2.weight, fc2.bias, attn.heads, attn.window, shift=attn.shift, m=attn.m,
            opts=attn.opts, attention=att, workspace=ws)
        # A residual sum lays its result out as x lies (densely, in x's order
        # of the dimensions), so the fused result does too.
        return y if xc is x else torch.empty_like(x).copy_(y)

    @torch.no_grad()
    def forward(self, x):
        if self._fusable(x):
            return self._forward_fused(x)
        x = x + self.attn(self.norm1(x))
        return x + self.mlp(self.norm2(x))
