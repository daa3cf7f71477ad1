"""One global-attention transformer block of a VGGT-like aggregator around the bsga library
(Sec. 3.1 for the alternating-attention design, Sec. 4.1 / 4.2 for what replaces the dense global
attention; the appendix "Theoretical FLOPs Reduction" for the block's parts: attention with its
projections plus an MLP with d_ff = 4 d).

Integration shape only: random weights, timing and parity of the data path.  The projections, the
layer norms and the MLP run on the bsga kernels in bf16 and are plain torch ops otherwise; pooling, selection,
block-sparse attention and the reorderings of tokens and heads are the bsga kernels.
"""
from __future__ import annotations

from typing import Optional

import torch
import torch.nn.functional as F
import torch.utils._device
from torch.autograd import forward_ad

from . import binding as B

# Torch has no public names for these: without one of them no pass is taken past torch's operations.
_function_modes = getattr(torch.overrides, "_get_current_function_mode_stack", None)
_dispatch_modes = getattr(torch._C, "_len_torch_dispatch_stack", None)
_DeviceContext = getattr(torch.utils._device, "DeviceContext", None)


def _calls_are_watched() -> bool:
    """Whether torch's operations are more than their results just now: forward-mode tangents, function and dispatch modes (FLOP
    counters, fake tensors; a default device is a function mode as well, but one that asks for nothing here)."""
    if _function_modes is None or _dispatch_modes is None or getattr(forward_ad, "_current_level", 0) >= 0:
        return True
    return _dispatch_modes() > 0 or any(type(m) is not _DeviceContext for m in _function_modes())


class GlobalAttentionBlock(torch.nn.Module):
    """x [N, d_model] (all frames' tokens of one scene) -> x + Attn(LN(x)) -> + MLP(LN(.)).

    heads * 64 == d_model.  `special` (bool [N], optional) marks the camera / register tokens: with it
    the block map is predicted on patch tokens only and everything touching a special token stays
    dense (Sec. 4.2); without it all tokens are treated alike.  tau >= 1 with rho = 1 runs the dense
    kernel.
    """

    def __init__(self, d_model: int = 1024, heads: int = 16, block: int = 128, tau: float = 0.9, rho: float = 1.0,
                 special: Optional[torch.Tensor] = None, mlp: bool = True, dtype=torch.bfloat16, device="cuda",
                 seed: int = 0):
        super().__init__()
        assert d_model == heads * 64, "head dimension must be 64"
        g = torch.Generator(device="cpu").manual_seed(seed)

        def w(*shape, scale):
            return torch.nn.Parameter((torch.randn(*shape, generator=g) * scale).to(dtype).to(device), requires_grad=False)

        self.d_model, self.heads, self.block, self.tau, self.rho = d_model, heads, block, tau, rho
        self.w_qkv = w(3 * d_model, d_model, scale=d_model ** -0.5)
        self.b_qkv = w(3 * d_model, scale=0.02)
        self.w_out = w(d_model, d_model, scale=d_model ** -0.5)
        self.b_out = w(d_model, scale=0.02)
        self.ln1 = torch.nn.LayerNorm(d_model, device=device, dtype=dtype)
        self.mlp = mlp
        if mlp:
            self.ln2 = torch.nn.LayerNorm(d_model, device=device, dtype=dtype)
            self.w_fc1 = w(4 * d_model, d_model, scale=d_model ** -0.5)
            self.b_fc1 = w(4 * d_model, scale=0.02)
            self.w_fc2 = w(d_model, 4 * d_model, scale=(4 * d_model) ** -0.5)
            self.b_fc2 = w(d_model, scale=0.02)
        self.plan = None if special is None else B.SpecialTokenPlan(special, block, device)
        self.last = {}  # q, k, v, o of the last call ([H, N, 64], working order), for tests

    def _folds(self, x: torch.Tensor) -> bool:
        """Whether a pass takes this library's linear layers and layer norms, which fold in the reorderings, the residuals and the GELU
        (transformer block of 10,992 tokens: 583 -> 482 us), and not torch's: bf16 on one device, rows and sizes as these need them,
        plain tensors, and nothing attached to the layer norms that calling them would run."""
        D, N = self.d_model, x.shape[0] if x.dim() == 2 else 0
        if type(x) is not torch.Tensor or not x.is_cuda or N < 1 or x.shape[1] != D or torch.is_autocast_enabled():
            return False
        # The linear layers are laid out for widths about 1024.  Whole passes, torch's / own, us: d_model 1024 (37 to 33,000 tokens) all faster, 13,740
        # tokens 574 / 551, 16,488 822 / 646; 1280 13,740 907 / 754, 27,480 1700 / 1553; 2048 1,374 228 / 199, 4,122 545 / 540; but 1536 8,244 646 / 664, 1792
        # 8,244 740 / 782, 2048 6,870 767 / 850, 2304 6,870 896 / 987, 2560 3,435 652 / 710, 3072 2,748 700 / 834, 4096 64 177 / 244.
        if D > 1280 and (D > 2048 or N > 4096):
            return False
        if _calls_are_watched():
            return False
        tensors = [x, self.w_qkv, self.b_qkv, self.w_out, self.b_out]
        norms = [self.ln1]
        if self.mlp:
            tensors += [self.w_fc1, self.b_fc1, self.w_fc2, self.b_fc2]
            norms.append(self.ln2)
        for ln in norms:
            if (type(ln) is not torch.nn.LayerNorm or tuple(ln.normalized_shape) != (D,) or ln.weight is None or ln.bias is None
                    or ln._forward_hooks or ln._forward_pre_hooks or "forward" in ln.__dict__
                    or torch.nn.modules.module._global_forward_hooks or torch.nn.modules.module._global_forward_pre_hooks):
                return False
            tensors += [ln.weight, ln.bias]
        # (weights of a subclass have a say in what is done with them, and may have no storage of their own: quantised, sharded)
        if any(type(t) is not torch.Tensor and type(t) is not torch.nn.Parameter for t in tensors):
            return False
        if any(t.dtype != torch.bfloat16 or t.device != x.device or not t.is_contiguous() or t.data_ptr() % 16 for t in tensors):
            return False
        if self.w_qkv.shape != (3 * D, D) or self.w_out.shape != (D, D) or self.b_qkv.numel() != 3 * D or self.b_out.numel() != D:
            return False
        if self.mlp and (self.w_fc1.shape != (4 * D, D) or self.w_fc2.shape != (D, 4 * D) or self.b_fc1.numel() != 4 * D
                         or self.b_fc2.numel() != D):
            return False
        if self.plan is not None and (self.plan.perm.device != x.device or self.plan.n_tokens != N):
            return False
        return (N + 256) * 4 * D * 2 < 1 << 31 and (4 * D + 256) * 4 * D * 2 < 1 << 31

    def _attend(self, qkv: torch.Tensor) -> torch.Tensor:
        """[3, heads, N, 64] in working order -> [heads, N, 64]."""
        q, k, v = qkv[0], qkv[1], qkv[2]
        N = q.shape[1]
        if self.tau >= 1.0 and self.rho >= 1.0:
            o = B.bsga_dense_attn(q, k, v)
        else:
            # with the split, patch tokens and special tokens are blocked separately (n_first = N_p)
            n_first = N if self.plan is None else self.plan.n_patch
            q_pool, k_pool = B.bsga_pool_qk_split(q, k, self.block, n_first)
            fq = None if self.plan is None else self.plan.force_q
            fk = None if self.plan is None else self.plan.force_k
            _, kv_idx, kv_cnt = B.bsga_select_blocks(q_pool, k_pool, self.tau, self.rho, force_q=fq, force_k=fk,
                                                     want_bits=False)
            o = B.bsga_sparse_attn_split(q, k, v, self.block, n_first, kv_idx, kv_cnt)
        self.last = {"q": q, "k": k, "v": v, "o": o}
        return o

    @torch.no_grad()
    def attention(self, x: torch.Tensor) -> torch.Tensor:
        H = self.heads
        # working order: patch tokens first, special tokens last
        perm, inverse = (None, None) if self.plan is None else (self.plan.perm, self.plan.inverse)
        o = self._attend(B.bsga_split_heads(F.linear(self.ln1(x), self.w_qkv, self.b_qkv), 3, H, perm))
        return F.linear(B.bsga_merge_heads(o, inverse), self.w_out, self.b_out)

    @torch.no_grad()
    def forward(self, x: torch.Tensor) -> torch.Tensor:
        own = type(self).attention is _ATTENTION and "attention" not in self.__dict__
        if own and self._folds(x):
            perm = None if self.plan is None else self.plan.perm
            h = B.bsga_layer_norm(x, self.ln1.weight, self.ln1.bias, self.ln1.eps, perm)
            qkv = B.bsga_linear(h, self.w_qkv, self.b_qkv, out_heads=True).view(3, self.heads, x.shape[0], 64)
            del h
            x = B.bsga_linear(self._attend(qkv), self.w_out, self.b_out, residual=x, row_index=perm)
            if self.mlp:
                h = B.bsga_layer_norm(x, self.ln2.weight, self.ln2.bias, self.ln2.eps)
                h = B.bsga_linear(h, self.w_fc1, self.b_fc1, gelu=True)
                x = B.bsga_linear(h, self.w_fc2, self.b_fc2, residual=x)
            return x
        x = x + self.attention(x)
        if self.mlp:
            x = x + F.linear(F.gelu(F.linear(self.ln2(x), self.w_fc1, self.b_fc1)), self.w_fc2, self.b_fc2)
        return x


_ATTENTION = GlobalAttentionBlock.attention  # to tell whether another has been put in its place
