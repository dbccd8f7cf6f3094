"""Shared helpers for the GPU parity tests (comparison rules, device copies)."""

import numpy as np
import torch

import oracle

# Tolerances stated for the verification step: attention rtol 2e-2 / atol 2e-3
# (bf16 inputs, fp32 accumulation), confidences 1e-4 absolute, indices and
# acceptance decisions bit-exact outside the 1e-4 band around tau.
ATTN_RTOL = 2e-2
ATTN_ATOL = 2e-3
CONF_ATOL = 1e-4
TAU_EPS = 1e-4


def cuda(x, dtype=None):
    t = torch.as_tensor(x)
    if dtype is not None:
        t = t.to(dtype)
    return t.contiguous().cuda()


# The kernel rounds the softmax weights to bf16 before the P.V product (unit roundoff
# u = 2^-9) and rounds the output to bf16: |err| <= u * sum_i w_i |v_i| + u |out| + fp32
# terms.  For peaked ("sharp") inputs whose output cancels, that bound can exceed the
# stated tolerance, so sharp-input tests add 2u * sum_i w_i |v_i| (computed by the oracle
# with |V| in place of V) to it.
BF16_U = 2.0 ** -9


def attn_close(gpu, ref, abs_weighted=None):
    """Elementwise |gpu - ref| <= atol + rtol |ref| [+ 2u sum w|v|]; returns
    (ok, worst excess, fraction outside)."""
    g = gpu.float().cpu().numpy().astype(np.float64) if isinstance(gpu, torch.Tensor) else gpu
    err = np.abs(g - ref)
    lim = ATTN_ATOL + ATTN_RTOL * np.abs(ref)
    if abs_weighted is not None:
        lim = lim + 2 * BF16_U * abs_weighted
    bad = err > lim
    return (not bad.any()), float((err - lim).max()), float(bad.mean())


def np64(t):
    return t.detach().float().cpu().numpy().astype(np.float64) if t.dtype == torch.bfloat16 else \
        t.detach().cpu().numpy().astype(np.float64)


def compare_accept(gpu, ref, d, conf_ref, tau, B, N, L, k):
    """Bit-exact comparison of acceptance outputs with the near-tau exclusion.

    ``d`` holds the decode inputs; ``conf_ref`` the oracle's [B,N,L,k] conf.
    Returns (mismatch messages, excluded sequence count, excluded hi bits)."""
    msgs = []
    excl_seq = 0
    excl_hi = 0
    g = {key: v.cpu().numpy() for key, v in gpu.items()}
    for b in range(B):
        fr = oracle.fragile_states(d["tokens"][b], d["committed"][b], d["conf0"][b], conf_ref[b], tau, TAU_EPS)
        # states visited by the oracle's decisions: the committed state and its path
        path = [-1]
        j = int(ref["leaf"][b])
        chain = []
        while j != -1:
            chain.append(j)
            j = int(d["parent"][b][j])
        path += chain[::-1]
        if any(fr[q + 1] for q in path) or (fr.any() and d.get("traversal", "greedy") == "longest"):
            excl_seq += 1
        else:
            for key in ("leaf", "n_accepted"):
                if int(g[key][b]) != int(ref[key][b]):
                    msgs.append(f"b={b} {key}: gpu {g[key][b]} oracle {ref[key][b]}")
            if not np.array_equal(g["on_path"][b].astype(bool), ref["on_path"][b]):
                msgs.append(f"b={b} on_path differs")
            if not np.array_equal(g["out_tokens"][b], ref["out_tokens"][b]):
                msgs.append(f"b={b} out_tokens differ")
        near = np.abs(conf_ref[b][:, :, 0] - tau) < TAU_EPS
        excl_hi += int((near & (d["tokens"][b] == -1)).sum())
        hi_ok = (g["hi"][b].astype(bool) == ref["hi"][b]) | near
        if not hi_ok.all():
            msgs.append(f"b={b} hi differs at {np.argwhere(~hi_ok)[:4].tolist()}")
    return msgs, excl_seq, excl_hi


# Products (M, K, N) with the tiling and K split that each is to run with: every tiling of the projection
# GEMM, ragged in rows, columns or k.  A change of the plan that moves one of them off its tiling has to
# bring another shape for it.
GEMM_ONE_PASS = {
    (16, 200, 72): (64, 64, 1), (66, 1096, 8216): (64, 128, 1), (9, 240, 43696): (64, 256, 1),
    (130, 328, 11120): (128, 128, 1), (580, 200, 8312): (128, 192, 1), (2586, 160, 6080): (128, 256, 1),
    (523, 160, 10184): (192, 128, 1), (643, 200, 10912): (192, 192, 1), (521, 200, 11232): (192, 192, 1),
    (385, 200, 11144): (256, 96, 1), (321, 200, 11240): (256, 96, 1), (769, 200, 6936): (256, 128, 1),
    (968, 200, 11088): (256, 256, 1), (64, 512, 33000): (128, 192, 1), (2053, 2056, 904): (128, 128, 1),
    (261, 2056, 6616): (128, 128, 1), (193, 2056, 8344): (128, 128, 1),
}
GEMM_SPLIT = {
    (16, 1544, 72): (64, 64, 3), (67, 3488, 2760): (64, 128, 5), (9, 1632, 16520): (64, 256, 3),
    (68, 1544, 8296): (128, 128, 3), (581, 2384, 3216): (128, 192, 3), (65, 2392, 16568): (128, 256, 3),
    (130, 2160, 6184): (192, 128, 4), (130, 2456, 10968): (192, 192, 4), (129, 2056, 5472): (256, 96, 4),
    (4129, 2056, 392): (256, 96, 3), (194, 2384, 8400): (256, 128, 3),
}
# Layers (drafts, tokens, hidden, inter) whose gate / up projection applies SwiGLU in its epilogue on each
# tiling: rows not a multiple of the tile's, inter not one of its gate columns.
GEMM_SWIGLU = {
    (40, 13, 192, 168): (64, 64, 1), (40, 13, 192, 904): (64, 128, 1), (34, 17, 192, 1616): (128, 128, 1),
    (34, 17, 192, 4104): (128, 192, 1), (34, 17, 256, 6152): (128, 256, 1), (27, 19, 192, 4920): (192, 128, 1),
    (19, 27, 192, 6544): (192, 192, 1), (19, 27, 192, 3272): (256, 96, 1), (15, 43, 192, 4104): (256, 128, 1),
    (34, 17, 192, 6568): (256, 256, 1),
}
