"""Kernels at the sizes where their tiles, remainders and dispatch rules meet, through the
C ABI against float64."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import log, rel

pytestmark = pytest.mark.gpu


# widths and ranks on both sides of the 64 x 256 workgroup tile, the 16-byte stores and the
# matrix cores' four-deep steps; sums of at most 64 exact products in float64, rounded once to
# float: 2^-24 of each entry
@pytest.mark.parametrize("d,kp,r", [(5, 3, 2), (63, 8, 5), (64, 16, 16), (257, 24, 7), (260, 64, 64), (1031, 12, 12)])
def test_dense_truncation_product_edges(d, kp, r):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    nm = 3
    m = torch.randn((nm, d, kp), generator=g, device="cuda") * 0.8 ** torch.arange(kp, device="cuda")
    b = torch.randn((nm, kp, d), generator=g, device="cuda")
    kw = dict(dtype=torch.float32, device="cuda")
    a_o, b_o = torch.full((nm, r, d), float("nan"), **kw), torch.full((nm, d, r), float("nan"), **kw)
    sig, W = torch.empty((nm, kp), **kw), torch.full((nm, d, d), float("nan"), **kw)
    info = torch.zeros(nm, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_LOWRANK_TRUNCATE, nm, 0, d, kp, r_a=r))
    log("dense truncation product", d, kp, r)
    loca.loca_lowrank_truncate(m, b, r, a_o, b_o, sig, info, ws, w_dense_out=W)
    ref = np.einsum("bri,bjr->bij", a_o.double().cpu().numpy(), b_o.double().cpu().numpy())
    assert np.max(np.abs(W.double().cpu().numpy() - ref) - 2.0 ** -23 * np.abs(ref)) <= 1e-30


# the direct-to-LDS kernel at every width, but for the calls of few tokens (64 by 260 alone among
# these by their k): below one tile, its edges, ragged last chunks with NaN in the rows' padding
# (read, never used), fused (2k <= 64) and cross-tile targets, weights.
# S: float32 sums of exact products, error at most n 2^-24 sum|x_i x_j| and far below 1e-5 of S
# in practice; K: two bf16 parts of Y (2^-16) on top
@pytest.mark.parametrize("d,n,k,w", [(1, 40, 4, 0), (7, 33, 3, 1), (64, 500, 8, 0), (255, 100, 40, 0), (256, 257, 32, 1),
                                     (260, 64, 64, 1), (517, 300, 16, 0), (896, 1, 12, 0), (1030, 95, 128, 0)])
def test_statistics_at_every_width(d, n, k, w):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * d + n)
    nb, ld = 3, -(-d // 8) * 8
    buf = torch.full((nb, n, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[:, :, :d] = torch.randn((nb, n, d), generator=g, device="cuda")
    x = buf[:, :, :d]
    y = torch.randn((nb, n, k), generator=g, device="cuda")
    a = torch.rand(n, generator=g, device="cuda") if w else None
    mb = loca.new_mb(nb)
    mb[:, 0] = 7.0
    S = torch.full((nb, d, d), float("nan"), dtype=torch.float32, device="cuda")
    K = torch.full((nb, d, k), float("nan"), dtype=torch.float32, device="cuda")
    info = torch.zeros(nb, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_ACCUMULATE_STATS, nb, n, d, k))
    log("statistics at width", d, n, k, w)
    loca.loca_accumulate_stats(x, y, 0.5, mb, S, K, ws, a_w=a, dev_info=info, overwrite=True)
    X, Y = x.double().cpu().numpy(), y.double().cpu().numpy()
    aw = a.double().cpu().numpy()[None, :, None] if w else 1.0
    iu = np.triu_indices(d)
    assert info.eq(0).all()
    for b in range(nb):
        ref = X[b].T @ ((aw * X)[b] if w else X[b])
        assert rel(S[b].cpu().numpy()[iu], ref[iu]) < 1e-5
        eta = 0.5 * np.sqrt(((aw * X * X)[b] if w else X[b] ** 2).sum() / 7.0)
        assert rel(K[b].cpu().numpy(), -eta * X[b].T @ ((aw * Y)[b] if w else Y[b])) < 1e-5


# few tokens on few tiles take 128-wide register-staged tiles: both sides of the rule's lines in
# tokens, target columns, width and tiles, weighted and not, S and K overwritten and then added to.
# Float32 sums of exact products and two bf16 parts of Y as above
@pytest.mark.parametrize("nb,d,n,k", [(1, 1, 1, 1), (2, 129, 64, 16), (2, 129, 65, 16), (2, 129, 64, 17), (1, 1023, 33, 8),
                                      (6, 1023, 31, 8), (7, 1001, 31, 8), (9, 1000, 31, 8), (10, 1000, 31, 8),
                                      (1, 1024, 20, 4), (64, 41, 64, 3), (65, 41, 64, 3), (96, 40, 64, 3), (97, 40, 64, 3)])
def test_statistics_of_few_tokens(nb, d, n, k):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(d + n)
    buf = torch.full((2, nb, n, -(-d // 8) * 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[..., :d] = torch.randn((2, nb, n, d), generator=g, device="cuda")
    y, a = torch.randn((2, nb, n, k), generator=g, device="cuda"), torch.rand(n, generator=g, device="cuda")
    kw = dict(dtype=torch.float32, device="cuda")
    S, K = torch.full((nb, d, d), float("nan"), **kw), torch.full((nb, d, k), float("nan"), **kw)
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_ACCUMULATE_STATS, nb, n, d, k))
    ws.fill_(255)
    info = torch.zeros(nb, dtype=torch.int32, device="cuda")
    log("statistics of few tokens", nb, d, n, k)
    for w in (None, a):
        refS, refK = 0, 0
        for m in range(2):
            mb = loca.new_mb(nb)
            mb[:, 0] = 7.0
            loca.loca_accumulate_stats(buf[m][..., :d], y[m], 0.5, mb, S, K, ws, a_w=w, dev_info=info, overwrite=m == 0)
            X, Y = buf[m][..., :d].double(), y[m].double()
            aX = X if w is None else X * w.double()[None, :, None]
            refS = refS + aX.transpose(1, 2).contiguous() @ X
            eta = 0.5 * ((aX * X).sum((1, 2)) / 7.0).sqrt()[:, None, None]
            refK = refK - eta * (aX.transpose(1, 2).contiguous() @ Y)
        assert rel(torch.triu(S).cpu().numpy(), torch.triu(refS).cpu().numpy()) < 1e-5
        assert rel(K.cpu().numpy(), refK.cpu().numpy()) < 1e-5 and info.eq(0).all()


# split targets past 2 GB beside an X below it: their byte offsets leave 31 bits first when 2k >
# ldx, and 2^32 bytes at n = 2^23, k = 128.  The n / 16 additions into a float32 sum round by at most
# 2^-24 of the running sum each, and the entries that make up the norm grow steadily to their
# final value: n / 16 2^-24 of it (3e-2 at n = 2^23, where 1.3e-4 is seen); a target read as zero
# or from another row is off by its own size
@pytest.mark.parametrize("n,d,w", [(1 << 23, 64, 0), ((1 << 22) + 5, 20, 0), ((1 << 22) + 5, 20, 1)])
def test_statistics_with_split_targets_past_2gb(n, d, w):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(n + w)
    k, ld = 128, -(-d // 8) * 8
    x = torch.randn((1, n, ld), generator=g, device="cuda").bfloat16()[:, :, :d]
    y = torch.randn((1, n, k), generator=g, device="cuda")
    y += x[0, :, :1].float()  # a part that the sums keep
    a = torch.rand(n, generator=g, device="cuda") if w else None
    mb = loca.new_mb(1)
    mb[:, 0] = 7.0
    kw = dict(dtype=torch.float32, device="cuda")
    S, K = torch.full((1, d, d), float("nan"), **kw), torch.full((1, d, k), float("nan"), **kw)
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_ACCUMULATE_STATS, 1, n, d, k))
    log("statistics with split targets past 2 GB", n, d, w)
    loca.loca_accumulate_stats(x, y, 0.5, mb, S, K, ws, a_w=a, dev_info=info, overwrite=True)
    refS = torch.zeros((d, d), dtype=torch.float64, device="cuda")
    refK = torch.zeros((d, k), dtype=torch.float64, device="cuda")
    for lo in range(0, n, 1 << 20):
        X, Y = x[0, lo:lo + (1 << 20)].double(), y[0, lo:lo + (1 << 20)].double()
        aX = a[lo:lo + (1 << 20), None].double() * X if w else X
        refS += X.T @ aX
        refK += aX.T @ Y
    refK *= -0.5 * float(refS.trace() / 7.0) ** 0.5
    iu = np.triu_indices(d)
    e_s, e_k = rel(S[0].cpu().numpy()[iu], refS.cpu().numpy()[iu]), rel(K[0].cpu().numpy(), refK.cpu().numpy())
    log(f"  S {e_s:.1e} K {e_k:.1e}")
    assert int(info[0]) == 0 and max(e_s, e_k) < n / 16 * 2.0 ** -24
    once = S.clone()
    loca.loca_accumulate_stats(x, y, 0.5, mb, S, K, ws, a_w=a, dev_info=info)  # adds the same to itself
    assert torch.equal(torch.triu(S), 2 * torch.triu(once)) and int(info[0]) == 0


# widths at the edges of the 16-wide blocks, the 64- and 128-wide panels and the 512-wide
# super-panels.  S from 4 d Gaussian rows: the equilibrated matrix's condition number is about
# (1 + 1/2)^2 / (1 - 1/2)^2 = 9; a backward stable solve errs by a small multiple of
# 9 sqrt(d) 2^-24 (fp32, 1.3e-5 at d = 530) or 9 sqrt(d) 2^-53, then the float output's 2^-24
@pytest.mark.parametrize("acc", ["f32", "f64"])
@pytest.mark.parametrize("d", [1, 15, 16, 17, 63, 64, 65, 100, 127, 128, 129, 144, 260, 530])
def test_ridge_solve_block_edges(d, acc):
    import torch
    from paper_2608_03020_amd import loca
    g = np.random.default_rng(d)
    nb, k, lams = 2, 5, [1e-2, 1.0]
    dt = torch.float32 if acc == "f32" else torch.float64
    X = g.standard_normal((nb, 4 * d + 4, d))
    S = torch.from_numpy(X.transpose(0, 2, 1) @ X).to("cuda", dt)
    K = torch.from_numpy(g.standard_normal((nb, d, k))).to("cuda", dt)
    M = torch.full((nb, len(lams), d, k), float("nan"), dtype=torch.float32, device="cuda")
    info = torch.full((nb * len(lams),), 77, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_RIDGE_SOLVE, nb, 0, d, k, n_lambda=len(lams),
                                                  acc=loca.LOCA_F32 if acc == "f32" else loca.LOCA_F64))
    ws.fill_(255)
    ref_s = torch.triu(S).double().cpu().numpy()
    ref_s = ref_s + np.triu(ref_s, 1).transpose(0, 2, 1)
    S += torch.tril(torch.full_like(S, float("nan")), -1)  # never read
    log("ridge solve", d, acc)
    loca.loca_ridge_solve(S, K, lams, M, info, ws)
    assert info.eq(0).all()
    for b in range(nb):
        for i, lam in enumerate(lams):
            ref = np.linalg.solve(ref_s[b] + lam * np.eye(d), K[b].double().cpu().numpy())
            assert rel(M[b, i].cpu().numpy(), ref) < (9 * np.sqrt(d) * 2.0 ** -24 if acc == "f32" else 0) + 2.0 ** -23


# enough matrices for the panel kernel's workgroups of eight waves (at least 256 of them), with and
# without 16-byte rows, a ragged last panel, waves past the last column and right-hand sides on both
# sides of a wave's 32 columns; bound as above
@pytest.mark.parametrize("d,k", [(130, 5), (132, 33), (301, 8), (300, 40)])
def test_ridge_solve_of_many_matrices(d, k):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    nb, lams = 64, [1e-2, 0.1, 1.0, 10.0]
    X = torch.randn((nb, 4 * d, d), generator=g, device="cuda", dtype=torch.float64)
    S = (X.transpose(1, 2).contiguous() @ X).float()
    K = torch.randn((nb, d, k), generator=g, device="cuda")
    U = torch.triu(S).double().cpu()
    U = U + torch.triu(U, 1).transpose(1, 2)
    S += torch.tril(torch.full_like(S, float("nan")), -1)  # never read
    M = torch.full((nb, 4, d, k), float("nan"), device="cuda")
    info = torch.full((nb * 4,), 77, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_RIDGE_SOLVE, nb, 0, d, k, n_lambda=4))
    ws.fill_(255)
    log("ridge solve of many matrices", d, k)
    loca.loca_ridge_solve(S, K, lams, M, info, ws)
    assert info.eq(0).all()
    for i, lam in enumerate(lams):
        ref = torch.linalg.solve(U + lam * torch.eye(d, dtype=torch.float64), K.double().cpu())
        e = (M[:, i].double().cpu() - ref).norm(dim=(1, 2)) / ref.norm(dim=(1, 2))
        assert float(e.max()) < 9 * np.sqrt(d) * 2.0 ** -24 + 2.0 ** -23


# the float32 solve's errors lean neither way: <M - ref, ref> / ||ref||^2, averaged over eight blocks
# (the errors themselves are 5e-7, of either sign).  Every column of the factor and of the inverse
# takes a reciprocal root, and a root that leans by a part of its unit 2^-24 moves all of M by as
# much: half of 2^-24 tells it from the roundings' own lean of about 2e-8
@pytest.mark.parametrize("d", [512, 897])
def test_ridge_solve_errors_are_unbiased(d):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    nb, k, lam = 8, 64, 1e-2
    X = torch.randn((nb, 2 * d, d), generator=g, device="cuda", dtype=torch.float64)
    S = (X.transpose(1, 2).contiguous() @ X).float()
    K = (X.transpose(1, 2).contiguous() @ torch.randn((nb, 2 * d, k), generator=g, device="cuda", dtype=torch.float64)).float()
    M = torch.full((nb, 1, d, k), float("nan"), device="cuda")
    info = torch.full((nb,), 77, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_RIDGE_SOLVE, nb, 0, d, k, n_lambda=1))
    log("bias of the solve", d)
    loca.loca_ridge_solve(S, K, [lam], M, info, ws)
    U = torch.triu(S).double()
    T = U + torch.triu(U, 1).transpose(1, 2) + lam * torch.eye(d, device="cuda", dtype=torch.float64)
    ref = torch.linalg.solve(T.cpu(), K.double().cpu())
    D = M[:, 0].double().cpu() - ref
    bias = ((D * ref).sum((1, 2)) / (ref * ref).sum((1, 2))).mean()
    log(f"  bias {float(bias):+.1e} rel {float(D.norm() / ref.norm()):.1e}")
    assert info.eq(0).all() and abs(float(bias)) < 0.5 * 2.0 ** -24


# the dual fit at the edges of its 16-wide blocks and 32-row ranges, and the head fold on both
# sides of the 64-class split.  float32 outputs of float64 sums; the map's truncation at rank k
# amplifies rounding by sigma_k / (sigma_k - sigma_k+1), kept small by a rank-k probe map
@pytest.mark.parametrize("d,n_p,k,V,wu16", [(16, 16, 4, 1, 0), (33, 17, 5, 3, 1), (300, 63, 8, 64, 0),
                                            (1031, 64, 12, 65, 1), (2048, 31, 16, 40, 0), (65, 1, 1, 7, 0)])
def test_dual_fit_edges(d, n_p, k, V, wu16):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(d + n_p)
    nb, beta = 3, 0.1
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    E = rn(d, n_p)
    G = rn(nb, d, k) / d ** 0.5 @ (rn(nb, k, d) @ E) + 0.01 * rn(nb, d, n_p)
    Wu = rn(V, d) / d ** 0.5
    Wu = Wu.to(torch.bfloat16) if wu16 else Wu
    kw = dict(dtype=torch.float32, device="cuda")
    bt, at = torch.full((nb, k, d), float("nan"), **kw), torch.full((nb, V, k), float("nan"), **kw)
    sig, info = torch.empty((nb, n_p), **kw), torch.full((nb,), 9, dtype=torch.int32, device="cuda")
    alpha = torch.empty(nb, dtype=torch.float64, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_FEEDBACK_FIT, nb, n_p, d, k))
    ws.fill_(255)
    log("dual fit", d, n_p, k, V, wu16)
    loca.loca_feedback_fit(E, G, beta, bt, sig, alpha, info, ws, wu=Wu, at_out=at)
    assert info.eq(0).all()
    e = E.double().cpu().numpy()
    for b in range(nb):
        gb = G[b].double().cpu().numpy()
        F = gb @ np.linalg.solve(e.T @ e + beta * np.eye(n_p), e.T)
        U, s, Vt = np.linalg.svd(F, full_matrices=False)
        Fk = (U[:, :k] * s[:k]) @ Vt[:k]
        assert rel(sig[b].cpu().numpy()[:k], s[:k]) < 1e-6
        FE = Fk @ e
        assert abs(float(alpha[b]) - (FE * gb).sum() / np.linalg.norm(FE) / np.linalg.norm(gb)) < 1e-6
        assert rel((at[b].double() @ bt[b].double()).cpu().numpy(), Wu.double().cpu().numpy() @ Fk.T) < 5e-6


# one factorization serves all blocks: a NaN in the probes is every block's first failed pivot, also
# past the 64 lanes that spread it
@pytest.mark.parametrize("fit,col", [("loca_feedback_fit", 0), ("loca_feedback_fit", 17), ("loca_feedback_fit_primal", 0)])
def test_fit_status_reaches_every_block(fit, col):
    import torch
    from paper_2608_03020_amd import loca
    nb, d, n_p, k = 130, 48, 20, 3
    E, G = torch.randn((d, n_p), device="cuda"), torch.randn((nb, d, n_p), device="cuda")
    E[5, col] = float("nan")
    kw = dict(dtype=torch.float32, device="cuda")
    info = torch.full((nb,), 99, dtype=torch.int32, device="cuda")
    op = loca.LOCA_OP_FEEDBACK_FIT if fit == "loca_feedback_fit" else loca.LOCA_OP_FEEDBACK_FIT_PRIMAL
    ws = loca.alloc_workspace(loca.workspace_size(op, nb, n_p, d, k))
    log("fit status", fit, col)
    getattr(loca, fit)(E, G, 0.1, torch.empty((nb, k, d), **kw), torch.empty((nb, n_p), **kw),
                       torch.empty(nb, dtype=torch.float64, device="cuda"), info, ws)
    assert info.eq(col + 1 if fit == "loca_feedback_fit" else 6).all(), info


# the fused head at the edges of its token tiles (128, 256), 256-entry vocabulary chunks, 64-wide
# slices of d and 64-column tiles, with a maximum that rises late and an excluded tail.  The
# exponentials carry 2^-17 (two bf16 parts), far below the 1e-5 asked of the output's norm
@pytest.mark.parametrize("n,V,d,c", [(1, 1, 8, 1), (128, 255, 64, 64), (129, 257, 72, 33), (256, 256, 128, 65),
                                     (257, 1000, 200, 130), (60, 5000, 1096, 4), (300, 777, 2048, 64)])
def test_fused_head_edges(n, V, d, c):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(n + V + d)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    h, Wu, Vm = (2 * rn(n, d)).bfloat16(), (rn(V, d) / d ** 0.5).bfloat16(), rn(V, c).bfloat16()
    Wu[-1] *= 6  # the last entry moves many maxima
    y = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    w = torch.rand(n, generator=g, device="cuda")
    out = torch.full((n, c), float("nan"), device="cuda")
    info = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_FUSED_HEAD, 1, n, d, c, C=V))
    ws.fill_(255)
    log("fused head", n, V, d, c)
    loca.loca_fused_head(h, Wu, y, Vm, out, info, ws, w=w)
    assert int(info) == 0
    H, W, M = (t.double().cpu().numpy() for t in (h, Wu, Vm))
    z = H @ W.T
    e = np.exp(z - z.max(1, keepdims=True))
    e /= e.sum(1, keepdims=True)
    e[np.arange(n), y.cpu().numpy()] -= 1
    ref = (e @ M) * w.double().cpu().numpy()[:, None]
    scale = np.linalg.norm(M) * np.linalg.norm(w.double().cpu().numpy()) / np.sqrt(V)
    assert np.linalg.norm(out.double().cpu().numpy() - ref) < 1e-5 * max(scale, np.linalg.norm(ref))


# rows of h (and of W_u) at the ends of the 31-bit byte offsets: 256 rows of 2^23 values are 2^32
# bytes, 256 rows past 2^22 leave the out-of-range offset inside the buffer (d % 64 != 0 reads it;
# NaN in the gaps between the rows must stay unread).  float32 sums of d products: the logits are
# off by d / 16 2^-24 of their size (about 2) at worst, the output by as much of its norm;
# hidden states or head rows read as zero are off by the output itself
@pytest.mark.parametrize("n,ldh,d,V", [(256, 1 << 23, 64, 300), (200, 1 << 23, 72, 300), (256, (1 << 22) + 8, 72, 300),
                                       (130, 1 << 23, 1 << 23, 256), (3, 1 << 23, (1 << 23) - 8, 300)])
def test_fused_head_long_rows(n, ldh, d, V):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(n + V)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    c = 5
    buf = torch.empty((n * ldh,), dtype=torch.bfloat16, device="cuda").view(n, ldh)
    h, Wu = buf[:, :d], torch.empty((V, d), dtype=torch.bfloat16, device="cuda")
    for t in (h, Wu):
        for i in range(0, t.shape[0], 16):
            t[i:i + 16] = rn(t[i:i + 16].shape[0], d) * (2 * d ** -0.25 if t is h else d ** -0.25)
    if ldh > d:
        buf[:, d:] = float("nan")
    Vm = rn(V, c).bfloat16()
    y = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    out = torch.full((n, c), float("nan"), device="cuda")
    info = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_FUSED_HEAD, 1, n, d, c, C=V))
    log("fused head, long rows", n, ldh, d, V)
    loca.loca_fused_head(h, Wu, y, Vm, out, info, ws)
    z = torch.zeros((n, V), dtype=torch.float64, device="cuda")
    for lo in range(0, d, 1 << 17):
        z += h[:, lo:lo + (1 << 17)].double() @ Wu[:, lo:lo + (1 << 17)].double().T
    p = torch.softmax(z, 1)
    p[torch.arange(n), y.long()] -= 1
    e = rel(out.cpu().numpy(), (p @ Vm.double()).cpu().numpy())
    log(f"  out {e:.1e}")
    assert int(info) == 0 and e < max(1e-5, d / 16 * 2.0 ** -24)


# an operand of ones: sum P / sum P - 1 is 0, and what is left is the rounding of the float32 sums of
# one part of a vocabulary range against each other, averaged over the parts.  3/4 of 2^-24 (half a
# unit of the quotient, 1) holds while a wave's sums stay at 10 chunks of 128 entries (3.5e-8; sums
# twice as long leave 6.6e-8)
def test_fused_head_length_of_sums():
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(0)
    n, V, d, c = 4096, 151936, 64, 8
    h, Wu = (2 * torch.randn((n, d), generator=g, device="cuda")).bfloat16(), torch.randn((V, d), generator=g, device="cuda")
    y = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    out = torch.full((n, c), float("nan"), device="cuda")
    info = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_FUSED_HEAD, 1, n, d, c, C=V))
    ws.fill_(255)
    log("fused head, operand of ones")
    loca.loca_fused_head(h, (Wu * d ** -0.5).bfloat16(), y, torch.ones((V, c), device="cuda").bfloat16(), out, info, ws)
    rms = float(out.double().pow(2).mean().sqrt())
    log(f"  rms {rms:.2e}")
    assert int(info) == 0 and rms < 0.75 * 2.0 ** -24


# a right operand of 2^35 entries (64 GiB, and as much again laid out in the workspace): one wave per
# fragment of 512 would be 2^32 threads, which no launch holds.  P as two bf16 parts: 2^-17 of each
# term, far below 1e-5 of the output's norm
def test_fused_head_operand_of_64_gib():
    import torch
    from paper_2608_03020_amd import loca
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 170 << 30:
        pytest.skip("needs 170 GiB of free device memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    n, V, d, c = 2, 1 << 18, 8, 1 << 17
    h, Wu = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((n, d), (V, d)))
    y = torch.tensor([0, V - 1], dtype=torch.int32, device="cuda")
    out = torch.full((n, c), float("nan"), device="cuda")
    info = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_FUSED_HEAD, 1, n, d, c, C=V))
    Vm = torch.empty((V, c), dtype=torch.bfloat16, device="cuda")
    for i in range(0, V, 1 << 13):
        Vm[i:i + (1 << 13)].normal_(generator=g)
    log("fused head, operand of 64 GiB")
    loca.loca_fused_head(h, Wu, y, Vm, out, info, ws)
    p = torch.softmax(h.double() @ Wu.double().T, 1)
    p[torch.arange(n), y.long()] -= 1
    ref = torch.zeros((n, c), dtype=torch.float64, device="cuda")
    for i in range(0, V, 1 << 12):
        ref += p[:, i:i + (1 << 12)] @ Vm[i:i + (1 << 12)].double()
    e = rel(out.cpu().numpy(), ref.cpu().numpy())
    log(f"  out {e:.1e}")
    del Vm, ws
    torch.cuda.empty_cache()
    assert int(info) == 0 and e < 1e-5


# a vocabulary product whose scratch fits the fixed array only with the fewest ranges: taken by the
# allocation-free call, with the bits of the workspace call.  P as two bf16 parts: 2^-17 of each term
def test_allocation_free_vocabulary_product():
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(13)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    nb, n, C, k, d = 13, 608, 1680, 32, 64
    z, A, B = (3 * rn(n, C)).bfloat16(), rn(nb, C, k).bfloat16(), rn(nb, k, d)
    y = torch.randint(0, C, (n,), generator=g, device="cuda", dtype=torch.int32)
    Y, Yn = (torch.full((nb, n, k), float("nan"), device="cuda") for _ in range(2))
    mb, mbn = loca.new_mb(nb), loca.new_mb(nb)
    info, infon = (torch.full((1,), 5, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_ERROR_TARGETS, nb, n, d, k, C=C))
    ws.fill_(255)
    log("allocation-free vocabulary product")
    loca.loca_error_targets(z, y, A, B, Y, mb, info, ws)
    loca.loca_error_targets_noalloc(z, y, A, B, Yn, mbn, infon)
    assert int(info) == 0 and int(infon) == 0 and torch.equal(Y, Yn) and torch.equal(mb, mbn)
    E = torch.softmax(z.double(), 1)
    E[torch.arange(n), y.long()] -= 1
    for b in range(nb):
        assert rel(Y[b].cpu().numpy(), (E @ A[b].double()).cpu().numpy()) < 1e-5


# the paper-order head at the edges of its 128-token tiles, 64-entry blocks and column tiles
# (one to three of 32 to 256 columns, float and bf16 logits), NaN in the rows' padding, and the
# blocks' coordinates on both sides of 64 columns.  P as two bf16 parts: 2^-17 of each term
@pytest.mark.parametrize("n,V,d,k,bf", [(1, 5, 8, 1, 1), (127, 64, 40, 16, 0), (129, 65, 72, 33, 1), (130, 1003, 136, 64, 0),
                                        (64, 300, 200, 65, 1), (200, 130, 264, 128, 0), (33, 9000, 520, 12, 1)])
def test_paper_order_head_edges(n, V, d, k, bf):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(n + V + d)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    per = 8 if bf else 4
    buf = torch.full((n, -(-V // per) * per), float("nan"), device="cuda", dtype=torch.bfloat16 if bf else torch.float32)
    buf[:, :V] = 3 * rn(n, V)
    z, nb = buf[:, :V], 2
    if V > 8:
        z[:, 3] = float("-inf")  # an excluded class
    Wu, Vk, B = (rn(V, d) / d ** 0.5).bfloat16(), rn(nb, d, k) / d ** 0.5, rn(nb, k, d)
    y = torch.randint(4 if V > 8 else 0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    w, a = torch.rand(n, generator=g, device="cuda"), torch.rand(n, generator=g, device="cuda")
    e, Y = torch.full((n, d), float("nan"), device="cuda"), torch.full((nb, n, k), float("nan"), device="cuda")
    mb, info = loca.new_mb(nb), torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(max(loca.workspace_size(loca.LOCA_OP_TOP_ERROR, 1, n, d, 1, V),
                                  loca.workspace_size(loca.LOCA_OP_CREDIT_FROM_TOP_ERROR, nb, n, d, k)))
    ws.fill_(255)
    log("paper-order head", n, V, d, k, bf)
    loca.loca_top_error(z, y, Wu, e, info, ws, w=w)
    loca.loca_credit_from_top_error(e, Vk, B, Y, mb, ws, a_w=a)
    assert int(info) == 0
    Z, W = z.double().cpu().numpy(), Wu.double().cpu().numpy()
    E = np.exp(Z - Z.max(1, keepdims=True))
    E /= E.sum(1, keepdims=True)
    E[np.arange(n), y.cpu().numpy()] -= 1
    ref = (E @ W) * w.double().cpu().numpy()[:, None]
    scale = np.linalg.norm(W) * np.linalg.norm(w.double().cpu().numpy()) / np.sqrt(V)
    assert np.linalg.norm(e.double().cpu().numpy() - ref) < 1e-5 * max(scale, np.linalg.norm(ref))
    ed = e.double().cpu().numpy()
    for b in range(nb):  # float64 sums of exact products, rounded once; q2 from the rounded Y
        Yr = ed @ Vk[b].double().cpu().numpy()
        assert rel(Y[b].cpu().numpy(), Yr) < 2.0 ** -23
        Bd, Yd = B[b].double().cpu().numpy(), Y[b].double().cpu().numpy()
        q2 = (a.double().cpu().numpy() * ((Yd @ Bd) ** 2).sum(1)).sum()
        assert abs(float(mb[b, 0]) - q2) < 1e-12 * q2


# label sets of 1 to 17 classes (both sides of the 8-class form),
# tokens around the 256-token tiles, ranks on both sides of the column blocks and of the 16-byte
# stores, weights, and more tiles than the 512 partials of M.  float32 softmax (a few ulp of terms
# below 1) times float32 factors: 1e-6 of Y; ||Q||^2 from the same rows in float64: 2e-6
@pytest.mark.parametrize("n,C,k,nb,wt", [(1, 1, 1, 1, 0), (255, 2, 3, 3, 1), (256, 5, 64, 2, 0), (257, 8, 16, 5, 1),
                                         (300, 9, 18, 2, 1), (1000, 16, 33, 7, 0), (70, 17, 20, 2, 1),
                                         (131500, 3, 4, 1, 1)])
def test_label_set_head_edges(n, C, k, nb, wt):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(n + C + k)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    d = 40
    z, A, B = 3 * rn(n, C), rn(nb, C, k), rn(nb, k, d)
    if C > 3:
        z[0, 1] = float("-inf")
    y = torch.randint(2 if C > 3 else 0, C, (n,), generator=g, device="cuda", dtype=torch.int32)
    w = torch.rand(n, generator=g, device="cuda") if wt else None
    a = torch.rand(n, generator=g, device="cuda") if wt else None
    Y, e = torch.full((nb, n, k), float("nan"), device="cuda"), torch.full((n, C), float("nan"), device="cuda")
    mb, info = loca.new_mb(nb), torch.full((1,), 5, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_ERROR_TARGETS, nb, n, d, k, C=C))
    ws.fill_(255)
    log("label-set head", n, C, k, nb, wt)
    loca.loca_error_targets(z, y, A, B, Y, mb, info, ws, w=w, a_w=a, e_out=e)
    assert int(info) == 0
    Z = z.double().cpu().numpy()
    E = np.exp(Z - Z.max(1, keepdims=True))
    E /= E.sum(1, keepdims=True)
    E[np.arange(n), y.cpu().numpy()] -= 1
    if wt:
        E *= w.double().cpu().numpy()[:, None]
    aw = a.double().cpu().numpy() if wt else np.ones(n)
    assert np.max(np.abs(e.double().cpu().numpy() - E)) < 1e-6
    for b in range(nb):
        Ad, Bd = A[b].double().cpu().numpy(), B[b].double().cpu().numpy()
        Yr = E @ Ad
        assert np.linalg.norm(Y[b].double().cpu().numpy() - Yr) <= 1e-6 * np.linalg.norm(Yr)
        q2 = (aw * ((Yr @ Bd) ** 2).sum(1)).sum()
        assert abs(float(mb[b, 0]) - q2) <= 2e-6 * q2


# the truncation's small eigenproblem at the sizes where its column groups of four, its rows of
# eight in the Sturm counts and its 16 x 16 blocks end, over norms whose squares leave the float
# range, up to the switch to the larger core at kp = 65.  The factors are rounded to float, so
# each entry of W is off by about 2^-23 of its products, and so are the singular values; 1e-6
# leaves a factor of eight
@pytest.mark.parametrize("scale", [1.0, 1e-16, 1e14])
@pytest.mark.parametrize("kp,r", [(1, 1), (2, 1), (2, 2), (3, 3), (4, 4), (7, 5), (8, 8), (9, 2), (15, 15), (16, 8), (17, 17), (31, 16),
                                  (32, 32), (33, 12), (48, 32), (63, 63), (64, 64), (65, 20), (128, 64)])
def test_truncation_core_edges(kp, r, scale):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(kp)
    nm, d = 2, 150
    m = torch.randn((nm, d, kp), generator=g, device="cuda") * (0.9 ** torch.arange(kp, device="cuda") * scale)
    b = torch.randn((nm, kp, d), generator=g, device="cuda")
    kw = dict(dtype=torch.float32, device="cuda")
    a_o, b_o = torch.full((nm, r, d), float("nan"), **kw), torch.full((nm, d, r), float("nan"), **kw)
    sig, info = torch.full((nm, kp), float("nan"), **kw), torch.zeros(nm, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_LOWRANK_TRUNCATE, nm, 0, d, kp, r_a=r))
    log("truncation core", kp, r, scale)
    loca.loca_lowrank_truncate(m, b, r, a_o, b_o, sig, info, ws)
    W = np.einsum("bri,bjr->bij", a_o.double().cpu().numpy(), b_o.double().cpu().numpy())
    for i in range(nm):
        U, s, Vh = np.linalg.svd(m[i].double().cpu().numpy() @ b[i].double().cpu().numpy(), full_matrices=False)
        ref = (U[:, :r] * s[:r]) @ Vh[:r]
        e_w, e_s = rel(W[i], ref), rel(sig[i].double().cpu().numpy(), s[:kp])
        log(f"  W_r {e_w:.1e} sigma {e_s:.1e}")
        assert e_w < 1e-6 and e_s < 1e-6
    assert not info.any()


# two equal singular values: W itself at rank 2, and at rank 1 any unit direction of its column space.
# Factors rounded to float as above
@pytest.mark.parametrize("r", [1, 2])
def test_truncation_of_two_equal_values(r):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(r)
    d = 150
    orth = lambda: torch.linalg.qr(torch.randn((d, 2), generator=g, device="cuda").double())[0].float()
    m, b = orth().contiguous()[None], orth().T.contiguous()[None]
    kw = dict(dtype=torch.float32, device="cuda")
    a_o, b_o = torch.full((1, r, d), float("nan"), **kw), torch.full((1, d, r), float("nan"), **kw)
    sig, info = torch.full((1, 2), float("nan"), **kw), torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_LOWRANK_TRUNCATE, 1, 0, d, 2, r_a=r))
    log("truncation of two equal values", r)
    loca.loca_lowrank_truncate(m.contiguous(), b.contiguous(), r, a_o, b_o, sig, info, ws)
    A, B = a_o[0].double().cpu().numpy(), b_o[0].double().cpu().numpy()
    W = m[0].double().cpu().numpy() @ b[0].double().cpu().numpy()
    assert np.abs(A @ A.T - np.eye(r)).max() < 1e-6 and np.abs(sig.cpu().numpy() - 1.0).max() < 1e-6
    Wr = (B @ A).T  # A's rows lie in W's column space, B = W^T A^T
    assert np.linalg.norm(B - W.T @ A.T) < 1e-6 and (r == 1 or np.linalg.norm(Wr - W) < 1e-6)
    assert not info.any()


# the float64 statistics at the edges of their 32-token stages and 64-wide tiles: float64 sums of
# exact products, n 2^-53 of the sum of magnitudes, far below 1e-13
@pytest.mark.parametrize("d,n,k,w", [(1, 1, 1, 0), (63, 31, 5, 1), (64, 32, 64, 0), (65, 33, 65, 1), (200, 64, 8, 0), (130, 97, 3, 1)])
def test_float64_statistics_edges(d, n, k, w):
    import torch
    from paper_2608_03020_amd import loca
    g = torch.Generator(device="cuda")
    g.manual_seed(d + n)
    nb, ld = 2, -(-d // 4) * 4
    buf = torch.full((nb, n, ld), float("nan"), dtype=torch.float32, device="cuda")
    buf[:, :, :d] = torch.randn((nb, n, d), generator=g, device="cuda")
    x, y = buf[:, :, :d], torch.randn((nb, n, k), generator=g, device="cuda")
    a = torch.rand(n, generator=g, device="cuda") if w else None
    mb = loca.new_mb(nb)
    mb[:, 0] = 7.0
    S = torch.full((nb, d, d), float("nan"), dtype=torch.float64, device="cuda")
    K = torch.full((nb, d, k), float("nan"), dtype=torch.float64, device="cuda")
    info = torch.zeros(nb, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_ACCUMULATE_STATS, nb, n, d, k, acc=loca.LOCA_F64))
    log("float64 statistics", d, n, k, w)
    loca.loca_accumulate_stats(x, y, 0.5, mb, S, K, ws, a_w=a, dev_info=info, overwrite=True)
    aw = (a.double() if w else torch.ones(n, dtype=torch.float64, device="cuda"))[:, None].cpu()
    for b in range(nb):
        X, Y = x[b].double().cpu(), y[b].double().cpu()
        eta = 0.5 * float(np.sqrt(float((aw * X * X).sum()) / 7.0))
        iu = np.triu_indices(d)
        assert rel(S[b].cpu().numpy()[iu], (X.T @ (aw * X)).numpy()[iu]) < 1e-13
        assert rel(K[b].cpu().numpy(), (-eta * (X.T @ (aw * Y))).numpy()) < 1e-13
    assert not info.any()


# S_sym L at the edges of its 64-row tiles and 16- and 32-column chunks, L along its rows (the
# current adapters of the solve) and along its columns (the projected form in float64); entries of
# S below the diagonal are NaN.  As for the solve alone: float32 rounding of the result, and with
# float32 statistics the solve's own 9 sqrt(d) 2^-24
@pytest.mark.parametrize("acc", ["f32", "f64"])
@pytest.mark.parametrize("d,r", [(1, 1), (63, 1), (64, 16), (65, 17), (129, 32), (130, 33), (200, 60)])
def test_symmetric_product_edges(d, r, acc):
    import torch
    from paper_2608_03020_amd import loca
    g = np.random.default_rng(d + r)
    nb, k, lam = 2, 3, 0.7
    dt = torch.float32 if acc == "f32" else torch.float64
    lacc = loca.LOCA_F32 if acc == "f32" else loca.LOCA_F64
    X = g.standard_normal((nb, 4 * d + 4, d))
    S = torch.triu(torch.from_numpy(X.transpose(0, 2, 1) @ X).to("cuda", dt))
    ref_s = S.double().cpu().numpy()
    ref_s = ref_s + np.triu(ref_s, 1).transpose(0, 2, 1)
    S += torch.tril(torch.full_like(S, float("nan")), -1)
    kw = dict(dtype=torch.float32, device="cuda")
    K = torch.from_numpy(g.standard_normal((nb, d, k))).to("cuda", dt)
    lp, rp = (torch.from_numpy(g.standard_normal(s)).to(**kw) for s in ((nb, d, r), (nb, r, d)))
    B = torch.from_numpy(g.standard_normal((nb, k, d))).to(**kw)
    M = torch.full((nb, 1, d, r + k), float("nan"), **kw)
    info = torch.full((nb,), 77, dtype=torch.int32, device="cuda")
    ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_RIDGE_SOLVE, nb, 0, d, r + k, n_lambda=1, acc=lacc))
    log("symmetric product", d, r, acc)
    loca.loca_ridge_solve(S, K, [lam], M, info, ws, lp=lp, rp=rp)
    assert info.eq(0).all()
    bound = (9 * np.sqrt(d) * 2.0 ** -24 if acc == "f32" else 0) + 2.0 ** -23
    for b in range(nb):
        rhs = np.concatenate([ref_s[b] @ lp[b].double().cpu().numpy(), K[b].double().cpu().numpy()], axis=1)
        assert rel(M[b, 0].cpu().numpy(), np.linalg.solve(ref_s[b] + lam * np.eye(d), rhs)) < bound
    if acc == "f64" and r <= min(d, 64):
        Bp = torch.full((nb, 1, d, r), float("nan"), **kw)
        ws = loca.alloc_workspace(loca.workspace_size(loca.LOCA_OP_RIDGE_SOLVE_PROJECTED, nb, 0, d, k, r_a=r, n_lambda=1,
                                                      acc=lacc))
        loca.loca_ridge_solve_projected(S, K, B, rp, [lam], Bp, info, ws)
        assert info.eq(0).all()
        for b in range(nb):
            P = rp[b].double().cpu().numpy()
            G = P @ ref_s[b] @ P.T + lam * np.eye(r)
            ref = np.linalg.solve(G, P @ K[b].double().cpu().numpy() @ B[b].double().cpu().numpy()).T
            assert rel(Bp[b, 0].cpu().numpy(), ref) < 2.0 ** -23
