"""GPU parity of the gradient transformation G Q, Q = T^T T (Sec. 3.1) against the CPU oracle."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_common import b, dev, ora, relF, workspace, DEV

pytestmark = pytest.mark.gpu
rng = np.random.default_rng(77)


def sym_Q(M, seed):
    r = np.random.default_rng(seed)
    T = np.eye(M) + 0.2 * r.standard_normal((M, M)) / np.sqrt(M)
    return T.astype(np.float32), (T.astype(np.float32).astype(np.float64).T @ T.astype(np.float32).astype(np.float64))


@pytest.mark.parametrize("S,M", [(32, 64), (5, 7), (64, 576), (70, 200), (1, 129), (130, 147), (256, 300), (40, 260), (200, 1156),
                                 (256, 2304), (96, 1024), (17, 4608)])
def test_f32_with_Q(S, M):
    T32, Q64 = sym_Q(M, M)
    Q32 = Q64.astype(np.float32)
    G = (rng.standard_normal((S, M)) * 0.1).astype(np.float32)
    out = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out)
    torch.cuda.synchronize()
    want = ora.grad_transform(G, Q32)
    assert relF(out.cpu().numpy(), want) < 1e-5


@pytest.mark.parametrize("S,M", [(32, 64), (64, 576), (70, 200), (256, 2304), (96, 1024), (17, 4608), (1, 2052), (33, 1156), (512, 1152)])
def test_f32_with_Q_and_the_workspace(S, M):
    """With the whole workspace a product with few output tiles cuts its contraction index into runs (ragged last run
    included) and adds them in a fixed order: same result to float32 rounding, and the same bits on a second call."""
    T32, Q64 = sym_Q(M, M + 5)
    Q32 = Q64.astype(np.float32)
    G = (rng.standard_normal((S, M)) * 0.1).astype(np.float32)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S))
    out = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out, ws)
    torch.cuda.synchronize()
    assert relF(out.cpu().numpy(), ora.grad_transform(G, Q32)) < 1e-5
    out2 = torch.full((S, M), float("nan"), device=DEV)
    ws.fill_(0xFF)                     # nothing in the workspace may matter between calls
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out2, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    # bfloat16 gradient through the same path (widened, product in float32, rounded on the way out)
    Gb = wl.round_to_bf16(G)
    wsb = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S, None, b.FW_BF16))
    outb = torch.zeros(S, M, device=DEV, dtype=torch.bfloat16)
    b.fw_grad_transform(dev(Gb, torch.bfloat16), b.FW_BF16, S, M, None, dev(Q32), outb, wsb)
    torch.cuda.synchronize()
    assert relF(outb.float().cpu().numpy(), ora.grad_transform(Gb, Q32)) < 3e-3


@pytest.mark.parametrize("S,M", [(512, 4608), (400, 3076), (384, 3072), (1000, 3200), (1100, 1536), (2100, 1028)])
def test_f32_split_form_for_many_features(S, M):
    """float32 gradients past the size rule of the split form, with the whole workspace: G and Q as bfloat16 hi + lo planes on the
    bfloat16 matrix cores (three products per term, float32 accumulation), the contraction index cut into runs when S
    gives few tiles.  Operands carry 16 significant bits: tolerance 2e-5 (float32 form: 1e-5); reproducible bit for bit."""
    T32, Q64 = sym_Q(M, M + 9)
    Q32 = Q64.astype(np.float32)
    G = (rng.standard_normal((S, M)) * 0.1).astype(np.float32)
    want = ora.grad_transform(G, Q32)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S))
    out = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out, ws)
    torch.cuda.synchronize()
    e = relF(out.cpu().numpy(), want)
    print(f"S={S} M={M}: rel-F = {e:.2e}")
    assert 1e-6 < e < 2e-5            # the split form ran (float32 would be below 1e-6) and is inside its tolerance
    ws.fill_(0xFF)
    out2 = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out2, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    # without the workspace: plain float32
    out3 = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out3)
    torch.cuda.synchronize()
    assert relF(out3.cpu().numpy(), want) < 1e-6
    # bfloat16 gradients of the same size: widened, split form, one rounding at the end
    if M % 4 == 0:
        Gb = wl.round_to_bf16(G)
        wsb = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S, None, b.FW_BF16))
        outb = torch.zeros(S, M, device=DEV, dtype=torch.bfloat16)
        b.fw_grad_transform(dev(Gb, torch.bfloat16), b.FW_BF16, S, M, None, dev(Q32), outb, wsb)
        torch.cuda.synchronize()
        wantb = ora.grad_transform(Gb, Q32)
        assert relF(outb.float().cpu().numpy(), wantb) < 3e-3
        assert np.all(np.abs(outb.float().cpu().numpy() - wantb) <= np.abs(wantb) * 2.0 ** -8 + 1e-5 * np.abs(wantb).max())


@pytest.mark.parametrize("S,M", [(32, 64), (5, 7), (64, 576), (70, 200), (130, 147), (33, 260)])
def test_bf16_with_Q(S, M):
    T32, Q64 = sym_Q(M, M + 1)
    Q32 = Q64.astype(np.float32)
    G = wl.round_to_bf16((rng.standard_normal((S, M)) * 0.1).astype(np.float32))
    out = torch.zeros(S, M, device=DEV, dtype=torch.bfloat16)
    b.fw_grad_transform(dev(G, torch.bfloat16), b.FW_BF16, S, M, None, dev(Q32), out)
    torch.cuda.synchronize()
    want = ora.grad_transform(G, Q32)
    assert relF(out.float().cpu().numpy(), want) < 2e-2
    # against the same computation with Q rounded to bf16 the only error left is accumulation order and output rounding
    want_r = ora.grad_transform(G, wl.round_to_bf16(Q32))
    assert relF(out.float().cpu().numpy(), want_r) < 4e-3
    # with the workspace G is widened and Q is used as it is: only the rounding of the output is left
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S, None, b.FW_BF16))
    out2 = torch.zeros(S, M, device=DEV, dtype=torch.bfloat16)
    b.fw_grad_transform(dev(G, torch.bfloat16), b.FW_BF16, S, M, None, dev(Q32), out2, ws)
    torch.cuda.synchronize()
    assert relF(out2.float().cpu().numpy(), want) < 3e-3
    assert np.array_equal(out2.float().cpu().numpy(), wl.round_to_bf16(ora.grad_transform(G, Q32).astype(np.float32))) or \
        relF(out2.float().cpu().numpy(), wl.round_to_bf16(ora.grad_transform(G, Q32).astype(np.float32))) < 1e-3


@pytest.mark.parametrize("S,M", [(8, 64), (33, 150), (64, 576)])
def test_f32_from_nonsymmetric_T(S, M):
    """Q is built as T^T T (eq. (vQ)); a transposed product would fail for this non-symmetric T."""
    T32, Q64 = sym_Q(M, 3 * M)
    assert not np.allclose(T32, T32.T)
    G = (rng.standard_normal((S, M)) * 0.1).astype(np.float32)
    out = torch.zeros(S, M, device=DEV)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S))
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, dev(T32), None, out, ws)
    torch.cuda.synchronize()
    want = ora.grad_transform(G, ora.Q_from_T(T32))
    assert relF(out.cpu().numpy(), want) < 1e-5
    wrong = ora.grad_transform(G, T32.astype(np.float64) @ T32.astype(np.float64).T)
    assert relF(out.cpu().numpy(), wrong) > 1e-3


@pytest.mark.parametrize("S,M", [(40, 1536), (24, 1670), (160, 3072)])
def test_f32_from_nonsymmetric_T_split_build(S, M):
    """From FW_REFRESH_SPLIT_MIN_M features on Q = T^T T (eq. (vQ)) is built on the bfloat16 matrix cores from the hi + lo
    planes of T's columns (the product G Q stays in float32 at these sizes): float32-grade results,
    and still T^T T, not T T^T."""
    T32, Q64 = sym_Q(M, 5 * M)
    G = (rng.standard_normal((S, M)) * 0.1).astype(np.float32)
    out = torch.zeros(S, M, device=DEV)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S))
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, dev(T32), None, out, ws)
    torch.cuda.synchronize()
    want = ora.grad_transform(G, ora.Q_from_T(T32))
    err = relF(out.cpu().numpy(), want)
    print(f"raw T, split build: S={S} M={M} rel-F {err:.2e}")
    assert err < 2e-5
    wrong = ora.grad_transform(G, T32.astype(np.float64) @ T32.astype(np.float64).T)
    assert relF(out.cpu().numpy(), wrong) > 1e-3


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_large_feature_count(dtype):
    """M = 9216: Q = I + u u^T keeps the float64 reference cheap."""
    S, M = 24, 9216
    r = np.random.default_rng(9)
    u = (r.standard_normal(M) / np.sqrt(M)).astype(np.float32)
    Q32 = (np.eye(M, dtype=np.float32) + np.outer(u, u)).astype(np.float32)
    Q32 = np.maximum(Q32, Q32.T)   # exactly symmetric
    G = (r.standard_normal((S, M)) * 0.1).astype(np.float32)
    want = ora.grad_transform(wl.round_to_bf16(G) if dtype == "bf16" else G, Q32)
    if dtype == "f32":
        out = torch.zeros(S, M, device=DEV)
        b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out)
        torch.cuda.synchronize()
        assert relF(out.cpu().numpy(), want) < 1e-5
    else:
        ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S, None, b.FW_BF16))
        out = torch.zeros(S, M, device=DEV, dtype=torch.bfloat16)
        b.fw_grad_transform(dev(wl.round_to_bf16(G), torch.bfloat16), b.FW_BF16, S, M, None, dev(Q32), out, ws)
        torch.cuda.synchronize()
        assert relF(out.float().cpu().numpy(), want) < 3e-3


def test_config1_gradient_with_identity_is_copy():
    L = wl.config1()
    S, M = L.G.shape
    out = torch.zeros(S, M, device=DEV)
    b.fw_grad_transform(dev(L.G), b.FW_F32, S, M, None, torch.eye(M, device=DEV), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), L.G)


def test_largest_feature_count():
    """M = 16384, the library's limit (Q is 1 GiB): Q = I + u u^T + v v^T keeps the float64 reference a few dot products."""
    S, M = 40, 16384
    r = np.random.default_rng(12)
    u = (r.standard_normal(M) / np.sqrt(M)).astype(np.float32)
    v = (r.standard_normal(M) / np.sqrt(M)).astype(np.float32)
    Q = torch.eye(M, device=DEV)
    ud, vd = dev(u), dev(v)
    Q += torch.outer(ud, ud) + torch.outer(vd, vd)
    Q = torch.maximum(Q, Q.T).contiguous()                       # exactly symmetric
    G = (r.standard_normal((S, M)) * 0.1).astype(np.float32)
    out = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, Q, out)
    torch.cuda.synchronize()
    # the reference from the same float32 Q, block of columns by block of columns
    G64 = G.astype(np.float64)
    num = den = 0.0
    for c0 in range(0, M, 2048):
        want = G64 @ Q[:, c0:c0 + 2048].cpu().numpy().astype(np.float64)
        got = out[:, c0:c0 + 2048].cpu().numpy().astype(np.float64)
        num += float(((got - want) ** 2).sum()); den += float((want ** 2).sum())
    assert (num / den) ** 0.5 < 1e-5
    with pytest.raises(b.FwError):
        b.fw_grad_transform(dev(G[:, :64]), b.FW_F32, S, M + 4, None, Q, out)


# The three-plane form: tiles of 64 x 64 and chunks of 32 entries with one row, column or entry too many and too few, contraction
# shorter than a chunk, sizes that are no multiple of 4 (from 192 features and 28 rows on; bfloat16 from 96 on) and multiples of 4 where it
# takes over from the strips.  Operands carry 24 bits and the chain of a result has M / 32 links: 2^-24 sqrt(M / 32) and the final
# additions stay below 1e-6; bfloat16 results (8 significant bits) are rounded once, at most 2^-8 relative.
@pytest.mark.parametrize("S,M", [(17, 193), (27, 193), (28, 193), (64, 223), (65, 225), (63, 255), (130, 321), (50, 525), (200, 1023), (900, 896), (2304, 256), (384, 2304)])
def test_three_planes_f32(S, M):
    T32, Q64 = sym_Q(M, M + 9)
    Q32 = Q64.astype(np.float32)
    G = (rng.standard_normal((S, M)) * np.exp(rng.uniform(-8, 8, (S, 1)))).astype(np.float32)
    out = torch.full((S, M), float("nan"), device=DEV)
    b.fw_grad_transform(dev(G), b.FW_F32, S, M, None, dev(Q32), out)
    torch.cuda.synchronize()
    want = G.astype(np.float64) @ Q32.astype(np.float64)
    err = np.linalg.norm(out.cpu().numpy() - want, axis=1) / np.linalg.norm(want, axis=1)
    assert err.max() < 1e-6                   # every row against its own size


@pytest.mark.parametrize("S,M", [(3, 97), (64, 99), (65, 129), (50, 525), (1000, 256), (384, 512), (1000, 1156)])
def test_three_planes_bf16(S, M):
    T32, Q64 = sym_Q(M, M + 11)
    Q32 = Q64.astype(np.float32)
    G = wl.round_to_bf16((rng.standard_normal((S, M)) * 0.1).astype(np.float32))
    want = G.astype(np.float64) @ Q32.astype(np.float64)
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S, None, b.FW_BF16))
    out = torch.zeros(S, M, device=DEV, dtype=torch.bfloat16)
    b.fw_grad_transform(dev(G, torch.bfloat16), b.FW_BF16, S, M, None, dev(Q32), out, ws)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    assert np.max(np.abs(got - want) / np.maximum(np.abs(want), 1e-3 * np.abs(want).max())) < 1.001 * 2.0 ** -8
    W0 = rng.standard_normal((S, M)).astype(np.float32)
    W, V = dev(W0.copy()), torch.zeros(S, M, device=DEV)
    wsu = workspace(b.fw_workspace_bytes(b.FW_OP_SGD_UPDATE, M, S, None, b.FW_BF16))
    b.fw_sgd_update(dev(G, torch.bfloat16), b.FW_BF16, S, M, 1, dev(Q32), b.sgd_params(0.1, 0.9, 5e-4), W, V, wsu)
    torch.cuda.synchronize()
    d = want + 5e-4 * W0
    assert relF(V.cpu().numpy(), d) < 1e-6 and relF(W.cpu().numpy(), W0 - 0.1 * d) < 1e-6


# Numbers of any size in the three-plane form.  Rows of G (or all of Q) at 2^-k, up to where a tile is multiplied in float32 and down to where entries are subnormal: 24 bits of
# an operand and float32 sums leave the 1e-6 of above; a subnormal result is rounded to 2^-150, 2^-26 of a row at 2^-124.
@pytest.mark.parametrize("S,M", [(50, 525), (900, 896)])
@pytest.mark.parametrize("gdt", [b.FW_F32, b.FW_BF16])
def test_three_planes_numbers_of_any_size(S, M, gdt):
    T32, Q64 = sym_Q(M, M + 13)
    k = np.array([0, 60, -100, -118, 112, 116, 120, 124])
    tdt = torch.bfloat16 if gdt == b.FW_BF16 else torch.float32
    for gk, qk in ((k[np.arange(S) % 8][:, None], 0), (0, 116), (0, 124)):
        Q32 = (Q64 * 2.0 ** -float(qk)).astype(np.float32)
        G = (rng.standard_normal((S, M)) * 2.0 ** -gk.astype(float) if qk == 0 else rng.standard_normal((S, M))).astype(np.float32)
        if gdt == b.FW_BF16:
            G = wl.round_to_bf16(G)
        want = G.astype(np.float64) @ Q32.astype(np.float64)
        W, V = torch.zeros(S, M, device=DEV), torch.zeros(S, M, device=DEV)
        ws = workspace(b.fw_workspace_bytes(b.FW_OP_SGD_UPDATE, M, S, None, gdt))
        b.fw_sgd_update(dev(G, tdt), gdt, S, M, 1, dev(Q32), b.sgd_params(0.5, 0.9, 0.0), W, V, ws)
        got = {"V": V.cpu().numpy(), "W": -2.0 * W.cpu().numpy().astype(np.float64)}
        if gdt == b.FW_F32:
            out = torch.full((S, M), float("nan"), device=DEV)
            b.fw_grad_transform(dev(G), gdt, S, M, None, dev(Q32), out)
            got["out"] = out.cpu().numpy()
        for name, x in got.items():
            err = np.linalg.norm(x - want, axis=1) / np.linalg.norm(want, axis=1)
            assert err.max() < 1e-6, (name, int(err.argmax()))


# Infinite entries, NaN, and finite ones above the largest bfloat16 number: what float32 arithmetic gives, and only in the rows (of G) and
# columns (of Q) that they enter.
@pytest.mark.parametrize("S,M", [(50, 525), (130, 193), (900, 896)])
@pytest.mark.parametrize("gdt", [b.FW_F32, b.FW_BF16])
def test_three_planes_infinite_and_huge(S, M, gdt):
    T32, Q64 = sym_Q(M, M + 17)
    Q32 = (0.25 * Q64).astype(np.float32)
    Q32[7, 11] = Q32[11, 7] = 0.0
    tdt = torch.bfloat16 if gdt == b.FW_BF16 else torch.float32
    ws = workspace(b.fw_workspace_bytes(b.FW_OP_SGD_UPDATE, M, S, None, gdt))
    wst = workspace(b.fw_workspace_bytes(b.FW_OP_GRAD_TRANSFORM, M, S, None, gdt))
    for kind in ("G", "Q"):
        G = rng.standard_normal((S, M)).astype(np.float32)
        Q = Q32.copy()
        if kind == "G":
            G[3, 7], G[33, M - 1], G[S - 1, 0], G[5, 2] = np.inf, -np.inf, np.nan, 3.4e38 if gdt == b.FW_F32 else 3.3e38
        else:
            Q[9, 40] = Q[40, 9] = -np.inf
            Q[M - 1, M - 1] = 3.4e38
            G[:, M - 1] *= 0.1
        if gdt == b.FW_BF16:
            G = np.where(np.isfinite(G), wl.round_to_bf16(np.where(np.isfinite(G), G, 0).astype(np.float32)), G)
        with np.errstate(invalid="ignore"):
            want = G.astype(np.float64) @ Q.astype(np.float64)
        want = np.where(np.isnan(G).any(1)[:, None], np.nan, want)
        V, W = torch.zeros(S, M, device=DEV), torch.zeros(S, M, device=DEV)
        b.fw_sgd_update(dev(G, tdt), gdt, S, M, 1, dev(Q), b.sgd_params(0.0, 0.9, 0.0), W, V, ws)
        out = torch.zeros(S, M, device=DEV, dtype=tdt)
        b.fw_grad_transform(dev(G, tdt), gdt, S, M, None, dev(Q), out, wst)
        for got, bound in ((V.cpu().numpy(), 1e-6), (out.float().cpu().numpy(), 1e-6 if gdt == b.FW_F32 else 2.0 ** -8)):
            assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
            assert np.array_equal(np.isneginf(got), np.isneginf(want))
            ok = np.isfinite(want)
            # every row (and every huge column) against its own size
            for x, y in ((got, want), (got.T, want.T)):
                f = np.isfinite(y)
                for r in range(len(y)):
                    if f[r].any():
                        assert relF(x[r][f[r]].astype(np.float64), y[r][f[r]]) < bound
            assert ok.any()
