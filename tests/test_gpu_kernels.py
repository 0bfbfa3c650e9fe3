"""Kernel-level GPU parity through the C ABI's fusion_test_* entry points:
each kernel of the pipeline runs on caller-supplied packed ragged buffers
and is compared with the oracle's function for that step, at random ragged
lengths that include the degenerate cases (T = 1, T = 2, odd N, r = 0,
r = floor(N/2), k = 0, k = N, every sample exiting).

Merge and learned-score prune decisions follow the oracle's near-tie rule
(the GPU's choice may differ only where the oracle's margin is below 1e-3;
any other difference fails); CLS-attention prune scores are bit-identical
on both sides, so those decisions must match exactly.
"""
import numpy as np
import pytest

from oracle import fusion_oracle as fo

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _kern():
    from paper_2607_02612_amd import kernels
    return kernels


def _bf16(rng, shape, scale=1.0):
    return fo.bf16_round((rng.standard_normal(shape) * scale).astype(np.float32))


def _to_dev_bf16(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


# ------------------------------------------------------------------ GEMM --
GEMM_SHAPES = [(1, 1152, 384), (37, 1152, 384), (300, 1536, 384), (1000, 384, 1536),
               (129, 384, 384), (70, 1000, 384), (2049, 384, 384)]


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
@pytest.mark.parametrize("epi", ["store", "gelu", "resid", "f32"])
def test_gemm_bf16(torch_cuda, M, N, K, epi):
    torch = torch_cuda
    if epi in ("store", "gelu") and N % 8:
        pytest.skip("bf16 outputs need N % 8 == 0")
    print(f"[gemm bf16] M={M} N={N} K={K} epi={epi}", flush=True)
    rng = np.random.default_rng(M * 7 + N + K)
    A, W = _bf16(rng, (M, K)), _bf16(rng, (N, K), 0.05)
    bias = rng.standard_normal(N).astype(np.float32) * 0.1
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    bound = np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T
    dA, dW = _to_dev_bf16(torch, A), _to_dev_bf16(torch, W)
    db = torch.from_numpy(bias).cuda()
    k = _kern()
    if epi in ("store", "gelu"):
        out = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
        k.gemm(dA, dW, db, epi, out)
        g = out.float().cpu().numpy()
        pre = ref.astype(np.float32)
        r = fo.gelu(pre) if epi == "gelu" else pre
        # one bf16 rounding of a value that differs only by the fp32
        # accumulation order (and, for GELU, the 7e-7 approximation)
        err = np.abs(g - r) - (2.0 ** -8 * np.abs(r) + 1e-5 * bound + 1e-6)
        assert (err <= 0).all(), float(err.max())
        return
    rows = None
    nrow = M
    if epi in ("resid", "f32"):
        nrow = M + 5
        perm = rng.permutation(nrow)[:M].astype(np.int32)
        rows = torch.from_numpy(perm).cuda()
    x0 = rng.standard_normal((nrow, N)).astype(np.float32)
    out = torch.from_numpy(x0.copy()).cuda()
    k.gemm(dA, dW, db, epi, out, rows=rows)
    g = out.cpu().numpy()
    want = x0.astype(np.float64).copy()
    idx = perm
    want[idx] = (want[idx] if epi == "resid" else 0.0) + ref
    tol = 1e-5 * (bound + np.abs(x0[idx])) + 1e-6
    assert np.all(np.abs(g[idx] - want[idx]) <= tol)
    untouched = np.setdiff1d(np.arange(nrow), idx)
    assert np.array_equal(g[untouched], x0[untouched])


@pytest.mark.parametrize("M,N,K,epi", [
    (1, 64, 64, "store"), (33, 72, 192, "gelu"), (31, 36, 320, "resid"), (257, 1000, 64, "f32"),
    (197, 384, 1536, "resid"),                                  # one block per workgroup
    (300, 1152, 384, "store"), (511, 1004, 128, "resid"),       # two blocks
    (1000, 1536, 384, "gelu"), (2047, 384, 448, "resid"), (2017, 1000, 64, "f32"),  # four blocks
])
def test_gemm_bf16_small_launches(torch_cuda, M, N, K, epi):
    """Launches with few tiles: against float64, and bit for bit the rows that
    a launch with thousands of tiles gives (N % 8 == 4 included)."""
    torch = torch_cuda
    print(f"[gemm bf16 small] M={M} N={N} K={K} epi={epi}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A, W = _bf16(rng, (M, K)), _bf16(rng, (N, K), 0.05)
    bias = rng.standard_normal(N).astype(np.float32) * 0.1
    dA, dW = _to_dev_bf16(torch, A), _to_dev_bf16(torch, W)
    db = torch.from_numpy(bias).cuda()
    x0 = rng.standard_normal((M, N)).astype(np.float32)
    fp32 = epi in ("resid", "f32")

    def run(times):
        rows = torch.randperm(M * times, device="cuda").int() if fp32 else None
        out = torch.from_numpy(x0).cuda().to(torch.float32 if fp32 else torch.bfloat16)
        out = out.repeat(times, 1)
        if fp32:
            out[rows.long()] = out.clone()  # the row of A's row r is rows[r]
        _kern().gemm(dA.repeat(times, 1), dW, db, epi, out, rows)
        return (out[rows.long()] if fp32 else out).float().cpu().numpy()

    g = run(1)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    bound = np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T
    if fp32:
        want = ref + (x0 if epi == "resid" else 0.0)
        tol = 1e-5 * (bound + np.abs(x0)) + 1e-6
    else:
        want = fo.gelu(ref.astype(np.float32)) if epi == "gelu" else ref
        tol = 2.0 ** -8 * np.abs(want) + 1e-5 * bound + 1e-6
    assert (np.abs(g - want) <= tol).all()
    times = 2400 * 32 * 32 // (M * N) + 1  # beyond the small launches
    assert np.array_equal(run(times).reshape(times, M, N), np.broadcast_to(g, (times, M, N)))


@pytest.mark.parametrize("M,N,K,epi", [
    (2113, 1000, 64, "f32"), (2300, 1004, 192, "resid"), (2561, 840, 128, "store"),
    (4097, 520, 1536, "gelu"), (5000, 384, 384, "resid"),            # 64-row tiles, three stages
    (4225, 1000, 64, "store"), (4300, 1004, 192, "f32"), (9000, 520, 128, "gelu"),
    (12608, 384, 1536, "resid"),                                    # 128-row tiles, two stages
    (12300, 1000, 64, "gelu"), (33000, 384, 128, "resid"), (25000, 1000, 64, "store"),  # more rounds
    (300, 384, 96, "resid"), (2500, 1000, 32, "store"),             # K not a multiple of 64:
    (1, 64, 32, "store"), (65, 1004, 160, "f32"), (1573, 520, 96, "gelu"),  # 32-row waves
    (4097, 1500, 96, "resid"),                                      # 64-row waves
    (1049, 520, 64, "store"), (1700, 384, 192, "resid"), (3100, 384, 320, "f32"),  # short K
    (1084, 3072, 64, "gelu"), (10431, 768, 64, "resid"),            # 9 and 11 panels on an XCD
])
def test_gemm_bf16_medium_launches(torch_cuda, M, N, K, epi):
    """Launches whose tiles fit the chip once or in even rounds: against
    float64, and bit for bit the rows of a launch with thousands of tiles."""
    torch = torch_cuda
    print(f"[gemm bf16 medium] M={M} N={N} K={K} epi={epi}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    A, W, bias = rnd(M, K).bfloat16(), (0.05 * rnd(N, K)).bfloat16(), 0.1 * rnd(N)
    fp32 = epi in ("resid", "f32")
    x0 = rnd(M, N)

    def run(times):
        rows = torch.randperm(M * times, generator=g, device="cuda").int() if fp32 else None
        out = x0.repeat(times, 1).to(torch.float32 if fp32 else torch.bfloat16)
        if fp32:
            out[rows.long()] = out.clone()  # the row of A's row r is rows[r]
        _kern().gemm(A.repeat(times, 1), W, bias, epi, out, rows)
        return out[rows.long()] if fp32 else out

    got = run(1)
    ref = A.double() @ W.double().t() + bias.double()
    bound = A.double().abs() @ W.double().abs().t()
    if fp32:
        want = ref + (x0.double() if epi == "resid" else 0.0)
        tol = 1e-5 * (bound + x0.double().abs()) + 1e-6
    else:
        want = ref * 0.5 * (1 + torch.erf(ref / 2 ** 0.5)) if epi == "gelu" else ref
        tol = 2.0 ** -8 * want.abs() + 1e-5 * bound + 1e-6
    assert ((got.double() - want).abs() <= tol).all()
    times = 2100 * 128 * 128 // (M * N) + 1  # beyond the medium launches
    assert torch.equal(run(times).view(times, M, N), got.expand(times, M, N))


@pytest.mark.parametrize("M,N,K", [(6000, 1536, 384), (20000, 1536, 384), (12000, 768, 192),
                                   (6000, 3072, 768)])
def test_gemm_gelu_fc1_shapes(torch_cuda, M, N, K):
    """fc1 shapes of DeiT-Ti / S / B (K = 192, 384, 768) with hundreds to
    thousands of 128-row tiles and a ragged last row tile: every output
    against the float64 product + exact GELU."""
    torch = torch_cuda
    print(f"[gemm gelu fc1] M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A, W = _bf16(rng, (M, K)), _bf16(rng, (N, K), 0.05)
    bias = rng.standard_normal(N).astype(np.float32) * 0.1
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    bound = np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T
    out = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
    _kern().gemm(_to_dev_bf16(torch, A), _to_dev_bf16(torch, W), torch.from_numpy(bias).cuda(),
                 "gelu", out)
    g = out.float().cpu().numpy()
    r = fo.gelu(ref.astype(np.float32))
    err = np.abs(g - r) - (2.0 ** -8 * np.abs(r) + 1e-5 * bound + 1e-6)
    assert (err <= 0).all(), float(err.max())


@pytest.mark.parametrize("M,N,K,epi", [(1, 64, 64, "store"), (65, 256, 64, "gelu"),
                                       (130, 64, 256, "resid"), (9, 10, 64, "f32")])
def test_gemm_fp32(torch_cuda, M, N, K, epi):
    torch = torch_cuda
    rng = np.random.default_rng(N + K + M)
    A = rng.standard_normal((M, K)).astype(np.float32)
    W = (rng.standard_normal((N, K)) * 0.1).astype(np.float32)
    bias = rng.standard_normal(N).astype(np.float32)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    x0 = rng.standard_normal((M, N)).astype(np.float32)
    out = torch.from_numpy(x0.copy()).cuda()
    _kern().gemm(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda(),
                 torch.from_numpy(bias).cuda(), epi, out)
    g = out.cpu().numpy()
    want = {"store": ref, "gelu": fo.gelu(ref.astype(np.float32)), "resid": x0 + ref,
            "f32": ref}[epi]
    assert np.abs(g - want).max() <= 1e-4


@pytest.mark.parametrize("M,N,K,epi,shift", [
    (33, 68, 16, "store", 0),      # one K step, edges of 32-row tiles
    (31, 36, 144, "resid", 0),     # more K steps than ring stages
    (95, 70, 48, "gelu", 0),       # columns that 16-byte stores do not fit
    (2100, 1025, 32, "f32", 0),    # 64-row tiles, scalar stores
    (4200, 516, 80, "resid", 0),   # 64-row tiles with edges
    (33, 36, 32, "store", 0),      # K steps of 32: fewer than, and more than, the stages
    (65, 68, 160, "resid", 0),
    (4300, 1100, 32, "gelu", 0),   # the same with more tiles
    (4300, 1090, 96, "f32", 0),
    (6400, 1150, 96, "f32", 0),    # 64-row tiles: from 1792 of them at K = 96,
    (4100, 1180, 512, "resid", 0),  # 1152 at K = 512
    (40, 64, 40, "store", 0),      # K not a multiple of 16: general kernel
    (40, 64, 64, "store", 1),      # operands off 16-byte alignment: general kernel
])
def test_gemm_fp32_tiles(torch_cuda, M, N, K, epi, shift):
    """Each route of the fp32 product against float64 (K rounded products and
    sums), rows through a map, and a row alone equal to the same row in M."""
    torch = torch_cuda
    print(f"[gemm fp32] M={M} N={N} K={K} epi={epi} shift={shift}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    W = rng.standard_normal((N, K)).astype(np.float32)
    bias = rng.standard_normal(N).astype(np.float32)
    dA = torch.zeros(M * K + shift, device="cuda")[shift:].view(M, K)
    dA.copy_(torch.from_numpy(A))
    dW, db = torch.from_numpy(W).cuda(), torch.from_numpy(bias).cuda()
    mapped = epi in ("resid", "f32")
    rows = rng.permutation(M + 3)[:M].astype(np.int32) if mapped else np.arange(M)
    x0 = rng.standard_normal((M + 3 if mapped else M, N)).astype(np.float32)
    out = torch.from_numpy(x0.copy()).cuda()
    _kern().gemm(dA, dW, db, epi, out, torch.from_numpy(rows).cuda() if mapped else None)
    g = out.cpu().numpy()
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    bound = (np.abs(A).astype(np.float64) @ np.abs(W).astype(np.float64).T + np.abs(bias)
             + np.abs(x0[rows])) * (K + 4) * 2.0 ** -24 + 1e-6
    want = fo.gelu(ref.astype(np.float32)) if epi == "gelu" else ref
    if epi == "resid":
        want = want + x0[rows]
    assert (np.abs(g[rows] - want) <= 2 * bound).all()
    if mapped:
        rest = np.setdiff1d(np.arange(M + 3), rows)
        assert np.array_equal(g[rest], x0[rest])
    one = torch.from_numpy(x0[rows[M - 1]][None].copy()).cuda()
    _kern().gemm(dA[M - 1:], dW, db, epi, one)
    assert np.array_equal(one.cpu().numpy()[0], g[rows[M - 1]])


def test_gemm_fp32_rows_past_4_gib(torch_cuda):
    """An operand of more than 4 GiB: rows at its start, on both sides of the
    limit and at its end have the bits they have in a small product."""
    torch = torch_cuda
    M, N, K = (1 << 20) + 4099, 36, 1024
    print(f"[gemm fp32] M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn(M, K, generator=g, device="cuda")
    W, bias = torch.randn(N, K, generator=g, device="cuda"), torch.randn(N, generator=g, device="cuda")
    out = torch.empty(M, N, device="cuda")
    _kern().gemm(A, W, bias, "store", out)
    for i in (0, (1 << 20) - 70, M - 130):
        part = torch.empty(130, N, device="cuda")
        _kern().gemm(A[i:i + 130], W, bias, "store", part)
        assert torch.equal(out[i:i + 130], part), i


# ------------------------------------------------------------- attention --
ATT_CASES = [
    # lengths, heads, dh, precision, prop_attn
    ([1, 2, 17, 64, 197, 250, 33], 6, 64, "bf16", True),
    ([1, 2, 17, 64, 197, 250, 33], 6, 64, "bf16", False),
    ([577, 1, 300, 129, 2, 400], 6, 64, "bf16", True),   # long resident kernel (<= 592)
    ([640, 17, 3, 599], 6, 64, "bf16", True),             # chunked kernel (593 .. 640)
    ([260, 33, 272], 6, 64, "bf16", False),               # 17 key tiles
    ([1, 2, 33, 65, 7], 2, 32, "fp32", True),
]


@pytest.mark.parametrize("lengths,H,dh,prec,prop", ATT_CASES)
def test_attention_ragged(torch_cuda, lengths, H, dh, prec, prop):
    torch = torch_cuda
    print(f"[attention] T={lengths} H={H} {prec} prop={prop}", flush=True)
    rng = np.random.default_rng(sum(lengths) + H)
    cu = _offsets(lengths)
    M, d = int(cu[-1]), H * dh
    mode = "bf16emu" if prec == "bf16" else "fp32"
    qkv = fo._rnd((rng.standard_normal((M, 3 * d)) * 1.2).astype(np.float32), mode)
    size = rng.integers(1, 5, size=M).astype(np.float32) if prop else np.ones(M, np.float32)
    tmax = max(lengths) + 3
    dq = _to_dev_bf16(torch, qkv) if prec == "bf16" else torch.from_numpy(qkv).cuda()
    out, cls = _kern().attention(dq, torch.from_numpy(size).cuda(), cu, H, prop, cls_tmax=tmax)
    O = out.float().cpu().numpy()
    C = cls.cpu().numpy()
    worst = 0.0
    for i, T in enumerate(lengths):
        a, b = cu[i], cu[i + 1]
        Oref, cref = fo.attention_heads(qkv[a:b], size[a:b], H, int(prop), mode, True)
        e = np.abs(O[a:b] - Oref)
        if prec == "bf16":
            # exp in base 2 with folded constants and one bf16 rounding of E
            # and of O on each side
            assert (e <= 1e-2 + 2.0 ** -7 * np.abs(Oref)).all(), (i, T, float(e.max()))
        else:
            assert e.max() <= 1e-5, (i, T, float(e.max()))
        worst = max(worst, float(e.max()))
        cmean = C[i, :, :T].mean(axis=0)
        assert np.abs(cmean - cref).max() <= 2e-6, (i, T)
        assert np.all(C[i, :, T:] == -1.0), "entries past the sample untouched"
        assert np.abs(C[i, :, :T].sum(axis=1) - 1.0).max() <= 1e-5
    print(f"  max |dO| = {worst:.3e}")



@pytest.mark.parametrize("T", [1, 128, 129, 144, 256, 257, 400, 592])
def test_attention_split_queries(torch_cuda, T):
    """One sample, whose query tiles are split over workgroups, gives the bits
    that it gives inside a batch that fills the chip (CLS rows included)."""
    torch = torch_cuda
    print(f"[attention split] T={T}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T)
    H, n = 3, 180
    qkv = torch.randn(T, 3 * 64 * H, generator=g, device="cuda").bfloat16()
    size = torch.randint(1, 4, (T,), generator=g, device="cuda").float()
    one, cls1 = _kern().attention(qkv, size, [0, T], H, True, T)
    many, cls = _kern().attention(qkv.repeat(n, 1), size.repeat(n), [T * i for i in range(n + 1)],
                                  H, True, T)
    assert torch.equal(many.view(n, T, -1), one.expand(n, T, -1))
    assert torch.equal(cls, cls1.expand(n, H, T))


@pytest.mark.parametrize("lengths,H,dh", [
    ([64, 65, 1, 16, 17, 128], 2, 64),    # chunk and query-block edges
    ([256, 255, 63, 193], 3, 20),         # head padded from 20 to 32 dims
    ([257, 640, 2, 320], 1, 128),         # longest samples, widest heads
    ([130, 66], 2, 36),                   # padded from 36 to 64 dims
    ([40, 3], 2, 6),                      # width without 16-byte pieces: general kernel
    ([50, 7], 1, 132),                    # wider than the matrix kernel takes
])
def test_attention_fp32_widths(torch_cuda, lengths, H, dh):
    """fp32 attention over head widths, sample lengths and (shifted by one
    float) unaligned buffers: every form against float64.  E and the two
    products are fp32 sums of at most max(T, dh) terms."""
    torch = torch_cuda
    print(f"[attention fp32] T={lengths} H={H} dh={dh}", flush=True)
    rng = np.random.default_rng(sum(lengths) + dh)
    cu = _offsets(lengths)
    M, d = int(cu[-1]), H * dh
    qkv = rng.standard_normal((M, 3 * d)).astype(np.float32)
    size = rng.integers(1, 5, size=M).astype(np.float32)
    base = torch.zeros(M * 3 * d + 1, device="cuda")
    for shift in (0, 1):
        dq = base[shift:shift + M * 3 * d].view(M, 3 * d)
        dq.copy_(torch.from_numpy(qkv))
        out, cls = _kern().attention(dq, torch.from_numpy(size).cuda(), cu, H, True,
                                     cls_tmax=max(lengths))
        out, cls = out.cpu().numpy(), cls.cpu().numpy()
        for i, T in enumerate(lengths):
            q, k, v = (qkv[cu[i]:cu[i + 1], j * d:(j + 1) * d].astype(np.float64)
                       .reshape(T, H, dh).transpose(1, 0, 2) for j in range(3))
            S = q @ k.transpose(0, 2, 1) / np.sqrt(dh) + np.log(size[cu[i]:cu[i + 1]])
            P = np.exp(S - S.max(-1, keepdims=True))
            P /= P.sum(-1, keepdims=True)
            want = (P @ v).transpose(1, 0, 2).reshape(T, d)
            tol = 2.0 ** -24 * max(T, dh) * 4
            assert np.abs(out[cu[i]:cu[i + 1]] - want).max() <= tol * np.abs(v).max(), (shift, i)
            assert np.abs(cls[i, :, :T] - P[:, 0]).max() <= tol, (shift, i)
            assert (cls[i, :, T:] == -1).all()


@pytest.mark.parametrize("T", [65, 400, 640])
def test_attention_fp32_sum_of_small_terms(torch_cuda, T):
    """One key of weight 1 and T - 1 of weight 2^-25: summed one after the
    other onto the 1 they vanish (5e-6 of the probability at 640 keys), summed
    in pairs at most the few that meet it first do."""
    torch = torch_cuda
    print(f"[attention fp32 sum] T={T}", flush=True)
    qkv = np.zeros((T, 192), np.float32)
    qkv[0, 0] = 8.0  # times 1 / sqrt(64): the score is the key's first entry
    qkv[1:, 64] = -25 * np.log(2.0)
    _, cls = _kern().attention(torch.from_numpy(qkv).cuda(), torch.ones(T, device="cuda"), [0, T], 1,
                               True, T)
    S = qkv[:, 64].astype(np.float64)
    P = np.exp(S) / np.exp(S).sum()
    # 2 + 2 levels in a chunk of 64 keys, up to 10 chunks, 2 lane swaps, exp and
    # the division: 16 roundings of half an ulp, and two of the exp's own
    tol = 18 * 2.0 ** -24
    assert np.abs(cls[0, 0].cpu().numpy() / P - 1).max() <= tol


# ----------------------------------------------------------------- merge --
def _tokens(rng, T, d, rank=8):
    """Hidden states with a low-rank structure (cosines spread over [-1, 1])."""
    basis = rng.standard_normal((rank, d))
    c = rng.standard_normal((T, rank))
    return (c @ basis + 0.4 * rng.standard_normal((T, d))).astype(np.float32)


MERGE_CASES = [
    # lengths, d
    ([1, 2, 3, 4, 17, 64, 97, 128], 384),     # size class T <= 128
    ([1, 2, 3, 18, 129, 197, 256, 65], 384),  # T <= 256
    ([577, 300, 1, 2, 451], 384),             # T <= 640
    ([197, 5, 66, 31], 192),
    ([130, 257, 258, 260, 40], 768),          # 128 / 129 / 130 A tokens, wide rows
]


@pytest.mark.parametrize("lengths,d", MERGE_CASES)
def test_merge_ragged(torch_cuda, lengths, d):
    torch = torch_cuda
    print(f"[merge] T={lengths} d={d}", flush=True)
    rng = np.random.default_rng(len(lengths) * 1000 + d + lengths[0])
    cu = _offsets(lengths)
    M = int(cu[-1])
    x = np.concatenate([_tokens(rng, T, d) for T in lengths])
    size = rng.integers(1, 4, size=M).astype(np.float32)
    id_stride = max(lengths) + 7
    origin = np.concatenate([np.sort(rng.permutation(id_stride)[:T]) for T in lengths]).astype(np.int32)
    r = []
    for j, T in enumerate(lengths):
        N = T - 1
        r.append([0, N // 2, N // 2, rng.integers(0, N // 2 + 1)][j % 4])
    r = np.array(r, dtype=np.int32)
    dx = torch.from_numpy(x.copy()).cuda()
    o, md = _kern().merge(dx, torch.from_numpy(size).cuda(), torch.from_numpy(origin).cuda(),
                          cu, r, id_stride)
    torch.cuda.synchronize()
    xg = dx.cpu().numpy()
    o = {k: v.cpu().numpy() for k, v in o.items()}
    md = md.cpu().numpy()
    B = len(lengths)
    assert list(o["counts"]) == [B, int(M - r.sum())]
    assert list(o["live"]) == list(range(B))
    assert np.array_equal(o["cu"], _offsets([T - int(rr) for T, rr in zip(lengths, r)]))
    adopted = []
    for i, T in enumerate(lengths):
        a, b = cu[i], cu[i + 1]
        xs, ss, og = x[a:b], size[a:b], origin[a:b].astype(np.int64)
        plan = fo.merge_plan(xs, int(r[i]))
        gmap = {int(s_): int(t_) for s_, t_ in enumerate(md[i]) if t_ >= 0}
        chosen, dst = fo._follow_merge(1, plan, int(r[i]), og, gmap, fo.TOL, adopted)
        if r[i] > 0:
            xr, sr, _, orr = fo.apply_merge(xs, ss, None, og, plan["A"], plan["B"], chosen, dst)
        else:
            xr, sr, orr = xs, ss, og
        p, q = o["cu"][i], o["cu"][i + 1]
        assert np.array_equal(o["origin"][p:q], orr), i
        assert np.array_equal(o["size"][p:q], sr), i
        rows = o["rows"][p:q]
        assert np.all((rows >= a) & (rows < b))
        got = xg[rows]
        assert np.abs(got - xr).max() <= 2e-6 * max(1.0, float(np.abs(xr).max())), i
    n_dec = int(r.sum())
    print(f"  merges={n_dec} near-tie adoptions={len(adopted)}")
    assert len(adopted) <= max(2, n_dec // 20)


def _axis_tokens(rng, T, d, n_axes=3):
    """Tokens c e_j with c = +-2^k and j among a few axes: every cosine is
    exactly -1, 0 or 1 in any arithmetic (and the merge weights exact), so
    the best matches and the top-r tie massively and identically on both
    sides; ties go to the lower B slot and the lower A slot."""
    x = np.zeros((T, d), np.float32)
    j = rng.integers(0, n_axes, size=T)
    c = rng.choice([-2.0, -1.0, 0.5, 1.0, 2.0, 4.0], size=T).astype(np.float32)
    x[np.arange(T), j] = c
    return x


@pytest.mark.parametrize("lengths", [[97, 128, 3, 2], [197, 256, 130, 1], [577, 640, 300, 514]])
def test_merge_exact_ties(torch_cuda, lengths):
    """Selections among exactly equal similarities: identical to the oracle
    with no near-tie adoption (every size class, long samples through the
    similarity passes)."""
    torch = torch_cuda
    print(f"[merge ties] T={lengths}", flush=True)
    rng = np.random.default_rng(sum(lengths))
    d = 192
    cu = _offsets(lengths)
    M = int(cu[-1])
    x = np.concatenate([_axis_tokens(rng, T, d) for T in lengths])
    size = rng.integers(1, 4, size=M).astype(np.float32)
    id_stride = max(lengths) + 1
    origin = np.concatenate([np.arange(T) for T in lengths]).astype(np.int32)
    r = np.array([min([(T - 1) // 2, (T - 1) // 3, (T - 1) // 5, 1][j % 4], (T - 1) // 2)
                  for j, T in enumerate(lengths)], dtype=np.int32)
    dx = torch.from_numpy(x.copy()).cuda()
    o, md = _kern().merge(dx, torch.from_numpy(size).cuda(), torch.from_numpy(origin).cuda(),
                          cu, r, id_stride)
    torch.cuda.synchronize()
    xg = dx.cpu().numpy()
    o = {k: v.cpu().numpy() for k, v in o.items()}
    md = md.cpu().numpy()
    adopted = []
    for i, T in enumerate(lengths):
        a, b = cu[i], cu[i + 1]
        xs, ss, og = x[a:b], size[a:b], origin[a:b].astype(np.int64)
        plan = fo.merge_plan(xs, int(r[i]))
        gmap = {int(s_): int(t_) for s_, t_ in enumerate(md[i]) if t_ >= 0}
        chosen, dst = fo._follow_merge(1, plan, int(r[i]), og, gmap, 0.0, adopted)
        if r[i] > 0:
            assert np.array_equal(np.sort(chosen), np.sort(plan["chosen"])), i
            assert np.array_equal(dst[np.argsort(chosen)], plan["best"][np.sort(chosen)]), i
            xr, sr, _, orr = fo.apply_merge(xs, ss, None, og, plan["A"], plan["B"], chosen, dst)
        else:
            xr, sr, orr = xs, ss, og
        p, q = o["cu"][i], o["cu"][i + 1]
        assert np.array_equal(o["origin"][p:q], orr), i
        assert np.array_equal(o["size"][p:q], sr), i
        assert np.abs(xg[o["rows"][p:q]] - xr).max() <= 2e-6 * max(1.0, float(np.abs(xr).max())), i
    assert not adopted


# --------------------------------------------------------- prune, compact --
def _cls_scores(rng, lengths, H, tmax):
    S = np.full((len(lengths), H, tmax), -3.0, dtype=np.float32)
    for i, T in enumerate(lengths):
        e = rng.random((H, T)).astype(np.float32) ** 3 + 1e-3
        S[i, :, :T] = e / e.sum(axis=1, keepdims=True)
    return S


@pytest.mark.parametrize("keep,rho", [(0.7, 1.0), (0.7, 1.5), (0.0, 1.0), (1.0, 1.0)])
def test_topk_compact_cls_attention(torch_cuda, keep, rho):
    torch = torch_cuda
    lengths = [1, 2, 3, 10, 65, 197, 128, 300, 4]
    print(f"[topk cls] tau={keep} rho={rho}", flush=True)
    rng = np.random.default_rng(int(keep * 100 + rho * 10))
    H, d = 6, 384
    cu = _offsets(lengths)
    M, B = int(cu[-1]), len(lengths)
    x = np.concatenate([_tokens(rng, T, d) for T in lengths])
    size = rng.integers(1, 4, size=M).astype(np.float32)
    origin = np.concatenate([np.arange(T) for T in lengths]).astype(np.int32)
    tmax = max(lengths)
    S = _cls_scores(rng, lengths, H, tmax)
    C = 10
    lg = rng.standard_normal((B, C)).astype(np.float32)
    lg[::3, 2] += 6.0                                  # confident: exits
    delta = 0.5
    g = (1 + 0.1 * rng.standard_normal(d)).astype(np.float32)
    bb = (0.1 * rng.standard_normal(d)).astype(np.float32)
    tau_eff = min(1.0, max(0.0, 1.0 - rho * (1.0 - keep)))
    T_ = torch.from_numpy
    o, logits, eb, ln_out = _kern().topk_compact(
        T_(x).cuda(), T_(size).cuda(), T_(origin).cuda(), cu, tau_eff, scores=T_(S).cuda(),
        heads=H, exit_logits=T_(lg).cuda(), delta=delta, ln=(T_(g).cuda(), T_(bb).cuda()))
    o = {k: v.cpu().numpy() for k, v in o.items()}
    logits, eb, ln_out = logits.cpu().numpy(), eb.cpu().numpy(), ln_out.float().cpu().numpy()
    j = 0
    for i, T in enumerate(lengths):
        c = fo.max_softmax(lg[i])
        assert abs(float(c) - delta) > 1e-4
        if c >= delta:
            assert eb[i] == 1 and np.array_equal(logits[i], lg[i])
            assert i not in o["live"][:o["counts"][0]]
            continue
        assert eb[i] == -1 and np.all(logits[i] == -7.0)
        assert o["live"][j] == i
        a = cu[i]
        acc = S[i, 0, :T].copy()
        for h in range(1, H):
            acc = acc + S[i, h, :T]
        score = (acc / np.float32(H)).astype(np.float32)
        k = fo.keep_count(T - 1, keep, rho)
        kept, _, _ = fo.prune_plan(score, k)
        rows = np.concatenate([[0], 1 + kept])
        p, q = o["cu"][j], o["cu"][j + 1]
        assert q - p == k + 1
        assert np.array_equal(o["origin"][p:q], origin[a + rows])
        assert np.array_equal(o["rows"][p:q], a + rows)
        assert np.array_equal(o["size"][p:q], size[a + rows])
        ref = fo.bf16_round(fo.layer_norm(x[a + rows], g, bb))
        assert np.abs(ln_out[p:q] - ref).max() <= 2.0 ** -7 * max(1.0, float(np.abs(ref).max()))
        j += 1
    assert o["counts"][0] == j
    assert o["counts"][1] == o["cu"][j]


@pytest.mark.parametrize("lengths", [[640, 513, 514, 200, 2], [600, 97, 1, 639]])
def test_topk_compact_exact_ties(torch_cuda, lengths):
    """CLS-attention scores on a grid of a few values (and signed zeros,
    which compare equal): the kept sets are decided by the lower-slot tie
    rule on both sides and must be identical, including samples of more
    than 513 tokens (two candidates per thread)."""
    torch = torch_cuda
    print(f"[topk ties] T={lengths}", flush=True)
    rng = np.random.default_rng(len(lengths) + lengths[0])
    H, d = 3, 64
    cu = _offsets(lengths)
    M, B = int(cu[-1]), len(lengths)
    x = rng.standard_normal((M, d)).astype(np.float32)
    size = np.ones(M, np.float32)
    origin = np.concatenate([np.arange(T) for T in lengths]).astype(np.int32)
    tmax = max(lengths)
    S = np.full((B, H, tmax), -3.0, dtype=np.float32)
    for i, T in enumerate(lengths):
        S[i, :, :T] = rng.integers(0, 4, size=(H, T)).astype(np.float32) / 8.0
        z = rng.random(T) < 0.3
        S[i, :, :T][:, z] = rng.choice([0.0, -0.0], size=(H, int(z.sum()))).astype(np.float32)
    T_ = torch.from_numpy
    o, _, _, _ = _kern().topk_compact(T_(x).cuda(), T_(size).cuda(), T_(origin).cuda(), cu, 0.7,
                                      scores=T_(S).cuda(), heads=H)
    o = {k: v.cpu().numpy() for k, v in o.items()}
    for i, T in enumerate(lengths):
        acc = S[i, 0, :T].copy()
        for h in range(1, H):
            acc = acc + S[i, h, :T]
        score = (acc / np.float32(H)).astype(np.float32)
        k = fo.keep_count(T - 1, 0.7, 1.0)
        kept, _, _ = fo.prune_plan(score, k)
        rows = np.concatenate([[0], 1 + kept])
        p, q = o["cu"][i], o["cu"][i + 1]
        assert np.array_equal(o["rows"][p:q], cu[i] + rows), i


@pytest.mark.parametrize("lengths", [[128, 127, 66], [256, 130, 129, 65], [640, 258, 257, 130, 129]])
@pytest.mark.parametrize("H,keep", [(1, 0.5), (2, 1.0), (4, 0.02), (12, 0.9)])
def test_topk_selection_edges(torch_cuda, lengths, H, keep):
    """Selection sizes around the wave width and the change from the rank
    count to the wave search (129 tokens), with few distinct scores, equal
    scores throughout and infinities: the kept sets are identical to the
    lower-slot tie rule."""
    torch = torch_cuda
    print(f"[topk edges] T={lengths} H={H} keep={keep}", flush=True)
    rng = np.random.default_rng(H + lengths[0])
    cu = _offsets(lengths)
    M, B, tmax = int(cu[-1]), len(lengths), max(lengths)
    x = rng.standard_normal((M, 64)).astype(np.float32)
    origin = np.concatenate([np.arange(T) for T in lengths]).astype(np.int32)
    for kind in ("few", "equal", "inf"):
        S = rng.integers(1, 4, size=(B, 1, tmax)).astype(np.float32) / 8
        if kind == "equal":
            S[:] = 0.25
        if kind == "inf":
            S[rng.random(S.shape) < 0.2] = np.inf
            S[rng.random(S.shape) < 0.2] = -np.inf
        S = np.repeat(S, H, axis=1)  # equal heads: their mean is exact for these values
        T_ = torch.from_numpy
        o, _, _, _ = _kern().topk_compact(T_(x).cuda(), T_(np.ones(M, np.float32)).cuda(),
                                          T_(origin).cuda(), cu, keep, scores=T_(S).cuda(), heads=H)
        o = {k: v.cpu().numpy() for k, v in o.items()}
        for i, T in enumerate(lengths):
            k = int(np.floor(keep * (T - 1)))
            order = np.argsort(-S[i, 0, 1:T], kind="stable")[:k]
            rows = np.concatenate([[0], 1 + np.sort(order)])
            assert np.array_equal(o["origin"][o["cu"][i]:o["cu"][i + 1]], rows), (kind, i)


def test_topk_compact_learned_scorer_fp32_ln(torch_cuda):
    torch = torch_cuda
    lengths = [1, 2, 9, 64, 197, 5]
    rng = np.random.default_rng(11)
    d = 256
    cu = _offsets(lengths)
    M = int(cu[-1])
    x = np.concatenate([_tokens(rng, T, d) for T in lengths])
    size = np.ones(M, np.float32)
    origin = np.concatenate([np.arange(T) for T in lengths]).astype(np.int32)
    w = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    beta = np.array([0.3], np.float32)
    g = np.ones(d, np.float32)
    bb = np.zeros(d, np.float32)
    T_ = torch.from_numpy
    o, _, _, ln_out = _kern().topk_compact(
        T_(x).cuda(), T_(size).cuda(), T_(origin).cuda(), cu, 0.7, prune_w=T_(w).cuda(),
        prune_b=T_(beta).cuda(), ln=(T_(g).cuda(), T_(bb).cuda()), precision=0)
    o = {k: v.cpu().numpy() for k, v in o.items()}
    ln_out = ln_out.cpu().numpy()
    assert list(o["counts"]) == [len(lengths), int(sum(1 + int(np.floor(0.7 * (T - 1))) for T in lengths))]
    adopted = []
    for i, T in enumerate(lengths):
        a = cu[i]
        score = fo.learned_scores(x[a:a + T], w, beta[0])
        k = fo.keep_count(T - 1, 0.7, 1.0)
        kept, _, order = fo.prune_plan(score, k, 1.0)
        p, q = o["cu"][i], o["cu"][i + 1]
        kept = fo._follow_prune(1, score, k, kept, order, origin[a:a + T].astype(np.int64),
                                list(o["origin"][p:q]), fo.TOL, adopted, 1.0)
        rows = np.concatenate([[0], 1 + kept])
        assert np.array_equal(o["rows"][p:q], a + rows)
        ref = fo.layer_norm(x[a + rows], g, bb)
        assert np.abs(ln_out[p:q] - ref).max() <= 1e-5
    assert len(adopted) <= 1


def test_topk_compact_every_sample_exits(torch_cuda):
    torch = torch_cuda
    lengths = [3, 1, 20]
    rng = np.random.default_rng(5)
    cu = _offsets(lengths)
    M, B = int(cu[-1]), len(lengths)
    x = rng.standard_normal((M, 64)).astype(np.float32)
    S = _cls_scores(rng, lengths, 2, 20)
    lg = rng.standard_normal((B, 4)).astype(np.float32)
    T_ = torch.from_numpy
    o, logits, eb, _ = _kern().topk_compact(
        T_(x).cuda(), T_(np.ones(M, np.float32)).cuda(),
        T_(np.zeros(M, np.int32)).cuda(), cu, 0.7, scores=T_(S).cuda(), heads=2,
        exit_logits=T_(lg).cuda(), delta=0.0)
    assert list(o["counts"].cpu().numpy()) == [0, 0]
    assert np.all(eb.cpu().numpy() == 1)
    assert np.array_equal(logits.cpu().numpy(), lg)


# ------------------------------------------ the caller's workspace variants --
@pytest.mark.parametrize("B", [1, 63, 64, 128, 447, 448, 895, 896])
def test_workspace_entries_equal_allocating_ones(torch_cuda, B):
    """The binding (workspace entries; offsets as a kernel argument of two
    sizes, or copied) gives what the allocating entries write into buffers
    that hold the documented values before the call, on a side stream and
    with the arguments reused right after the call."""
    import ctypes
    torch = torch_cuda
    from paper_2607_02612_amd import _native
    print(f"[workspace] samples={B}", flush=True)
    L, kern = _native.lib(), _kern()
    rng = np.random.default_rng(B)
    lengths = [int(v) for v in rng.integers(1, 12 if B > 64 else 80, size=B)]
    cu = _offsets(lengths)
    M, d, H, C, tmax = int(cu[-1]), 128, 2, 7, max(lengths) + 3
    f = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda()
    x, size = f(M, d), torch.from_numpy(rng.integers(1, 4, size=M).astype(np.float32)).cuda()
    origin = torch.from_numpy(np.concatenate([np.arange(T) for T in lengths]).astype(np.int32)).cuda()
    r = np.array([(T - 1) // 3 for T in lengths], np.int32)
    qkv, scores, logits_in = f(M, 3 * d).bfloat16(), f(B, H, tmax).abs(), 3 * f(B, C)
    ln = (f(d), f(d))
    cp = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        cu_b, r_b, xb = cu.copy(), r.copy(), x.clone()
        at, cls = kern.attention(qkv, size, cu_b, H, True, tmax)
        om, md = kern.merge(xb, size, origin, cu_b, r_b, tmax)
        ot, lg, eb, lo = kern.topk_compact(x, size, origin, cu_b, 0.6, scores=scores, heads=H,
                                           exit_logits=logits_in, delta=0.6, ln=ln)
        cu_b[:], r_b[:] = -1, -1
    stream.synchronize()
    full = lambda v, dt, *s: torch.full(s, v, dtype=dt, device="cuda")
    i32, f32 = torch.int32, torch.float32

    def packed():
        o = dict(rows=full(-1, i32, M), size=full(-1, f32, M), origin=full(-1, i32, M),
                 cu=full(-1, i32, B + 1), live=full(-1, i32, B), counts=full(-1, i32, 2))
        return o, _native.FusionPackedOut(*(o[k].data_ptr() for k in ("rows", "size", "origin", "cu",
                                                                      "live", "counts")))
    s0 = torch.cuda.current_stream().cuda_stream
    at0, cls0 = full(0, torch.bfloat16, M, d), full(-1, f32, B, H, tmax)
    _native.check(L.fusion_test_attention(1, qkv.data_ptr(), size.data_ptr(), cp(cu), B, H, d, 1,
                                          at0.data_ptr(), cls0.data_ptr(), tmax, s0))
    assert torch.equal(at, at0) and torch.equal(cls, cls0)
    xa = x.clone()
    o0, po = packed()
    md0 = full(-1, i32, B, tmax)
    rg = _native.FusionRagged(xa.data_ptr(), size.data_ptr(), origin.data_ptr(), cp(cu), B, d)
    _native.check(L.fusion_test_merge(ctypes.byref(rg), cp(r), tmax, md0.data_ptr(),
                                      ctypes.byref(po), s0))
    assert torch.equal(xb, xa) and torch.equal(md, md0)
    assert all(torch.equal(om[k], o0[k]) for k in o0)
    o0, po = packed()
    lg0, eb0, lo0 = full(-7, f32, B, C), full(-1, i32, B), full(0, torch.bfloat16, M, d)
    rg = _native.FusionRagged(x.data_ptr(), size.data_ptr(), origin.data_ptr(), cp(cu), B, d)
    _native.check(L.fusion_test_topk_compact(
        ctypes.byref(rg), scores.data_ptr(), H, tmax, None, None, 0.6, logits_in.data_ptr(), C, 0.6,
        lg0.data_ptr(), eb0.data_ptr(), 1, ln[0].data_ptr(), ln[1].data_ptr(), lo0.data_ptr(),
        ctypes.byref(po), s0))
    assert torch.equal(lg, lg0) and torch.equal(eb, eb0) and torch.equal(lo, lo0)
    assert all(torch.equal(ot[k], o0[k]) for k in o0)


def test_workspace_entries_refuse_capture(torch_cuda):
    """Offsets and counts belong to one call: no recording into a graph."""
    torch = torch_cuda
    from paper_2607_02612_amd import FusionError
    qkv, size = torch.zeros(4, 192, device="cuda"), torch.ones(4, device="cuda")
    _kern().attention(qkv, size, [0, 4], 1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        size.add_(0)
        with pytest.raises(FusionError):
            _kern().attention(qkv, size, [0, 4], 1)


def test_calls_record_the_tensors_they_use(torch_cuda, monkeypatch):
    """The calls return before their kernels ran, so each tensor of the caller
    that they use is recorded on the stream: one that belongs to another stream
    keeps its memory until then (gemm leaves that to the caller)."""
    torch = torch_cuda
    used = set()
    record = torch.Tensor.record_stream
    monkeypatch.setattr(torch.Tensor, "record_stream",
                        lambda t, s: (used.add((t.data_ptr(), s.cuda_stream)), record(t, s))[1])
    f = lambda *s: torch.rand(*s, device="cuda")
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    x, size, origin, qkv = f(5, 64), f(5) + 1, i32(0, 1, 2, 0, 1), f(5, 192)
    scores, lg, ln = f(2, 1, 3), f(2, 7), (f(64), f(64))
    pw, pb = f(64), f(1)
    side.wait_stream(torch.cuda.current_stream())
    cu, k = [0, 3, 5], _kern()
    calls = [(lambda: k.attention(qkv, size, cu, 1), (qkv, size)),
             (lambda: k.merge(x, size, origin, cu, [1, 0], 3), (x, size, origin)),
             (lambda: k.merge(x, size, origin, cu, [1, 0], 3, noalloc=True), (x, size, origin)),
             (lambda: k.topk_compact(x, size, origin, cu, 0.5, scores=scores, exit_logits=lg, delta=0.9,
                                     ln=ln), (x, size, origin, scores, lg, *ln)),
             (lambda: k.topk_compact(x, size, origin, cu, 0.5, prune_w=pw, prune_b=pb), (x, pw, pb))]
    for n, (call, tensors) in enumerate(calls):
        used.clear()
        with torch.cuda.stream(side):
            call()
        assert {(t.data_ptr(), side.cuda_stream) for t in tensors} <= used, n
    torch.cuda.synchronize()
