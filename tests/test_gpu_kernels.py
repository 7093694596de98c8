"""GPU parity of every single-kernel entry point of the C ABI against the fp64
oracle, element by element, on seeded inputs spanning several tiles and ragged
tails.  Metric: max|x - ref| / max|ref| per tensor.  Tolerances: fp32 path 1e-4
(2e-5 for pure elementwise ops); bf16 path 2e-2."""
import math

import numpy as np
import pytest
import torch

from oracle import model as om
from paper_2202_01306_amd import synth
from tests.helpers import max_rel_err

pytestmark = pytest.mark.gpu

B = None


@pytest.fixture(scope="module", autouse=True)
def _binding():
    global B
    from paper_2202_01306_amd import binding
    B = binding
    yield
    torch.cuda.synchronize()


PRECS = [("fp32", 0, torch.float32, 1e-4), ("bf16", 1, torch.bfloat16, 2e-2)]


def rnd(rng, shape, prec, scale=1.0):
    """Random fp32 values, rounded to bf16 first in bf16 mode so both sides start equal."""
    a = (rng.standard_normal(shape) * scale).astype(np.float32)
    return synth.round_bf16(a) if prec == "bf16" else a


def dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype)


def host(t):
    torch.cuda.synchronize()
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
@pytest.mark.parametrize("T,d", [(5, 128), (130, 1024), (67, 1600), (33, 4096), (1037, 1600), (70, 2056), (9, 8192)])
def test_layernorm_fwd_bwd(prec, pc, dt, tol, T, d):
    say(f"layernorm {prec} T={T} d={d}")
    rng = np.random.default_rng(T * 1000 + d)
    # the residual stream (x, res, dx) is fp32 in every precision; dy, gamma, beta and y have the element type
    x = (rng.standard_normal((T, d)) * 2.0 + 0.5).astype(np.float32)
    g, bt = rnd(rng, (d,), prec) + 1, rnd(rng, (d,), prec, 0.1)
    g = synth.round_bf16(g) if prec == "bf16" else g
    dy, res = rnd(rng, (T, d), prec), rng.standard_normal((T, d)).astype(np.float32)
    xd, gd, bd = dev(x, torch.float32), dev(g, dt), dev(bt, dt)
    y = torch.empty(T, d, device="cuda", dtype=dt)
    mean = torch.empty(T, device="cuda")
    rstd = torch.empty(T, device="cuda")
    B.hmy_k_layernorm_fwd(pc, xd, gd, bd, y, mean, rstd, T, d, synth.LN_EPS)
    yr, (xhat, rs) = om.layernorm_fwd(x.astype(np.float64), g.astype(np.float64), bt.astype(np.float64), synth.LN_EPS)
    assert max_rel_err(host(y), yr) < (tol if prec == "bf16" else 2e-5)
    assert max_rel_err(host(mean), x.astype(np.float64).mean(axis=1)) < 1e-5
    assert max_rel_err(host(rstd), rs[:, 0]) < 1e-5
    # backward, accumulating onto non-zero dgamma / dbeta, residual added, in place over res
    dg0, db0 = rng.standard_normal(d).astype(np.float32), rng.standard_normal(d).astype(np.float32)
    dgd, dbd = dev(dg0, torch.float32), dev(db0, torch.float32)
    resd = dev(res, torch.float32)
    low = torch.zeros(T, d, device="cuda", dtype=dt)
    B.hmy_k_layernorm_bwd(pc, dev(dy, dt), xd, mean, rstd, gd, resd, resd, dgd, dbd, T, d, dx_e=low)
    dxr, dgr, dbr = om.layernorm_bwd(dy.astype(np.float64), (xhat, rs), g.astype(np.float64))
    assert max_rel_err(host(resd), dxr + res) < (tol if prec == "bf16" else 2e-5)
    assert torch.equal(low, resd.to(dt))        # the element-typed copy is the rounding of what was stored
    assert max_rel_err(host(dgd) - dg0, dgr) < (tol if prec == "bf16" else 2e-5)
    assert max_rel_err(host(dbd) - db0, dbr) < (tol if prec == "bf16" else 2e-5)
    # without residual
    dxd = torch.empty_like(xd)
    B.hmy_k_layernorm_bwd(pc, dev(dy, dt), xd, mean, rstd, gd, None, dxd, dgd, dbd, T, d)
    assert max_rel_err(host(dxd), dxr) < tol
    # with a workspace: partial sums per workgroup, added up by a second kernel
    dgd2, dbd2 = dev(dg0, torch.float32), dev(db0, torch.float32)
    ws = torch.full((256 * 2 * d,), float("nan"), device="cuda")
    B.hmy_k_layernorm_bwd(pc, dev(dy, dt), xd, mean, rstd, gd, None, dxd, dgd2, dbd2, T, d, workspace=ws)
    assert max_rel_err(host(dxd), dxr) < tol
    assert max_rel_err(host(dgd2) - dg0, dgr) < (tol if prec == "bf16" else 2e-5)
    assert max_rel_err(host(dbd2) - db0, dbr) < (tol if prec == "bf16" else 2e-5)
    # the column sums of the residual gradient taken along (a bias gradient), in place over res, with and
    # without the workspace; everything else as before
    for ws in (None, torch.full((256 * 3 * d,), float("nan"), device="cuda")):
        dgd3, dbd3 = dev(dg0, torch.float32), dev(db0, torch.float32)
        s0 = rng.standard_normal(d).astype(np.float32)
        sd, resd = dev(s0, torch.float32), dev(res, torch.float32)
        B.hmy_k_layernorm_bwd(pc, dev(dy, dt), xd, mean, rstd, gd, resd, resd, dgd3, dbd3, T, d, workspace=ws, dres_sum=sd)
        assert max_rel_err(host(sd) - s0, res.astype(np.float64).sum(axis=0)) < 1e-5
        assert max_rel_err(host(resd), dxr + res) < (tol if prec == "bf16" else 2e-5)
        assert max_rel_err(host(dgd3) - dg0, dgr) < (tol if prec == "bf16" else 2e-5)
        assert max_rel_err(host(dbd3) - db0, dbr) < (tol if prec == "bf16" else 2e-5)
    with pytest.raises(B.HmyError):      # sums of a residual that is not there
        B.hmy_k_layernorm_bwd(pc, dev(dy, dt), xd, mean, rstd, gd, None, dxd, dgd, dbd, T, d, dres_sum=dgd2)


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
def test_gelu_fwd_bwd(prec, pc, dt, tol):
    say(f"gelu {prec}")
    rng = np.random.default_rng(1)
    n = 8 * 12345
    u, dg = rnd(rng, (n,), prec, 2.5), rnd(rng, (n,), prec)
    ud = dev(u, dt)
    g = torch.empty_like(ud)
    B.hmy_k_gelu_fwd(pc, ud, g, n)
    assert max_rel_err(host(g), om.gelu_fwd(u.astype(np.float64))) < (tol if prec == "bf16" else 2e-6)
    dgd = dev(dg, dt)
    B.hmy_k_gelu_bwd(pc, dgd, ud, dgd, n)     # in place
    assert max_rel_err(host(dgd), om.gelu_bwd(dg.astype(np.float64), u.astype(np.float64))) < (tol if prec == "bf16" else 2e-6)


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
@pytest.mark.parametrize("T,N", [(3, 8), (257, 3072), (1000, 136), (4096, 4096)])
def test_gelu_bwd_with_column_sums(prec, pc, dt, tol, T, N):
    say(f"gelu backward + column sums {prec} {T}x{N}")
    rng = np.random.default_rng(T * 3 + N)
    u, dg = rnd(rng, (T, N), prec, 2.5), rnd(rng, (T, N), prec)
    db0 = rng.standard_normal(N).astype(np.float32)
    ud, dgd, dbd = dev(u, dt), dev(dg, dt), dev(db0, torch.float32)
    B.hmy_k_gelu_bwd_colsum(pc, dgd, ud, dgd, dbd, T, N)     # in place, as the engine runs it
    ref = om.gelu_bwd(dg.astype(np.float64), u.astype(np.float64))
    assert max_rel_err(host(dgd), ref) < (tol if prec == "bf16" else 2e-6)
    # the sums are those of the stored values, exactly what a separate pass over du would have added
    assert max_rel_err(host(dbd) - db0, host(dgd).astype(np.float64).sum(axis=0)) < 1e-5
    same = dev(dg, dt)
    B.hmy_k_gelu_bwd(pc, same, ud, same, T * N)
    assert torch.equal(same, dgd)


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
@pytest.mark.parametrize("T,N", [(3, 8), (257, 3072), (1000, 136)])
def test_colsum_accumulates(prec, pc, dt, tol, T, N):
    say(f"colsum {prec} {T}x{N}")
    rng = np.random.default_rng(T + N)
    a = rnd(rng, (T, N), prec)
    out0 = rng.standard_normal(N).astype(np.float32)
    out = dev(out0, torch.float32)
    B.hmy_k_colsum(pc, dev(a, dt), out, T, N)
    assert max_rel_err(host(out) - out0, a.astype(np.float64).sum(axis=0)) < 1e-5


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
def test_embedding_fwd_bwd_with_repeated_ids(prec, pc, dt, tol):
    say(f"embed {prec}")
    rng = np.random.default_rng(2)
    b, s, d, V = 3, 40, 64, 50
    T = b * s
    ids = rng.integers(0, V, size=(b, s), dtype=np.int32)       # 120 draws from 50 ids: many repeats
    wte, wpe = rnd(rng, (V, d), prec), rnd(rng, (s, d), prec)
    x = torch.empty(T, d, device="cuda", dtype=torch.float32)     # the residual stream starts here: fp32
    idd = torch.from_numpy(ids.reshape(-1)).cuda()
    B.hmy_k_embed_fwd(pc, idd, dev(wte, dt), dev(wpe, dt), x, T, d, s, V)
    params = {"wte": wte.astype(np.float64), "wpe": wpe.astype(np.float64)}
    spec = om.Spec(1, d, 1, 8, s, V)
    xr, cache = om.embed_fwd(ids, params, spec)
    assert max_rel_err(host(x), xr) < 1e-6         # a sum of two exactly representable values
    dx = rng.standard_normal((T, d)).astype(np.float32)
    dwte = torch.zeros(V, d, device="cuda")
    dwpe = torch.zeros(s, d, device="cuda")
    B.hmy_k_embed_bwd(pc, idd, dev(dx, torch.float32), dwte, dwpe, T, d, s, V)
    _, g = om.embed_bwd(dx.astype(np.float64), cache, params, spec)
    assert max_rel_err(host(dwte), g["wte"]) < 1e-5
    assert max_rel_err(host(dwpe), g["wpe"]) < 1e-5


# runs of one id: none, exactly as many as one wave sums, one more, all tokens alike; then more tokens than the search
# through the ids is used for (32 per column); few tokens of wide rows, on both sides of that line
@pytest.mark.parametrize("counts,d", [([60, 3], 1024), ([60, 3], 1032), ([250, 5], 1032), ([250, 6], 1032), ([1], 8), ([16, 1, 3], 264), ([17, 16], 64), ([33, 1] * 3, 1024), ([700], 128), ([130, 125, 2], 8)])
def test_embedding_bwd_runs(counts, d):
    say(f"embed runs {counts} d={d}")
    rng = np.random.default_rng(sum(counts) + d)
    ids = rng.permutation(np.repeat(np.arange(len(counts)) * 3, counts)).astype(np.int32)
    T, V = len(ids), 3 * len(counts)
    dx = rng.standard_normal((T, d)).astype(np.float32)
    w0 = rng.standard_normal((V, d)).astype(np.float32)
    dwte, dwpe = dev(w0, torch.float32), torch.zeros(T, d, device="cuda")
    B.hmy_k_embed_bwd(PRECS[1][1], torch.from_numpy(ids).cuda(), dev(dx, torch.float32), dwte, dwpe, T, d, T, V)
    ref = w0.astype(np.float64)
    np.add.at(ref, ids, dx.astype(np.float64))
    assert max_rel_err(host(dwte), ref) < 1e-5      # up to 700 terms in fp32
    assert max_rel_err(host(dwpe), dx) == 0


def _gemm_case(prec, pc, dt, tol, M, N, K, ta, tb, c_fp32, accumulate, bias, res, gelu, use_mfma, pad=0, res_fp32=0,
               row_pad=0, ldc=None, tiles=None):
    rng = np.random.default_rng(M * 7 + N * 3 + K + ta * 2 + tb)
    lda = M + row_pad if ta else K + pad        # pad: rows whose contiguous axis is K; row_pad: A stored [K, M]
    ldb = N if tb else K + pad
    A = rnd(rng, (K, lda) if ta else (M, lda), prec)
    Bm = rnd(rng, (K, ldb) if tb else (N, ldb), prec)
    A64 = (A[:, :M].T if ta else A[:, :K]).astype(np.float64)         # [M,K]
    B64 = (Bm[:, :N] if tb else Bm[:, :K].T).astype(np.float64)       # [K,N]
    ref = A64 @ B64
    biasv = rnd(rng, (N,), prec) if bias else None
    resv = (rng.standard_normal((M, N)).astype(np.float32) if res_fp32 else rnd(rng, (M, N), prec)) if res else None
    if bias:
        ref = ref + biasv
    if res:
        ref = ref + resv
    ldc = ldc or N + (8 if pad else 0)
    cdt = torch.float32 if c_fp32 else dt
    c0 = rng.standard_normal((M, ldc)).astype(np.float32)
    Cd = dev(c0, cdt)
    if accumulate:
        ref = ref + host(Cd)[:, :N]
    gout = torch.zeros(M, ldc, device="cuda", dtype=dt) if gelu else None
    if gelu == "in place":
        gout = Cd                       # only gelu(C) is wanted: it replaces C
    B.hmy_set_kernel_path(use_mfma)
    try:
        B.hmy_k_gemm(pc, M, N, K, dev(A, dt), lda, dev(Bm, dt), ldb, Cd, ldc, ta=ta, tb=tb, c_fp32=c_fp32,
                     accumulate=accumulate, bias=dev(biasv, dt) if bias else None,
                     res=dev(resv, torch.float32 if res_fp32 else dt) if res else None, ldr=N, gelu_out=gout,
                     res_fp32=res_fp32, tiles=tiles)
        got = host(Cd)
    finally:
        B.hmy_set_kernel_path(True)
    scale = math.sqrt(K)   # entries are sums of K unit-variance products
    if gelu == "in place":
        gref = om.gelu_fwd(synth.round_bf16(ref.astype(np.float32)).astype(np.float64) if prec == "bf16" else ref)
        # where the rounding of C falls on the other side the activation moves by one bf16 step of C
        assert np.abs(got[:, :N] - gref).max() / max(np.abs(gref).max(), scale) < tol, "gelu in place"
        return
    assert np.abs(got[:, :N] - ref).max() / max(np.abs(ref).max(), scale) < tol, "C"
    if ldc > N:   # columns beyond N are never written
        assert np.array_equal(got[:, N:], host(dev(c0, cdt))[:, N:])
    if gelu:
        gref = om.gelu_fwd(got[:, :N])          # gelu of the stored (rounded) C
        assert max_rel_err(host(gout)[:, :N], gref) < tol


GEMM_SHAPES = [(200, 136, 72), (128, 128, 32), (130, 257, 1001), (136, 264, 1001), (1, 8, 8), (384, 128, 512)]


@pytest.mark.parametrize("use_mfma", [True, False])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_bf16_all_layouts(use_mfma, ta, tb, M, N, K):
    say(f"gemm bf16 mfma={use_mfma} ta={ta} tb={tb} {M}x{N}x{K}")
    pad = 7 if K == 1001 else 0     # makes every leading dimension a multiple of 8
    ragged_rows = (ta and M % 8) or (tb and N % 8)     # an operand stored [K, rows] whose rows are not 16-byte multiples
    if ragged_rows and use_mfma:
        # the matrix-core kernels cannot take it, and the library says so instead of quietly running the plain kernel
        with pytest.raises(B.HmyError) as e:
            _gemm_case("bf16", 1, torch.bfloat16, 2e-2, M, N, K, ta, tb, 0, 0, False, False, False, use_mfma, pad)
        assert e.value.code == B.HMY_E_INVALID and "16-byte aligned" in str(e.value)
        return
    _gemm_case("bf16", 1, torch.bfloat16, 2e-2, M, N, K, ta, tb, 0, 0, False, False, False, use_mfma, pad)


@pytest.mark.parametrize("use_mfma", [True, False])
def test_gemm_bf16_epilogues(use_mfma):
    say(f"gemm bf16 epilogues mfma={use_mfma}")
    args = ("bf16", 1, torch.bfloat16, 2e-2)
    _gemm_case(*args, 200, 136, 72, 0, 0, 0, 0, True, False, False, use_mfma)       # bias
    _gemm_case(*args, 200, 136, 72, 0, 0, 0, 0, True, True, False, use_mfma)        # bias + residual
    _gemm_case(*args, 200, 136, 72, 0, 0, 1, 0, True, True, False, use_mfma, res_fp32=1)    # ... on the fp32 residual stream
    _gemm_case(*args, 384, 256, 128, 0, 0, 1, 0, True, True, False, use_mfma, res_fp32=1)   # ... whole tiles (16-byte accesses)
    _gemm_case(*args, 256, 128, 1024, 0, 0, 1, 0, True, True, False, use_mfma, res_fp32=1)  # ... one tile per workgroup, K tile 64
    _gemm_case(*args, 200, 136, 72, 0, 0, 0, 0, True, False, True, use_mfma)        # bias + gelu output
    _gemm_case(*args, 200, 136, 72, 0, 0, 0, 0, True, False, "in place", use_mfma)  # bias + gelu, the only output
    _gemm_case(*args, 384, 256, 128, 0, 0, 0, 0, True, False, "in place", use_mfma) # ... on whole tiles (16-byte stores)
    _gemm_case(*args, 200, 136, 72, 0, 0, 1, 0, False, False, False, use_mfma)      # fp32 C (logits)
    _gemm_case(*args, 136, 72, 200, 1, 1, 1, 1, False, False, False, use_mfma)      # wgrad: fp32 C +=
    _gemm_case(*args, 100, 1001, 64, 0, 0, 1, 0, False, False, False, use_mfma, 8)  # ragged N, padded ldc and lda
    _gemm_case(*args, 1000, 64, 96, 1, 1, 1, 1, False, False, False, use_mfma)      # ragged M (vocab-like), K=96


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("K", [96, 320])
def test_gemm_bf16_large_outputs_all_layouts(ta, tb, K):
    """256x256 tiles, one workgroup per compute unit or nearly, with a ragged last tile row and column; K of fewer and of
    more tiles than the ring has stages."""
    say(f"gemm bf16 large ta={ta} tb={tb} K={K}")
    _gemm_case("bf16", 1, torch.bfloat16, 2e-2, 3600, 3336, K, ta, tb, 0, 0, False, False, False, True, tiles=(256, 256))


def test_gemm_bf16_large_outputs_epilogues():
    args, big = ("bf16", 1, torch.bfloat16, 2e-2), dict(tiles=(256, 256))
    say("gemm bf16 large: bias + gelu")
    _gemm_case(*args, 4096, 3072, 64, 0, 0, 0, 0, True, False, True, True, **big)
    say("gemm bf16 large: bias + gelu in place")
    _gemm_case(*args, 4096, 3072, 64, 0, 0, 0, 0, True, False, "in place", True, **big)
    say("gemm bf16 large: bias + fp32 residual stream")
    _gemm_case(*args, 4096, 3072, 160, 0, 0, 1, 0, True, True, False, True, res_fp32=1, **big)
    say("gemm bf16 large: bias + bf16 residual")
    _gemm_case(*args, 4096, 3072, 64, 0, 0, 0, 0, True, True, False, True, **big)
    say("gemm bf16 large: fp32 C +=")
    _gemm_case(*args, 3072, 4096, 128, 1, 1, 1, 1, False, False, False, True, **big)
    _gemm_case(*args, 50257, 1024, 96, 1, 1, 1, 1, False, False, False, True, row_pad=47, **big)   # vocabulary rows, ragged
    say("gemm bf16: fp32 C +=, contraction split over workgroups (128x128 tiles)")
    _gemm_case(*args, 1024, 1024, 4096, 1, 1, 1, 1, False, False, False, True)
    _gemm_case(*args, 1536, 1024, 2048 + 32, 0, 1, 1, 1, False, False, False, True)    # the last split has two K tiles
    say("gemm bf16 large: fp32 logits, ragged vocabulary, padded leading dimensions")
    _gemm_case(*args, 512, 50257, 64, 0, 0, 1, 0, False, False, False, True, 8, **big)


@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 1)])
@pytest.mark.parametrize("K", [257, 289, 300, 319])
def test_gemm_bf16_sums_with_a_ragged_contraction(ta, tb, K):
    """More outputs than any product takes on 64x64 tiles: the multiple of 32 on larger tiles, the 1, 12 or 31 steps behind it on
    those."""
    say(f"gemm bf16 sums ta={ta} tb={tb} K={K}")
    _gemm_case("bf16", 1, torch.bfloat16, 2e-2, 3080, 3336, K, ta, tb, 1, 1, False, False, False, True, -K % 8)


def test_gemm_bf16_tiles_that_stick_out_of_c():
    """Outputs whose width is no multiple of the block tile, with 16-byte aligned rows: whole groups of 8 columns of an
    edge tile leave through the vector path, a ragged last group element by element; nothing beyond N is written."""
    args = ("bf16", 1, torch.bfloat16, 2e-2)
    say("gemm bf16 edge tiles: fp32 C, ragged width, aligned rows")
    _gemm_case(*args, 200, 333, 128, 0, 0, 1, 0, False, False, False, True, ldc=336)
    _gemm_case(*args, 200, 333, 128, 0, 0, 1, 1, False, False, False, True, ldc=336)      # +=
    say("gemm bf16 edge tiles: bf16 C, bias + gelu, ragged width")
    _gemm_case(*args, 200, 333, 128, 0, 0, 0, 0, True, False, True, True, ldc=336)
    say("gemm bf16 edge tiles: 1600 wide, bias + fp32 residual stream")
    _gemm_case(*args, 2048, 1600, 64, 0, 0, 1, 0, True, True, False, True, res_fp32=1)
    _gemm_case(*args, 1600, 1608, 256, 1, 1, 1, 1, False, False, False, True)            # weight gradient, ragged rows too
    say("gemm bf16 edge tiles, 256x256: fp32 C with a ragged width; bf16 C with bias + gelu")
    big = dict(tiles=(256, 256))
    _gemm_case(*args, 4096, 2999, 64, 0, 0, 1, 0, False, False, False, True, ldc=3008, **big)
    _gemm_case(*args, 4000, 3000, 96, 0, 0, 0, 0, True, False, True, True, **big)
    _gemm_case(*args, 4000, 3000, 64, 0, 1, 0, 0, True, True, False, True, **big)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
def test_gemm_bf16_256x128_tiles(ta, tb):
    """One round of them, with edge tiles that stick out of C in both directions, three rounds; every output stage.  Bounds as
    for the other tiles, of which these have the order of sums."""
    args, wide = ("bf16", 1, torch.bfloat16, 2e-2), dict(tiles=(256, 128))
    for M, N, K in ((2040, 2296, 1024), (2104, 3840, 1088)):
        say(f"gemm bf16 256x128 ta={ta} tb={tb} {M}x{N}x{K}")
        _gemm_case(*args, M, N, K, ta, tb, 0, 0, True, True, False, True, **wide)
        _gemm_case(*args, M, N, K, ta, tb, 0, 0, True, False, True, True, **wide)
        _gemm_case(*args, M, N, K, ta, tb, 1, 0, True, True, False, True, res_fp32=1, **wide)
    _gemm_case(*args, 2040, 2296, 512, ta, tb, 1, 1, False, False, False, True, **wide)      # sums into C: few tiles, and many
    _gemm_case(*args, 2048, 4096, 2048, ta, tb, 1, 1, False, False, False, True, **wide)
    # rows of C that allow no 16-byte access
    N = 2296 if tb else 2300
    _gemm_case(*args, 2048, N, 1024, ta, tb, 1, 0, False, False, False, True, ldc=N + 2, **wide)
    _gemm_case(*args, 2048, 8968, 2048, ta, tb, 0, 0, True, False, False, True, **wide)      # three rounds


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(1992, 1000, 18432), (1992, 1000, 18560), (264, 3200, 23104)])
def test_gemm_bf16_256x128_tiles_split(ta, tb, M, N, K):
    """Sums so long that they are split over 256x128 tiles: parts of equal length, and a shorter last one; edge tiles in both
    directions."""
    say(f"gemm bf16 256x128 split ta={ta} tb={tb} {M}x{N}x{K}")
    rows, cols, parts, tail = B.hmy_gemm_tiles(1, M, N, K, ta=ta, tb=tb, c_fp32=1, accumulate=1)
    assert (rows, cols, tail) == (256, 128, 0) and parts > 1
    _gemm_case("bf16", 1, torch.bfloat16, 2e-2, M, N, K, ta, tb, 1, 1, False, False, False, True)


@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb,N", [(1, 1), (1, 64), (1, 96), (1, 120), (1, 128), (0, 1), (0, 2), (0, 72)])
def test_gemm_bf16_long_sums_of_narrow_outputs(ta, tb, N):
    """The same split where the second operand is narrow (rows of 16 to 256 bytes if it is stored contraction-major, a single row
    if not), against 64 bits: a row of the contraction that is not read moves an element by about one standard deviation of a
    product.  Bound: one 16-deep multiply after the other adds to a sum of at most 6 sqrt(K) in 32 bits, K/16 of them."""
    say(f"gemm bf16 256x128 split, narrow: ta={ta} tb={tb} N={N}")
    M, K, ld = 8192, 36864, (N + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(N + ta)
    A = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g).bfloat16()
    Bm = torch.randn((K, ld) if tb else (N, K), device="cuda", generator=g).bfloat16()
    C = torch.randn(M, N, device="cuda", generator=g)
    ref = C.double() + (A.t() if ta else A).double() @ (Bm[:, :N] if tb else Bm.t()).double()
    B.hmy_k_gemm(1, M, N, K, A, M if ta else K, Bm, ld if tb else K, C, N, ta=ta, tb=tb, c_fp32=1, accumulate=1)
    assert float((C.double() - ref).abs().max()) < 6 * math.sqrt(K) * (K / 16) * 2.0 ** -24


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (1, 8, 7), (72, 136, 63), (65, 57, 65), (200, 264, 250), (480, 256, 321),
                                   (128, 128, 1100), (1288, 1928, 96), (768, 776, 2047), (768, 776, 2048), (768, 776, 2049),
                                   (2048, 1024, 2080),
                                   (200, 264, 576), (200, 264, 640), (200, 264, 960), (200, 264, 1000), (768, 776, 1728),
                                   (768, 776, 1792), (65, 57, 128), (72, 72, 192), (768, 776, 4096), (264, 200, 4224),
                                   (65, 57, 256),
                                   (72, 72, 320), (200, 264, 4672), (1000, 1200, 320), (1000, 1200, 384), (1000, 1200, 512),
                                   (768, 768, 4608), (1280, 1024, 2304)])
def test_gemm_bf16_small_tiles(ta, tb, M, N, K):
    """64x64 tiles: one tile, its edges, contractions shorter and longer than the ring of four K tiles, whole (an odd and
    an even number of K tiles), cut at a multiple of 8 and inside a group of 8, split (4672: the last part is one K tile); the
    smallest output that is left to 128x128 tiles, and both sides of the length of contraction that is and of those from which
    a kernel without branches takes multiples of 64.  What lies behind K in memory must not matter."""
    say(f"gemm bf16 {M}x{N}x{K} ta={ta} tb={tb}")
    if (ta and M % 8) or (tb and N % 8):
        M, N = (M + 7) // 8 * 8, (N + 7) // 8 * 8
    args = ("bf16", 1, torch.bfloat16, 2e-2)
    pad = -K % 8
    _gemm_case(*args, M, N, K, ta, tb, 0, 0, True, True, False, True, pad)
    _gemm_case(*args, M, N, K, ta, tb, 0, 0, True, False, True, True, pad)
    _gemm_case(*args, M, N, K, ta, tb, 1, 1, False, False, False, True, pad)
    _gemm_case(*args, M, N, K, ta, tb, 1, 0, True, True, False, True, pad, res_fp32=1)
    if pad and not ta and not tb:
        g = torch.Generator(device="cuda").manual_seed(K)
        a, b = (torch.randn(r, K + pad, device="cuda", generator=g).bfloat16() for r in (M, N))
        c = [torch.zeros(M, N, device="cuda") for _ in range(2)]
        B.hmy_k_gemm(1, M, N, K, a, K + pad, b, K + pad, c[0], N, c_fp32=1)
        a[:, K:], b[:, K:] = float("nan"), float("inf")
        B.hmy_k_gemm(1, M, N, K, a, K + pad, b, K + pad, c[1], N, c_fp32=1)
        assert torch.equal(c[0], c[1])


@pytest.mark.parametrize("M,N,K", [(64, 64, 257), (264, 200, 300), (768, 3072, 600), (1000, 1208, 481), (72, 136, 999),
                                   (1024, 1024, 2047), (1160, 1024, 2080), (2048, 2048, 1801), (4352, 1024, 2381),
                                   (4352, 1024, 2393)])
def test_gemm_bf16_weight_gradients_of_any_length(M, N, K):
    """Contractions that are no multiple of 64 on 64x64 tiles: the rows behind K, which lie in memory and are undefined numbers
    here, count as zeros; one part, several, more than 512 tiles, and either side of where more than 1024 of them give way to
    tiles of 256 rows and a tail."""
    say(f"gemm bf16 weight gradient {M}x{N}x{K}")
    g = torch.Generator(device="cuda").manual_seed(K)
    a, b = (torch.full((K + 192, n), float("nan"), device="cuda").bfloat16() for n in (M, N))
    a[:K], b[:K] = (torch.randn(K, n, device="cuda", generator=g) for n in (M, N))
    c = torch.randn(M, N, device="cuda", generator=g)
    ref = c.double() + a[:K].double().t() @ b[:K].double()
    B.hmy_k_gemm(1, M, N, K, a, M, b, N, c, N, ta=1, tb=1, c_fp32=1, accumulate=1)
    assert float((c.double() - ref).abs().max()) < 6 * math.sqrt(K) * (K / 16 + 2) * 2.0 ** -24


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("K", [32, 288, 512, 1024])
def test_gemm_bf16_small_tiles_sum_like_the_larger_ones(ta, tb, K):
    """The first 256 rows of a product that takes 128x128 tiles, and of one that takes 256x256 tiles, against the same rows as
    a product of their own (64x64 tiles): equal bits where no contraction is split and it is a multiple of 32."""
    say(f"gemm bf16 small against large tiles, K={K} ta={ta} tb={tb}")
    g = torch.Generator(device="cuda").manual_seed(K)
    for N in (1024, 2048):
        M = 8192
        a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g).bfloat16()
        b = torch.randn((K, N) if tb else (N, K), device="cuda", generator=g).bfloat16()
        bias = torch.randn(N, device="cuda", generator=g).bfloat16()
        for kw in (dict(c_fp32=1, accumulate=1), dict(c_fp32=1), dict(bias=bias)):
            # sums take small tiles in a weight gradient's layout alone, and are split from sixteen K tiles on
            if kw.get("accumulate") and not (ta and tb and K <= 512):
                continue
            got = []
            for rows in (M, 256):
                c = torch.ones(rows, N, device="cuda", dtype=torch.float32 if "c_fp32" in kw else torch.bfloat16)
                B.hmy_k_gemm(1, rows, N, K, a, a.shape[1], b, b.shape[1], c, N, ta=ta, tb=tb, **kw)
                got.append(c[:256])
            assert torch.equal(got[0], got[1]), (N, sorted(kw))


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(400, 8248, 480), (400, 8248, 512), (3256, 2528, 736), (1080, 7208, 480), (3664, 3360, 736),
                                   (1352, 8144, 480), (1352, 8144, 1024), (1352, 8144, 32), (1352, 8144, 64), (1352, 8144, 96)])
def test_gemm_bf16_large_products_a_few_rows_at_a_time(ta, tb, M, N, K):
    """Large products on the tiles that the rule picks for them and their output stage: edge tiles in both directions,
    contractions that end in half a K tile, of one and of two K tiles.  The rows a few at a time go to 64x64 tiles, which sum in
    the same order: equal bits."""
    say(f"gemm bf16 256 rows ta={ta} tb={tb} {M}x{N}x{K}")
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g).bfloat16()
    b = torch.randn((K, N) if tb else (N, K), device="cuda", generator=g).bfloat16()
    bias, low = torch.randn(N, device="cuda", generator=g).bfloat16(), torch.randn(M, N, device="cuda", generator=g)
    tiles_n = (N + 63) // 64
    rows = 64 * ((129 + tiles_n - 1) // tiles_n)       # more than 128 tiles: no sum is split
    for kind in ("res", "gelu", "stream", "sum"):
        if kind == "sum" and not (ta and tb):
            continue
        c32 = kind in ("stream", "sum")
        c = low.clone() if c32 else torch.zeros(M, N, device="cuda", dtype=torch.bfloat16)
        act, res = torch.zeros_like(c), low if c32 else low.bfloat16()
        want, want_act = c.clone(), act.clone()

        def product(r0, n, c, act):
            kw = dict(c_fp32=1, accumulate=1) if kind == "sum" else dict(bias=bias)
            if kind in ("res", "stream"):
                kw.update(c_fp32=int(c32), res=res[r0:], ldr=N, res_fp32=int(c32))
            if kind == "gelu":
                kw.update(gelu_out=act[r0:])
            B.hmy_k_gemm(1, n, N, K, a[:, r0:] if ta else a[r0:], a.shape[1], b, b.shape[1], c[r0:], N, ta=ta, tb=tb, **kw)

        product(0, M, c, act)
        for r0 in range(0, M, rows):
            product(r0, min(rows, M - r0), want, want_act)
        assert torch.equal(c, want) and torch.equal(act, want_act), kind
        if kind == "stream":
            ref = (a.t() if ta else a).double() @ (b if tb else b.t()).double() + bias.double() + low.double()
            assert float((c.double() - ref).abs().max()) < 6 * math.sqrt(K) * (K / 32 + 2) * 2.0 ** -24


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("cols", [128, 160, 192, 224, 256])
@pytest.mark.parametrize("aligned", [True, False])
def test_gemm_bf16_tiles_of_every_width(aligned, cols, ta, tb):
    """Tiles of 256 rows and every width, with every output stage: edge tiles in both directions, contractions of one K tile, of
    half a one, of one and a half, and longer ones that end in half a one.  Rows of C, of the residual and of the activation that
    allow 16-byte accesses, and ones that allow none and end inside a group of 8 columns.  64x64 tiles sum in the same order and
    have the same output stages: equal bits, and nothing beyond the last column changes."""
    M, N = 520, 2 * cols + (72 if aligned else 75)
    ld, up8 = N + (8 if aligned else 2), (N + 7) // 8 * 8
    for K in (32, 64, 96, 480, 736):
        say(f"gemm bf16 256x{cols} ta={ta} tb={tb} {M}x{N}x{K} ld={ld}")
        g = torch.Generator(device="cuda").manual_seed(N + K)
        a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g).bfloat16()
        b = torch.randn((K, up8) if tb else (N, K), device="cuda", generator=g).bfloat16()
        bias, low = torch.randn(up8, device="cuda", generator=g).bfloat16(), torch.randn(M, ld, device="cuda", generator=g)
        for kind in ("bias", "res", "gelu", "gelu alone", "fp32", "stream", "sum", "sum, bias and stream"):
            c32 = kind in ("fp32", "stream") or "sum" in kind
            kw = dict(c_fp32=int(c32), accumulate=int("sum" in kind))
            if kind not in ("fp32", "sum"):
                kw["bias"] = bias
            if kind == "res" or "stream" in kind:
                kw.update(res=low if c32 else low.bfloat16(), ldr=ld, res_fp32=int(c32))
            out = []
            for tiles in ((256, cols), (64, 64)):
                c = low.clone() if c32 else low.bfloat16()
                act = c if kind == "gelu alone" else low.bfloat16() if kind == "gelu" else None
                B.hmy_k_gemm(1, M, N, K, a, a.shape[1], b, b.shape[1], c, ld, ta=ta, tb=tb, gelu_out=act, tiles=tiles, **kw)
                out.append((c, c if act is None else act))
            for x, y in zip(*out):
                assert torch.equal(x, y), (kind, K)
                assert torch.equal(x[:, N:], low.to(x.dtype)[:, N:]), (kind, K)
            if kind == "stream":
                ref = (a.t() if ta else a).double() @ (b[:, :N] if tb else b.t()).double() + bias[:N].double() + low[:, :N].double()
                assert float((out[0][0][:, :N].double() - ref).abs().max()) < 6 * math.sqrt(K) * (K / 32 + 2) * 2.0 ** -24


def us_of(call, reps=20):
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(reps):
        call()
    end.record()
    torch.cuda.synchronize()
    return start.elapsed_time(end) * 1e3 / reps


def assert_takes_at_most(limit, call, reference, what):
    """The shortest of five times of each, in turn, in any of five attempts."""
    ratios = []
    for _ in range(5):
        times = [(us_of(call), us_of(reference)) for _ in range(5)]
        ratios.append(min(t[0] for t in times) / min(t[1] for t in times))
        if ratios[-1] < limit:
            return
    raise AssertionError(f"{what}: {ratios}")


def test_gemm_bf16_edge_tiles_cost_no_more_than_whole_ones():
    """4096x2816 on 192 columns: the last of fifteen columns of tiles has 128 of its columns inside C.  Beside 4096x2880, as many
    tiles and all of them whole, it took 1.23 times as long when groups of columns beyond C went through the element-by-element
    loop, and takes as long without that."""
    say("gemm bf16 edge tiles of 192 columns: time")
    K, calls = 832, []
    for N in (2816, 2880):
        a, b = (torch.randn(n, K, device="cuda").bfloat16() for n in (4096, N))
        c, bias = torch.empty(4096, N, device="cuda", dtype=torch.bfloat16), torch.randn(N, device="cuda").bfloat16()
        calls.append(lambda a=a, b=b, c=c, bias=bias, N=N: B.hmy_k_gemm(1, 4096, N, K, a, K, b, K, c, N, bias=bias, tiles=(256, 192)))

    assert_takes_at_most(1.1, *calls, "edge tiles over whole tiles")


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1)])
def test_gemm_fp32(ta, tb):
    say(f"gemm fp32 ta={ta} tb={tb}")
    args = ("fp32", 0, torch.float32, 1e-5)
    _gemm_case(*args, 130, 72, 100, ta, tb, 0, 0, True, True, False, True)
    _gemm_case(*args, 64, 200, 33, ta, tb, 1, 1, False, False, False, True)
    _gemm_case(*args, 128, 512, 128, ta, tb, 0, 0, True, False, True, True)
    _gemm_case(*args, 128, 512, 128, ta, tb, 0, 0, True, False, "in place", True)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(1, 8, 1), (33, 31, 129), (32, 32, 128), (900, 840, 70), (832, 1024, 32), (4100, 2050, 33),
                                   (4096, 2048, 64), (72, 520, 513), (256, 500, 800), (1500, 520, 130), (1408, 1472, 64),
                                   (2050, 1050, 96), (1000, 1040, 32), (1000, 1040, 36), (1000, 1040, 2052),
                                   (72, 520, 640), (72, 520, 644), (72, 520, 1092), (72, 520, 1540)])
def test_gemm_fp32_every_split(ta, tb, M, N, K):
    """One 32x32 tile and its edges, 64x64 tiles, 128x128 tiles, on four and on eight waves (272 tiles: eight where something is
    added and for long sums; 51 of 32x32: unless that leaves the last K tile nearly empty); ragged and whole in all three
    directions, contractions of one to a few K tiles; leading dimensions that allow 16-byte accesses and ones that do not.  Bound:
    sums of K rounded fp32 products."""
    say(f"gemm fp32 {M}x{N}x{K} ta={ta} tb={tb}")
    args = ("fp32", 0, torch.float32, 1e-5)
    _gemm_case(*args, M, N, K, ta, tb, 0, 0, True, True, False, True, pad=3)
    _gemm_case(*args, M, N, K, ta, tb, 1, 1, False, False, False, True)
    _gemm_case(*args, M, N, K, ta, tb, 1, 1, False, False, False, True, pad=-K % 4, row_pad=-M % 4)
    _gemm_case(*args, M, N, K, ta, tb, 0, 0, True, False, False, True, pad=-K % 4, row_pad=-M % 4)


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("b,s,H,dh", [(32, 130, 8, 32), (32, 129, 8, 64), (32, 140, 8, 128), (1, 2, 1, 64), (1, 33, 2, 128)])
def test_attention_fp32_one_and_several_waves(causal, b, s, H, dh):
    """Four waves per workgroup (512 workgroups), with a ragged last tile, and the shortest sequences."""
    say(f"attention fp32 causal={causal} b={b} s={s} H={H} dh={dh}")
    _attention_case("fp32", 0, torch.float32, 1e-5, causal, b, s, H, dh)


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("b,s,H,dh", [(1, 32, 3, 64), (3, 33, 2, 32), (2, 64, 2, 128), (2, 65, 3, 64), (1, 97, 2, 128),
                                      (4, 65, 24, 32),
                                      (2, 140, 40, 64), (2, 130, 40, 128), (6, 66, 60, 32)])
def test_attention_fp32_tiles_split_over_waves(causal, b, s, H, dh):
    """One, two and four waves per 32 rows: a single tile, waves without one, a ragged last tile, and launches on either side of
    the numbers of rows from which fewer waves share them (288, 400 and 1080 groups)."""
    say(f"attention fp32 split causal={causal} b={b} s={s} H={H} dh={dh}")
    _attention_case("fp32", 0, torch.float32, 1e-5, causal, b, s, H, dh)


def test_gemm_rejects_bad_arguments():
    a = torch.zeros(64, 64, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(B.HmyError) as e:
        B.hmy_k_gemm(1, 64, 64, 64, a, 32, a, 64, a, 64)       # lda < K
    assert e.value.code == B.HMY_E_INVALID
    with pytest.raises(B.HmyError):
        B.hmy_k_gemm(1, 64, 64, 64, a, 64, a, 64, a, 64, accumulate=1)   # accumulate needs fp32 C
    with pytest.raises(B.HmyError):
        B.hmy_k_gemm(1, 0, 64, 64, a, 64, a, 64, a, 64)


@pytest.mark.parametrize("prec,pc,dt,tol,use_mfma", [p + (True,) for p in PRECS] + [PRECS[1] + (False,)])
@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("b,s,H,dh", [(2, 64, 2, 32), (1, 100, 3, 64), (2, 256, 1, 128), (1, 7, 2, 64),
                                      (1, 333, 2, 64), (2, 130, 2, 32), (1, 161, 1, 128)])
def test_attention_fwd_bwd(prec, pc, dt, tol, use_mfma, causal, b, s, H, dh):
    say(f"attention {prec} mfma={use_mfma} causal={causal} b={b} s={s} H={H} dh={dh}")
    B.hmy_set_kernel_path(use_mfma)
    try:
        _attention_case(prec, pc, dt, tol, causal, b, s, H, dh)
    finally:
        B.hmy_set_kernel_path(True)


def _attention_case(prec, pc, dt, tol, causal, b, s, H, dh):
    rng = np.random.default_rng(s * 10 + dh + causal)
    d = H * dh
    T = b * s
    qkv = rnd(rng, (T, 3 * d), prec, 1.5)
    spec = om.Spec(1, d, H, 8, s, 16, bool(causal))
    oref, cache = om.attention_fwd(qkv.astype(np.float64), spec, b)
    qd = dev(qkv, dt)
    o = torch.empty(T, d, device="cuda", dtype=dt)
    lse = torch.empty(b * H * s, device="cuda")
    B.hmy_k_attn_fwd(pc, qd, o, lse, b, s, H, dh, causal)
    assert max_rel_err(host(o), oref) < tol
    # logsumexp of the scaled, masked scores
    q, k, v, P = cache
    S = (q @ k.transpose(0, 1, 3, 2)) / math.sqrt(dh)
    if causal:
        S = np.where(np.triu(np.ones((s, s), bool), 1), -np.inf, S)
    mx = S.max(-1)
    lref = mx + np.log(np.exp(S - mx[..., None]).sum(-1))
    assert np.abs(host(lse).reshape(b, H, s) - lref).max() < (3e-2 if prec == "bf16" else 1e-4)
    # backward consumes the kernel's own o and lse (as the executor does)
    do = rnd(rng, (T, d), prec)
    dqkv = torch.full((T, 3 * d), float("nan"), device="cuda", dtype=dt)
    delta = torch.empty(b * H * s, device="cuda")
    B.hmy_k_attn_bwd(pc, qd, o, dev(do, dt), lse, delta, dqkv, b, s, H, dh, causal)
    ref = om.attention_bwd(do.astype(np.float64), cache, spec, b)
    got = host(dqkv)
    for name, sl in (("dq", slice(0, d)), ("dk", slice(d, 2 * d)), ("dv", slice(2 * d, 3 * d))):
        assert max_rel_err(got[:, sl], ref[:, sl]) < tol, name
    # once more with the bias gradient of the QKV projection taken along: the column sums of dqkv as stored, added
    # onto what is there; dqkv and delta as before
    db0 = rng.standard_normal(3 * d).astype(np.float32)
    dbd = dev(db0, torch.float32)
    dqkv2 = torch.full((T, 3 * d), float("nan"), device="cuda", dtype=dt)
    delta2 = torch.full((b * H * s,), float("nan"), device="cuda")
    B.hmy_k_attn_bwd(pc, qd, o, dev(do, dt), lse, delta2, dqkv2, b, s, H, dh, causal, dbias=dbd)
    assert torch.equal(dqkv2, dqkv)
    assert max_rel_err(host(delta2), host(delta)) < 1e-5
    assert max_rel_err(host(delta2).reshape(b, H, s), (do.astype(np.float64) * host(o)).reshape(b, s, H, dh).sum(-1).transpose(0, 2, 1)) < 1e-4
    sums = got.astype(np.float64).sum(axis=0)
    assert np.abs(host(dbd) - db0 - sums).max() < 1e-4 * max(np.abs(sums).max(), np.abs(db0).max(), 1.0)


# the eight-wave kernels and the four-wave ones on both sides of their rules: few and many workgroups, long causal rows
@pytest.mark.parametrize("causal,b,s,H,dh", [(1, 1, 1030, 2, 64), (0, 1, 1030, 2, 64), (0, 33, 130, 4, 64), (1, 33, 130, 4, 64),
                                             (0, 17, 130, 8, 128), (1, 17, 130, 8, 128), (1, 1, 2050, 1, 128), (0, 1, 33, 1, 128),
                                             (1, 17, 2050, 1, 128), (1, 3, 64, 2, 64), (0, 3, 65, 2, 64), (0, 2, 111, 2, 128),
                                             (1, 2, 112, 2, 128), (0, 2, 191, 2, 128), (0, 2, 192, 2, 128), (1, 1, 383, 2, 128),
                                             (0, 1, 384, 2, 128), (0, 40, 31, 8, 128)])
def test_attention_eight_and_four_waves(causal, b, s, H, dh):
    prec, pc, dt, tol = PRECS[1]
    say(f"attention split causal={causal} b={b} s={s} H={H} dh={dh}")
    _attention_case(prec, pc, dt, tol, causal, b, s, H, dh)


# head dimension 64: rows of one streamed tile and of two; 256 workgroups and 258; causal, more than 256 of them on either side of
# 1024 rows, and 513 beyond it
@pytest.mark.parametrize("causal,b,s,H,dh", [(0, 2, 64, 3, 64), (0, 2, 65, 3, 64), (0, 8, 130, 16, 64), (0, 43, 130, 3, 64),
                                             (1, 1, 1020, 40, 64), (1, 1, 1030, 40, 64), (1, 1, 1030, 57, 64),
                                             (1, 3, 111, 2, 128), (0, 3, 112, 2, 128), (0, 2, 67, 3, 32)])
def test_attention_backward_either_side_of_eight_waves(causal, b, s, H, dh):
    """dK/dV on four and on eight waves from either side of the lengths and numbers of workgroups that part them, the edges' masks
    in both."""
    say(f"attention backward causal={causal} b={b} s={s} H={H} dh={dh}")
    _attention_case(*PRECS[1], causal, b, s, H, dh)


@pytest.mark.parametrize("causal,b,s", [(0, 32, 128), (1, 8, 1024)])
def test_attention_backward_bias_gradient_at_head_dimension_32_waits_for_no_queue_of_atomics(causal, b, s):
    """1024 workgroups and more that add to the same columns: 1.84 and 1.46 times the backward without the bias gradient with
    eight atomics per column and workgroup, 1.10 and 1.05 with one."""
    say(f"attention backward with the bias gradient, time: causal={causal} b={b} s={s}")
    H, dh, T, d = 32, 32, b * s, 1024
    qkv, do = torch.randn(T, 3 * d, device="cuda").bfloat16(), torch.randn(T, d, device="cuda").bfloat16()
    o, dqkv = torch.empty_like(do), torch.empty_like(qkv)
    lse, delta, db = torch.empty(T * H, device="cuda"), torch.empty(T * H, device="cuda"), torch.zeros(3 * d, device="cuda")
    B.hmy_k_attn_fwd(1, qkv, o, lse, b, s, H, dh, causal)
    with_sums, without = (lambda x=x: B.hmy_k_attn_bwd(1, qkv, o, do, lse, delta, dqkv, b, s, H, dh, causal, dbias=x) for x in (db, None))
    assert_takes_at_most(1.25, with_sums, without, "with the bias gradient over without")


# 160 workgroups and 162; causal, rows of 255 and 256 beyond 160 of them, 256 of them and 258; as many rows as their delta has room
# for in LDS, and one more
@pytest.mark.parametrize("causal,b,s,H", [(0, 10, 130, 8), (0, 27, 130, 3), (1, 10, 130, 8), (1, 41, 255, 2), (1, 41, 256, 2),
                                          (1, 32, 256, 4), (1, 43, 256, 3), (0, 1, 66, 1), (1, 1, 7168, 1), (1, 1, 7169, 1)])
def test_attention_backward_in_one_launch_and_in_two(causal, b, s, H):
    """dQ and dK/dV side by side, where dK/dV makes its own delta, and one after the other."""
    say(f"attention backward in one launch or two causal={causal} b={b} s={s} H={H}")
    _attention_case(*PRECS[1], causal, b, s, H, 64)


@pytest.mark.parametrize("causal,b,s,H,dh", [(1, 2, 60, 8, 32), (0, 1, 250, 16, 64), (1, 1, 1100, 4, 64), (0, 4, 500, 16, 64), (1, 2, 60, 8, 128),
                                             (0, 1, 500, 8, 128), (0, 17, 130, 8, 128), (1, 1, 2050, 2, 128)])
def test_attention_bf16_against_64_bits_element_by_element(causal, b, s, H, dh):
    """Each element against what bf16 roundings (eight significant bits: u = 2^-8 at most) can do to it at most, so that one wrong element shows:
    o: its own, the probabilities' and their sum's; lse: that sum's; dV: its own, the probabilities' and (through lse) the row's;
    delta: o's; dS: its own, lse's and delta's; dQ, dK: their own and dS's."""
    say(f"attention bf16 against 64 bits causal={causal} b={b} s={s} H={H} dh={dh}")
    T, d, u = b * s, H * dh, 2.0 ** -8
    g = torch.Generator(device="cuda").manual_seed(s + dh)
    qkv, do = (torch.randn(T, n, device="cuda", generator=g).bfloat16() for n in (3 * d, d))
    o, dqkv = torch.empty_like(do), torch.empty_like(qkv)
    lse, delta = torch.empty(b * H * s, device="cuda"), torch.empty(b * H * s, device="cuda")
    B.hmy_k_attn_fwd(1, qkv, o, lse, b, s, H, dh, causal)
    B.hmy_k_attn_bwd(1, qkv, o, do, lse, delta, dqkv, b, s, H, dh, causal)
    heads = lambda x: x.double().view(b, s, -1, H, dh).permute(2, 0, 3, 1, 4).contiguous()   # [.., b, H, s, dh]
    t = lambda x: x.transpose(-1, -2).contiguous()
    q, k, v = heads(qkv)
    G, scale = heads(do)[0], 1.0 / math.sqrt(dh)
    S = q @ t(k) * scale
    if causal:
        S = S.masked_fill(torch.ones(s, s, device="cuda", dtype=torch.bool).triu(1), -math.inf)
    P, ref_lse = S.softmax(-1), torch.logsumexp(S, -1)
    ref_o = P @ v
    off_o = u * (2 * ref_o.abs() + P @ v.abs())
    dS = P * (G @ t(v) - (G * ref_o).sum(-1, keepdim=True))
    off_dS = 2 * u * dS.abs() + P * (G.abs() * off_o).sum(-1, keepdim=True)
    ref = [("o", ref_o, off_o, heads(o)[0])]
    for (name, r, off), got in zip((("dq", dS @ k * scale, off_dS @ k.abs() * scale), ("dk", t(dS) @ q * scale, t(off_dS) @ q.abs() * scale),
                                    ("dv", t(P) @ G, 2 * u * (t(P) @ G.abs()))), heads(dqkv)):
        ref.append((name, r, off + u * r.abs(), got))
    assert float((lse.double().view(b, H, s) - ref_lse).abs().max()) < 1.05 * u
    for name, r, off, got in ref:
        rel = float((got - r).norm() / r.norm())
        share = float(((got - r).abs() / (off + 1e-6)).max())    # 1e-6: fp32 sums of a few hundred terms of size 1
        say(f"  {name}: 2-norm {rel:.2e}, largest error {share:.2f} of its bound")
        assert share < 1.05 and rel < u, name     # independent roundings: two or three of 0.4 u each in the 2-norm


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
@pytest.mark.parametrize("T,V", [(9, 1000), (33, 50257), (4, 2)] + [(2, v + k) for v in (4096, 14336, 32768, 57344) for k in (0, 1)])
def test_cross_entropy(prec, pc, dt, tol, T, V):
    say(f"xent {prec} T={T} V={V}")
    rng = np.random.default_rng(V)
    ldl = (V + 7) // 8 * 8
    logits = np.zeros((T, ldl), np.float32)
    logits[:, :V] = rng.standard_normal((T, V)).astype(np.float32) * 3
    tg = rng.integers(0, V, size=T).astype(np.int32)
    tg[::3] = -1
    n_tgt = 57                                  # a minibatch-wide count, not this chunk's
    dl = torch.full((T, ldl), float("nan"), device="cuda", dtype=dt)
    acc = torch.zeros(1, device="cuda", dtype=torch.float64)
    B.hmy_k_xent(pc, dev(logits, torch.float32), torch.from_numpy(tg).cuda(), acc, dl, T, V, ldl, 1.0 / n_tgt)
    l64 = logits[:, :V].astype(np.float64)
    lse = np.log(np.exp(l64 - l64.max(1, keepdims=True)).sum(1)) + l64.max(1)
    rows = np.nonzero(tg >= 0)[0]
    loss_ref = (lse[rows] - l64[rows, tg[rows]]).sum() / n_tgt
    assert abs(host(acc)[0] - loss_ref) < 1e-5 * abs(loss_ref)
    ref = np.zeros((T, V))
    ref[rows] = np.exp(l64[rows] - lse[rows, None])
    ref[rows, tg[rows]] -= 1
    ref /= n_tgt
    got = host(dl)
    assert np.all(got[:, V:] == 0)              # the row padding is zeroed
    assert max_rel_err(got[:, :V], ref) < (tol if prec == "bf16" else 1e-5)


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
@pytest.mark.parametrize("V", [1000, 9000, 20000, 40000])
def test_cross_entropy_of_infinities(prec, pc, dt, tol, V):
    """Rows in registers against the general kernel (rows that allow no 16-byte access): infinite and undefined logits
    give the same loss and the same gradient.  Rows: ordinary, +inf beside the target, +inf at it, most of the row -inf,
    NaN."""
    say(f"xent infinities {prec} V={V}")
    inf = float("inf")
    x = torch.randn(5, V, generator=torch.Generator().manual_seed(V))
    tgt = torch.tensor([3, 5, 7, 11, 13], dtype=torch.int32)
    x[1, V // 2], x[2, 7], x[3, 12:], x[4, V - 1] = inf, inf, -inf, float("nan")
    for row in range(5):
        got = []
        for ldl in (V, V + 1):
            logits = torch.full((1, ldl), 5.0, device="cuda")
            logits[:, :V] = x[row].cuda()
            loss, d = torch.zeros(1, dtype=torch.float64, device="cuda"), torch.full((1, ldl), 9.0, device="cuda", dtype=dt)
            B.hmy_k_xent(pc, logits, tgt[row:row + 1].cuda(), loss, d, 1, V, ldl, 0.5)
            got.append((loss.cpu(), d[:, :V].float().cpu()))
        # sums of V fp32 terms in two orders; a gradient on either side of a bf16 rounding boundary
        assert torch.allclose(got[0][0], got[1][0], rtol=1e-5, equal_nan=True), row
        assert torch.allclose(got[0][1], got[1][1], rtol=1e-2 if prec == "bf16" else 1e-4, atol=1e-9, equal_nan=True), row


@pytest.mark.parametrize("prec,pc,dt,tol", PRECS)
@pytest.mark.parametrize("step", [1, 10])
def test_adam(prec, pc, dt, tol, step):
    say(f"adam {prec} step={step}")
    rng = np.random.default_rng(step)
    n = 4 * 1000 + 3
    w = rng.standard_normal(n).astype(np.float32) * 0.02
    g = rng.standard_normal(n).astype(np.float32) * 1e-3
    m0 = (rng.standard_normal(n).astype(np.float32) * 1e-3) if step > 1 else np.zeros(n, np.float32)
    v0 = ((rng.standard_normal(n).astype(np.float32) * 1e-3) ** 2) if step > 1 else np.zeros(n, np.float32)
    f32 = lambda x: float(np.float32(x))     # the C ABI carries fp32 hyper-parameters
    hp = om.AdamHP(lr=f32(1e-3), beta1=f32(0.9), beta2=f32(0.999), eps=f32(1e-8), step=step)
    wr, mr, vr = om.adam_update(w.astype(np.float64), g.astype(np.float64), m0.astype(np.float64),
                                v0.astype(np.float64), hp)
    gd, md, vd = dev(g, torch.float32), dev(m0, torch.float32), dev(v0, torch.float32)
    if prec == "bf16":
        master = dev(w, torch.float32)
        wout = torch.zeros(n, device="cuda", dtype=torch.bfloat16)
        B.hmy_k_adam(pc, gd, master, md, vd, wout, n, hp.lr, hp.beta1, hp.beta2, hp.eps, step)
        new_master = host(master)
        # the compute copy is exactly the RNE rounding of the fp32 master
        assert np.array_equal(host(wout), synth.round_bf16(new_master.astype(np.float32)).astype(np.float64))
    else:
        wd = dev(w, torch.float32)
        B.hmy_k_adam(pc, gd, None, md, vd, wd, n, hp.lr, hp.beta1, hp.beta2, hp.eps, step)
        new_master = host(wd)
    assert max_rel_err(new_master - w, wr - w) < 1e-4     # the update itself, not w (which barely moves)
    assert max_rel_err(host(md), mr) < 1e-6
    assert max_rel_err(host(vd), vr) < 1e-6
