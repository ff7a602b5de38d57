"""Per-kernel parity of the HIP library against the CPU oracle.

Both sides take the same seeded inputs; the GPU result is compared element
by element with the oracle's fp64 result.  Tolerances: fp32 storage max-abs
1e-4 (plus 1e-5 relative); bf16 storage max-abs 2e-2 with 1e-2 relative,
the bar for bf16 activations.  Integer work (selection, gathers, scatters)
is compared bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2503_12450_amd import binding as B
from paper_2503_12450_amd.device import to_device
from paper_2503_12450_amd.workload import normal_rows, random_index_sets, to_storage

pytestmark = pytest.mark.gpu

TOL = {"f32": dict(atol=1e-4, rtol=1e-5), "bf16": dict(atol=2e-2, rtol=1e-2)}
DEV = "cuda"


def _host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def _close(got, want, dtype, what=""):
    np.testing.assert_allclose(_host(got) if torch.is_tensor(got) else got, want, err_msg=what, **TOL[dtype])


def _cache_layout(rows, H):
    """[slots, S, D] rows -> [slots, H, S, dh]"""
    s, S, D = rows.shape
    return np.ascontiguousarray(rows.reshape(s, S, H, D // H).transpose(0, 2, 1, 3))


# --------------------------------------------------------------------------
# LayerNorm (with and without the row gather)
# --------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,D", [(1, 64), (300, 256), (77, 1280), (5, 2048)])
def test_layernorm_dense(dtype, M, D):
    src = normal_rows((M, D), seed=11, std=2.0) + 0.5
    w = 1.0 + normal_rows((D,), seed=12, std=0.2)
    b = normal_rows((D,), seed=13, std=0.2)
    out = torch.empty((M, D), dtype=to_device(src[:1], dtype).dtype, device=DEV)
    B.k_layernorm(dtype, to_device(src, "f32"), to_device(w, "f32"), to_device(b, "f32"), 1e-6, out)
    torch.cuda.synchronize()
    _close(out, O.layer_norm(src, w, b, 1e-6), dtype)


@pytest.mark.parametrize("dtype,src_dtype", [("f32", "f32"), ("bf16", "f32"), ("bf16", "bf16")])
def test_layernorm_gather(dtype, src_dtype):
    slots, S, D, N = 3, 50, 256, 7
    src = normal_rows((slots, S, D), seed=14, dtype=src_dtype)
    idx = random_index_sets(slots, S, N, seed=15)
    w = 1.0 + normal_rows((D,), seed=16, std=0.2)
    b = normal_rows((D,), seed=17, std=0.2)
    out = torch.empty((slots * N, D), dtype=to_device(src[:1, :1], dtype).dtype, device=DEV)
    copy = torch.full((slots * N, D), 7.0, dtype=torch.float32, device=DEV)
    B.k_layernorm(dtype, to_device(src, src_dtype), to_device(w, "f32"), to_device(b, "f32"), 1e-6, out,
                  idx=torch.from_numpy(idx).to(DEV), per_slot=N, seq=S, copy_f32=copy)
    torch.cuda.synchronize()
    gathered = np.concatenate([src[s, idx[s]] for s in range(slots)])
    np.testing.assert_array_equal(copy.cpu().numpy(), gathered)   # the gather is exact
    _close(out, O.layer_norm(gathered, w, b, 1e-6), dtype)


# --------------------------------------------------------------------------
# Matrix products with their epilogues
# --------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(1, 64, 64), (300, 320, 256), (129, 1024, 1024), (1000, 192, 3072),
                                   (65, 264, 128), (7, 8, 64)])  # columns ending mid-tile, by 8
@pytest.mark.parametrize("gelu", [False, True])
def test_linear(dtype, M, N, K, gelu):
    a = normal_rows((M, K), seed=21, dtype=dtype)
    w = normal_rows((N, K), seed=22, std=0.05, dtype=dtype)
    bias = normal_rows((N,), seed=23, std=0.5)
    out = torch.empty((M, N), dtype=to_device(a[:1], dtype).dtype, device=DEV)
    B.k_linear(dtype, to_device(a, dtype), to_device(w, dtype), to_device(bias, "f32"), out, gelu=gelu)
    torch.cuda.synchronize()
    ref = O.linear(a, w, bias)
    if gelu:
        ref = O.gelu(ref)
    _close(out, ref, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gelu_over_wide_range(dtype):
    """GELU epilogue against the exact erf form for pre-activations from -12
    to 12 (tails where Phi saturates, zero, and both signs)."""
    M, N, K = 64, 1024, 64
    a = np.zeros((M, K), np.float32)
    a[:, 0] = 1.0
    w = np.zeros((N, K), np.float32)
    bias = np.linspace(-12, 12, N, dtype=np.float32)
    out = torch.empty((M, N), dtype=to_device(a[:1], dtype).dtype, device=DEV)
    B.k_linear(dtype, to_device(a, dtype), to_device(w, dtype), to_device(bias, "f32"), out, gelu=True)
    torch.cuda.synchronize()
    want = O.gelu(np.broadcast_to(bias.astype(np.float64), (M, N)))
    tol = dict(atol=2e-6, rtol=2e-6) if dtype == "f32" else TOL["bf16"]
    np.testing.assert_allclose(_host(out), want, **tol)


@pytest.mark.parametrize("variant", [-1, 4])  # the few-row kernel and the tiled one
def test_gelu_negative_tail(variant):
    """bf16 GELU for pre-activations from -6 to 0, where the result is far
    smaller than its argument: the approximation's absolute error of 2.4e-4
    |x| (evaluated over the formula; 2.5e-4 here for its fp32 arithmetic) and
    half a bf16 step of the result."""
    M, N, K = 48, 2048, 64
    bias = np.linspace(-6, 0, N, dtype=np.float32)
    out = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    try:
        B.k_gemm_variant(variant)
        B.k_linear("bf16", torch.zeros((M, K), dtype=torch.bfloat16, device=DEV),
                   torch.zeros((N, K), dtype=torch.bfloat16, device=DEV), to_device(bias, "f32"), out, gelu=True)
    finally:
        B.k_gemm_variant(-1)
    torch.cuda.synchronize()
    want = np.broadcast_to(O.gelu(bias.astype(np.float64)), (M, N))
    bound = 2.5e-4 * np.abs(bias.astype(np.float64))
    bound = bound + 2.0 ** -8 * (np.abs(want) + bound) + 1e-12
    assert np.all(np.abs(_host(out) - want) <= bound)


@pytest.mark.parametrize("variant", list(range(16)))
def test_tile_variants_are_bitwise_identical(variant):
    """Every tile configuration visits k in the same order: same bits."""
    M, N, K = 700, 640, 512
    a = to_device(normal_rows((M, K), seed=91, dtype="bf16"), "bf16")
    w = to_device(normal_rows((N, K), seed=92, std=0.05, dtype="bf16"), "bf16")
    bias = to_device(normal_rows((N,), seed=93), "f32")
    ref = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    out = torch.empty_like(ref)
    B.k_gemm_variant(-1)
    B.k_linear("bf16", a, w, bias, ref)
    try:
        B.k_gemm_variant(variant)
        B.k_linear("bf16", a, w, bias, out)
    finally:
        B.k_gemm_variant(-1)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


# sizes that reach every few-row tile (16 x 16, 32 x 32, 32 x 64, 64 x 48, 64 x
# 64, 64 x 96, 128 x 64), with rows and columns that end mid-tile, and K of one
# slice, of an odd number of slices, shorter and longer than the load rings
FEW_ROW_SHAPES = [(1, 64, 64), (10, 1024, 320), (17, 1000, 1024), (224, 1024, 1024), (100, 776, 192),
                  (640, 768, 3072), (509, 1288, 1216), (768, 1280, 64), (401, 2104, 640), (1023, 1528, 1536),
                  (1600, 1032, 1024)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", FEW_ROW_SHAPES)
def test_few_row_products_are_bitwise_the_tiled_ones(dtype, M, N, K):
    """The products on few rows take kernels of their own, which sum k in the
    order of the tiled kernel: the bits of the 128 x 128 tiles, for every
    epilogue (bias, GELU, residual in place and scattered, key/value cache)."""
    a = to_device(normal_rows((M, K), seed=101, dtype=dtype), dtype)
    w = to_device(normal_rows((N, K), seed=102, std=0.05, dtype=dtype), dtype)
    bias = to_device(normal_rows((N,), seed=103), "f32")
    resid = to_device(normal_rows((M, N), seed=104), "f32")
    seq = M + 3
    idx = torch.from_numpy(random_index_sets(1, seq, M, seed=105)).to(DEV)
    D = 64 * (K // 64)
    wq = to_device(normal_rows((3 * D, D), seed=106, std=0.05, dtype=dtype), dtype)
    bq = to_device(normal_rows((3 * D,), seed=107), "f32")

    def products():
        outs = [torch.full((M, N), 7.0, dtype=a.dtype, device=DEV) for _ in range(2)]
        B.k_linear(dtype, a, w, bias, outs[0])
        B.k_linear(dtype, a, w, bias, outs[1], gelu=True)
        h = resid.clone()
        B.k_linear_residual(dtype, a, w, bias, h, h)
        y = torch.full((seq, N), 7.0, dtype=torch.float32, device=DEV)
        copy = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
        B.k_linear_residual(dtype, a, w, bias, resid, y, out_idx=idx, per_slot=M, seq=seq, resid_copy=copy)
        q = torch.full((M, D), 7.0, dtype=a.dtype, device=DEV)
        kc, vc, v2 = (torch.full((1, D // 32, seq, 32), 7.0, dtype=a.dtype, device=DEV) for _ in range(3))
        B.k_qkv(dtype, a, wq, bq, D, D // 32, seq, M, q_out=q, k_cache=kc, v_cache=vc, v_copy=v2, idx=idx)
        torch.cuda.synchronize()
        return outs + [h, y, copy, q, kc, vc, v2]

    got = products()
    try:
        B.k_gemm_variant(4)
        want = products()
    finally:
        B.k_gemm_variant(-1)
    for g, r in zip(got, want):
        assert torch.equal(g, r)
    rows = np.linspace(0, M - 1, 5).astype(int)
    ref = O.linear(_host(a)[rows], _host(w), _host(bias))
    _close(_host(got[0])[rows], ref, dtype)


FEW_TILES = ["16x16", "32x32", "32x64", "64x48", "64x64", "64x96", "128x64"]
FEW_F32 = 4  # the tiles that exist for fp32


def _few_row_tile(tile):
    """Forces a few-row tile for every product (None: by shape), which the
    tuning hook of the C ABI cannot name."""
    B.load()["_ZN8marcache16set_gemm_variantEi"](-1 if tile is None else 100 + tile)


def _awkward(shape, seed, dtype):
    """Values spread over 2^24, the second half of every row nearly minus the
    first: sums whose rounding shows in which order they were formed."""
    g = np.random.Generator(np.random.Philox(seed))
    a = np.ldexp(g.standard_normal(shape), g.integers(-12, 12, shape)).astype(np.float32)
    k = shape[1] // 2
    a[:, k:2 * k] = -a[:, :k] * (1.0 + 0.01 * g.standard_normal((shape[0], k)).astype(np.float32))
    return to_storage(a, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tile", range(len(FEW_TILES)), ids=FEW_TILES)
def test_every_few_row_tile_is_bitwise_the_tiled_kernel(dtype, tile):
    """Each tile of the few-row kernel under every epilogue of the per-kernel
    entry points: rows and columns that end mid-tile, three slots with ragged
    rows, K from one slice to past the deepest ring, operands of one magnitude
    and of many."""
    if dtype == "f32" and tile >= FEW_F32:
        a = torch.zeros((16, 64), device=DEV)
        try:
            _few_row_tile(tile)
            with pytest.raises(B.MarError):
                B.k_linear(dtype, a, a, torch.zeros(16, device=DEV), torch.empty((16, 16), device=DEV))
        finally:
            _few_row_tile(None)
        return
    for n, (slots, per, N, D, dh, awkward) in enumerate([(1, 1, 8, 64, 16, False), (3, 45, 200, 192, 48, True),
                                                         (3, 70, 328, 320, 80, False), (2, 131, 136, 640, 64, True),
                                                         (3, 43, 1032, 1152, 32, True)]):
        M, seq, K = slots * per, per + 7, D
        a_h = _awkward((M, K), 300 + n, dtype) if awkward else normal_rows((M, K), seed=300 + n, dtype=dtype)
        a = to_device(a_h, dtype)
        w = to_device(_awkward((N, K), 310 + n, dtype) if awkward else normal_rows((N, K), seed=310 + n, std=0.05,
                                                                                   dtype=dtype), dtype)
        wq = to_device(normal_rows((3 * D, D), seed=320 + n, std=0.05, dtype=dtype), dtype)
        bias, bq = to_device(normal_rows((N,), seed=330 + n), "f32"), to_device(normal_rows((3 * D,), seed=340 + n), "f32")
        resid = to_device(normal_rows((M, N), seed=350 + n), "f32")
        idx = torch.from_numpy(random_index_sets(slots, seq, per, seed=360 + n).reshape(-1)).to(DEV)
        H = D // dh

        def products():
            out, act = (torch.full((M, N), 7.0, dtype=a.dtype, device=DEV) for _ in range(2))
            B.k_linear(dtype, a, w, bias, out)
            B.k_linear(dtype, a, w, bias, act, gelu=True)
            h = resid.clone()
            B.k_linear_residual(dtype, a, w, bias, h, h)
            y = torch.full((slots * seq, N), 7.0, device=DEV)
            copy = torch.full((M, N), 7.0, device=DEV)
            B.k_linear_residual(dtype, a, w, bias, resid, y, out_idx=idx, per_slot=per, seq=seq, resid_copy=copy)
            outs = [out, act, h, y, copy]
            for at, S in ((idx, seq), (None, per)):  # scattered and dense rows
                q = torch.full((M, D), 7.0, dtype=a.dtype, device=DEV)
                kv = [torch.full((slots, H, S, dh), 7.0, dtype=a.dtype, device=DEV) for _ in range(3)]
                B.k_qkv(dtype, a, wq, bq, D, H, S, per, q_out=q, k_cache=kv[0], v_cache=kv[1], v_copy=kv[2], idx=at)
                outs += [q, *kv]
            torch.cuda.synchronize()
            return outs

        try:
            _few_row_tile(tile)
            got = products()
            B.k_gemm_variant(4)
            want = products()
        finally:
            B.k_gemm_variant(-1)
        for g, r in zip(got, want):
            assert torch.equal(g, r)


@pytest.mark.parametrize("tile", range(len(FEW_TILES)), ids=FEW_TILES)
def test_every_few_row_tile_is_bitwise_the_tiled_kernel_in_the_head(tile):
    """The SiLU and gated-residual epilogues of every tile, through the
    diffusion head with all its products forced."""
    from paper_2503_12450_amd.device import upload_head
    from paper_2503_12450_amd.workload import HeadDims, head_weights
    hd = HeadDims(width=448, depth=2, cond_dim=64, token_dim=16, steps=4, train_steps=40, freq_dim=64, max_rows=90)
    W = upload_head(head_weights(hd, seed=81), hd.dtype)
    y = to_device(normal_rows((77, hd.cond_dim), seed=82), "f32")
    idx = torch.arange(77, dtype=torch.int32, device=DEV)
    x0 = to_device(normal_rows((77, hd.token_dim), seed=83), "f32")
    xi = to_device(normal_rows((hd.steps, 77, hd.token_dim), seed=84), "f32")
    out = [torch.empty((77, hd.token_dim), device=DEV) for _ in range(2)]
    try:
        _few_row_tile(tile)
        B.MarHead(hd, W).sample(y, y, idx, idx, x0, xi, 3.0, out[0])
        B.k_gemm_variant(4)
        B.MarHead(hd, W).sample(y, y, idx, idx, x0, xi, 3.0, out[1])
        torch.cuda.synchronize()
    finally:
        B.k_gemm_variant(-1)
    assert torch.equal(*out)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("variant", list(range(8, 16)))
def test_persistent_workgroups_walk_several_tiles(dtype, variant):
    """Persistent launches run one or two workgroups per CU; with 264 tiles
    of 256 x 256 (1056 of 128 x 128) each workgroup carries its load ring
    and bias across tile boundaries.  Same bits as one workgroup per tile,
    and within tolerance of the oracle on sampled rows."""
    M, N, K = 8448, 2048, 384
    a_h = normal_rows((M, K), seed=95, dtype=dtype)
    w_h = normal_rows((N, K), seed=96, std=0.05, dtype=dtype)
    bias_h = normal_rows((N,), seed=97)
    a, w, bias = to_device(a_h, dtype), to_device(w_h, dtype), to_device(bias_h, "f32")
    ref = torch.empty((M, N), dtype=a.dtype, device=DEV)
    out = torch.empty_like(ref)
    try:
        B.k_gemm_variant(variant - 8)
        B.k_linear(dtype, a, w, bias, ref, gelu=True)
        B.k_gemm_variant(variant)
        B.k_linear(dtype, a, w, bias, out, gelu=True)
    finally:
        B.k_gemm_variant(-1)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    rows = np.array([0, 1, 255, 256, 4095, 4096, 8191, 8192, M - 1])
    want = O.gelu(O.linear(a_h[rows], w_h, bias_h))
    _close(out[torch.from_numpy(rows).to(DEV)], want, dtype)


@pytest.mark.parametrize("kind,M,N", [("residual", 33280, 1024), ("gelu", 41216, 2048)])
def test_balanced_last_round_is_bitwise_identical(kind, M, N):
    """By shape, a persistent 256 x 256 launch whose last round would leave
    CUs idle runs its whole rounds with 256 x 256 tiles and the rows left
    over with 256 x 128 tiles (a second launch).  Same bits as one
    workgroup per 256 x 256 tile, and within tolerance of the oracle on rows
    of both parts."""
    K = 256
    a_h = normal_rows((M, K), seed=81, dtype="bf16")
    w_h = normal_rows((N, K), seed=82, std=0.05, dtype="bf16")
    bias_h = normal_rows((N,), seed=83)
    a, w, bias = to_device(a_h, "bf16"), to_device(w_h, "bf16"), to_device(bias_h, "f32")
    if kind == "residual":
        r_h = normal_rows((M, N), seed=84)
        ref, out = to_device(r_h, "f32"), to_device(r_h, "f32")
        run = lambda o: B.k_linear_residual("bf16", a, w, bias, o, o)  # noqa: E731
    else:
        ref = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        out = torch.empty_like(ref)
        run = lambda o: B.k_linear("bf16", a, w, bias, o, gelu=True)  # noqa: E731
    try:
        B.k_gemm_variant(0)
        run(ref)
        B.k_gemm_variant(-1)
        run(out)
    finally:
        B.k_gemm_variant(-1)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    rows = np.array([0, 255, 32767, 32768, M - 257, M - 1])
    want = O.linear(a_h[rows], w_h, bias_h)
    want = want + r_h[rows] if kind == "residual" else O.gelu(want)
    _close(out[torch.from_numpy(rows).to(DEV)], want, "bf16")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(200, 256, 512), (200, 264, 128)])
def test_linear_residual_in_place_and_scatter(dtype, M, N, K):
    a = normal_rows((M, K), seed=31, dtype=dtype)
    w = normal_rows((N, K), seed=32, std=0.05, dtype=dtype)
    bias = normal_rows((N,), seed=33, std=0.5)
    resid = normal_rows((M, N), seed=34)
    r = to_device(resid, "f32")
    B.k_linear_residual(dtype, to_device(a, dtype), to_device(w, dtype), to_device(bias, "f32"), r, r)
    torch.cuda.synchronize()
    ref = resid + O.linear(a, w, bias)
    _close(r, ref, dtype)
    # scatter into an output cache [slots, S, N] at per-slot token indices
    slots, S = 4, 120
    per = M // slots
    idx = random_index_sets(slots, S, per, seed=35)
    ycache = torch.full((slots, S, N), -3.0, dtype=torch.float32, device=DEV)
    copy = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    r2 = to_device(resid, "f32")
    B.k_linear_residual(dtype, to_device(a, dtype), to_device(w, dtype), to_device(bias, "f32"), r2, ycache,
                        out_idx=torch.from_numpy(idx.reshape(-1)).to(DEV), per_slot=per, seq=S, resid_copy=copy)
    torch.cuda.synchronize()
    yc = ycache.cpu().numpy()
    for s in range(slots):
        _close(yc[s, idx[s]], ref[s * per:(s + 1) * per], dtype)
        untouched = np.setdiff1d(np.arange(S), idx[s])
        assert np.all(yc[s, untouched] == -3.0)
    _close(copy, ref, dtype)
    np.testing.assert_array_equal(r2.cpu().numpy(), resid)  # resid is read only here


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,H", [(128, 2), (320, 4), (256, 16)])
def test_qkv_dense_and_scattered(dtype, D, H):
    slots, S = 3, 70
    dh = D // H
    M = slots * S
    a = normal_rows((M, D), seed=41, dtype=dtype)
    w = normal_rows((3 * D, D), seed=42, std=0.05, dtype=dtype)
    bias = normal_rows((3 * D,), seed=43, std=0.5)
    ref = O.linear(a, w, bias)
    td = to_device(a[:1], dtype).dtype
    q = torch.empty((M, D), dtype=td, device=DEV)
    kc = torch.zeros((slots, H, S, dh), dtype=td, device=DEV)
    vc = torch.zeros((slots, H, S, dh), dtype=td, device=DEV)
    vcopy = torch.zeros((slots, H, S, dh), dtype=td, device=DEV)
    B.k_qkv(dtype, to_device(a, dtype), to_device(w, dtype), to_device(bias, "f32"), D, H, S, S,
            q_out=q, k_cache=kc, v_cache=vc, v_copy=vcopy)
    torch.cuda.synchronize()
    _close(q, ref[:, :D], dtype)
    _close(kc, _cache_layout(ref[:, D:2 * D].reshape(slots, S, D), H), dtype)
    # values: the cache and the copy share the key layout [slot, head, token, d]
    _close(vc, _cache_layout(ref[:, 2 * D:].reshape(slots, S, D), H), dtype)
    np.testing.assert_array_equal(_host(vcopy), _host(vc))
    # compact rows: keys/values land at their tokens, other rows untouched
    N = 9
    idx = random_index_sets(slots, S, N, seed=44)
    ac = normal_rows((slots * N, D), seed=45, dtype=dtype)
    refc = O.linear(ac, w, bias)
    kc2 = torch.full((slots, H, S, dh), 5.0, dtype=td, device=DEV)
    vc2 = torch.full((slots, H, S, dh), 5.0, dtype=td, device=DEV)
    qc = torch.empty((slots * N, D), dtype=td, device=DEV)
    B.k_qkv(dtype, to_device(ac, dtype), to_device(w, dtype), to_device(bias, "f32"), D, H, S, N,
            q_out=qc, k_cache=kc2, v_cache=vc2, idx=torch.from_numpy(idx.reshape(-1)).to(DEV))
    torch.cuda.synchronize()
    _close(qc, refc[:, :D], dtype)
    k2, v2 = _host(kc2), _host(vc2)
    for s in range(slots):
        rows = refc[s * N:(s + 1) * N]
        _close(k2[s][:, idx[s]], rows[:, D:2 * D].reshape(N, H, dh).transpose(1, 0, 2), dtype)
        _close(v2[s][:, idx[s]], rows[:, 2 * D:].reshape(N, H, dh).transpose(1, 0, 2), dtype)
        other = np.setdiff1d(np.arange(S), idx[s])
        assert np.all(k2[s][:, other] == 5.0) and np.all(v2[s][:, other] == 5.0)
    # value columns only (the scoring pass when no block is always computed)
    vonly = torch.zeros((slots, H, S, dh), dtype=td, device=DEV)
    wd = to_device(w, dtype)
    bd = to_device(bias, "f32")
    B.k_qkv(dtype, to_device(a, dtype), wd[2 * D:], bd[2 * D:], D, H, S, S, v_cache=vonly,
            n_offset=2 * D, n_cols=D)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(_host(vonly), _host(vc))


# --------------------------------------------------------------------------
# Attention (Eq. 3), dense and partial
# --------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("S,dh,H,per", [(64, 64, 2, 64), (100, 64, 2, 100), (320, 64, 3, 50),
                                        (320, 80, 2, 32), (131, 16, 2, 131), (1088, 64, 1, 218),
                                        (70, 128, 1, 5), (200, 48, 2, 1)])
def test_attention(dtype, S, dh, H, per):
    slots = 2
    D = H * dh
    q = normal_rows((slots * per, D), seed=51, dtype=dtype)
    k = normal_rows((slots, H, S, dh), seed=52, dtype=dtype)
    v = normal_rows((slots, H, S, dh), seed=53, dtype=dtype)
    td = to_device(q[:1], dtype).dtype
    out = torch.empty((slots * per, D), dtype=td, device=DEV)
    B.k_attention(dtype, to_device(q, dtype), to_device(k, dtype), to_device(v, dtype), out, slots, H, S, dh, per)
    torch.cuda.synchronize()
    ref = np.empty((slots * per, D))
    for s in range(slots):
        for h in range(H):
            ref[s * per:(s + 1) * per, h * dh:(h + 1) * dh] = O.attention(
                q[s * per:(s + 1) * per, h * dh:(h + 1) * dh], k[s, h], v[s, h])
    _close(out, ref, dtype)


@pytest.mark.parametrize("S,dh,per", [(1, 16, 1), (15, 48, 15), (16, 64, 17), (17, 64, 16), (63, 80, 33), (65, 128, 1),
                                      (130, 112, 130)])
def test_attention_f32_key_and_query_edges(S, dh, per):
    """fp32: sequences shorter than the four waves' key tiles, one key or
    query past a tile, one short of it; infinite values of the last key stay
    infinite (the padding past it adds nothing)."""
    slots, H = 2, 3
    q = normal_rows((slots * per, H * dh), seed=61)
    k = normal_rows((slots, H, S, dh), seed=62)
    v = normal_rows((slots, H, S, dh), seed=63)
    v[1, 2, S - 1, 3] = np.inf
    out = torch.empty((slots * per, H * dh), dtype=torch.float32, device=DEV)
    B.k_attention("f32", to_device(q, "f32"), to_device(k, "f32"), to_device(v, "f32"), out, slots, H, S, dh, per)
    torch.cuda.synchronize()
    ref = np.empty((slots * per, H * dh))
    for s in range(slots):
        for h in range(H):
            ref[s * per:(s + 1) * per, h * dh:(h + 1) * dh] = O.attention(
                q[s * per:(s + 1) * per, h * dh:(h + 1) * dh], k[s, h], v[s, h])
    assert np.all(np.isinf(ref[per:, 2 * dh + 3]))
    _close(out, ref, "f32")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("per", [320, 50])
def test_attention_spiky_keys(dtype, per):
    """Keys past the first blocks that score far above (or below) all
    earlier ones move the running softmax maxima mid-sequence; against the
    oracle for the dense and a partial launch."""
    slots, H, S, dh = 2, 2, 320, 64
    D = H * dh
    q = normal_rows((slots * per, D), seed=58, dtype=dtype)
    k = normal_rows((slots, H, S, dh), seed=59, dtype=dtype)
    k[:, :, 200:204] *= 12.0
    k[:, :, 290:292] *= 20.0
    k = to_storage(k, dtype)
    v = normal_rows((slots, H, S, dh), seed=60, dtype=dtype)
    td = to_device(q[:1], dtype).dtype
    out = torch.empty((slots * per, D), dtype=td, device=DEV)
    B.k_attention(dtype, to_device(q, dtype), to_device(k, dtype), to_device(v, dtype), out, slots, H, S, dh, per)
    torch.cuda.synchronize()
    ref = np.empty((slots * per, D))
    for s in range(slots):
        for h in range(H):
            ref[s * per:(s + 1) * per, h * dh:(h + 1) * dh] = O.attention(
                q[s * per:(s + 1) * per, h * dh:(h + 1) * dh], k[s, h], v[s, h])
    _close(out, ref, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("spiky", [False, True])
def test_attention_query_rows_independent(dtype, spiky):
    """A query's result does not depend on the other queries of the launch:
    the partial launch (other queries per workgroup and wave) reproduces the
    dense launch's rows bit for bit.  With spiky keys, a few keys past the
    first block score far above everything before them for some queries and
    far below for others, so the running maxima move mid-sequence for only
    part of each wave."""
    slots, H, S, dh = 2, 2, 200, 64
    D = H * dh
    q = normal_rows((slots * S, D), seed=54, dtype=dtype)
    k = normal_rows((slots, H, S, dh), seed=55, dtype=dtype)
    v = normal_rows((slots, H, S, dh), seed=56, dtype=dtype)
    if spiky:
        k[:, :, 130:136] *= 12.0
        k = to_storage(k, dtype)
    kd, vd = to_device(k, dtype), to_device(v, dtype)
    td = kd.dtype
    dense = torch.empty((slots * S, D), dtype=td, device=DEV)
    B.k_attention(dtype, to_device(q, dtype), kd, vd, dense, slots, H, S, dh, S)
    N = 37
    idx = random_index_sets(slots, S, N, seed=57)
    qs = np.concatenate([q[s * S + idx[s]] for s in range(slots)])
    part = torch.empty((slots * N, D), dtype=td, device=DEV)
    B.k_attention(dtype, to_device(qs, dtype), kd, vd, part, slots, H, S, dh, N)
    torch.cuda.synchronize()
    dh_ = _host(dense)
    want = np.concatenate([dh_[s * S + idx[s]] for s in range(slots)])
    np.testing.assert_array_equal(_host(part), want)


# --------------------------------------------------------------------------
# Eq. (8): scores and selection
# --------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("slots,H,S,dh", [(2, 12, 320, 64), (3, 16, 100, 80), (1, 1, 7, 16)])
def test_scores_bitwise(dtype, slots, H, S, dh):
    v = normal_rows((slots, H, S, dh), seed=61, dtype=dtype)
    r = to_storage(v + normal_rows((slots, H, S, dh), seed=62, std=0.3), dtype)
    r[0, :, 1] = v[0, :, 1]          # identical row: score exactly 1
    if S > 4:
        r[0, :, 2] = 0.0              # one zero row: score 0
        v[0, :, 3] = 0.0
        r[0, :, 3] = 0.0              # both zero: score 1
    vd, rd = to_device(v, dtype), to_device(r, dtype)
    scores = torch.empty((slots, S), dtype=torch.float64, device=DEV)
    B.k_scores(dtype, vd, rd, scores, update_ref=True)
    torch.cuda.synchronize()
    rows = lambda a: a.transpose(0, 2, 1, 3).reshape(slots, S, H * dh)  # noqa: E731
    want = O.cosine_scores(rows(v), rows(r))
    got = scores.cpu().numpy()
    np.testing.assert_array_equal(got, want)
    assert got[0, 1] == 1.0
    np.testing.assert_array_equal(_host(rd), v)   # the reference now holds v


@pytest.mark.parametrize("slots", [2, 450])  # one wave per token; runs of tokens per wave
@pytest.mark.parametrize("H,dh", [(16, 64), (1, 8), (5, 48), (16, 80), (2, 256)])
def test_scores_bitwise_over_magnitudes(slots, H, dh):
    """bf16 rows whose vectors fall on both sides of the range that sums
    without rounding: single values far below or above their neighbours,
    denormals, zeros, and rows of one magnitude; bit for bit, in the first
    and last slots, and the reference replaced everywhere."""
    S, D = 25, H * dh
    g = np.random.Generator(np.random.Philox(77))
    v, r = (g.standard_normal((slots, S, D)).astype(np.float32) for _ in range(2))
    for s in (0, slots - 1):
        for t in range(S):
            kind = t % 6
            e = np.zeros(D, np.int64)
            if kind == 1:
                e = g.integers(-40, 40, D)
            elif kind == 2:
                e[g.integers(0, D, 2)] = -17 - t
            elif kind == 3:
                e = np.full(D, -125)
            elif kind == 4:
                e = -g.integers(0, 17, D)
            v[s, t] = np.ldexp(v[s, t], e)
            r[s, t] = np.ldexp(r[s, t], e)
            if kind == 5:
                v[s, t, g.random(D) < 0.5] = 0.0
    v, r = to_storage(v, "bf16"), to_storage(r, "bf16")
    dev = lambda a: to_device(_cache_layout(a, H), "bf16")  # noqa: E731
    scores = torch.empty((slots, S), dtype=torch.float64, device=DEV)
    dv, dr = dev(v), dev(r)
    B.k_scores("bf16", dv, dr, scores, update_ref=True)
    torch.cuda.synchronize()
    ends = [0, slots - 1]
    np.testing.assert_array_equal(scores.cpu().numpy()[ends], O.cosine_scores(v[ends], r[ends]))
    assert torch.equal(dr, dv)


@pytest.mark.parametrize("slots", [2, 450])  # one wave per token; runs of tokens per wave
@pytest.mark.parametrize("H,dh", [(16, 64), (5, 48), (16, 80), (2, 128), (3, 8)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_scores_bitwise_without_update(dtype, slots, H, dh):
    """Both kernels in both types over chunks per row that are no power of two
    and leave lanes over (fp32 48: 12 chunks, 80: 20), rows of many magnitudes
    among them; without update_ref the reference stays as it was."""
    S, D = 25, H * dh
    g = np.random.Generator(np.random.Philox(78))
    v, r = (g.standard_normal((slots, S, D)).astype(np.float32) for _ in range(2))
    for s in (0, slots - 1):
        v[s, ::3] = np.ldexp(v[s, ::3], g.integers(-30, 30, v[s, ::3].shape))
        r[s, ::4] = np.ldexp(r[s, ::4], g.integers(-30, 30, r[s, ::4].shape))
    v, r = to_storage(v, dtype), to_storage(r, dtype)
    dv, dr = (to_device(_cache_layout(a, H), dtype) for a in (v, r))
    before = dr.clone()
    scores = torch.empty((slots, S), dtype=torch.float64, device=DEV)
    B.k_scores(dtype, dv, dr, scores)
    torch.cuda.synchronize()
    ends = [0, slots - 1]
    np.testing.assert_array_equal(scores.cpu().numpy()[ends], O.cosine_scores(v[ends], r[ends]))
    assert torch.equal(dr, before)


@pytest.mark.parametrize("slots,S,n", [(4, 320, 50), (2, 320, 0), (2, 320, 320), (1, 1, 1), (3, 1088, 218),
                                       (2, 4096, 1000), (5, 33, 31)])
@pytest.mark.parametrize("most", [False, True])
def test_select_bit_exact(slots, S, n, most):
    """Both ranking rules (least similar: strategy V; most similar: strategy
    IV of Table 3) bit for bit, with exact ties, NaN and signed zeros."""
    g = np.random.Generator(np.random.Philox(71))
    s = 1.0 - np.abs(g.standard_normal((slots, S))) * 1e-3
    s[0, : S // 3] = np.round(s[0, : S // 3], 4)   # many exact ties
    if S > 10:
        s[-1, 5] = np.nan
        s[-1, 6] = -0.0
        s[-1, 7] = 0.0
    idx = torch.full((slots, n), -1, dtype=torch.int32, device=DEV)
    B.k_select(torch.from_numpy(s).to(DEV), n, idx, most_similar=most)
    torch.cuda.synchronize()
    rule = O.select_most_similar if most else O.select_least_similar
    want = np.stack([rule(s[b], n) for b in range(slots)])
    np.testing.assert_array_equal(idx.cpu().numpy(), want)


@pytest.mark.parametrize("S", [1, 64, 511, 512, 513, 1024, 1025, 4096])
@pytest.mark.parametrize("kind", ["equal", "ties", "range", "close"])
def test_select_over_sizes_and_score_ranges(S, kind):
    """Sizes around the workgroup's tokens per thread; scores that are all
    equal, of few values, of every magnitude and sign (denormals, infinities,
    signed zeros, NaN), and a few units in the last place apart."""
    g = np.random.Generator(np.random.Philox(S))
    s = {"equal": lambda: np.full((2, S), -0.25),
         "ties": lambda: g.integers(-2, 3, (2, S)) * np.where(g.random((2, S)) < 0.5, 0.5, -0.5),
         "range": lambda: g.standard_normal((2, S)) * np.exp2(g.integers(-1070, 1000, (2, S)).astype(np.float64)),
         "close": lambda: 1.0 - g.integers(0, 40, (2, S)) * 2.0 ** -53}[kind]()
    if kind == "range":
        s[0, ::7] = g.choice([np.inf, -np.inf, np.nan, 0.0, -0.0], s[0, ::7].shape)
    d = torch.from_numpy(np.ascontiguousarray(s, dtype=np.float64)).to(DEV)
    for n in sorted({1, (S + 1) // 2, max(1, S - 1), S}):
        for most in (False, True):
            idx = torch.full((2, n), -1, dtype=torch.int32, device=DEV)
            B.k_select(d, n, idx, most_similar=most)
            torch.cuda.synchronize()
            rule = O.select_most_similar if most else O.select_least_similar
            for b in range(2):
                np.testing.assert_array_equal(idx[b].cpu().numpy(), rule(s[b], n))


@pytest.mark.parametrize("S", [1, 63, 64, 65, 128, 129, 256, 257, 1024, 1025, 2048, 2049, 4096])
def test_select_of_many_sequences(S):
    """Several hundred sequences per launch at the edges of every workgroup
    size and of the tokens per thread; scores a few units in the last place
    apart, with one far below, so that a selection takes up to eight passes."""
    slots = 400
    g = np.random.Generator(np.random.Philox(1000 + S))
    s = 1.0 - g.integers(0, 3 * S, (slots, S)) * 2.0 ** -53
    s[np.arange(slots), g.integers(0, S, slots)] = -1e300
    d = torch.from_numpy(s).to(DEV)
    n = max(1, (2 * S) // 5)
    for most in (False, True):
        idx = torch.full((slots, n), -1, dtype=torch.int32, device=DEV)
        B.k_select(d, n, idx, most_similar=most)
        torch.cuda.synchronize()
        rule = O.select_most_similar if most else O.select_least_similar
        np.testing.assert_array_equal(idx.cpu().numpy(), np.stack([rule(s[b], n) for b in range(slots)]))


def test_select_of_more_sequences_than_one_launch_takes():
    """2^23 sequences and more: a launch of that many workgroups of 512 threads
    would be of 2^32 threads, which the runtime refuses."""
    slots, S = (1 << 23) + 3, 257
    s = torch.rand((slots, S), generator=torch.Generator(device=DEV).manual_seed(7), device=DEV, dtype=torch.float64)
    idx = torch.full((slots, 1), -1, dtype=torch.int32, device=DEV)
    B.k_select(s, 1, idx)
    torch.cuda.synchronize()
    assert torch.equal(idx[:, 0].long(), s.argmin(1))


def test_attention_f32_of_more_blocks_than_one_launch_takes():
    """2^24 heads and more, one query and one key each: 256 threads per head
    would be a launch of 2^32.  The softmax of one key is 1."""
    slots, H, dh = (1 << 20) + 1, 16, 16
    g = torch.Generator(device=DEV).manual_seed(8)
    q, k, v = (torch.randn((slots, H, 1, dh), generator=g, device=DEV) for _ in range(3))
    out = torch.empty((slots, H * dh), device=DEV)
    B.k_attention("f32", q.view(slots, H * dh), k, v, out, slots, H, 1, dh, 1)
    torch.cuda.synchronize()
    assert torch.equal(out, v.view(slots, H * dh))


@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 29807, 128, 128), ("bf16", 1268, 4424, 64), ("bf16", 1593, 1720, 320),
                                         ("bf16", 554, 6016, 128), ("bf16", 11558, 416, 128), ("bf16", 6, 2440, 1024),
                                         ("bf16", 1111, 3080, 768), ("f32", 1626, 448, 64), ("f32", 74, 7080, 128)])
def test_product_choice_is_near_the_fastest(dtype, M, N, K):
    """The kernel chosen by shape against every other one, in launches of a
    captured graph (no host time): products of a short K once took three times
    the fastest in thousands of small tiles.  The bound leaves room for the
    spread of timings of a few microseconds."""
    a = to_device(normal_rows((M, K), seed=201, dtype=dtype), dtype)
    w = to_device(normal_rows((N, K), seed=202, std=0.05, dtype=dtype), dtype)
    bias = to_device(normal_rows((N,), seed=203), "f32")
    out = torch.empty((M, N), dtype=a.dtype, device=DEV)
    few = range(FEW_F32 if dtype == "f32" else len(FEW_TILES))
    graphs = {}
    try:
        for v in (-1, 0, 4, 6, 7, *(100 + t for t in few)):
            _few_row_tile(None) if v < 0 else _few_row_tile(v - 100)
            B.k_linear(dtype, a, w, bias, out)
            torch.cuda.synchronize()
            graphs[v] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graphs[v]):
                for _ in range(20):
                    B.k_linear(dtype, a, w, bias, out)
    finally:
        _few_row_tile(None)
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    us = {}
    for _ in range(4):
        for v, g in graphs.items():
            t0.record()
            g.replay()
            t1.record()
            t1.synchronize()
            us[v] = min(us.get(v, 1e9), t0.elapsed_time(t1) * 1e3 / 20)
    assert us[-1] <= 1.35 * min(us.values()), us
