"""Per-kernel parity of the HIP kernels (through the C ABI's per-kernel entry
points) against the oracle's building blocks / the plain definition."""
import numpy as np
import pytest

import oracle
from paper_2206_04959_amd import binding as B
from paper_2206_04959_amd import synth
from tests.gpu_util import need_gpu, rel_err

pytestmark = pytest.mark.gpu


def _rand(shape, dtype, seed, std=1.0, mean=0.0):
    rng = np.random.default_rng(seed)
    v = (rng.standard_normal(size=shape, dtype=np.float32) * np.float32(std) + np.float32(mean))
    if dtype == "bf16":
        bits = synth.f32_to_bf16_bits(v)
        return bits, synth.bf16_bits_to_f64(bits)
    return v, v.astype(np.float64)


def _dev(payload):
    return B.to_device(payload)


GEMM_SHAPES = [(192, 320, 128), (2048, 8192, 128), (320, 192, 512)]


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("mnk", GEMM_SHAPES)
def test_gemm_layouts(dtype, a_t, b_t, mnk):
    torch = need_gpu()
    M, N, K = mnk
    if dtype == "fp32" and M * N > 4_000_000:
        pytest.skip("large fp32 case not needed")
    print(f"[gemm] {dtype} a_t={a_t} b_t={b_t} {mnk}", flush=True)
    a_p, a = _rand((K, M) if a_t else (M, K), dtype, 1)
    b_p, b = _rand((K, N) if b_t else (N, K), dtype, 2)
    A = a.T if a_t else a
    Bm = b if b_t else b.T
    ref = A @ Bm
    c = torch.empty((M, N), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    B.gemm(_dev(a_p), _dev(b_p), c, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_STORE)
    torch.cuda.synchronize()
    tol = 1e-2 if dtype == "bf16" else 1e-5
    assert rel_err(B.to_host_f64(c), ref) < tol
    # fp32 output (the weight-gradient epilogue), overwrite then accumulate
    c32 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    B.gemm(_dev(a_p), _dev(b_p), c32, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_F32,
           dtype=B.BF16 if dtype == "bf16" else B.FP32)
    B.gemm(_dev(a_p), _dev(b_p), c32, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_F32, accumulate=True,
           dtype=B.BF16 if dtype == "bf16" else B.FP32)
    torch.cuda.synchronize()
    assert rel_err(c32.cpu().numpy(), 2 * ref) < 2e-5


@pytest.mark.parametrize("cfg", list(range(1, 11)))
@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1), (1, 0)])
def test_gemm_smallest_problem_on_every_tile(cfg, a_t, b_t):
    """M = N = K = 64, the smallest problem the boundary accepts: one partial
    tile of every shape (up to 256 x 256), one K stage."""
    torch = need_gpu()
    M = N = K = 64
    print(f"[gemm 64^3] tile {cfg} a_t={a_t} b_t={b_t}", flush=True)
    a_p, a = _rand((K, M) if a_t else (M, K), "bf16", 23)
    b_p, b = _rand((K, N) if b_t else (N, K), "bf16", 24)
    ref = (a.T if a_t else a) @ (b if b_t else b.T)
    c32 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    prev = B.gemm_tile_override(cfg)
    try:
        B.gemm(_dev(a_p), _dev(b_p), c32, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_F32, dtype=B.BF16)
        torch.cuda.synchronize()
    finally:
        B.gemm_tile_override(prev)
    assert rel_err(c32.cpu().numpy(), ref) < 2e-5


@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("mnk", [(64, 64, 64), (128, 192, 192), (64, 320, 1024)])
def test_gemm_fp32_k_split(mnk, a_t, b_t):
    """fp32 kernel: K split over four waves in groups of 16 (one group each at K
    = 64).  Tolerance: fp32 sums of up to 1024 products, as in the layout test."""
    torch = need_gpu()
    M, N, K = mnk
    print(f"[gemm fp32] a_t={a_t} b_t={b_t} {mnk}", flush=True)
    a_p, a = _rand((K, M) if a_t else (M, K), "fp32", 27)
    b_p, b = _rand((K, N) if b_t else (N, K), "fp32", 28)
    ref = (a.T if a_t else a) @ (b if b_t else b.T)
    c = torch.empty((M, N), dtype=torch.float32, device="cuda")
    B.gemm(_dev(a_p), _dev(b_p), c, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_STORE)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(c), ref) < 1e-5


@pytest.mark.parametrize("a_t,b_t", [(0, 0), (1, 1)])
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_BIAS, B.EPI_BIAS_GELU, B.EPI_BIAS_RESID, B.EPI_GELU_BWD, B.EPI_F32])
def test_gemm_fp32_large_tiles(epi, a_t, b_t):
    """fp32 kernel at the first number of 64x64 tiles that takes them (800), with
    every epilogue: the bits of the same rows as a call with one row of tiles less,
    which takes 32x32 tiles."""
    torch = need_gpu()
    M, N, K = 1280, 2560, 192
    print(f"[gemm fp32 large] a_t={a_t} b_t={b_t} epi={epi}", flush=True)
    a_p, _ = _rand((K, M) if a_t else (M, K), "fp32", 61)
    b_p, _ = _rand((K, N) if b_t else (N, K), "fp32", 62)
    bias, resid, aux0 = (_dev(_rand(s, "fp32", i)[0]) for i, s in ((63, (N,)), (64, (M, N)), (65, (M, N))))
    a, b, out = _dev(a_p), _dev(b_p), []
    for m in (M, M - 64):
        c, aux = torch.full((m, N), 0.5, device="cuda"), aux0[:m].clone()
        B.gemm(a, b, c, m, N, K, a_trans=a_t, b_trans=b_t, lda=M if a_t else K, epilogue=epi,
               bias=bias if epi in (B.EPI_BIAS, B.EPI_BIAS_GELU, B.EPI_BIAS_RESID) else None,
               resid=resid if epi == B.EPI_BIAS_RESID else None,
               aux=aux if epi in (B.EPI_BIAS_GELU, B.EPI_BIAS_RESID, B.EPI_GELU_BWD) else None,
               accumulate=epi == B.EPI_F32)
        out.append((c, aux))
    torch.cuda.synchronize()
    assert torch.equal(out[0][0][:M - 64], out[1][0]) and torch.equal(out[0][1][:M - 64], out[1][1])
    if epi == B.EPI_STORE:  # and the values of the last rows
        A, Bm = a_p.astype(np.float64), b_p.astype(np.float64)
        ref = (A.T if a_t else A)[M - 64:] @ (Bm if b_t else Bm.T)
        assert rel_err(out[0][0][M - 64:].cpu().numpy(), ref) < 1e-5


# The tile that a lone launch of each (M, N, K) takes (64x128 tiles need A with K
# contiguous; where it is read transposed another is taken), each with ragged last tiles and
# more K stages than the ring holds; and the fewest stages that the two small shapes
# are chosen at, one and two.  test_tile_choice.py holds the choice to this table.
LONE_TILES = {(960, 1088, 320): "64x128", (1984, 1600, 320): "128x128", (3008, 1984, 576): "192x128",
              (1984, 3008, 576): "128x192", (3840, 1984, 576): "256x128", (960, 1088, 64): "128x128",
              (1984, 1600, 64): "128x128", (320, 448, 128): "64x128"}


@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("mnk", LONE_TILES)
def test_gemm_lone_launch_tiles(mnk, a_t, b_t):
    """fp32 output, so the tolerance is that of fp32 sums of up to 576 products
    of bf16 values (2e-5 of the largest, as for every tile shape below)."""
    torch = need_gpu()
    M, N, K = mnk
    print(f"[gemm lone] a_t={a_t} b_t={b_t} {mnk}", flush=True)
    a_p, a = _rand((K, M) if a_t else (M, K), "bf16", 25)
    b_p, b = _rand((K, N) if b_t else (N, K), "bf16", 26)
    ref = (a.T if a_t else a) @ (b if b_t else b.T)
    c32 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    B.gemm(_dev(a_p), _dev(b_p), c32, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_F32, dtype=B.BF16)
    torch.cuda.synchronize()
    assert rel_err(c32.cpu().numpy(), ref) < 2e-5


# bf16: the automatic tile choice, the forced shapes the stage's choice can make
# (7, 8 and 10: 256x256, 256x128 and 256x192) and 9 (128x192 on four waves, by
# override only); fp32 has one kernel at this size.  The shapes that only the choice
# itself reaches are in the test after it.
EPI_CASES = [("bf16", 0), ("bf16", 7), ("bf16", 8), ("bf16", 9), ("bf16", 10), ("fp32", 0)]


@pytest.mark.parametrize("dtype,tile", EPI_CASES)
def test_gemm_epilogues(dtype, tile):
    torch = need_gpu()
    print(f"[gemm epilogues] {dtype} tile {tile}", flush=True)
    prev = B.gemm_tile_override(tile)
    try:
        _gemm_epilogues(torch, dtype)
    finally:
        B.gemm_tile_override(prev)


@pytest.mark.parametrize("mnk", [k for k in LONE_TILES if k[2] > 128])
def test_gemm_epilogues_lone_launch(mnk):
    """Every fused epilogue on each tile that only a lone launch's choice reaches
    (the stage's narrow launches take the 128x128 one too), GeLU' also with the
    weight read in place, as the input gradient does."""
    torch = need_gpu()
    print(f"[gemm epilogues] lone launch {mnk}: {LONE_TILES[mnk]}", flush=True)
    _gemm_epilogues(torch, "bf16", mnk)


def _gemm_epilogues(torch, dtype, mnk=(320, 448, 192)):
    M, N, K = mnk
    a_p, a = _rand((M, K), dtype, 3)
    w_p, w = _rand((N, K), dtype, 4, std=0.1)
    bias_p, bias = _rand((N,), dtype, 5, std=0.5)
    res_p, res = _rand((M, N), dtype, 6)
    acc = a @ w.T
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tol = 1e-2 if dtype == "bf16" else 1e-5
    A, W, Bi, R = _dev(a_p), _dev(w_p), _dev(bias_p), _dev(res_p)
    c = torch.empty((M, N), dtype=tdt, device="cuda")
    aux = torch.empty((M, N), dtype=tdt, device="cuda")
    B.gemm(A, W, c, M, N, K, epilogue=B.EPI_BIAS, bias=Bi)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(c), acc + bias) < tol
    B.gemm(A, W, c, M, N, K, epilogue=B.EPI_BIAS_GELU, bias=Bi, aux=aux)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(aux), acc + bias) < tol
    assert rel_err(B.to_host_f64(c), oracle.gelu(acc + bias)) < tol
    B.gemm(A, W, c, M, N, K, epilogue=B.EPI_BIAS_RESID, bias=Bi, resid=R, aux=aux)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(aux), acc) < tol
    assert rel_err(B.to_host_f64(c), res + acc + bias) < tol
    B.gemm(A, W, c, M, N, K, epilogue=B.EPI_BIAS_RESID, bias=Bi, resid=R, aux=None)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(c), res + acc + bias) < tol
    u_p, u = _rand((M, N), dtype, 7, std=2.0)
    U = _dev(u_p)
    B.gemm(A, W, c, M, N, K, epilogue=B.EPI_GELU_BWD, aux=U)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(c), acc * oracle.gelu_grad(u)) < tol
    B.gemm(A, W.t().contiguous(), c, M, N, K, b_trans=True, epilogue=B.EPI_GELU_BWD, aux=U)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(c), acc * oracle.gelu_grad(u)) < tol


# widths: the smallest (one 8-wide chunk, one active lane), ragged chunk counts,
# the workloads' widths and the largest the kernels take (8192)
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("h", [8, 256, 520, 1600, 3072, 6144, 8192])
def test_layernorm_fwd_bwd(dtype, h):
    torch = need_gpu()
    print(f"[layernorm] {dtype} h={h}", flush=True)
    rows = 203  # a partial workgroup of rows and a partial 64-row reduction segment
    x_p, x = _rand((rows, h), dtype, 8, std=2.0, mean=0.5)
    g_p, g = _rand((h,), dtype, 9, std=0.1, mean=1.0)
    b_p, b = _rand((h,), dtype, 10, std=0.1)
    do_p, do = _rand((rows, h), dtype, 11)
    dr_p, dr = _rand((rows, h), dtype, 12)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X = _dev(x_p)
    y = torch.empty((rows, h), dtype=tdt, device="cuda")
    mean = torch.empty(rows, dtype=torch.float32, device="cuda")
    rstd = torch.empty(rows, dtype=torch.float32, device="cuda")
    B.layernorm_fwd(X, _dev(g_p), _dev(b_p), y, mean, rstd, eps=1e-5)
    ref, xhat, rs = oracle.layer_norm_forward(x, g, b, 1e-5)
    dx = torch.empty((rows, h), dtype=tdt, device="cuda")
    dg = torch.empty(h, dtype=torch.float32, device="cuda")
    db = torch.empty(h, dtype=torch.float32, device="cuda")
    scratch = torch.empty(2 * B.reduce_scratch_elems(rows, h), dtype=torch.float32, device="cuda")
    B.layernorm_bwd(_dev(do_p), X, mean, rstd, _dev(g_p), _dev(dr_p), dx, dg, db, scratch)
    torch.cuda.synchronize()
    dz, dgr, dbr = oracle.layer_norm_backward(do, xhat, rs, g)
    tol = 1e-2 if dtype == "bf16" else 1e-5
    assert rel_err(B.to_host_f64(y), ref) < tol
    assert rel_err(rstd.cpu().numpy(), rs[:, 0]) < 1e-5
    assert rel_err(B.to_host_f64(dx), dr + dz) < tol
    assert rel_err(dg.cpu().numpy(), dgr) < 1e-4
    assert rel_err(db.cpu().numpy(), dbr) < 1e-5


# one row; one segment of 64 rows and one row more; nine segments (one XCD gets
# two of them) over widths of one, two and three 512-column slices; and the widths
# whose sums keep four and eight rows in flight, with rows left over by either
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,h", [(1, 64), (64, 512), (65, 520), (575, 1344), (83, 4104), (575, 6144), (83, 6152),
                                    (575, 8192)])
def test_layernorm_bwd_one_launch_equals_parts(dtype, rows, h):
    """dx and the parameter sums made in one launch: dx against the oracle, the
    sums within fp32 rounding of the exact sums, and accumulate adds exactly the
    overwritten values."""
    torch = need_gpu()
    print(f"[layernorm bwd] {dtype} {rows}x{h}", flush=True)
    x_p, x = _rand((rows, h), dtype, 41, std=2.0, mean=0.5)
    g_p, g = _rand((h,), dtype, 42, std=0.1, mean=1.0)
    do_p, do = _rand((rows, h), dtype, 43)
    dr_p, dr = _rand((rows, h), dtype, 44)
    _, xhat, rs = oracle.layer_norm_forward(x, g, np.zeros(h), 1e-5)
    dz, dgr, dbr = oracle.layer_norm_backward(do, xhat, rs, g)
    mean = torch.from_numpy(x.mean(1).astype(np.float32)).cuda()
    rstd = torch.from_numpy(rs[:, 0].astype(np.float32)).cuda()
    dx = torch.empty((rows, h), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    dg = torch.full((h,), float("nan"), dtype=torch.float32, device="cuda")
    db = torch.full((h,), float("nan"), dtype=torch.float32, device="cuda")
    scratch = torch.full((2 * B.reduce_scratch_elems(rows, h),), float("nan"), dtype=torch.float32, device="cuda")
    args = (_dev(do_p), _dev(x_p), mean, rstd, _dev(g_p), _dev(dr_p), dx, dg, db, scratch)
    B.layernorm_bwd(*args)
    torch.cuda.synchronize()
    assert rel_err(B.to_host_f64(dx), dr + dz) < (1e-2 if dtype == "bf16" else 1e-5)
    assert rel_err(dg.cpu().numpy(), dgr) < 1e-4 and rel_err(db.cpu().numpy(), dbr) < 1e-5
    dg1, db1 = dg.clone(), db.clone()
    B.layernorm_bwd(*args, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(dg, dg1 + dg1) and torch.equal(db, db1 + db1)


# one row of one 8-column chunk, a ragged column count over a partial
# reduction segment, and a width past one workgroup's 512 columns
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,cols", [(1, 8), (1000, 776), (8192, 3072)])
def test_column_sum(dtype, rows, cols):
    torch = need_gpu()
    print(f"[column sum] {dtype} {rows}x{cols}", flush=True)
    x_p, x = _rand((rows, cols), dtype, 13)
    out = torch.empty(cols, dtype=torch.float32, device="cuda")
    scratch = torch.empty(B.reduce_scratch_elems(rows, cols), dtype=torch.float32, device="cuda")
    B.column_sum(_dev(x_p), out, scratch)
    B.column_sum(_dev(x_p), out, scratch, accumulate=True)
    torch.cuda.synchronize()
    assert rel_err(out.cpu().numpy(), 2 * x.sum(0)) < 1e-5


ATTN_CASES = [(dt, d, s, 2, 3) for dt in ("bf16", "fp32") for d in (64, 96, 128) for s in (128, 320)]
ATTN_CASES += [("bf16", 128, 2048, 1, 2), ("bf16", 96, 1024, 2, 2)]  # full-length rows of the workloads
ATTN_CASES += [("bf16", d, 64, 2, 3) for d in (64, 96, 128)]  # one block: the pair's second half is empty
ATTN_CASES += [("fp32", d, 64, 2, 3) for d in (64, 96, 128)]  # two tiles: two of the four waves have none


@pytest.mark.parametrize("dtype,d,seq,batch,heads", ATTN_CASES)
def test_attention_fwd_bwd(dtype, d, seq, batch, heads):
    torch = need_gpu()
    print(f"[attention] {dtype} d={d} seq={seq}", flush=True)
    qkv_p, qkv = _rand((batch, seq, 3, heads, d), dtype, 14 + d + seq)
    do_p, do = _rand((batch, seq, heads, d), dtype, 15 + d + seq)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    QKV = _dev(qkv_p)
    o = torch.empty((batch, seq, heads, d), dtype=tdt, device="cuda")
    lse = torch.empty((batch, heads, seq), dtype=torch.float32, device="cuda")
    B.attention_fwd(QKV, o, lse, batch, seq, heads, d)
    dqkv = torch.empty_like(QKV)
    delta = torch.empty((batch, heads, seq), dtype=torch.float32, device="cuda")
    B.attention_bwd(QKV, o, lse, _dev(do_p), dqkv, delta, batch, seq, heads, d)
    torch.cuda.synchronize()
    q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
    O, P = oracle.causal_attention_forward(q, k, v)
    S = np.einsum("bihd,bjhd->bhij", q, k) / np.sqrt(d)
    S = np.where(np.triu(np.ones((seq, seq), bool), 1), -np.inf, S)
    m = S.max(-1, keepdims=True)
    lse_ref = (m + np.log(np.exp(S - m).sum(-1, keepdims=True)))[..., 0]
    tol = 2e-2 if dtype == "bf16" else 1e-5
    assert rel_err(B.to_host_f64(o), O) < tol
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) < (2e-2 if dtype == "bf16" else 1e-5)
    # backward against the oracle with the GPU's own (rounded) forward output
    dq, dk, dv = oracle.causal_attention_backward(do, q, k, v, P)
    g = B.to_host_f64(dqkv)
    assert rel_err(g[:, :, 0], dq) < tol
    assert rel_err(g[:, :, 1], dk) < tol
    assert rel_err(g[:, :, 2], dv) < tol


# (d, seq, batch, heads): pairs of (sequence, head) below, at and above the eight
# XCDs' share, with and without leftovers; a grid beyond one resident round; and
# (the last two) more pairs per XCD than one chunk of the workgroup order holds.
@pytest.mark.parametrize("d,seq,batch,heads", [(64, 64, 1, 1), (96, 192, 2, 4), (64, 320, 2, 5), (128, 128, 3, 11),
                                               (96, 1024, 5, 11), (128, 1024, 4, 12)])
def test_attention_workgroup_order(d, seq, batch, heads):
    """Every (sequence, head) pair of a large launch equals, bit for bit, the
    same pair launched alone: the workgroup order covers each row block of each
    pair exactly once, and no result depends on it."""
    torch = need_gpu()
    print(f"[attention order] d={d} seq={seq} batch={batch} heads={heads}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(31 + d + seq)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    qkv, do = rnd(batch, seq, 3, heads, d), rnd(batch, seq, heads, d)

    def run(q, g_o, b, h):
        o = torch.empty((b, seq, h, d), dtype=torch.bfloat16, device="cuda")
        lse = torch.empty((b, h, seq), dtype=torch.float32, device="cuda")
        delta, dq = torch.empty_like(lse), torch.empty_like(q)
        B.attention_fwd(q, o, lse, b, seq, h, d)
        B.attention_bwd(q, o, lse, g_o, dq, delta, b, seq, h, d)
        return o, lse, dq

    o, lse, dqkv = run(qkv, do, batch, heads)
    for b in range(batch):
        for h in range(heads):
            o1, l1, d1 = run(qkv[b:b + 1, :, :, h:h + 1].contiguous(), do[b:b + 1, :, h:h + 1].contiguous(), 1, 1)
            assert torch.equal(o[b, :, h], o1[0, :, 0]) and torch.equal(lse[b, h], l1[0, 0])
            assert torch.equal(dqkv[b, :, :, h], d1[0, :, :, 0])


@pytest.mark.parametrize("cfg", list(range(1, 11)))
@pytest.mark.parametrize("a_t,b_t", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("K", [64, 192, 320])
def test_gemm_every_tile_shape(cfg, a_t, b_t, K):
    """Each tile shape of the bf16 kernel on a ragged problem (M, N not
    multiples of 128 or 256), fp32 output so the check is tight.  K spans 1,
    3 or 5 stages of 64: fewer stages than the LDS ring holds, as many as a
    3-stage ring, and more, so that every path of the load schedule (loads
    issued in the prologue only, split over the two sub-steps after a
    barrier, none for the last stages) runs."""
    torch = need_gpu()
    M, N = 320, 448
    print(f"[gemm tile {cfg}] a_t={a_t} b_t={b_t} K={K}", flush=True)
    a_p, a = _rand((K, M) if a_t else (M, K), "bf16", 21)
    b_p, b = _rand((K, N) if b_t else (N, K), "bf16", 22)
    ref = (a.T if a_t else a) @ (b if b_t else b.T)
    c32 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    prev = B.gemm_tile_override(cfg)
    try:
        B.gemm(_dev(a_p), _dev(b_p), c32, M, N, K, a_trans=a_t, b_trans=b_t, epilogue=B.EPI_F32, dtype=B.BF16)
        torch.cuda.synchronize()
    finally:
        B.gemm_tile_override(prev)
    assert rel_err(c32.cpu().numpy(), ref) < 2e-5


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("n", [0, 5, 4099, (1 << 20) + 7])
def test_count_nonfinite(dtype, n):
    """NaN and +-Inf planted at seeded positions (the ragged tail included),
    beside the largest finite values and subnormals, are counted exactly."""
    torch = need_gpu()
    print(f"[nonfinite] {dtype} n={n}", flush=True)
    rng = np.random.default_rng(90 + n)
    v = rng.standard_normal(n).astype(np.float32)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    big = float(torch.finfo(tdt).max)
    tiny = float(torch.finfo(tdt).tiny) / 4  # subnormal
    if n:
        idx = rng.choice(n, size=min(n, 37), replace=False)
        kinds = [np.nan, np.inf, -np.inf, big, -big, tiny]
        for j, i in enumerate(idx):
            v[i] = kinds[j % len(kinds)]
        v[n - 1] = np.nan  # the last element sits in the tail for most n
    x = torch.from_numpy(v).to(tdt).to("cuda")
    expect = int((~torch.isfinite(x.cpu().float())).sum().item())
    count = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    B.count_nonfinite(x, count)
    torch.cuda.synchronize()
    assert int(count.item()) == expect
    # a second call overwrites the count rather than adding to it
    B.count_nonfinite(x, count)
    torch.cuda.synchronize()
    assert int(count.item()) == expect
