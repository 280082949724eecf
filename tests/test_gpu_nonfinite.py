"""Non-finite values in attention stay where causality lets them: a token's NaN or
infinity reaches no other row than those that attend to it (or that it attends to).
Rows beyond its reach keep the bits of the clean call."""
import pytest

from paper_2206_04959_amd import binding as B
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

SEQ, HEADS = 192, 2


def _call(torch, d, dtype, seed=51):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + d)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dtype)  # noqa: E731
    qkv, do = rnd(1, SEQ, 3, HEADS, d), rnd(1, SEQ, HEADS, d)
    o = torch.empty((1, SEQ, HEADS, d), dtype=dtype, device="cuda")
    lse = torch.empty((1, HEADS, SEQ), dtype=torch.float32, device="cuda")
    B.attention_fwd(qkv, o, lse, 1, SEQ, HEADS, d)
    torch.cuda.synchronize()
    return qkv, do, o, lse


def _backward(torch, d, qkv, do, o, lse):
    dqkv, delta = torch.empty_like(qkv), torch.empty_like(lse)
    B.attention_bwd(qkv, o, lse, do, dqkv, delta, 1, SEQ, HEADS, d)
    torch.cuda.synchronize()
    return dqkv[0, :, 0], dqkv[0, :, 1], dqkv[0, :, 2]


# a row in the middle of a 32-row tile, and the first and last of a 64-row block
@pytest.mark.parametrize("row", [74, 64, 127])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_row_statistic_nan_reaches_no_masked_key(d, dtype, row):
    """A query whose stored log-sum-exp is NaN: the keys after it are masked for
    it, so their gradients and every other query's are those of the clean call."""
    torch = need_gpu()
    print(f"[non-finite] lse {dtype} d={d} row={row}", flush=True)
    qkv, do, o, lse = _call(torch, d, torch.bfloat16 if dtype == "bf16" else torch.float32)
    dq, dk, dv = _backward(torch, d, qkv, do, o, lse)
    for bad in (float("nan"), -float("inf")):
        lse_bad = lse.clone()
        lse_bad[0, :, row] = bad
        nq, nk, nv = _backward(torch, d, qkv, do, o, lse_bad)
        assert torch.equal(nv[row + 1:], dv[row + 1:]) and torch.equal(nk[row + 1:], dk[row + 1:])
        assert torch.equal(nq[:row], dq[:row]) and torch.equal(nq[row + 1:], dq[row + 1:])
        assert not torch.isfinite(nq[row]).any() and not torch.isfinite(nv[row]).any()


def _close(got, want):
    """fp32 sums of up to 192 terms in another order, as for the finite cases of
    test_gpu_kernels.py; a NaN fails."""
    return bool((got - want).abs().max() <= 1e-5 * want.abs().max())


# a row in the middle of a 32-row tile, the first and the last of one
@pytest.mark.parametrize("bad", ["nan", "inf"])
@pytest.mark.parametrize("row", [74, 64, 95])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_fp32_token_reaches_only_rows_that_see_it(d, row, bad):
    """fp32: one non-finite element in a token's q, k, v or dO.  The rows before the
    token (for the gradients of k and v: after it) are those of the clean call."""
    torch = need_gpu()
    print(f"[non-finite] fp32 token d={d} row={row} {bad}", flush=True)
    qkv, do, o, lse = _call(torch, d, torch.float32)
    dq, dk, dv = _backward(torch, d, qkv, do, o, lse)
    for which in range(3):
        poisoned = qkv.clone()
        poisoned[0, row, which, :, d // 3] = float(bad)
        o1, lse1 = torch.empty_like(o), torch.empty_like(lse)
        B.attention_fwd(poisoned, o1, lse1, 1, SEQ, HEADS, d)
        torch.cuda.synchronize()
        assert _close(o1[0, :row], o[0, :row]) and torch.equal(lse1[0, :, :row], lse[0, :, :row])
        sees = torch.isfinite(o1[0, row:]).all(-1).all(-1)
        if bad == "nan" or which == 2:  # (an infinite score can also be a weight of exactly 0)
            assert not sees[0] and (which == 0 or not sees.any())
        if which == 2:  # a value: one column only
            keep = [c for c in range(d) if c != d // 3]
            assert torch.equal(o1[..., keep], o[..., keep])
        nq, nk, nv = _backward(torch, d, poisoned, do, o, lse)
        assert _close(nq[:row], dq[:row])
        assert _close(nk[row + 1:], dk[row + 1:]) and _close(nv[row + 1:], dv[row + 1:])
        if which == 0:  # a query: only its own dq, and dk and dv of the keys up to it
            assert _close(nq[row + 1:], dq[row + 1:]) and not torch.isfinite(nk[: row + 1]).all()
        else:  # a key or value: only its own dk and dv, and dq of the queries from it on
            assert _close(nk[:row], dk[:row]) and _close(nv[:row], dv[:row])
            assert not torch.isfinite(nq[row:]).all()
    bad_do = do.clone()
    bad_do[0, row, :, d // 3] = float(bad)
    nq, nk, nv = _backward(torch, d, qkv, bad_do, o, lse)
    assert _close(nq[:row], dq[:row]) and _close(nq[row + 1:], dq[row + 1:])
    assert _close(nk[row + 1:], dk[row + 1:]) and _close(nv[row + 1:], dv[row + 1:])
    assert not torch.isfinite(nv[: row + 1, :, d // 3]).any()
