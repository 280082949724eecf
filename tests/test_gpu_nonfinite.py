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
