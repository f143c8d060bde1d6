"""The vocabulary scans over rows that start at any element: vocabularies
around whole 16-byte chunks and load rounds, first rows 0 to 16 bytes past an
aligned address, and the largest logits at the rows' two ends, where the
elements outside the chunks lie.  Against the oracle: argmaxes and top-W
tokens bit for bit; log-probabilities within 1e-5 (their sums are at most a
few thousand fp32 terms, each a few ulp off, so 1e-6 in the logarithm)."""
import numpy as np
import pytest
import torch

import oracle
from oracle.tree_accept_sampled import tree_accept_sampled as oracle_sampled
from paper_2606_18394_amd import synth
from helpers import dev_i32

pytestmark = pytest.mark.gpu

# below one chunk, around one chunk, around 256 and 512 chunks of both
# dtypes, and around one whole load round of a split (2048 chunks)
VOCABS = [1, 3, 7, 8, 9, 15, 17, 1023, 2047, 2049, 4095, 4097, 8191, 8195, 16383, 16391]


def _rows(rng, B, N, V, dtype, offset):
    """Logits [B, N, V] whose storage starts `offset` elements past an
    allocation, with each row's maximum at its first or last element (equal
    there in every third row); device tensor and fp64 values."""
    x = rng.standard_normal((B, N, V), dtype=np.float32) * 2
    x[:, 0::3, 0] = x[:, 0::3, -1] = 9.0
    x[:, 1::3, -1] = 9.5
    x[:, 2::3, 0] = 9.25
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    flat = torch.empty(B * N * V + offset, dtype=td, device="cuda")
    lg = flat[offset:].view(B, N, V)
    lg.copy_(torch.from_numpy(x))
    return lg, lg.double().cpu().numpy()


@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_from_any_element(dtype, offset):
    from paper_2606_18394_amd import draft_topw, tree_accept, tree_accept_sampled
    B, N = 2, 5
    par = np.tile(np.array([-1, 0, 0, 1, 3], np.int32), (B, 1))
    for V in VOCABS:
        print(f"V={V} {dtype} offset={offset}", flush=True)
        rng = np.random.default_rng(V)
        lg, ref = _rows(rng, B, N, V, dtype, offset)
        tgt = oracle.target_argmax(ref)
        tok = synth.draft_tokens(par, tgt, rng.random((B, N)) < 0.7,
                                 rng.integers(0, V, (B, N)).astype(np.int32))
        got = [t.cpu().numpy() for t in tree_accept(lg, dev_i32(tok), dev_i32(par), N)]
        for g, r in zip(got, oracle.tree_accept(ref, tok, par, N)):
            np.testing.assert_array_equal(g, r, err_msg=f"V={V}")

        W = min(V, 4)
        t, lp = (y.cpu().numpy() for y in draft_topw(lg, W))
        rt, rlp = oracle.draft_topw(ref, W)
        np.testing.assert_array_equal(t, rt, err_msg=f"V={V}")
        assert np.abs(lp - rlp).max() <= 1e-5, V

        u = rng.random((B, N), dtype=np.float32)
        for _ in range(20):
            res = oracle_sampled(ref, tok, par, u.astype(np.float64), 7, 1.0, N, detail=True)
            close = res[3]["margin"] < 1e-4
            if not close.any():
                break
            u[close] = rng.random(int(close.sum()), dtype=np.float32)
        ln, path, corr = (y.cpu().numpy() for y in tree_accept_sampled(
            lg, dev_i32(tok), dev_i32(par), torch.from_numpy(u).cuda(), 7, 1.0, N))
        np.testing.assert_array_equal(ln, res[0], err_msg=f"V={V}")
        np.testing.assert_array_equal(path, res[1], err_msg=f"V={V}")
        for b in range(B):
            if res[3]["gap"][b] >= 1e-3:
                assert corr[b] == res[2][b], (V, b)


@pytest.mark.parametrize("shape", [
    # (B, Nd, V, dtype): 3, 5 and 8 (6, 10 and 16) loads per thread in one
    # round, then several rounds
    (1, 3, 90000, "bf16"), (2, 4, 151937, "bf16"), (1, 2, 262140, "bf16"), (1, 2, 262200, "bf16"),
    (1, 3, 90001, "f32"), (2, 4, 151937, "f32"), (1, 2, 262143, "f32"), (1, 2, 300003, "f32"),
    (40, 16, 16391, "bf16"), (40, 16, 32800, "f32"),
])
def test_topw_rounds(shape):
    from paper_2606_18394_amd import draft_topw
    B, Nd, V, dtype = shape
    print(shape, flush=True)
    lg, ref = _rows(np.random.default_rng(V), B, Nd, V, dtype, 0)
    t, lp = (y.cpu().numpy() for y in draft_topw(lg, 8))
    rt, rlp = oracle.draft_topw(ref, 8)
    np.testing.assert_array_equal(t, rt)
    assert np.abs(lp - rlp).max() <= 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_topw_less_workspace(dtype):
    """2048 rows: the query asks for the splits of the plan; half of that, one
    split per row, is enough for the same result, and less is refused."""
    from paper_2606_18394_amd import draft_topw
    from paper_2606_18394_amd.binding import load_library
    B, Nd, V, W = 32, 64, 16640, 4
    print(dtype, flush=True)
    x = torch.randn(B, Nd, V, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    x = x if dtype == "f32" else x.to(torch.bfloat16)
    v, i = torch.sort(x.double(), dim=-1, descending=True, stable=True)
    ref = v[..., :W] - torch.logsumexp(v, -1, keepdim=True)
    need, least = load_library().tv_draft_topw_workspace(B, Nd, V), B * Nd * 136
    assert need >= 2 * least
    for size in (least, 2 * least - 1, need):
        tok, lp = draft_topw(x, W, workspace_tensor=torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert torch.equal(tok.long(), i[..., :W])
        assert (lp.double() - ref).abs().max().item() <= 1e-5
    with pytest.raises(RuntimeError, match="WORKSPACE"):
        draft_topw(x, W, workspace_tensor=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
