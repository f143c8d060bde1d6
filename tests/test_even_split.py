"""The even split of a batch into chunks of one size, which the kernels find
from the kv_lens: its work order on the host, and parity on the GPU where the
lengths leave sequences of no, one and many chunks."""
import itertools
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2606_18394_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_work_order(tmp_path):
    exe = tmp_path / "even_check"
    subprocess.run(["g++", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2606_18394_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "even_check.cpp"), "-o", str(exe)],
                   check=True)
    lines = [f"{c} {s} {rb} {h}" for s, rb, h in itertools.product(
        [1, 2, 7, 8, 42, 64], [1, 2, 3, 32], [1, 2, 3, 8, 12]) for c in sorted({1, s // 2 + 1, s})]
    res = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[-500:]


LENGTHS = {
    "empty": lambda B, L: [0] * B,
    "short": lambda B, L: [5] * B,                                    # far below the capacity
    "full": lambda B, L: [L] * B,
    "one long": lambda B, L: [L] + [0] * (B - 1),
    "last long": lambda B, L: [33] * (B - 1) + [L - 1],
    "spread": lambda B, L: [(i * 977 + 31) % (L + 1) for i in range(B)],
}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", sorted(LENGTHS))
@pytest.mark.parametrize("shape", [
    # (B, N, Hq, Hkv, D, capacity): one sequence; few; a lane for each; several
    # to a lane (4, above 256 16), the last lanes with fewer or none
    (1, 33, 8, 2, 128, 3000), (1, 200, 8, 1, 64, 4000), (2, 40, 4, 2, 128, 2500),
    (5, 70, 12, 3, 64, 1500), (16, 9, 8, 4, 128, 1200), (64, 3, 4, 2, 64, 700),
    (65, 3, 4, 2, 64, 700), (130, 2, 4, 1, 128, 900), (255, 1, 2, 1, 64, 500), (257, 1, 1, 1, 64, 700),
    (600, 1, 1, 1, 64, 500),
])
def test_lengths(shape, kind):
    """Max-abs error at most 1.5e-2: rounding the softmax weights and the
    output to bf16 costs up to 2^-9 of |out| each, and a row of few visible
    keys has outputs up to about 3.5 here (2^-8 * 3.5 = 1.4e-2).  The padded,
    the paged and the tree-tail call agree where they hold the same keys, and
    one workspace serves them all."""
    import torch
    from helpers import dev_bf16, dev_i32, oracle_attention
    from paper_2606_18394_amd import tree_verify_attention, tree_verify_attention_paged
    B, N, Hq, Hkv, D, L = shape
    rng = np.random.default_rng(B * 1000 + N)
    trees = np.stack([synth.random_tree(rng, N, depth=9, branching=4) for _ in range(B)])
    inp = synth.make_inputs(rng, B=B, N=N, Hq=Hq, Hkv=Hkv, D=D, Lmax=L, V=8, trees=trees,
                            kv_len=np.array(LENGTHS[kind](B, L)), with_logits=False)
    print(f"{shape} {kind}", flush=True)
    ref = oracle_attention(inp)
    q, kt, vt = (dev_bf16(inp[k]) for k in ("q", "k_tree", "v_tree"))
    par, kvl = dev_i32(inp["parent"]), dev_i32(inp["kv_len"])
    out = torch.empty_like(q)
    tree_verify_attention(q, dev_bf16(inp["k_cache"]), dev_bf16(inp["v_cache"]), kt, vt, par, out,
                          kv_len=kvl)
    padded = out.float().cpu().numpy()
    assert np.abs(padded - ref).max() <= 1.5e-2
    # the tree's rows behind the context of a larger cache
    cap = L + N
    tail = {}
    for c, t in (("k_cache", "k_tree"), ("v_cache", "v_tree")):
        a = np.zeros((B, cap, Hkv, D), np.uint16)
        a[:, :L] = inp[c]
        for b in range(B):
            n = int(inp["kv_len"][b])
            a[b, n:n + N] = inp[t][b]
        tail[c] = a
    tree_verify_attention(q, dev_bf16(tail["k_cache"]), dev_bf16(tail["v_cache"]), None, None, par,
                          out, kv_len=kvl)
    assert np.abs(out.float().cpu().numpy() - ref).max() <= 1.5e-2
    # pages of 32 rows
    per = -(-cap // 32)
    bt, nb = synth.block_table(rng, B, per, spare=2)
    pools = [synth.scatter_pool(rng, np.pad(tail[c], ((0, 0), (0, per * 32 - cap), (0, 0), (0, 0))),
                                bt, nb, 32) for c in ("k_cache", "v_cache")]
    tree_verify_attention_paged(q, dev_bf16(pools[0]), dev_bf16(pools[1]), dev_i32(bt), None, None,
                                par, out, kv_len=kvl)
    torch.cuda.synchronize()
    assert np.abs(out.float().cpu().numpy() - ref).max() <= 1.5e-2


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [
    # (B, N, Hq, Hkv, D, rows): 1 to 16 rows per KV head, merged by the last chunk
    # and by a second kernel
    (1, 1, 2, 2, 128, 4000), (1, 4, 4, 1, 64, 3000), (1, 2, 64, 8, 128, 30000), (2, 1, 1, 1, 128, 9000),
])
def test_partials_hold_the_rows_only(shape):
    """At most 16 rows per KV head, in row blocks of at least 32: no more than
    half of the workspace's partials are written."""
    import torch
    from paper_2606_18394_amd import tree_verify_attention
    from paper_2606_18394_amd.binding import load_library
    B, N, Hq, Hkv, D, L = shape
    print(shape, flush=True)
    g = torch.Generator(device="cuda").manual_seed(N)

    def normal(*s):
        return torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    q, kc, vc = normal(B, N, Hq, D), normal(B, L, Hkv, D), normal(B, L, Hkv, D)
    kt, vt = normal(B, N, Hkv, D), normal(B, N, Hkv, D)
    par = torch.arange(-1, N - 1, dtype=torch.int32, device="cuda").repeat(B, 1)
    need = load_library().tv_tree_verify_attention_workspace(B, N, Hq, Hkv, D, L)
    assert need > 32768, "the plan does not split"
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    ws[:32768] = 0
    tree_verify_attention(q, kc, vc, kt, vt, par, torch.empty_like(q), workspace_tensor=ws)
    torch.cuda.synchronize()
    written = int((ws[32768:] != 0xA5).sum())
    print(f"{written} of {need - 32768} bytes", flush=True)
    assert 0 < written <= (need - 32768) // 2


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [
    # (B, N, Hq, Hkv, D, rows): the fixed split's plan needs no workspace (one, several
    # and more than 64 sequences, longest first), then less than the even split's (a
    # lane of chunks per XCD of 1, 2, 4 and 8, and none)
    (1, 39, 3, 3, 128, 353), (2, 2, 16, 4, 128, 437), (35, 8, 16, 8, 64, 790),
    (174, 6, 3, 3, 128, 168), (2, 6, 16, 8, 128, 459), (2, 14, 4, 4, 128, 458),
    (8, 3, 8, 2, 64, 2097), (2, 3, 8, 1, 64, 4165), (1, 18, 3, 3, 64, 5465), (3, 9, 2, 1, 64, 2655),
    # both ask for more than a smaller split, or none, once needed
    (22, 4, 64, 8, 128, 975), (77, 5, 4, 1, 128, 951), (65, 9, 4, 1, 64, 3000),
])
def test_less_workspace(shape):
    """A call with less workspace than the query says is computed: with the fixed
    split where that fits, else with what fits.  Refused are only sizes that hold
    no split, where the fixed split needs one and the batch is not above 64."""
    import torch
    from helpers import dev_bf16, dev_i32, oracle_attention
    from paper_2606_18394_amd import tree_verify_attention
    from paper_2606_18394_amd.binding import load_library
    B, N, Hq, Hkv, D, L = shape
    rng = np.random.default_rng(B * 100 + L)
    trees = np.stack([synth.random_tree(rng, N, depth=min(N - 1, 9), branching=4) for _ in range(B)])
    inp = synth.make_inputs(rng, B=B, N=N, Hq=Hq, Hkv=Hkv, D=D, Lmax=L, V=8, trees=trees,
                            kv_len=np.array([L - (i * 61) % (L + 1) for i in range(B)]),
                            with_logits=False)
    print(shape, flush=True)
    ref = oracle_attention(inp)
    q, kc, vc, kt, vt = (dev_bf16(inp[k]) for k in ("q", "k_cache", "v_cache", "k_tree", "v_tree"))
    par, kvl = dev_i32(inp["parent"]), dev_i32(inp["kv_len"])
    need = load_library().tv_tree_verify_attention_workspace(B, N, Hq, Hkv, D, L)
    full = torch.zeros(need, dtype=torch.uint8, device="cuda")

    def call(size):
        out = torch.zeros_like(q)
        try:
            tree_verify_attention(q, kc, vc, kt, vt, par, out, kv_len=kvl, workspace_tensor=full[:size])
        except RuntimeError as e:
            assert "WORKSPACE" in str(e)
            return None
        torch.cuda.synchronize()
        return out.float().cpu().numpy()
    lo, hi = -1, need  # the smallest size that is accepted
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if call(mid) is None:
            lo = mid
        else:
            hi = mid
    print(f"{hi} of {need} bytes", flush=True)
    assert need > 32768 and hi == 0 if B > 64 else hi in (0, 32768)
    for size in (hi, hi, (32768 + need) // 2, need - 1, need):
        assert np.abs(call(size) - ref).max() <= 1.5e-2
        assert not full[:32768].any(), "sync words left non-zero"
