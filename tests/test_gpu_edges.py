"""GPU parity at the sizes where a launch changes its shape: edges of tiles, remainders, the lines of the
dispatch rules.  Same oracle, same tolerances as test_gpu_parity.py."""

import numpy as np
import pytest

from oracle import ppmoe_oracle as O
from paper_2304_11414_amd import binding as B
from paper_2304_11414_amd import synth
from tests.gpu_util import GRAD_ELEM_FACTOR, TOL, DeviceLayer, assert_close, to_np, torch_dtype
from tests.test_gpu_parity import check_dispatch, compare_layer_full, ragged_offsets, small_cfg
from tests.test_gpu_parity import test_expert_ffn_on_oracle_rows as check_ffn
from tests.test_gpu_parity import test_gate_router as check_router

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------- permutation and balance loss

@pytest.mark.parametrize("kw", [
    dict(T=64 * 4096, E=8, top_k=1),                                # 4096 segments: the last the placing kernel scans
    dict(T=64 * 4096 + 1, E=8, top_k=1, capacity_factor=1.0),       # one more: the scan is a launch of its own
    dict(T=64 * 15 + 1, E=17, top_k=1),                             # 16 segments = one block; two rounds of experts
    dict(T=64 * 16 + 1, E=33, top_k=1, local_begin=1, local_count=32),   # one more block; the most experts it scans
    dict(T=64 * 16 + 1, E=33, top_k=2),                             # one expert more: the scan is a launch of its own
    dict(T=32769, E=130, top_k=2, local_begin=1, local_count=129),
])
def test_dispatch_at_the_lines_of_the_scan(kw):
    lc = small_cfg(d=64, **kw)
    idx = O.top_k_picks(synth.random_logits(lc.T, lc.E, seed=lc.T), lc.top_k)
    check_dispatch(lc, idx)


@pytest.mark.parametrize("kw", [
    dict(T=3000, d=128, F=128, E=12, top_k=2, renorm_topk=True, seed=61),    # slices of 12 threads, some idle
    dict(T=700, d=128, F=128, E=100, top_k=2, local_begin=20, local_count=10, seed=62),
    dict(T=130, d=128, F=128, E=256, top_k=1, local_begin=0, local_count=16, seed=63),
])
def test_balance_loss_inside_the_layer(kw):
    lc = small_cfg(**kw)
    compare_layer_full(lc, synth.make_inputs(lc))


# ---------------------------------------------------------------- router gradients

@pytest.mark.parametrize("kw", [
    dict(T=1, d=8, F=64, E=1, top_k=1, seed=70),                        # one token, one 16-byte piece of columns
    dict(T=257, d=136, F=128, E=17, top_k=1, seed=71),                  # second group of 16 experts, nine pieces
    dict(T=149, d=1032, F=64, E=33, top_k=8, renorm_topk=True, seed=70),    # as many picks as are allowed
    dict(T=133, d=64, F=64, E=200, top_k=4, local_begin=0, local_count=200, seed=70),   # four rounds of 64 experts
])
def test_router_gradients(kw):
    """dx, dWg and dbias only.  (With two or three rows per expert an element of an expert weight gradient is a
    single product of two factors with heavy tails, which the elementwise bound of a sum over many rows does not
    cover; those products are tested on layers with many rows.)"""
    lc = small_cfg(**kw)
    inp = synth.make_inputs(lc)
    mv = synth.math_views(inp)
    d_out = np.random.default_rng(lc.seed).standard_normal((lc.T, lc.d)).astype(np.float32)
    synth.round_to_bf16(d_out)
    ref = O.layer_backward(inp["x"], mv["Wg"], inp["bias"], mv["W1"], mv["W2"], d_out, E=lc.E, k=lc.top_k,
                           local_begin=lc.local_begin, local_count=lc.n_local,
                           capacity_factor=lc.capacity_factor, renorm=lc.renorm_topk)
    got = DeviceLayer(lc, inp).run_layer_backward(d_out)
    tol = TOL[lc.in_dtype]
    et = GRAD_ELEM_FACTOR * tol
    assert_close(got["dWg"], ref["dWg"].T, tol, "dWg", et)
    assert_close(got["dbias"], ref["dbias"], tol, "dbias", et)
    assert_close(got["dx"], ref["dx"], tol, "dx", et)


# ---------------------------------------------------------------- rows that are not whole k-tiles of 64

@pytest.mark.parametrize("kw", [
    dict(T=300, d=8, F=72, E=2, top_k=1, in_dtype="f16", out_dtype="f16", seed=80),         # one piece, one past a tile
    dict(T=515, d=200, F=824, E=3, top_k=2, renorm_topk=True, seed=81),                     # gathered rows and placed rows
    dict(T=700, d=136, F=1000, E=5, top_k=1, out_dtype="f32", seed=82),                     # cut tiles, packed results
    dict(T=1100, d=1000, F=4000, E=4, top_k=2, local_begin=2, local_count=2, in_dtype="f16", out_dtype="f16", seed=83),
    dict(T=600, d=440, F=1000, E=4, top_k=1, seed=84),                      # the first product on the tile-per-block kernel
    dict(T=600, d=456, F=440, E=4, top_k=2, renorm_topk=True, seed=85),     # the second
])
def test_layer_with_rows_of_no_whole_tiles(kw):
    lc = small_cfg(**kw)
    compare_layer_full(lc, synth.make_inputs(lc))


@pytest.mark.parametrize("dtype,d,F,counts", [
    ("bf16", 456, 3000, [700, 300, 0, 129]),      # 8 k-tiles: the first taken; 47: cut
    ("f16", 1288, 1000, [700]),                   # big tiles in the stream, 21 and 16 k-tiles, dealt out whole
    ("bf16", 1240, 2568, [40, 60, 128, 7]),       # small tiles alone: 20 k-tiles whole, 41 cut
    ("bf16", 1992, 4000, [257] * 6),              # a partial round beside 96 small tiles of 32 k-tiles
    ("f16", 520, 136, [1500, 1000, 30]),          # more tiles than 16-k-tile shares of a short contraction
])
def test_expert_ffn_with_rows_of_no_whole_tiles(dtype, d, F, counts):
    check_ffn(dtype, d, F, counts)


@pytest.mark.parametrize("K", [(1 << 22) + 8, 8421600])   # the first too long for the persistent kernel; 255 K > 2^31
@pytest.mark.parametrize("product,rows,cols", [("up", 33, 256), ("down", 256, 8)])
def test_products_of_very_long_contractions(product, rows, cols, K):
    """256 rows or 256 columns: the last row of a tile starts more than 2^31 elements behind the first.  Reference: float64
    sums over pieces of the contraction (torch)."""
    import torch
    F, d = (cols, K) if product == "up" else (K, cols)
    cfg = B.make_config(rows, d, F, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(9)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    a, w = draw(1.0, rows, K), draw(K ** -0.5, 1, cols, K)
    got = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty((B.moe_ffn_workspace_bytes(cfg),), dtype=torch.uint8, device="cuda")
    run = B.moe_expert_ffn_up if product == "up" else B.moe_expert_ffn_down
    run(cfg, a, torch.tensor([0, rows], dtype=torch.int32, device="cuda"), w, got, ws)
    ref = sum(x.double() @ y.double().t() for x, y in zip(a.split(1 << 18, dim=1), w[0].split(1 << 18, dim=1)))
    if product == "up":
        ref = torch.nn.functional.gelu(ref, approximate="tanh")
    assert_close(to_np(got), to_np(ref), TOL["bf16"], product)


# ---------------------------------------------------------------- few rows

@pytest.mark.parametrize("kw", [
    dict(T=1, d=8, F=8, E=4, top_k=2, renorm_topk=True, seed=90),                       # one row, one 16-byte piece
    dict(T=17, d=1160, F=1024, E=1, top_k=1, seed=91),                                  # 16 rows and one, row ends inside a span
    dict(T=33, d=1024, F=1992, E=2, top_k=2, renorm_topk=True, in_dtype="f16", out_dtype="f16", seed=92),   # 66 rows of 2 experts: too many
    dict(T=128, d=136, F=264, E=8, top_k=1, out_dtype="f32", seed=93),                  # as many rows as are taken
    dict(T=129, d=136, F=264, E=8, top_k=1, seed=94),                                   # one more
    dict(T=32, d=256, F=512, E=16, top_k=4, renorm_topk=True, local_begin=3, local_count=8, seed=95),
    dict(T=64, d=320, F=640, E=8, top_k=2, capacity_factor=0.5, seed=96),               # dropped picks, rows of zeros
    # nearly all rows on one or two experts: rows read and placed through the permutation, more than one pass
    dict(T=64, d=328, F=640, E=8, top_k=2, renorm_topk=True, bias_kind="zipf", bias_s=40.0, seed=97),
    dict(T=128, d=136, F=264, E=8, top_k=1, bias_kind="zipf", bias_s=40.0, in_dtype="f16", out_dtype="f16", seed=98),
    dict(T=64, d=136, F=520, E=9, top_k=2, bias_kind="zipf", bias_s=40.0, local_begin=1, local_count=8, seed=99),
])
def test_layer_on_few_rows(kw):
    lc = small_cfg(**kw)
    compare_layer_full(lc, synth.make_inputs(lc))


def run_ffn_and_see_the_kernel(lc, x, offsets, W1, W2):
    """moe_expert_ffn on device tensors; returns H, y and whether the kernel of the large tiles has worked: its
    blocks lower their hand-over flags (256 words before the other 257 words and 256 bytes that end the workspace)."""
    import torch
    cfg = B.config_from(lc)
    ws = torch.full((B.moe_ffn_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda")
    rows = int(offsets[-1])
    H = torch.empty((rows, lc.F), dtype=x.dtype, device="cuda")
    y = torch.empty((rows, lc.d), dtype=x.dtype, device="cuda")
    B.moe_expert_ffn(cfg, x, torch.from_numpy(offsets).cuda(), W1, W2, H, y, ws)
    assert B.moe_ffn_check(cfg, ws, False) == 0
    flags = ws[-(513 * 4 + 256):][: 256 * 4].view(torch.int32)
    return H, y, bool((flags != -1).any())


@pytest.mark.parametrize("counts,few", [
    ([32], True), ([33], False),
    ([0, 1, 0], True), ([31, 0, 17], True), ([32, 0, 17], False),               # 16 rows per expert, and one more
    ([128, 0, 0, 0, 0, 0, 0, 0], True),                                         # two passes of 64 rows
    ([0, 0, 65, 0, 0, 0, 0, 63], True),
    ([33, 0, 1, 31, 32, 17, 14, 0], True), ([33, 0, 1, 31, 32, 17, 15, 0], False),   # 128 rows, and one more
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_expert_ffn_on_few_rows(dtype, counts, few):
    check_ffn(dtype, 1160, 1032, counts)
    lc = small_cfg(T=sum(counts), d=1160, F=1032, E=len(counts), top_k=1, in_dtype=dtype, out_dtype=dtype, seed=3)
    dl = DeviceLayer(lc, synth.make_inputs(lc, parts=("x", "W1_t", "W2_t")))
    assert run_ffn_and_see_the_kernel(lc, dl.x, ragged_offsets(counts), dl.W1, dl.W2)[2] != few


@pytest.mark.parametrize("counts,few", [
    ([16] * 8, True),
    ([0, 1, 127, 0, 0, 0, 0, 0], True),            # 2^31 / (4096 * 4104) = 127 rows: the most one expert may have
    ([128, 0, 0, 0, 0, 0, 0, 0], False),           # one more
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_few_rows_decided_by_the_counts(dtype, counts, few):
    """Weights so large that an expert with many rows is better off on the large tiles: both kernels are launched,
    one of them leaves.  Reference: the same products in float64 (torch)."""
    import torch
    d, F, n = 4096, 4104, len(counts)
    lc = small_cfg(T=128, d=d, F=F, E=n, top_k=1, in_dtype=dtype, out_dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch_dtype(dtype), device="cuda").normal_(0.0, std, generator=g)
    x, W1, W2 = draw(1.0, 128, d), draw(0.02, n, F, d), draw(0.02, n, d, F)
    offsets = ragged_offsets(counts)
    H, y, large = run_ffn_and_see_the_kernel(lc, x, offsets, W1, W2)
    assert large != few
    for i in range(n):
        rows = slice(int(offsets[i]), int(offsets[i + 1]))
        if counts[i]:
            h_ref = torch.nn.functional.gelu(x[rows].double() @ W1[i].double().t(), approximate="tanh")
            assert_close(to_np(H[rows]), to_np(h_ref), TOL[dtype], "H")
            assert_close(to_np(y[rows]), to_np(H[rows].double() @ W2[i].double().t()), TOL[dtype], "y_sliced")


FIRST_CALL_SETS_UP = """
import sys, torch
from paper_2304_11414_amd import binding as B
T, d, F, E = int(sys.argv[1]), int(sys.argv[2]), int(sys.argv[3]), 4
cfg = B.make_config(T, d, F, E, 1)
x = torch.randn(T, d, device="cuda").bfloat16()
Wg = torch.randn(E, d, device="cuda").bfloat16()
W1 = torch.randn(E, F, d, device="cuda").bfloat16()
W2 = torch.randn(E, d, F, device="cuda").bfloat16()
out = torch.empty_like(x)
ws = torch.empty(B.moe_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
start.record()
torch.cuda._sleep(1000000)
end.record()
torch.cuda.synchronize()
second = int(1000000 * 1000.0 / start.elapsed_time(end))      # cycles of a kernel that runs for a second
waited = []
for call in range(2):
    done = torch.cuda.Event()
    torch.cuda._sleep(second)
    done.record()
    B.moe_layer_forward(cfg, x, Wg, None, W1, W2, out, ws)
    waited.append(done.query())
    torch.cuda.synchronize()
print("WAITED", waited, flush=True)
"""


@pytest.mark.parametrize("T,d,F", [(4, 64, 128), (500, 72, 136)])
def test_first_call_of_a_process_sets_up(T, d, F):
    """Without moe_init the first 16-bit layer call does the set-up and waits for it, also where its products take the
    kernel for few rows or the one for short contractions (a later capture of a large batch relies on it)."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-u", "-c", FIRST_CALL_SETS_UP, str(T), str(d), str(F)], cwd=root,
                       capture_output=True, text=True, timeout=100)
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0 and "WAITED [True, False]" in r.stdout


@pytest.mark.parametrize("counts", [[0, 5, 0], [0, 0, 1], [20, 0, 3]])
def test_clock_of_a_product_on_few_rows(counts):
    """The block whose counters are read back is one with work, also where the first expert has none: it fetches 512 KiB
    of weights, which takes more than a microsecond at any clock."""
    import torch
    lc = small_cfg(T=sum(counts), d=64, F=8192, E=3, top_k=1)
    dl = DeviceLayer(lc, synth.make_inputs(lc, parts=("x", "W1_t", "W2_t")))
    ws = torch.zeros((B.moe_ffn_workspace_bytes(dl.cfg),), dtype=torch.uint8, device="cuda")
    H = torch.empty((sum(counts), lc.F), dtype=dl.x.dtype, device="cuda")
    y = torch.empty_like(dl.x)
    B.moe_expert_ffn(dl.cfg, dl.x, torch.from_numpy(ragged_offsets(counts)).cuda(), dl.W1, dl.W2, H, y, ws)
    ghz, us = B.moe_ffn_clock(dl.cfg, ws, False)
    assert us > 1.0 and 0.1 < ghz < 3.0, (us, ghz)


# ---------------------------------------------------------------- float32 products

@pytest.mark.parametrize("d,F,counts", [
    (8, 40, [1, 0, 33]),                  # one piece per half-wavefront, partial column tile
    (264, 136, [31, 32, 65]),             # contraction past two rounds of the four wavefronts, remainders
    (256, 2048, [1000, 0, 25]),           # split form (F = 2048) beside wide tiles in one layer
    (72, 4104, [513, 64, 63]),            # wide tiles with a partial quarter along rows and columns
])
def test_expert_ffn_in_float32(d, F, counts):
    check_ffn("f32", d, F, counts)


# ---------------------------------------------------------------- router on few tokens

@pytest.mark.parametrize("T,d,E,k,dtype", [
    (1, 8, 16, 1, "bf16"),                # as many experts as stay on the kernel of whole rows
    (1, 8, 17, 1, "bf16"),                # one more: all wavefronts but one without a span
    (1, 8, 64, 2, "f16"),
    (17, 1032, 17, 2, "f16"),             # two blocks, a span past the end of the row
    (16, 4104, 33, 8, "bf16"),            # a second round of spans
    (4096, 136, 64, 1, "bf16"),           # the last size the kernel of few tokens takes
    (4097, 136, 64, 1, "f16"),            # the first of the next
    (4097, 136, 20, 2, "bf16"),
])
def test_router_on_few_tokens(T, d, E, k, dtype):
    check_router(dict(T=T, d=d, F=64, E=E, top_k=k, renorm_topk=k > 1, in_dtype=dtype, out_dtype=dtype, seed=101))


# ---------------------------------------------------------------- many rows on a small layer

def test_weight_gradients_over_more_than_two_to_the_31_elements():
    """One expert with so many rows that its last rows of H and dU start more than 2^31 elements behind the first, on a
    layer so small that the 128 x 128 tiles are taken.  Reference: float64 sums over pieces of the rows (torch)."""
    import torch
    rows, d, F = 524288 + 520, 8, 4096
    cfg = B.make_config(rows, d, F, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(11)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, dY, W1, W2 = draw(1.0, rows, d), draw(1.0, rows, d), draw(0.35, 1, F, d), draw(0.35, 1, d, F)
    dX = torch.empty_like(x)
    dW1, dW2 = (torch.empty(s, dtype=torch.float32, device="cuda") for s in ((1, F, d), (1, d, F)))
    ws = torch.empty((B.moe_ffn_backward_workspace_bytes(cfg),), dtype=torch.uint8, device="cuda")
    B.moe_expert_ffn_backward(cfg, x, torch.tensor([0, rows], dtype=torch.int32, device="cuda"), W1, W2, dY, dX, dW1, dW2, ws)
    w1, w2 = W1[0].double(), W2[0].double()
    ref1, ref2 = torch.zeros_like(w1), torch.zeros_like(w2)
    for xs, dy, dx in zip(x.split(1 << 15), dY.split(1 << 15), dX.split(1 << 15)):
        u = (xs.double() @ w1.t()).requires_grad_()
        h = torch.nn.functional.gelu(u, approximate="tanh")
        (du,) = torch.autograd.grad(h, u, dy.double() @ w2)
        ref1 += du.t() @ xs.double()
        ref2 += dy.double().t() @ h.detach()
    assert_close(to_np(dx), to_np(du @ w1), TOL["bf16"], "dX_sliced", GRAD_ELEM_FACTOR * TOL["bf16"])   # (the last piece)
    assert_close(to_np(dW1[0]), to_np(ref1), TOL["bf16"], "dW1", GRAD_ELEM_FACTOR * TOL["bf16"])
    assert_close(to_np(dW2[0]), to_np(ref2), TOL["bf16"], "dW2", GRAD_ELEM_FACTOR * TOL["bf16"])


def test_gradients_past_2_24_columns():
    """Operands by rows of so many columns that 63 of them pass 2^31 bytes: the persistent kernels' 32-bit offsets do not
    reach the last rows of a k-tile.  Reference: the chain rule in float64, at some of the columns, dX at all."""
    import torch
    T, d, F = 64, 64, 17_200_000
    cfg = B.config_from(small_cfg(T=T, d=d, F=F, E=1, top_k=1))
    g = torch.Generator(device="cuda").manual_seed(24)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, dY, W1, W2 = draw(1.0, T, d), draw(1.0, T, d), draw(0.1, 1, F, d), draw(0.1, 1, d, F)
    dX = torch.empty_like(x)
    dW1, dW2 = torch.empty(W1.shape, device="cuda"), torch.empty(W2.shape, device="cuda")
    ws = torch.empty(B.moe_ffn_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    B.moe_expert_ffn_backward(cfg, x, torch.tensor([0, T], dtype=torch.int32, device="cuda"), W1, W2, dY, dX, dW1, dW2, ws)

    def columns(f):
        u = (x.double() @ W1[0, f].double().t()).requires_grad_()
        h = torch.nn.functional.gelu(u, approximate="tanh")
        (du,) = torch.autograd.grad(h, u, dY.double() @ W2[0, :, f].double())
        return h.detach(), du

    ref = sum(columns(slice(f, f + (1 << 20)))[1] @ W1[0, f:f + (1 << 20)].double() for f in range(0, F, 1 << 20))
    assert_close(to_np(dX), to_np(ref), TOL["bf16"], "dX_sliced", GRAD_ELEM_FACTOR * TOL["bf16"])
    f = torch.cat([torch.arange(512), torch.randint(0, F, (2000,)), torch.arange(F - 512, F)]).cuda()
    h, du = columns(f)
    assert_close(to_np(dW1[0, f]), to_np(du.t() @ x.double()), TOL["bf16"], "dW1", 1.0)   # (elementwise only over many rows)
    assert_close(to_np(dW2[0][:, f]), to_np(dY.double().t() @ h), TOL["bf16"], "dW2", 1.0)


# ---------------------------------------------------------------- data gradient of a rank with some of the experts

@pytest.mark.parametrize("counts", [
    [60, 0, 300, 33],        # an even share and less: the 128 x 128 launch has the rows
    [4000, 60, 0, 36],       # one expert with nearly all: the 256 x 256 launch has them
    [3840, 0, 0, 0],         # 15 row tiles x 8 column tiles: one fewer than would fill half of 256 CUs
    [3841, 0, 0, 0],
])
def test_data_gradient_tiles_follow_the_rows(counts):
    d, F = 2048, 256
    lc = small_cfg(T=4096, d=d, F=F, E=64, top_k=1, local_begin=4, local_count=4, seed=110)
    inp = synth.make_inputs(lc, parts=("x", "W1_t", "W2_t"))
    inp["W1_t"] *= 8.0
    inp["W2_t"] *= 8.0
    mv = synth.math_views(inp)
    A = sum(counts)
    x = inp["x"][:A]
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dY = np.random.default_rng(7).standard_normal((A, d)).astype(np.float32)
    synth.round_to_bf16(dY)
    ref = O.expert_ffn_backward(x, offsets, mv["W1"], mv["W2"], dY)
    dX = DeviceLayer(lc, inp).run_ffn_backward(x, offsets, dY)[0]
    assert_close(dX, ref["dX"], TOL["bf16"], "dX_sliced", GRAD_ELEM_FACTOR * TOL["bf16"])


@pytest.mark.parametrize("counts", [
    [1200, 0, 31, 33],       # dX (8 column tiles, 64 k-tiles) and dH (16, 32) on the 128 x 128 launch: 7 row tiles
    [2000, 0, 31, 33],       # 10 row tiles: dX on the 128 x 128 launch, dH on the 256 x 256 one
    [60, 100, 128, 9],       # dX: mostly empty tiles, 256 x 256 all the same; dH (K = 2048): 128 x 128
    [3840, 0, 0, 0],         # dX: 15 row tiles, the last size on the 128 x 128 launch; dH on 256 x 256
    [4000, 60, 0, 36],       # 18 row tiles, both on 256 x 256; two small tiles
    [8192, 20, 0, 0],        # dX: a round of 256 CUs; the 20 rows are small tiles, one an XCD
    [8192, 0, 200, 0],       # dX: 33 x 8 big tiles: one an XCD behind the round, cut into the stream (64 k-tiles)
    [44, 8000, 0, 300],      # small tiles of 44, 64 and 44 rows beside 32 row tiles
])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_data_gradient_tiles_of_a_long_contraction(dtype, counts):
    """A long contraction on a rank with some of the experts: two launches (256 x 256, 128 x 128) take one decision from
    the row counts, each by itself.  Reference: the chain rule in float64 (torch)."""
    import torch
    d, F, T = 2048, 4096, 8448
    lc = small_cfg(T=T, d=d, F=F, E=64, top_k=1, local_begin=4, local_count=4, in_dtype=dtype, out_dtype=dtype)
    cfg = B.config_from(lc)
    g = torch.Generator(device="cuda").manual_seed(17)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch_dtype(dtype), device="cuda").normal_(0.0, std, generator=g)
    x, dY, W1, W2 = draw(1.0, T, d), draw(1.0, T, d), draw(0.02, 4, F, d), draw(0.02, 4, d, F)
    offsets = ragged_offsets(counts)
    A = int(offsets[-1])
    x[A:], dY[A:] = float("nan"), float("nan")               # rows past the last packed row must not be read
    dX = torch.full_like(x, 5.0)
    dW1, dW2 = (torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((4, F, d), (4, d, F)))
    ws = torch.full((B.moe_ffn_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda")
    B.moe_expert_ffn_backward(cfg, x, torch.from_numpy(offsets).cuda(), W1, W2, dY, dX, dW1, dW2, ws)
    assert bool((dX[A:] == 5.0).all()), "rows past the last packed row were written"
    et = GRAD_ELEM_FACTOR * TOL[dtype]
    for i in range(4):
        rows = slice(int(offsets[i]), int(offsets[i + 1]))
        xs, dy, w1, w2 = x[rows].double(), dY[rows].double(), W1[i].double(), W2[i].double()
        u = (xs @ w1.t()).requires_grad_()
        h = torch.nn.functional.gelu(u, approximate="tanh")
        (du,) = torch.autograd.grad(h, u, dy @ w2)
        many = et if counts[i] >= 256 else 1.0   # (elementwise only over many rows: see test_router_gradients)
        assert_close(to_np(dX[rows]), to_np(du @ w1), TOL[dtype], "dX_sliced", et)
        assert_close(to_np(dW1[i]), to_np(du.t() @ xs), TOL[dtype], "dW1", many)
        assert_close(to_np(dW2[i]), to_np(dy.t() @ h.detach()), TOL[dtype], "dW2", many)


# ---------------------------------------------------------------- the persistent kernels' tiles

@pytest.mark.parametrize("dtype,d,F,counts", [
    ("bf16", 64, 320, [3] * 130 + [300]),              # lookups past 64 experts; one k-tile; a last column tile of 64
    ("bf16", 128, 264, [32, 33, 64, 65, 128, 129]),    # every kind of small tile at its last size; a column tile of 8
    ("bf16", 192, 256, [288, 289, 320, 321, 384, 385, 512, 0, 513]),    # the same behind whole tiles; three k-tiles
    ("f16", 1280, 512, [257, 256, 0, 255]),            # 20 k-tiles, the last dealt whole
    ("bf16", 1344, 2560, [256, 40, 300]),              # 21, and 40 in the second product: the last with big tiles in the stream
    ("f16", 2624, 256, [700, 1]),                      # 41: cut again
    ("bf16", 64, 8192, [5000, 3300, 41]),              # more than a round of one k-tile each, 128 k-tiles in the second product
])
def test_tiles_of_the_persistent_kernel(dtype, d, F, counts):
    check_ffn(dtype, d, F, counts)


@pytest.mark.parametrize("dtype,d,F,counts", [
    ("bf16", 512, 2048, [0, 1, 63, 64, 65, 300, 1000, 700]),   # dH with weights by rows, all kinds of tiles; 128 tiles of weight gradients
    ("f16", 512, 2048, [513, 0, 255, 128, 127, 33, 1100, 0]),
    ("bf16", 520, 2056, [0, 1, 63, 64, 65, 191]),              # weight gradients: 3 x 9 tiles, the last ones of 8 columns
    ("f16", 2112, 1032, [1200, 0, 130, 700]),                  # 128 x 128 data gradients: 65 x 5 tiles for dH, K of no whole k-tiles for dX
    # dH on the persistent kernel with a last column tile of 8 (its loads run on into the next k-row, and past the expert's last
    # one at the end), whole tiles and small ones of up to 32, 64 and 128 rows; dX of no whole k-tiles
    ("bf16", 1088, 2056, [1044, 0, 1080, 1124, 1500, 1]),
    ("f16", 2752, 1288, [2324, 60, 128, 1, 4000]),             # the same, 43 k-tiles: the small tiles are cut
])
def test_gradient_tiles_by_rows(dtype, d, F, counts):
    """Expert-FFN backward against the chain rule in float64 (torch); rows past the last packed one hold NaN."""
    import torch
    n, A = len(counts), int(sum(counts))
    T = A + 70
    lc = small_cfg(T=T, d=d, F=F, E=n, top_k=1, in_dtype=dtype, out_dtype=dtype)
    cfg = B.config_from(lc)
    g = torch.Generator(device="cuda").manual_seed(d + F)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch_dtype(dtype), device="cuda").normal_(0.0, std, generator=g)
    x, dY, W1, W2 = draw(1.0, T, d), draw(1.0, T, d), draw(0.02, n, F, d), draw(0.02, n, d, F)
    offsets = ragged_offsets(counts)
    x[A:], dY[A:] = float("nan"), float("nan")
    dX = torch.full_like(x, 5.0)
    dW1, dW2 = (torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((n, F, d), (n, d, F)))
    ws = torch.full((B.moe_ffn_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda")
    B.moe_expert_ffn_backward(cfg, x, torch.from_numpy(offsets).cuda(), W1, W2, dY, dX, dW1, dW2, ws)
    assert bool((dX[A:] == 5.0).all()), "rows past the last packed row were written"
    et = GRAD_ELEM_FACTOR * TOL[dtype]
    for i in range(n):
        rows = slice(int(offsets[i]), int(offsets[i + 1]))
        if counts[i] == 0:
            assert float(dW1[i].abs().max()) == 0.0 and float(dW2[i].abs().max()) == 0.0
            continue
        xs, dy, w1, w2 = x[rows].double(), dY[rows].double(), W1[i].double(), W2[i].double()
        u = (xs @ w1.t()).requires_grad_()
        h = torch.nn.functional.gelu(u, approximate="tanh")
        (du,) = torch.autograd.grad(h, u, dy @ w2)
        many = et if counts[i] >= 256 else 1.0   # (elementwise only over many rows: see test_router_gradients)
        assert_close(to_np(dX[rows]), to_np(du @ w1), TOL[dtype], "dX_sliced", et)
        assert_close(to_np(dW1[i]), to_np(du.t() @ xs), TOL[dtype], "dW1", many)
        assert_close(to_np(dW2[i]), to_np(dy.t() @ h.detach()), TOL[dtype], "dW2", many)


@pytest.mark.parametrize("dtype,T,d,F,E,k", [
    ("bf16", 300, 64, 328, 2, 1),       # both sides of the activation from one product: one k-tile, a column tile of 72
    ("f16", 1100, 256, 512, 4, 2),      # whole tiles and tails
    ("bf16", 700, 2688, 256, 2, 1),     # 42 k-tiles: tiles cut between CUs
    ("bf16", 24, 128, 256, 4, 1),       # few rows: the pass over U
    ("f16", 300, 72, 136, 2, 1),        # d no multiple of 64: the pass over U
])
def test_training_pair_against_the_recomputing_calls(dtype, T, d, F, E, k):
    """out of moe_layer_forward_train against moe_layer_forward: they differ by the rounding of U (tests/gpu_util.py).  Gradients from
    its kept intermediates against moe_layer_backward, which computes the same U and H again: the same bits."""
    import torch
    lc = small_cfg(T=T, d=d, F=F, E=E, top_k=k, renorm_topk=k > 1, in_dtype=dtype, out_dtype=dtype)
    cfg = B.config_from(lc)
    g = torch.Generator(device="cuda").manual_seed(T + d)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch_dtype(dtype), device="cuda").normal_(0.0, std, generator=g)
    x, Wg, W1, W2, d_out = draw(1.0, T, d), draw(0.1, E, d), draw(0.05, E, F, d), draw(0.05, E, d, F), draw(1.0, T, d)
    raw = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
    ws, bws, saved = raw(B.moe_workspace_bytes(cfg)), raw(B.moe_layer_backward_workspace_bytes(cfg)), raw(B.moe_layer_saved_bytes(cfg))
    out = [torch.empty_like(x) for _ in range(2)]
    grads = [[torch.empty_like(x)] + [torch.empty(s, device="cuda") for s in ((E, d), (E,), (E, F, d), (E, d, F))] for _ in range(2)]
    B.moe_layer_forward(cfg, x, Wg, None, W1, W2, out[0], ws)
    B.moe_layer_backward(cfg, x, Wg, None, W1, W2, d_out, *grads[0], bws)
    B.moe_layer_forward_train(cfg, x, Wg, None, W1, W2, out[1], None, None, None, saved, ws)
    B.moe_layer_backward_saved(cfg, x, Wg, W1, W2, d_out, saved, *grads[1], bws)
    assert_close(to_np(out[1]), to_np(out[0]), TOL[dtype], "out", GRAD_ELEM_FACTOR * TOL[dtype])
    for name, a, b in zip(("dx", "dWg", "dbias", "dW1", "dW2"), *grads):
        differ = int((a != b).sum())
        assert differ == 0, f"{name}: {differ} elements"


# ---------------------------------------------------------------- hand-over of partial sums between CUs

def expert_chain(x, dY, W1, W2, offsets):
    """H, y and the gradients of the expert FFN in float64 (torch), expert by expert."""
    import torch
    H, y, dX = (torch.zeros((x.shape[0], n), dtype=torch.float64, device="cuda") for n in (W1.shape[1], x.shape[1], x.shape[1]))
    dW1, dW2 = (torch.zeros(W.shape, dtype=torch.float64, device="cuda") for W in (W1, W2))
    for i in range(W1.shape[0]):
        rows = slice(int(offsets[i]), int(offsets[i + 1]))
        xs, dy, w1, w2 = x[rows].double(), dY[rows].double(), W1[i].double(), W2[i].double()
        u = (xs @ w1.t()).requires_grad_()
        h = torch.nn.functional.gelu(u, approximate="tanh")
        (du,) = torch.autograd.grad(h, u, dy @ w2)
        H[rows], y[rows], dX[rows] = h.detach(), h.detach() @ w2.t(), du @ w1
        dW1[i], dW2[i] = du.t() @ xs, dy.t() @ h.detach()
    return H, y, dX, dW1, dW2


HANDOVER_SETTINGS = [(B.MOE_OPT_HANDOVER_DEVICE_SCOPE, 1, 0), (B.MOE_OPT_HANDOVER_SPIN_LIMIT, 0, 1 << 17)]   # (option, value, default)


@pytest.mark.parametrize("dtype,counts", [
    ("bf16", [300, 3, 0, 257, 40, 100]),   # big and small tiles in one cut stream, up to four CUs a tile
    ("f16", [2048, 2048, 2048]),           # 24 x 11 big tiles: a round of 256 CUs, then one cut big tile per XCD
])
def test_cut_tiles_have_the_same_bits_however_they_are_handed_over(dtype, counts):
    """Partial sums through the shared L2, with device-scope fences, or never waited for and computed by the CU that needs
    them: the expert FFN and its backward (weights by columns and by rows) give the same bits.  42 and 43 k-tiles, past every
    line below which a stream is dealt out in whole tiles, so all settings cut the same tiles."""
    import torch
    d, F, n, A = 2688, 2752, len(counts), sum(counts)
    T = A + 800                              # (the data gradients go to the persistent kernel by this bound)
    cfg = B.config_from(small_cfg(T=T, d=d, F=F, E=n, top_k=1, in_dtype=dtype, out_dtype=dtype))
    g = torch.Generator(device="cuda").manual_seed(A)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch_dtype(dtype), device="cuda").normal_(0.0, std, generator=g)
    x, dY, W1, W2 = draw(1.0, T, d), draw(1.0, T, d), draw(0.02, n, F, d), draw(0.02, n, d, F)
    offsets = ragged_offsets(counts)
    off = torch.from_numpy(offsets).cuda()

    def run():
        ws = torch.full((B.moe_ffn_workspace_bytes(cfg),), 0x11, dtype=torch.uint8, device="cuda")
        bws = torch.full((B.moe_ffn_backward_workspace_bytes(cfg),), 0x11, dtype=torch.uint8, device="cuda")
        H, y, dX = (torch.zeros((T, w), dtype=torch_dtype(dtype), device="cuda") for w in (F, d, d))
        dW1, dW2 = torch.empty(W1.shape, device="cuda"), torch.empty(W2.shape, device="cuda")
        B.moe_expert_ffn(cfg, x, off, W1, W2, H, y, ws)
        B.moe_expert_ffn_backward(cfg, x, off, W1, W2, dY, dX, dW1, dW2, bws)
        return [t[:A] for t in (H, y, dX)] + [dW1, dW2], (B.moe_ffn_check(cfg, ws, False), B.moe_backward_check(cfg, bws, False))

    names = ("H", "y_sliced", "dX_sliced", "dW1", "dW2")
    first, status = run()
    assert status == (0, 0)
    for name, a, b in zip(names, first, expert_chain(x[:A], dY[:A], W1, W2, offsets)):
        et = TOL[dtype] if name in ("H", "y_sliced") else GRAD_ELEM_FACTOR * TOL[dtype] if min(counts) >= 256 else 1.0
        assert_close(to_np(a), to_np(b), TOL[dtype], name, et)   # (weight gradients elementwise only over many rows)
    for option, value, default in HANDOVER_SETTINGS:
        B.moe_set_option(option, value)
        try:
            again, status = run()
        finally:
            B.moe_set_option(option, default)
        assert status == ((1, 1) if option == B.MOE_OPT_HANDOVER_SPIN_LIMIT else (0, 0))
        for name, a, b in zip(names, first, again):
            assert bool((a == b).all()), f"{name}, option {option}: {int((a != b).sum())} elements"


@pytest.mark.parametrize("dtype,k", [("bf16", 1), ("f16", 2)])
def test_layers_with_cut_tiles_have_the_same_bits_however_they_are_handed_over(dtype, k):
    """The same for the products of a layer (rows gathered by the loads, placed by the stores) and of a training step, whose
    first product stores two results."""
    import torch
    T, d, F, E = 1800, 2688, 2752, 4         # (the fewest tokens, to the hundred, whose data gradients are cut)
    cfg = B.config_from(small_cfg(T=T, d=d, F=F, E=E, top_k=k, renorm_topk=k > 1, in_dtype=dtype, out_dtype=dtype))
    g = torch.Generator(device="cuda").manual_seed(k)
    draw = lambda std, *shape: torch.empty(shape, dtype=torch_dtype(dtype), device="cuda").normal_(0.0, std, generator=g)
    x, Wg, W1, W2, d_out = draw(1.0, T, d), draw(0.02, E, d), draw(0.02, E, F, d), draw(0.02, E, d, F), draw(1.0, T, d)

    def run():
        raw = lambda n: torch.full((n,), 0x11, dtype=torch.uint8, device="cuda")
        ws, tws, bws, saved = (raw(f(cfg)) for f in (B.moe_workspace_bytes, B.moe_workspace_bytes,
                                                     B.moe_layer_backward_workspace_bytes, B.moe_layer_saved_bytes))
        out, out_t, dx = (torch.empty_like(x) for _ in range(3))
        dWg, dbias, dW1, dW2 = (torch.empty(s, device="cuda") for s in ((E, d), (E,), (E, F, d), (E, d, F)))
        B.moe_layer_forward(cfg, x, Wg, None, W1, W2, out, ws)
        B.moe_layer_forward_train(cfg, x, Wg, None, W1, W2, out_t, None, None, None, saved, tws)
        B.moe_layer_backward_saved(cfg, x, Wg, W1, W2, d_out, saved, dx, dWg, dbias, dW1, dW2, bws)
        return [out, out_t, saved, dx, dWg, dbias, dW1, dW2], (B.moe_ffn_check(cfg, ws, True), B.moe_ffn_check(cfg, tws, True),
                                                                        B.moe_backward_check(cfg, bws, True))

    first, status = run()
    assert status == (0, 0, 0)
    assert_close(to_np(first[1]), to_np(first[0]), TOL[dtype], "out", GRAD_ELEM_FACTOR * TOL[dtype])
    for option, value, default in HANDOVER_SETTINGS:
        B.moe_set_option(option, value)
        try:
            again, status = run()
        finally:
            B.moe_set_option(option, default)
        assert status == ((1, 1, 1) if option == B.MOE_OPT_HANDOVER_SPIN_LIMIT else (0, 0, 0))
        for name, a, b in zip(("out", "out (train)", "saved", "dx", "dWg", "dbias", "dW1", "dW2"), first, again):
            assert bool((a == b).all()), f"{name}, option {option}: {int((a != b).sum())} elements"
