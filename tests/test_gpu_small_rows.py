"""GPU parity of the projection GEMMs at the edges of their tiles.

bf16 up to 192 rows runs with K split over a workgroup's waves (one kernel instance per number of
32-row blocks, tiles of 1 to 4 column blocks, 1 to 8 K splits); fp32 projections of up to 1024
tiles of 16 x 32 run on those; bf16 tiles of 288 rows split k between two groups of waves.  Every element is held to what its arithmetic allows: fp32 sums of
K products in any order lie within K 2^-24 sum |x w| of the exact value, and storing in bf16 adds
at most 2^-8 of it.
"""
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu

af = pytest.importorskip("paper_2512_20276_amd")


def _check(M, N, K, dt):
    x = wl.draw(("t_rows_x", M, K), (M, K), dtype=dt, device="cuda")
    w = wl.draw(("t_rows_w", N, K), (N, K), std=0.02, dtype=dt, device="cuda")
    y = torch.full((M, N), float("nan"), dtype=dt, device="cuda")
    af.op_linear(x, w, y)
    torch.cuda.synchronize()
    xd, wd = x.cpu().double(), w.cpu().double()
    ref = xd @ wd.t()
    bound = (K + 8) * 2.0 ** -24 * (xd.abs() @ wd.abs().t())
    if dt == torch.bfloat16:
        bound = bound + ref.abs() * 2.0 ** -8
    err = (y.cpu().double() - ref).abs()
    assert bool((err <= bound).all()), (M, N, K, float((err - bound).max()))


@pytest.mark.parametrize("M", [1, 2, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193])
@pytest.mark.parametrize("N,K", [(48, 256), (608, 4096), (4096, 1024)])
def test_bf16_row_block_edges(M, N, K):
    """Every instance's first and last row count; a last column block half past N (48), tiles past
    the last column block (608 = 19 blocks), split and unsplit K."""
    _check(M, N, K, torch.bfloat16)


@pytest.mark.parametrize("M", [7, 135, 192])
@pytest.mark.parametrize("N,K", [(4096, 11008), (12288, 4096), (22016, 256), (32000, 512)])
def test_bf16_projection_widths(M, N, K):
    """The 7B projections' widths with their K splits (11008: shares of 43 k units), and widths
    that take three and four column blocks per tile."""
    _check(M, N, K, torch.bfloat16)


@pytest.mark.parametrize("M", [257, 288, 385, 543, 576, 577, 2264])
@pytest.mark.parametrize("N,K", [(48, 256), (608, 1024), (4096, 512)])
def test_bf16_two_k_groups(M, N, K):
    """288 x 128 tiles with two k groups: row tiles of one row and of 288, a last column block
    half past N, a last column tile partly past it, K split over workgroups (48, 608) and not."""
    _check(M, N, K, torch.bfloat16)


@pytest.mark.parametrize("M", [1, 15, 16, 17, 34, 200])
@pytest.mark.parametrize("N,K", [(16, 4), (48, 252), (768, 256), (256, 688), (1376, 260), (512, 1600)])
def test_f32_small_tiles(M, N, K):
    """Row and column remainders of the 16 x 32 tile; K below, at and past what a wave requests at
    once (two steps of 32 at K <= 256, six beyond, and more than one such share)."""
    _check(M, N, K, torch.float32)


@pytest.mark.parametrize("M,N,K", [(32, 16384, 512), (24, 6144, 1024), (80, 6144, 2048), (144, 3072, 2048)])
def test_f32_wide_tiles_of_few_rows(M, N, K):
    """Few rows that the 32- and 96-row fp32 tiles do faster than the 16 x 32 ones, K split and not."""
    _check(M, N, K, torch.float32)


@pytest.mark.parametrize("M", [1, 34])
@pytest.mark.parametrize("K", [256, 512, 1024, 2048])
def test_f32_small_tiles_infinite_weight(M, K):
    """An infinite weight in the last k of a column, where a wave's last batch of six steps is not
    full (K = 512, 1024 and 2048: four, two and four steps): the column is infinite with the sign
    of its activation and no other column is touched."""
    N, col = 48, 20
    x = wl.draw(("t_inf_x", M, K), (M, K), dtype=torch.float32, device="cuda")
    w = wl.draw(("t_inf_w", N, K), (N, K), std=0.02, dtype=torch.float32, device="cuda")
    y, clean = torch.empty((M, N), device="cuda"), torch.empty((M, N), device="cuda")
    af.op_linear(x, w, clean)
    w[col, K - 1] = float("inf")
    af.op_linear(x, w, y)
    torch.cuda.synchronize()
    assert torch.equal(y[:, col], torch.sign(x[:, K - 1]) * float("inf"))
    keep = [c for c in range(N) if c != col]
    assert torch.equal(y[:, keep], clean[:, keep])


def test_step_tables_of_calls_in_flight():
    """Calls whose tables differ, sent without waiting, twice round the staging buffers and with
    tables that outgrow them on the way: every call reads its own tables."""
    shape = wl.TINY
    g, layers = wl.model_weights(shape, seed=3, device="cuda")
    n_req, rows = 12, 2500
    order = [[(5 * i + j) % n_req for j in range(1 + i % n_req)] for i in range(72)]

    def all_calls(wait):
        w = af.Weights(shape, g, layers)
        ring = af.Ring(shape.n_layers, n_req + 1, 2560, shape.n_heads, shape.head_dim, dtype=torch.float32)
        segs = {}
        for r in range(n_req):
            slot = ring.append(r, 3 + r).slot
            kv = [wl.draw(("t_tab", n, r), (3 + r, shape.n_heads, shape.head_dim), dtype=torch.float32,
                          device="cuda") for n in "kv"]
            ring.write_kv(0, slot, 0, *kv)
            segs[r] = ring.append(r, 1)
        long = ring.append(n_req, rows)
        out = []
        for i, reqs in enumerate(order):
            call = [segs[r] for r in reqs] if i != 40 else [long]
            for row, s in enumerate(call):
                s.q_start, s.flags = row, af.AF_SEG_EMIT
            # a request's row is the same in every call, so are the keys and values it writes
            ids = reqs if i != 40 else range(100, 100 + rows)
            h = torch.stack([base[r] for r in ids])
            af.packed_layer_forward(w, 0, h, af.segments_array(call), ring)
            z = torch.empty((len(call), shape.vocab), dtype=torch.float32, device="cuda")
            af.op_lm_head_argmax(w, h, af.segments_array(call), z)
            if wait:
                torch.cuda.synchronize()
            out += [h, z]
        torch.cuda.synchronize()
        return out

    base = wl.draw(("t_tab_x",), (100 + rows, shape.d_model), dtype=torch.float32, device="cuda")
    for i, (a, b) in enumerate(zip(all_calls(True), all_calls(False))):
        assert torch.equal(a, b), i
