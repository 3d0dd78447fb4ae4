"""GPU parity of the projection GEMMs at the edges of their tiles.

bf16 up to 192 rows runs with K split over a workgroup's waves where that is faster (one kernel
instance per number of 32-row blocks and of column blocks; every one is run here, unsplit and with
K split over workgroups, the planner saying which one a shape takes); fp32 projections run on 16 x
32 tiles where those are faster; bf16 tiles of 288 rows split k between two groups of waves.  Every
element is held to what its arithmetic allows: fp32 sums of K products in any order lie within
K 2^-24 sum |x w| of the exact value, and storing in bf16 adds at most 2^-8 of it.
"""
import pytest
import torch

import workload as wl
from tests.plans import EPI_STORE, EPI_STORE_F32, f32_small, stream_plan

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


@pytest.mark.parametrize("V", [16, 4080, 4096, 4112, 16384, 16400, 32768, 32784, 65552])
def test_argmax_widths(V):
    """Tokens at the widths where a thread's share of chunks changes: ties at the first and the last
    column, rows of equal, of infinite and of NaN logits."""
    D = 64
    shape = wl.ModelShape(n_layers=0, d_model=D, n_heads=1, head_dim=64, d_ff=64, vocab=V, dtype="f32")
    head = wl.draw(("t_argmax_w", V), (V, D), dtype=torch.float32, device="cuda")
    head[V - 1] = head[0]  # the same logit in the first and the last column
    g = {"embed": torch.zeros((V, D), device="cuda"), "final_norm": torch.ones(D, device="cuda"), "lm_head": head}
    w = af.Weights(shape, g, [])
    n = 70
    hidden = wl.draw(("t_argmax_x", V), (n, D), dtype=torch.float32, device="cuda")
    hidden[0] = head[0] * 10    # the tied columns win
    hidden[1] = 0.0             # every logit equal
    hidden[2] = float("nan")    # no logit is comparable
    z = torch.empty((n, V), dtype=torch.float32, device="cuda")
    toks = torch.empty(n, dtype=torch.int32, device="cuda")
    af.op_lm_head_argmax(w, hidden, [af.Segment(i, 1, i, 0, 100 + i, af.AF_SEG_EMIT, 0) for i in range(n)], z, toks)
    torch.cuda.synchronize()
    best = z.max(dim=1, keepdim=True).values
    want = torch.argmax((z == best).float(), dim=1)
    assert want[0] == 0 and want[1] == 0 and want[2] == 0  # the lowest index; 0 where nothing compares
    assert torch.equal(toks.long(), want)
    w.close()


def _bound(x, w, ref, dt):
    """What the exact value and a result may differ by (float64 on the GPU)."""
    b = (x.shape[1] + 8) * 2.0 ** -24 * (x.abs() @ w.abs().t())
    return b + ref.abs() * 2.0 ** -8 if dt == torch.bfloat16 else b


# (row blocks, column blocks, K splits) of an instance and a width and depth that take it
STREAMED = [
    (1, 1, 1, 48, 3072), (1, 1, 8, 48, 11008), (1, 2, 1, 9200, 512), (1, 2, 4, 3072, 5632), (1, 3, 1, 20464, 512),
    (2, 1, 1, 48, 2048), (2, 1, 8, 48, 11008), (2, 2, 1, 9200, 256), (2, 2, 4, 3072, 3072), (2, 3, 1, 20464, 512),
    (2, 3, 2, 9200, 4096), (2, 4, 1, 27632, 3072),
    (3, 1, 1, 48, 1536), (3, 1, 8, 48, 11008), (3, 2, 1, 9200, 256), (3, 2, 4, 3072, 2816), (3, 3, 1, 20464, 512),
    (3, 3, 4, 6128, 4096), (3, 4, 1, 27632, 3072), (3, 4, 2, 15344, 11008),
    (4, 1, 1, 48, 1280), (4, 1, 8, 48, 11008), (4, 2, 1, 9200, 256), (4, 2, 4, 3072, 2048), (4, 3, 1, 20464, 1536),
    (4, 3, 4, 6128, 2816), (4, 4, 1, 27632, 3072), (4, 4, 2, 15344, 5632),
    (5, 1, 1, 48, 1280), (5, 1, 8, 48, 11008), (5, 2, 1, 9200, 256), (5, 2, 4, 3072, 2048), (5, 3, 1, 20464, 1536),
    (5, 3, 4, 6128, 2816), (5, 4, 1, 27632, 3072), (5, 4, 2, 15344, 4096),
    (6, 1, 1, 48, 1280), (6, 1, 4, 48, 11008), (6, 2, 1, 9200, 512), (6, 2, 3, 5104, 2048), (6, 3, 1, 20464, 8192),
    (6, 3, 4, 6128, 2048),
]


@pytest.mark.parametrize("fm,cb,S,N,K", STREAMED)
def test_bf16_streamed_instances(fm, cb, S, N, K):
    """Every reachable instance, unsplit and split, at its first and last row count; N ends inside a
    column block or a tile."""
    for M in (32 * fm - 31, 32 * fm):
        assert stream_plan(EPI_STORE, M, N, K) == (fm, cb, S)
        x = wl.draw(("t_inst_x", M, K), (M, K), device="cuda")
        w = wl.draw(("t_inst_w", N, K), (N, K), std=0.02, device="cuda")
        y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        af.op_linear(x, w, y)
        xd, wd = x.double(), w.double()
        ref = xd @ wd.t()
        err = (y.double() - ref).abs()
        assert bool((err <= _bound(xd, wd, ref, torch.bfloat16)).all()), (M, N, K)


# rows, d_model, vocabulary and the streaming instance of an LM head (None: the tiles)
HEADS = [
    (1, 3072, 48, (1, 1, 1)), (33, 2048, 48, (2, 1, 1)), (64, 256, 9200, (2, 2, 1)), (50, 5632, 20464, (2, 3, 1)),
    (64, 3072, 3072, (2, 2, 4)), (96, 1536, 48, (3, 1, 1)), (65, 256, 9200, (3, 2, 1)), (96, 5632, 20464, (3, 3, 1)),
    (66, 8192, 27632, (3, 4, 1)), (97, 1280, 48, (4, 1, 1)), (128, 256, 9200, (4, 2, 1)), (100, 5632, 20464, (4, 3, 1)),
    (128, 2816, 6128, (4, 3, 4)), (129, 1280, 48, (5, 1, 1)), (160, 256, 9200, (5, 2, 1)), (140, 5632, 20464, (5, 3, 1)),
    (161, 1280, 48, (6, 1, 1)), (192, 512, 9200, (6, 2, 1)), (170, 2048, 6128, (6, 3, 4)),
    (33, 4096, 32000, (2, 4, 1)), (64, 4096, 32000, (2, 4, 1)), (96, 4096, 32000, None), (128, 4096, 32000, None),
    (192, 4096, 32000, None), (288, 4096, 32000, None),
]


@pytest.mark.parametrize("n,D,V,plan", HEADS)
def test_bf16_head_of_many_rows(n, D, V, plan):
    """fp32 logits of n emitting rows, streamed and on the tiles, and the greedy token of each."""
    assert stream_plan(EPI_STORE_F32, n, V, D) == plan
    shape = wl.ModelShape(n_layers=0, d_model=D, n_heads=D // 64, head_dim=64, d_ff=64, vocab=V)
    g = {"embed": torch.zeros((V, D), dtype=torch.bfloat16, device="cuda"),
         "final_norm": wl.draw(("t_head_g", D), (D,), std=0.1, mean=1.0, device="cuda"),
         "lm_head": wl.draw(("t_head_w", V, D), (V, D), std=0.02, device="cuda")}
    w = af.Weights(shape, g, [])
    hidden = wl.draw(("t_head_x", n, D), (n + 3, D), device="cuda")
    rows = [(i * 7 + 2) % (n + 3) for i in range(n)] if (n + 3) % 7 else list(range(3, n + 3))
    segs = [af.Segment(r, 1, i, 0, 1000 + i, af.AF_SEG_EMIT, 0) for i, r in enumerate(rows)]
    z = torch.full((n + 1, V), 7.0, dtype=torch.float32, device="cuda")
    toks = torch.empty(n, dtype=torch.int32, device="cuda")
    af.op_lm_head_argmax(w, hidden, segs, z, toks)
    # the normed rows as the library stores them
    xn = torch.empty((n, D), dtype=torch.bfloat16, device="cuda")
    af.op_rmsnorm(hidden[rows].contiguous(), g["final_norm"], xn, shape.rms_eps)
    torch.cuda.synchronize()
    xd, wd = xn.double(), g["lm_head"].double()
    ref = xd @ wd.t()
    err = (z[:n].double() - ref).abs()
    assert bool((err <= _bound(xd, wd, ref, torch.float32)).all())
    assert bool((z[n] == 7.0).all())  # nothing past the last row
    # ties between fp32 logits: the lowest index
    assert torch.equal(toks.long(), torch.argmax((z[:n] == z[:n].max(dim=1, keepdim=True).values).float(), dim=1))
    w.close()


@pytest.mark.parametrize("M", [1, 2, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193])
@pytest.mark.parametrize("N,K", [(48, 256), (608, 4096), (4096, 1024)])
def test_bf16_row_block_edges(M, N, K):
    """Row counts at the edges of row blocks; a last column block half past N (48), tiles past
    the last column block (608 = 19 blocks), split and unsplit K."""
    _check(M, N, K, torch.bfloat16)


@pytest.mark.parametrize("M", [7, 135, 192])
@pytest.mark.parametrize("N,K", [(4096, 11008), (12288, 4096), (22016, 256), (32000, 512)])
def test_bf16_projection_widths(M, N, K):
    """The 7B projections' widths with their K splits (11008: shares of 43 k units), and wide ones."""
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
    assert f32_small(M, N, K)
    _check(M, N, K, torch.float32)


@pytest.mark.parametrize("M,N,K", [(32, 16384, 512), (24, 6144, 1024), (80, 6144, 2048), (144, 3072, 2048)])
def test_f32_wide_tiles_of_few_rows(M, N, K):
    """Few rows that the 32- and 96-row fp32 tiles do faster than the 16 x 32 ones, K split and not."""
    assert not f32_small(M, N, K)
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


class _Busy:
    """A bounded stretch of work (products of 8192 x 8192, about 1 ms each) that holds the stream back."""

    def __init__(self):
        self.a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
        self.out = torch.empty_like(self.a)
        self.end = torch.cuda.Event()

    def start(self, n):
        for _ in range(n):
            torch.mm(self.a, self.a, out=self.out)
        self.end.record()

    def running(self):
        return not self.end.query()


def test_step_tables_of_calls_in_flight():
    """Calls whose tables differ, sent while the stream is held back: every staging buffer is in
    flight when the host comes round to the first again, which then has to wait.  Twice round the 32
    buffers, and after tables that outgrow them, of which there is room for 16 and for 4: every call
    reads its own tables."""
    shape = wl.TINY
    g, layers = wl.model_weights(shape, seed=3, device="cuda")
    n_req, rows, n_many = 12, 2500, 3300
    base = wl.draw(("t_tab_x",), (100 + n_many * 10, shape.d_model), dtype=torch.float32, device="cuda")
    # (requests of a call) ; "long" and "many" are the calls whose tables outgrow the buffers
    order = [[(5 * i + j) % n_req for j in range(1 + i % n_req)] for i in range(40)]

    def all_calls(wait):
        w = af.Weights(shape, g, layers)
        ring = af.Ring(shape.n_layers, n_req + 1, 2560, shape.n_heads, shape.head_dim, dtype=torch.float32)
        ring2 = af.Ring(shape.n_layers, n_many, 16, shape.n_heads, shape.head_dim, dtype=torch.float32)
        busy = _Busy()
        segs = {}
        for r in range(n_req):
            slot = ring.append(r, 3 + r).slot
            kv = [wl.draw(("t_tab", n, r), (3 + r, shape.n_heads, shape.head_dim), dtype=torch.float32,
                          device="cuda") for n in "kv"]
            ring.write_kv(0, slot, 0, *kv)
            segs[r] = ring.append(r, 1)
        long = ring.append(n_req, rows)
        many = [ring2.append(r, 10) for r in range(n_many)]
        for i, s in enumerate(many):
            s.q_start, s.flags = 10 * i, af.AF_SEG_EMIT
        many = af.segments_array(many)
        long.q_start, long.flags = 0, af.AF_SEG_EMIT
        long = af.segments_array([long])
        # a request's row is the same in every call, so are the keys and values it writes
        hidden = [base[torch.tensor(reqs, device="cuda")] for reqs in order]
        arrays = []
        for reqs in order:
            call = [segs[r] for r in reqs]
            for row, s in enumerate(call):
                s.q_start, s.flags = row, af.AF_SEG_EMIT
            arrays.append(af.segments_array(call))
        out = []

        def call(h, sa, r):
            af.packed_layer_forward(w, 0, h, sa, r)
            z = torch.empty((len(sa), shape.vocab), dtype=torch.float32, device="cuda")
            af.op_lm_head_argmax(w, h, sa, z)
            if wait:
                torch.cuda.synchronize()
            out.extend([h, z])

        for grow, buffers in ((None, 32), ((base[100:100 + rows], long, ring), 16), ((base[100:], many, ring2), 4)):
            if grow is None:
                call(hidden[0].clone(), arrays[0], ring)  # workspaces are allocated here
            else:
                call(grow[0].clone(), *grow[1:])
            torch.cuda.synchronize()
            if not wait:
                busy.start(60)
            # a call stages two tables (layer, head); the one above has taken the first two buffers
            for i, (h, sa) in enumerate(zip(hidden, arrays)):
                call(h.clone(), sa, ring)
                if not wait and 2 * i + 4 == buffers:
                    assert busy.running()  # the next call needs the first buffer again
        torch.cuda.synchronize()
        return out

    for i, (a, b) in enumerate(zip(all_calls(True), all_calls(False))):
        assert torch.equal(a, b), i
