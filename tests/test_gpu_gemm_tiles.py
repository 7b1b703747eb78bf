"""The tile form of a projection is picked by the size of the call; an output has the same bits in all of them."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2605_23296_amd import binding as B
from paper_2605_23296_amd.workloads import WORKLOADS, LayerConfig, to_numpy_f64
from oracle import layer as O
from tests.test_gpu_kernels import rnd
from tests.util import rel_err

pytestmark = pytest.mark.gpu
DENSE = WORKLOADS["dense_8x4096"].layer


# column tails of 8, K of an odd number of 64-wide k-tiles; whatever forms the rule picks for the row counts below
@pytest.mark.parametrize("N,K,epi,res", [(4104, 1088, 0, True), (2056, 576, 1, False), (4096, 64, 0, False), (4096, 192, 0, True)])
def test_rows_have_the_same_bits_in_every_tile_form(N, K, epi, res):
    lay = B.Layer(DENSE, None)
    Mmax = 4200
    a = rnd((Mmax, K), torch.bfloat16, 3)
    b = rnd(((2 if epi else 1) * N, K), torch.bfloat16, 4, std=0.05)
    r = rnd((Mmax, N), torch.bfloat16, 5) if res else None
    full = torch.empty((Mmax, N), dtype=torch.bfloat16, device="cuda")
    lay.compact_gemm(a, b, r, full, epi)
    rows = [0, 255, 256, 1000, Mmax - 1]
    A, Bm = to_numpy_f64(a[rows]), to_numpy_f64(b)
    ref = O.silu(O.linear(A, Bm[:N])) * O.linear(A, Bm[N:]) if epi else O.linear(A, Bm) + (to_numpy_f64(r[rows]) if res else 0.0)
    assert rel_err(to_numpy_f64(full[rows]), ref) < 1e-2
    for M in (65, 100, 129, 200, 300, 450, 600, 1000, 1652, 2100, 2600, 3100):
        c = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
        lay.compact_gemm(a[:M], b, None if r is None else r[:M], c[:M], epi)
        torch.cuda.synchronize()
        assert torch.equal(c[:M], full[:M]), M
        assert bool((c[M] == 7.0).all()), M     # nothing past the last row


FORMS = ["256x256", "128x256", "128x128", "128x64", "64x128", "64x64"]


def gemm_form(lay, form, a, b, r, c, epi):
    """The product in tile form `form` (-1: the picked one); returns the form that the rule picks."""
    picked = C.c_int32(-1)
    ptr = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    lay.check(lay.L.compact_test_gemm_form(lay.ctx, C.c_int32(form), ptr(a), ptr(b), ptr(r), ptr(c), C.c_int64(a.shape[0]),
                                           C.c_int32(c.shape[1]), C.c_int32(a.shape[1]), C.c_int32(epi), C.byref(picked),
                                           C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    return picked.value


# one to four k-tiles of 64 (shorter than the rings: their repeated loads), an odd and a long number of them; one row, rows and
# columns just under, at and over the tile edges
@pytest.mark.parametrize("K", [64, 128, 192, 256, 576, 1088])
@pytest.mark.parametrize("epi,res", [(0, True), (0, False), (1, False)])
def test_every_tile_form_at_its_edges(K, epi, res):
    lay = B.Layer(DENSE, None)
    for M, N in [(1, 8), (63, 136), (65, 56), (128, 64), (129, 264), (257, 520), (300, 128), (511, 1000)]:
        a, b = rnd((M, K), torch.bfloat16, 3), rnd(((2 if epi else 1) * N, K), torch.bfloat16, 4, std=0.05)
        r = rnd((M, N), torch.bfloat16, 5) if res else None
        A, Bm = to_numpy_f64(a), to_numpy_f64(b)
        ref = O.silu(O.linear(A, Bm[:N])) * O.linear(A, Bm[N:]) if epi else O.linear(A, Bm) + (to_numpy_f64(r) if res else 0.0)
        first = None
        for form in range(len(FORMS)):
            c = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
            gemm_form(lay, form, a, b, r, c[:M], epi)
            torch.cuda.synchronize()
            assert bool((c[M] == 7.0).all()), (M, N, FORMS[form])
            if first is None:
                assert rel_err(to_numpy_f64(c[:M]), ref) < 1e-2, (M, N)
                first = c
            assert torch.equal(c, first), (M, N, FORMS[form])


# whole tiles, halves of the other slots and a bottom row tile of at most 128 rows in one launch: no whole tile, one, several; last
# row tiles of 1, 76, 128, 129 and 255 rows, the first three a bottom strip beside whole and half tiles; workgroup counts that the
# XCDs do not share evenly
@pytest.mark.parametrize("epi,res", [(0, True), (1, False)])
@pytest.mark.parametrize("M,N,K", [(255, 264, 192), (385, 520, 64), (640, 1032, 256), (1153, 776, 320), (1791, 2056, 128), (200, 136, 64),
                                   (513, 1032, 192), (1100, 776, 128)])
def test_whole_and_half_tiles_in_one_launch(M, N, K, epi, res):
    lay = B.Layer(DENSE, None)
    a, b = rnd((M, K), torch.bfloat16, 3), rnd(((2 if epi else 1) * N, K), torch.bfloat16, 4, std=0.05)
    r = rnd((M, N), torch.bfloat16, 5) if res else None
    A, Bm = to_numpy_f64(a), to_numpy_f64(b)
    ref = O.silu(O.linear(A, Bm[:N])) * O.linear(A, Bm[N:]) if epi else O.linear(A, Bm) + (to_numpy_f64(r) if res else 0.0)
    first = None
    for form in (len(FORMS), 5):   # mixed, 64 x 64
        c = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
        gemm_form(lay, form, a, b, r, c[:M], epi)
        torch.cuda.synchronize()
        assert bool((c[M] == 7.0).all())
        if first is None:
            assert rel_err(to_numpy_f64(c[:M]), ref) < 1e-2
            first = c
        assert torch.equal(c, first)


# half tiles in one round, K of 2048 and more: eight workgroups share out the weight lines that are touched ahead; groups of four
# 256-row tiles with and without a rest, K whose last k-tiles nobody touches, columns past the last tile
@pytest.mark.parametrize("M,N,K,epi", [(1024, 1000, 2048, 0), (1153, 2056, 2112, 0), (1300, 264, 2240, 1), (2048, 520, 4160, 1)])
def test_half_tiles_that_touch_weight_lines_ahead(M, N, K, epi):
    lay = B.Layer(DENSE, None)
    a, b = rnd((M, K), torch.bfloat16, 3), rnd(((1 + epi) * N, K), torch.bfloat16, 4, std=0.05)
    out = []
    for form in (1, 5):   # 128 x 256, 64 x 64
        out.append(torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device="cuda"))
        gemm_form(lay, form, a, b, None, out[-1][:M], epi)
    torch.cuda.synchronize()
    rows = [0, 127, 128, 600, 1023, M - 1]
    A, Bm = to_numpy_f64(a[rows]), to_numpy_f64(b)
    ref = O.silu(O.linear(A, Bm[:N])) * O.linear(A, Bm[N:]) if epi else O.linear(A, Bm)
    assert rel_err(to_numpy_f64(out[0][rows]), ref) < 1e-2
    assert torch.equal(out[0], out[1]) and bool((out[0][M] == 7.0).all())


def test_the_swiglu_divides_to_half_a_unit():
    """silu(a) u with a and u exact products of two bf16 values, so that every step of the fp32 formula is known (the exponential
    is the hardware's exp2 of a * log2(e), which torch.exp2 calls too; division and products are rounded once each).  Every tile
    form has exactly those bits; a quotient off by one unit would change a bf16 result in about 2^-16 of the places."""
    lay = B.Layer(DENSE, None)
    M, N, K = 1152, 4104, 64
    a, b = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda"), torch.zeros((2 * N, K), dtype=torch.bfloat16, device="cuda")
    a[:, 0], b[:, 0] = rnd((M,), torch.bfloat16, 6, std=1.5), rnd((2 * N,), torch.bfloat16, 7, std=1.5)
    x, w = a[:, 0].float(), b[:, 0].float()
    g, up = x[:, None] * w[:N], x[:, None] * w[N:]
    den = (1.0 + torch.exp2(g * -1.44269504).cpu()).numpy()
    q, up = g.cpu().numpy() / den, up.cpu().numpy()
    bf = lambda v: torch.from_numpy(v).to(torch.bfloat16)
    want, off = bf(q * up), bf(np.nextafter(q, np.float32(0)) * up)
    assert int((off != want).sum()) > 20
    for form in range(len(FORMS) + 1):
        c = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        gemm_form(lay, form, a, b, None, c, 1)
        assert torch.equal(c.cpu(), want), (form, int((c.cpu() != want).sum()))


def test_the_rule_picks_every_tile_form():
    """Calls at which each form is the cheapest by the rule: a retuned table that drops one shows up here."""
    lay = B.Layer(DENSE, None)
    seen = set()
    for M, N, K, epi in [(8192, 4096, 4096, 0), (2048, 4096, 14336, 0), (1000, 4096, 14336, 0), (300, 4096, 14336, 0), (513, 1024, 2816, 1),
                         (126, 6144, 14336, 1), (65, 4096, 4096, 0), (300, 6144, 4096, 0), (20, 4096, 14336, 0), (200, 14336, 4096, 1)]:
        a, b = torch.empty((M, K), dtype=torch.bfloat16, device="cuda"), torch.empty(((1 + epi) * N, K), dtype=torch.bfloat16, device="cuda")
        seen.add(gemm_form(lay, -1, a.zero_(), b.zero_(), None, torch.empty((M, N), dtype=torch.bfloat16, device="cuda"), epi))
    assert sorted(FORMS[f] for f in seen) == sorted(FORMS)


def test_routed_rows_have_the_same_bits_at_every_row_tile_height():
    E, k, d, F, rows = 8, 4, 1024, 1408, 9000
    layer = LayerConfig(d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=F, n_experts=E, top_k=k, dtype="bf16")
    bf = torch.bfloat16
    w = dict(w_router=rnd((E, d), bf, 6, 0.05), w_exp_gate_up=rnd((E, 2 * F, d), bf, 1, 0.03), w_exp_down=rnd((E, d, F), bf, 2, 0.03),
             g_attn=rnd((d,), bf, 7), w_qkv=rnd((8, d), bf, 8), w_o=rnd((d, 8), bf, 9), g_ffn=rnd((d,), bf, 10))
    lay = B.Layer(layer, w)
    lay.ensure_workspace(rows, 1, 8, "cuda")
    m, h = rnd((rows, d), bf, 3), rnd((rows, d), bf, 4)
    g = torch.Generator(device="cpu")
    g.manual_seed(5)
    idx = torch.rand((rows, E), generator=g).topk(k, dim=1).indices.int().cuda()
    gate = torch.softmax(torch.randn((rows, k), generator=g), dim=1).cuda()
    full = torch.empty_like(h)
    lay.compact_moe_ffn(m, h, idx, gate, full)
    heights = set()
    for n in (70, 300, 1500, 3000, 6000):   # row tiles of 64, 128 and 256
        mt = C.c_int32(0)
        lay.check(lay.L.compact_test_group_mtile(lay.ctx, C.c_int64(n * k), C.c_int32(E), C.c_int32(F), C.c_int32(d), C.byref(mt)))
        heights.add(mt.value)
        y = torch.empty((n, d), dtype=bf, device="cuda")
        lay.compact_moe_ffn(m[:n], h[:n], idx[:n].contiguous(), gate[:n].contiguous(), y)
        torch.cuda.synchronize()
        assert torch.equal(y, full[:n]), n
    assert heights == {64, 128, 256}
