"""The tile form of a projection is picked by the size of the call; an output has the same bits in all of them."""
import pytest
import torch

from paper_2605_23296_amd import binding as B
from paper_2605_23296_amd.workloads import WORKLOADS, LayerConfig, to_numpy_f64
from oracle import layer as O
from tests.test_gpu_kernels import rnd
from tests.util import rel_err

pytestmark = pytest.mark.gpu
DENSE = WORKLOADS["dense_8x4096"].layer


# column tails of 8, K of an odd number of 64-wide k-tiles; the row counts below reach every tile form
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
    for n in (70, 300, 1500, 3000, 6000):   # row tiles of 64, 128 and 256
        y = torch.empty((n, d), dtype=bf, device="cuda")
        lay.compact_moe_ffn(m[:n], h[:n], idx[:n].contiguous(), gate[:n].contiguous(), y)
        torch.cuda.synchronize()
        assert torch.equal(y, full[:n]), n
