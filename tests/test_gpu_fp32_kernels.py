"""fp32 storage kernels at the edges of their pieces: k-chunks of 16 dealt to four or eight wavefronts, output tiles of 16, 32
and 64, keys 64 at a time."""
import pytest
import torch

from oracle import layer as O
from paper_2605_23296_amd import binding as B
from paper_2605_23296_amd.workloads import to_numpy_f64
from tests.test_gpu_kernels import attention_case, decode_case, fp32_variant, rnd, MOE, DENSE
from tests.util import rel_err

pytestmark = pytest.mark.gpu


# fp32 sums of K products of N(0, 1) x N(0, 0.05): the error is below 2^-24 sqrt(K) of the rms, K <= 2051: 3e-6
@pytest.mark.parametrize("M,N,K,epi,res", [
    (1, 17, 16, 0, True), (4, 256, 1024, 0, True), (16, 512, 256, 1, False), (17, 33, 1040, 0, False),   # 16 x 16 tiles
    (5, 40, 30, 0, False), (9, 23, 1027, 1, False),                                                     # rows that are not 16-byte aligned
    (700, 900, 272, 0, True), (1300, 700, 1024, 1, False),                                              # 32 x 32 tiles, tails
    (1200, 1300, 64, 0, True), (1030, 1100, 1040, 0, False), (1090, 1030, 79, 0, True),                 # 64 x 64
    (1100, 1110, 2048, 1, False), (1041, 1033, 2051, 1, False)])                                        # 64 x 32, SwiGLU
def test_gemm_fp32_tiles(M, N, K, epi, res):
    lay = B.Layer(fp32_variant(DENSE), None)
    a, b = rnd((M, K), torch.float32, 3), rnd(((2 if epi else 1) * N, K), torch.float32, 4, std=0.05)
    r = rnd((M, N), torch.float32, 5) if res else None
    c = torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda")
    lay.compact_gemm(a, b, r, c[:M], epi)
    one = torch.empty((1, N), dtype=torch.float32, device="cuda")
    lay.compact_gemm(a[M - 1:], b, None if r is None else r[M - 1:], one, epi)
    torch.cuda.synchronize()
    A, Bm = to_numpy_f64(a), to_numpy_f64(b)
    ref = O.silu(O.linear(A, Bm[:N])) * O.linear(A, Bm[N:]) if epi else O.linear(A, Bm) + (to_numpy_f64(r) if res else 0.0)
    assert rel_err(to_numpy_f64(c[:M]), ref) < 1e-5
    assert bool((c[M] == 7.0).all())
    assert torch.equal(one[0], c[M - 1])     # a row's bits do not depend on the rows beside it


@pytest.mark.parametrize("layer", [MOE, DENSE], ids=["hd64", "hd128"])
def test_prefill_attention_fp32_key_pieces(layer):
    # one key, one short of / exactly / one past a 64-key piece and a 16-key run, several pieces
    attention_case(fp32_variant(layer), [1, 2, 15, 17, 63, 64, 65, 130, 257], 61)


@pytest.mark.parametrize("layer", [MOE, DENSE], ids=["hd64", "hd128"])
def test_decode_attention_fp32_key_pieces(layer):
    # fewer pieces than wavefronts, exactly one each, a second round that only some wavefronts take part in
    decode_case(fp32_variant(layer), [1, 3, 63, 64, 65, 192, 255, 256, 257, 333, 600], 62)
