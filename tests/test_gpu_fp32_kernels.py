"""fp32 storage kernels at the edges of their pieces: k-chunks of 16 dealt to four or eight wavefronts, output tiles of 16, 32
and 64, keys 64 at a time."""
import copy

import numpy as np
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
    (1100, 1110, 2048, 1, False), (1041, 1033, 2051, 1, False),                                         # 64 x 32, SwiGLU
    # the same tiles where their loads go out one by one, or in a batch, as the other lines do not have them
    (17, 2100, 1040, 0, True), (500, 1000, 144, 1, False),                                              # 16 x 16
    (700, 900, 80, 0, True), (700, 900, 272, 1, False), (900, 1000, 272, 1, False),                     # 32 x 32
    (1024, 1023, 528, 0, True), (1500, 1600, 528, 0, False), (1030, 1100, 1552, 0, True)])              # 64 x 64
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
def test_prefill_attention_fp32_short_blocks(layer):
    # forms for 16 and 32 keys, and calls whose rows all have at most 32: a row's bits do not depend on a longer block beside it
    lay, short = fp32_variant(layer), [1, 2, 15, 16, 17, 20, 31, 32]
    attention_case(lay, short, 63)
    qkv = rnd((sum(short) + 33, lay.Dq + 2 * lay.Dkv), torch.float32, 64)
    out = []
    for lens in (short, short + [33]):
        cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
        rows = qkv[:cu[-1]].clone()
        kv = B.KVCache(lay, lens, "cuda", torch.float32)
        kv.k.fill_(float("nan"))
        kv.v.fill_(float("nan"))
        gpu = B.Layer(lay, None)
        gpu.compact_rope_kvwrite(cu, rows, kv)
        o = torch.empty((cu[-1], lay.Dq), dtype=torch.float32, device="cuda")
        gpu.compact_attn_prefill(cu, rows, kv, o)
        torch.cuda.synchronize()
        out.append(o[:sum(short)])
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("layer", [MOE, DENSE], ids=["hd64", "hd128"])
def test_decode_attention_fp32_key_pieces(layer):
    # fewer pieces than wavefronts, exactly one each, a second round that only some wavefronts take part in
    decode_case(fp32_variant(layer), [1, 3, 63, 64, 65, 192, 255, 256, 257, 333, 600], 62)


# 16-column tiles beyond 2048 leave the kernel that projects, rotates and appends in one launch; four wavefronts a tile below
# d_model 1024, eight from there on; both head sizes; row counts around a tile of 16
@pytest.mark.parametrize("d_model,head_dim,n_blocks", [(256, 64, 1100), (1088, 128, 700)])
def test_decode_rows_have_the_same_bits_in_the_fused_and_the_separate_projection(d_model, head_dim, n_blocks):
    from paper_2605_23296_amd.workloads import LayerConfig, Workload, make_inputs
    from tests import harness as H
    layer = LayerConfig(d_model=d_model, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, ffn_dim=128, rope_theta=10000.0, dtype="fp32")
    lens = [1 + (b * 5) % 3 for b in range(n_blocks)]
    big = make_inputs(Workload("many", layer, lens, n_blocks, 2), gain_jitter=True)
    lay = H.gpu_layer(big)
    full = H.gpu_forward(big, lay=lay)
    cu = big.cu_seqlens
    for n in (1, 15, 16, 17, 33):
        few = copy.copy(big)
        few.block_lens, few.cu_seqlens = lens[:n], cu[:n + 1]
        few.x_prefill, few.x_decode = big.x_prefill[:cu[n]].contiguous(), big.x_decode[:, :n].contiguous()
        g = H.gpu_forward(few, lay=lay)
        assert np.array_equal(g["y_decode"], full["y_decode"][:, :n]), n
        for b in (0, n - 1):
            assert np.array_equal(g["K"][b], full["K"][b]) and np.array_equal(g["V"][b], full["V"][b]), (n, b)
