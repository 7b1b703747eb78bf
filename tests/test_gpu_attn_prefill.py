"""Prefill attention as a prefill runs it (rotation, cache append, attention) against the fp64 definition: the edges of its
key tiles and halves, every share of the KV heads among the XCDs, references that move."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2605_23296_amd import binding as B
from paper_2605_23296_amd.workloads import LayerConfig, to_numpy_f64
from tests.test_gpu_kernels import rnd
from tests.util import rel_err, rms_err

pytestmark = pytest.mark.gpu


def run(layer, lens, qkv):
    lay = B.Layer(layer, None)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    kv = B.KVCache(layer, [L + 3 for L in lens], "cuda", torch.bfloat16)
    kv.k.fill_(float("nan"))   # rows past a block's length must never reach a result
    kv.v.fill_(float("nan"))
    o = torch.empty((int(cu[-1]), layer.Dq), dtype=torch.bfloat16, device="cuda")
    lay.check(lay.L.compact_test_rope_attn(lay.ctx, C.c_int32(len(lens)), cu.ctypes.data_as(C.POINTER(C.c_int32)),
                                           C.c_void_p(qkv.data_ptr()), C.byref(kv.c), C.c_void_p(o.data_ptr()),
                                           C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    return to_numpy_f64(o), cu


def check(layer, lens, qkv):
    x = to_numpy_f64(qkv)
    o, cu = run(layer, lens, qkv)
    Dq, Dkv, hd = layer.Dq, layer.Dkv, layer.head_dim
    for b, L in enumerate(lens):
        rows, pos = x[cu[b]:cu[b + 1]], np.arange(L)
        q = O.rope(rows[:, :Dq].reshape(L, -1, hd), pos, layer.rope_theta)
        k = O.rope(rows[:, Dq:Dq + Dkv].reshape(L, -1, hd), pos, layer.rope_theta)
        ref = O.gqa_attention(q, k, rows[:, Dq + Dkv:].reshape(L, -1, hd), visible=pos + 1).reshape(L, Dq)
        # q, k, the probabilities and the output are each rounded to 8 mantissa bits once: 0.3 % of the rms, the worst of
        # 10^6 values at five sigma (the bounds of the kernel tests beside this file)
        assert rms_err(o[cu[b]:cu[b + 1]], ref) < 6e-3, (b, L)
        assert rel_err(o[cu[b]:cu[b + 1]], ref) < 5e-2, (b, L)


# KV heads that the eight XCDs share 1, 2, 4 and 8 ways, and that they have several of; groups of 1, 2, 3, 8 and 16
@pytest.mark.parametrize("hq,hkv,hd", [(3, 1, 64), (16, 1, 64), (4, 2, 64), (9, 3, 64), (32, 4, 64), (8, 8, 64), (24, 12, 64),
                                       (2, 1, 128), (6, 2, 128), (5, 5, 128), (8, 4, 128), (16, 16, 128)])
def test_edges_of_key_tiles_and_halves(hq, hkv, hd):
    layer = LayerConfig(d_model=64, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=64, rope_theta=500000.0, dtype="bf16")
    lens = [1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 160, 191, 193, 257, 320, 449]
    check(layer, lens, rnd((sum(lens), layer.Dq + 2 * layer.Dkv), torch.bfloat16, 21))


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("step", [32, 64, 200])
def test_reference_that_moves(hd, step):
    """Scores that outgrow the reference by 2^9 every `step` keys, in the rotary pair that positions up to a thousand leave
    practically unrotated: whichever half of a tile it falls into, accumulators and the next half's scores follow."""
    layer = LayerConfig(d_model=64, n_q_heads=4, n_kv_heads=2, head_dim=hd, ffn_dim=64, rope_theta=500000.0, dtype="bf16")
    lens = [1, 70, 500, 777]
    qkv = rnd((sum(lens), layer.Dq + 2 * layer.Dkv), torch.bfloat16, 22)
    q, k = qkv[:, :layer.Dq].view(-1, 4, hd), qkv[:, layer.Dq:layer.Dq + layer.Dkv].view(-1, 2, hd)
    q[:, :, hd // 2 - 1], q[:, :, hd - 1], k[:, :, hd - 1] = 16.0, 0.0, 0.0
    j = torch.cat([torch.arange(n) for n in lens]).to(qkv.device)
    k[:, :, hd // 2 - 1] = ((j // step) * (9.0 / (16.0 * 1.4426950408889634 / np.sqrt(hd)))).to(qkv.dtype)[:, None]
    check(layer, lens, qkv)


@pytest.mark.parametrize("hq,hkv,hd,cap", [(2, 1, 128, 1 << 24), (3, 1, 128, (1 << 25) + 8), (2, 1, 64, 1 << 25), (1, 1, 64, (1 << 26) + 72)])
def test_slabs_of_4_gib_and_more_per_kv_head(hq, hkv, hd, cap):
    """Offsets inside a KV head's slab leave 32 bits at 4 GiB (2^24 rows of 128, 2^25 of 64): a block's result has the bits that it
    has in a small slab, wherever in the call the large slab stands."""
    layer = LayerConfig(d_model=64, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=64, rope_theta=500000.0, dtype="bf16")
    lens = [65, 333, 40]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    qkv = rnd((sum(lens), layer.Dq + 2 * layer.Dkv), torch.bfloat16, 23)
    out = []
    for caps in ([72, 336, 40], [72, cap, 40]):
        lay, kv = B.Layer(layer, None), B.KVCache(layer, caps, "cuda", torch.bfloat16)
        x, o = qkv.clone(), torch.empty((sum(lens), layer.Dq), dtype=torch.bfloat16, device="cuda")
        lay.compact_rope_kvwrite(cu, x, kv)
        lay.compact_attn_prefill(cu, x, kv, o)
        torch.cuda.synchronize()
        out.append(o)
        del kv
    torch.cuda.empty_cache()
    assert bool(torch.isfinite(out[0].float()).all()) and torch.equal(out[1], out[0])


def test_more_workgroups_than_one_grid_dimension_takes():
    """2^18 + 1 blocks of one token at 64 query heads are more than the 2^24 workgroups of 256 that a grid's first dimension holds.
    A token that attends itself alone gives its value row back, exactly."""
    layer = LayerConfig(d_model=64, n_q_heads=64, n_kv_heads=4, head_dim=64, ffn_dim=64, rope_theta=500000.0, dtype="bf16")
    n = (1 << 18) + 1
    qkv = rnd((n, layer.Dq + 2 * layer.Dkv), torch.bfloat16, 24)
    lay, kv = B.Layer(layer, None), B.KVCache(layer, [1] * n, "cuda", torch.bfloat16)
    o, cu = torch.zeros((n, layer.Dq), dtype=torch.bfloat16, device="cuda"), np.arange(n + 1, dtype=np.int32)
    lay.check(lay.L.compact_test_rope_attn(lay.ctx, C.c_int32(n), cu.ctypes.data_as(C.POINTER(C.c_int32)), C.c_void_p(qkv.data_ptr()),
                                           C.byref(kv.c), C.c_void_p(o.data_ptr()), C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    v = qkv[:, layer.Dq + layer.Dkv:].view(n, 4, 1, 64).expand(n, 4, 16, 64).reshape(n, layer.Dq)
    assert torch.equal(o, v)


def weight_of_one_key(hd, key, size=0.5, rivals=()):
    """A block of 160 tokens whose values are zero but for one key's, and whose scores are zero but for that key's, `size` times
    4 .. 12, and those of `rivals` (key, size): the query and key entries lie in the rotary pair that these positions leave where
    it is.  Returns output and its fp64 value."""
    layer = LayerConfig(d_model=64, n_q_heads=8, n_kv_heads=2, head_dim=hd, ffn_dim=64, rope_theta=500000.0, dtype="bf16")
    L, gen = 160, torch.Generator().manual_seed(25)
    qkv = torch.zeros((L, layer.Dq + 2 * layer.Dkv), dtype=torch.bfloat16, device="cuda")
    q, k = qkv[:, :layer.Dq].view(L, 8, hd), qkv[:, layer.Dq:layer.Dq + layer.Dkv].view(L, 2, hd)
    q[:, :, hd // 2 - 1] = (4.0 + 8.0 * torch.rand((L, 8), generator=gen)).to(torch.bfloat16).cuda()
    for j, f in ((key, size),) + tuple(rivals):
        k[j, :, hd // 2 - 1] = f * np.sqrt(hd)
    qkv[key, layer.Dq + layer.Dkv:] = rnd((layer.Dkv,), torch.bfloat16, 26)
    x = to_numpy_f64(qkv)
    o, _ = run(layer, [L], qkv)
    pos = np.arange(L)
    rot = lambda lo, hi: O.rope(x[:, lo:hi].reshape(L, -1, hd), pos, layer.rope_theta)
    ref = O.gqa_attention(rot(0, layer.Dq), rot(layer.Dq, layer.Dq + layer.Dkv), x[:, layer.Dq + layer.Dkv:].reshape(L, -1, hd), visible=pos + 1)
    return o[key:], ref.reshape(L, layer.Dq)[key:]


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("key", [0, 1, 13, 31])
def test_a_query_is_rounded_only_by_its_rotation(hd, key):
    """A query that its rotation leaves a bf16 value goes into the scores as it is, and the largest weight is the reference's own, 1:
    the output is the fp64 value rounded once, but for the fp32 sums (2^-21 of it; a rounding differs in one of 2^12 places) and
    the rotation (angles up to 5e-4 move score and value by 1e-6)."""
    o, ref = weight_of_one_key(hd, key)
    want = torch.from_numpy(ref).to(torch.float32).to(torch.bfloat16).double().numpy()
    assert float((o != want).mean()) < 5e-3


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("key", [32, 45, 63])
def test_the_largest_weight_of_the_first_key_tile_is_one(hd, key):
    """The softmax's first reference is the largest score of 64 keys, not of the first 32: the largest weight among them is 1 and is
    not rounded."""
    o, ref = weight_of_one_key(hd, key)
    want = torch.from_numpy(ref).to(torch.float32).to(torch.bfloat16).double().numpy()
    assert float((o != want).mean()) < 5e-3


@pytest.mark.parametrize("hd", [64, 128])
def test_probabilities_are_summed_tile_by_tile(hd):
    """Key 0 alone has a score and a value, and a rotation of none, so that every step in fp32 is known (the exponential is the
    hardware's exp2, which torch.exp2 calls too): a lane has the keys whose number's bit 3 is its own, sums a tile's 32 one after
    the other and adds the tiles.  The output has exactly those bits; sums of half tiles would change some."""
    layer = LayerConfig(d_model=64, n_q_heads=32, n_kv_heads=8, head_dim=hd, ffn_dim=64, rope_theta=500000.0, dtype="bf16")
    L, gen, f32 = 700, torch.Generator().manual_seed(27), np.float32
    qkv = torch.zeros((L, layer.Dq + 2 * layer.Dkv), dtype=torch.bfloat16, device="cuda")
    qv = (4.0 + 8.0 * torch.rand((L, 32), generator=gen)).to(torch.bfloat16)
    qkv[:, :layer.Dq].view(L, 32, hd)[:, :, hd // 2 - 1] = qv.cuda()
    qkv[0, layer.Dq:layer.Dq + layer.Dkv].view(8, hd)[:, hd // 2 - 1] = 4.0
    qkv[0, layer.Dq + layer.Dkv:] = rnd((layer.Dkv,), torch.bfloat16, 28)
    v0 = np.repeat(qkv[0, layer.Dq + layer.Dkv:].float().cpu().numpy().reshape(8, hd), 4, axis=0)

    scale = f32(f32(1.4426950408889634) / f32(np.sqrt(hd)))
    s = qv.double().numpy() * 4.0
    ref = (s * np.float64(scale)).astype(f32)
    exp2 = lambda x: torch.exp2(torch.from_numpy(x.astype(f32)).cuda()).cpu().numpy()
    first, others = exp2(s * np.float64(scale) - ref), exp2(-ref)
    got = qkv.clone()
    o, _ = run(layer, [L], got)

    def outputs(keys):   # sums of `keys` keys at a time
        total = []
        for lane in (0, 1):
            t = np.zeros((L, 32), f32)
            for k0 in range(0, L, keys):
                part = np.zeros((L, 32), f32)
                for k in (k for k in range(k0, min(k0 + keys, L)) if k >> 3 & 1 == lane):
                    part[k:] += first[k:] if k == 0 else others[k:]
                t += part
            total.append(t)
        inv = f32(1) / (total[0] + total[1])
        return torch.from_numpy(v0[None] * inv[:, :, None]).to(torch.bfloat16).double().numpy().reshape(L, -1)

    want = outputs(64)
    assert int((outputs(32) != want).sum()) > 5
    assert np.array_equal(o, want), int((o != want).sum())


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("key", [96, 104, 127])
def test_a_reference_that_moves_takes_the_whole_tile(hd, key):
    """The reference moves at the first half of the second tile, by a key 2^13 and more above what came before: to the largest
    score of the tile, which lies in its second half, so that this key's weight is 1."""
    o, ref = weight_of_one_key(hd, key, 2.5, ((70, 2.25),))
    want = torch.from_numpy(ref).to(torch.float32).to(torch.bfloat16).double().numpy()
    assert float((o != want).mean()) < 5e-3
