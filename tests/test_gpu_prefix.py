"""Prefix-aware target-at-end layout on the GPU (paper Sec. IV, Dispatch: worker
k's prompt is blocks 1..k): the history is prefilled once as one block, then
every worker decodes against its prefix of that shared cache plus its own tail.
Checked against the fp64 checker through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2605_23296_amd import binding as B
from paper_2605_23296_amd.workloads import WORKLOADS, LayerConfig, Workload, make_inputs, to_numpy_f64
from tests import harness as H
from tests.util import ErrLog, rel_err, vec_rel_err, BF16_VEC_TOL as TOL, BF16_ELEM_TOL as ELEM_TOL

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rnd(shape, seed, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (torch.randn(shape, generator=g, dtype=torch.float32) * scale).to(torch.bfloat16).to(DEV)


def fill_cache(kv, b, K, V):
    """K, V [len, Hkv, hd] into block b of a KVCache (V goes in transposed)."""
    kv.h_len[b] = K.shape[0]
    kv.block_k(b).copy_(K)
    kv.block_v(b).copy_(V)


@pytest.mark.parametrize("wl,prefix,tail", [
    ("dense_8x4096", [100, 256, 257, 700, 700], [1, 3, 260, 1, 17]),          # group of 4: 20 columns, two column groups
    ("dense_8x4096", [512] * 2 + [513] * 3 + [1000] * 4, [2] * 9),            # 9 workers: 36 columns, three groups
    ("moe_16x8192", [64, 300, 301], [5, 1, 257]),                             # head_dim 64, group of 8
    ("dense_8x4096", [0, 0, 40], [3, 1, 2]),                                  # workers without any prefix
    ("dense_8x4096", [90 * (b + 1) for b in range(24)], [1 + b % 3 for b in range(24)]),   # 24 workers: six column groups
    # prefixes on and around item boundaries, tails that reach into further items
    ("dense_8x4096", [255, 256, 1023, 1024, 1025, 2047, 2048, 2049, 2304, 3000], [1, 2, 1030, 1, 3, 1024, 1, 2, 1025, 5]),
    ("moe_16x8192", [1023, 1025, 2300] + [2560] * 10, [1, 260, 3] + [2] * 10),            # head_dim 64: 104 columns, seven groups
    ("dense_8x4096", [1500] * 30, [1 + b % 2 for b in range(30)]),                          # 120 columns: eight column groups
    ("dense_8x4096", [40 * (b // 2) for b in range(64)], [1 + b % 4 for b in range(64)]),   # 64 workers (the most a call takes): 256 columns
])
def test_prefix_decode_attention_kernel(wl, prefix, tail):
    prefix_kernel_case(WORKLOADS[wl].layer, prefix, tail)


@pytest.mark.parametrize("heads", [(4, 4, 128), (3, 1, 128), (16, 1, 64), (6, 2, 64), (1, 1, 64)],
                         ids=lambda h: "%dq%dkv_x%d" % h)
def test_prefix_decode_attention_kernel_head_groupings(heads):
    """No grouping, odd groups, the widest group (16 query heads per KV head) and a single head, with workers
    whose prefixes end on and off the chunk edges."""
    from paper_2605_23296_amd.workloads import LayerConfig
    hq, hkv, hd = heads
    layer = LayerConfig(d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=256, rope_theta=500000.0, dtype="bf16")
    prefix_kernel_case(layer, [0, 255, 256, 257, 600, 600, 1024], [1, 2, 300, 1, 5, 1, 257])


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_prefix_decode_attention_scores_that_grow_or_fall_along_the_history(sign):
    """2^8 more (or less) per 64 shared rows: the records of a worker's chunks differ by hundreds of binary orders
    when they are merged, and the private tails (plain random keys) drown or dominate."""
    layer = WORKLOADS["dense_8x4096"].layer
    per_key = 8.0 / 64.0 / (16.0 * 1.4426950408889634 / np.sqrt(layer.head_dim))
    prefix_kernel_case(layer, [0, 100, 256, 257, 700, 1500, 1500], [3, 1, 2, 300, 1, 5, 1], grow=sign * per_key)


@pytest.mark.parametrize("wl", ["dense_8x4096", "moe_16x8192"])
def test_prefix_decode_attention_kernel_tile_edges(wl):
    """Prefixes and tails on and around the 32-row tiles, the 64-row V pairs and item edges; enough workers that the query
    columns of an item (128) overflow into a second one."""
    edges = [1, 31, 32, 33, 63, 64, 65, 96, 127, 511, 512, 513, 543, 544, 545, 1023, 1024, 1025, 1057, 1057]
    prefix_kernel_case(WORKLOADS[wl].layer, edges + [1100] * 15, [1, 2, 31, 32, 33] * 6 + [64, 65, 512, 513, 96])


@pytest.mark.parametrize("hkv,hd,group,rows", [
    (8, 128, 4, 2048), (8, 128, 4, 4096), (8, 128, 4, 4097), (8, 128, 4, 12288), (8, 128, 4, 12289),   # the lines at head_dim 128
    (8, 64, 3, 8192), (8, 64, 8, 8193), (8, 64, 8, 16385), (2, 64, 16, 32769), (16, 128, 1, 2049)])
def test_prefix_decode_attention_kernel_item_heights(hkv, hd, group, rows):
    """Work items of 128, 256 and 512 rows, chosen by the length of the history and the layer: prefixes on and around the
    item edges in histories on both sides of the lines, more columns than an item takes.  A worker alone, and the workers of
    short prefixes alone (their workspace sized for those prefixes), have the same bits."""
    layer = LayerConfig(d_model=256, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=hd, ffn_dim=256, rope_theta=500000.0, dtype="bf16")
    prefix = [0, 1, 127, 128, 129, 255, 256, 257, 384, 511, 512, 513, 767, 768, 1024, 1025] + [1500] * 20 + [min(2048, rows), rows]
    tail = [1 + (37 * b) % 70 for b in range(len(prefix))]
    tail[3:9] = [127, 128, 129, 255, 256, 257]
    every = prefix_kernel_case(layer, prefix, tail, rows=rows)
    for pick in ([len(prefix) - 1], [11], list(range(16))):
        some = prefix_kernel_case(layer, prefix, tail, rows=rows, pick=pick)
        assert np.array_equal(some, every[pick])


@pytest.mark.parametrize("hkv,hd,rows", [(32, 128, 16384), (32, 128, 16385), (32, 128, 24576), (32, 128, 24577), (64, 64, 12289), (64, 64, 18500)])
def test_prefix_decode_attention_kernel_items_beyond_512_rows(hkv, hd, rows):
    """Long histories of layers with many KV heads, which keep items of 512 rows: the cases of the other heights."""
    test_prefix_decode_attention_kernel_item_heights(hkv, hd, 1, rows)


@pytest.mark.parametrize("hkv,hd,rows,item", [(8, 128, 65536, 512), (8, 128, 65537, 1088), (8, 128, 98305, 832), (8, 64, 98305, 1088)])
def test_prefix_decode_attention_kernel_items_of_whole_rounds(hkv, hd, rows, item):
    """The line to the items that make whole rounds of workgroups, and between one round of them and two: prefixes around an
    item boundary and the whole history; a worker has the same bits alone."""
    layer = LayerConfig(d_model=512, n_q_heads=hkv, n_kv_heads=hkv, head_dim=hd, ffn_dim=512, rope_theta=1e4, dtype="bf16")
    prefix, tail = [item, item + 1, rows], [1, 40, 257]
    every = prefix_kernel_case(layer, prefix, tail, rows=rows)
    assert np.array_equal(prefix_kernel_case(layer, prefix, tail, rows=rows, pick=[1])[0], every[1])


def prefix_kernel_case(layer, prefix, tail, grow=None, rows=None, pick=None):
    """rows: length of the shared history (default: the longest prefix); pick: the workers that take part (default: all)."""
    Hq, Hkv, hd = layer.n_q_heads, layer.n_kv_heads, layer.head_dim
    lay = B.Layer(layer, None)
    T = rows or max(prefix)
    pick = list(range(len(prefix))) if pick is None else pick
    seeds = pick
    prefix, tail, N = [prefix[b] for b in pick], [tail[b] for b in pick], len(pick)
    shared = B.KVCache(layer, [max(T, 8) + 9], DEV, torch.bfloat16)
    tails = B.KVCache(layer, [t + 5 for t in tail], DEV, torch.bfloat16)
    for c in (shared, tails):
        c.k.fill_(float("nan"))
        c.v.fill_(float("nan"))
    Kp, Vp = rnd((T, Hkv, hd), 1), rnd((T, Hkv, hd), 2)
    if grow is not None:   # scores that grow along the history: k[j][0] = grow * j against q[0] = 16
        Kp[:, :, 0] = (torch.arange(T, device=Kp.device, dtype=torch.float32) * grow).to(Kp.dtype)[:, None]
    fill_cache(shared, 0, Kp, Vp)
    Kt = [rnd((t, Hkv, hd), 10 + b) for b, t in zip(seeds, tail)]
    Vt = [rnd((t, Hkv, hd), 30 + b) for b, t in zip(seeds, tail)]
    for b in range(N):
        fill_cache(tails, b, Kt[b], Vt[b])
    q = rnd((64, Hq * hd), 3)[seeds].contiguous()
    if grow is not None:
        q.view(N, Hq, hd)[:, :, 0] = 16.0
    o = torch.full((N, Hq * hd), float("nan"), dtype=torch.bfloat16, device=DEV)
    lay.ws = torch.empty(lay.prefix_workspace_bytes(N, max(max(prefix), 1), max(tail)), dtype=torch.uint8, device=DEV)
    lay.compact_attn_decode_prefix(q, shared, prefix, tails, o)
    torch.cuda.synchronize()
    got = to_numpy_f64(o).reshape(N, Hq, hd)
    assert not np.isnan(got).any()
    for b in range(N):
        K = np.concatenate([to_numpy_f64(Kp)[:prefix[b]], to_numpy_f64(Kt[b])], axis=0)
        V = np.concatenate([to_numpy_f64(Vp)[:prefix[b]], to_numpy_f64(Vt[b])], axis=0)
        ref = O.gqa_attention(to_numpy_f64(q[b]).reshape(1, Hq, hd), K, V, visible=np.array([K.shape[0]]))[0]
        assert vec_rel_err(got[b], ref) < TOL, (b, vec_rel_err(got[b], ref))
        assert rel_err(got[b], ref) < ELEM_TOL
    return got


def run_prefix_layer(inp, n_steps):
    """History prefilled as ONE block, then n_steps prefix-aware decode steps."""
    layer, cu = inp.layer, inp.cu_seqlens
    N, T = len(inp.block_lens), cu[-1]
    lay = B.Layer(layer, {k: v.to(DEV).contiguous() for k, v in inp.weights.items()})
    dt = torch.bfloat16
    shared = B.KVCache(layer, [T], DEV, dt)
    tails = B.KVCache(layer, [n_steps + 3] * N, DEV, dt)
    tails.k.fill_(float("nan"))
    tails.v.fill_(float("nan"))
    lay.ensure_workspace(T, 1, T, DEV)
    x = inp.x_prefill.to(DEV)
    y_pre = torch.empty(T, layer.d_model, dtype=dt, device=DEV)
    lay.compact_prefill([0, T], x, shared, y_pre)
    need = lay.prefix_workspace_bytes(N, T, n_steps)
    if lay.ws.numel() < need:
        lay.ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    prefix = [int(c) for c in cu[1:]]
    y_dec = torch.empty(n_steps, N, layer.d_model, dtype=dt, device=DEV)
    xd = inp.x_decode.to(DEV).contiguous()
    out = dict(y_pre=y_pre, y_dec=y_dec, shared=shared, tails=tails)
    k = layer.top_k
    if layer.n_experts:
        out["idx"] = torch.empty(n_steps, N, k, dtype=torch.int32, device=DEV)
        out["gate"] = torch.empty(n_steps, N, k, dtype=torch.float32, device=DEV)
    for s in range(n_steps):
        route = (out["idx"][s], out["gate"][s]) if layer.n_experts else None
        lay.compact_prefix_decode_step(xd[s], shared, prefix, tails, y_dec[s], route)
    torch.cuda.synchronize()
    assert tails.lens() == [n_steps] * N and shared.lens() == [T]
    return out


def check_prefix_layer(inp, n_steps, workers=None, pre_rows=None):
    g = run_prefix_layer(inp, n_steps)
    ref = O.Layer(inp.layer.as_dict(), {k: to_numpy_f64(v) for k, v in inp.weights.items()})
    x = to_numpy_f64(inp.x_prefill)
    xd = to_numpy_f64(inp.x_decode[:n_steps])
    cu = inp.cu_seqlens
    N = len(inp.block_lens)
    workers = list(range(N)) if workers is None else workers
    log = ErrLog()
    cmp = log.cmp

    pre = ref.prefill_block(x, 0, pre_rows)
    cmp("y_pre", to_numpy_f64(g["y_pre"][pre["rows"]]), pre["y"])
    cmp("Kshared", to_numpy_f64(g["shared"].block_k(0)), pre["K"])
    cmp("Vshared", to_numpy_f64(g["shared"].block_v(0)), pre["V"])
    for b in workers:
        Kt = np.zeros((0, ref.Hkv, ref.hd))
        Vt = np.zeros((0, ref.Hkv, ref.hd))
        for s in range(n_steps):
            st = ref.decode_block_prefix(xd[s, b], pre["K"], pre["V"], int(cu[b + 1]), Kt, Vt)
            Kt, Vt = st["Kt"], st["Vt"]
            cmp("y_dec%d_%d" % (s, b), to_numpy_f64(g["y_dec"][s, b]), st["y"])
        cmp("Ktail%d" % b, to_numpy_f64(g["tails"].block_k(b)), Kt)
        cmp("Vtail%d" % b, to_numpy_f64(g["tails"].block_v(b)), Vt)
    log.check()
    return g


def test_prefix_aware_layer_small_history():
    inp = make_inputs(WORKLOADS["dense_8x4096"], block_lens=[100, 157, 43, 300], decode_steps=3, gain_jitter=True)
    check_prefix_layer(inp, 3)


def test_prefix_aware_equals_lone_runs_on_truncated_histories_bitwise_in_the_tails():
    """Worker k's tail K/V rows and outputs do not depend on the workers it is batched
    with: the same prefix-aware step run with worker k alone gives the same bits."""
    inp = make_inputs(WORKLOADS["dense_8x4096"], block_lens=[200, 70, 300], decode_steps=2)
    full = run_prefix_layer(inp, 2)
    cu = inp.cu_seqlens
    import copy
    for b in range(3):
        one = copy.copy(inp)
        one.block_lens, one.cu_seqlens = [cu[b + 1]], [0, cu[b + 1]]
        one.x_prefill = inp.x_prefill[:cu[b + 1]].contiguous()
        one.x_decode = inp.x_decode[:, b:b + 1].contiguous()
        g = run_prefix_layer(one, 2)
        assert torch.equal(g["y_dec"][:, 0], full["y_dec"][:, b])
        assert torch.equal(g["tails"].block_k(0), full["tails"].block_k(b))


def test_prefix_aware_dense_8x4096_full_history():
    """The named 32 k history in 8 blocks of 4096: one 32768-token prefill, then every
    worker decodes against 4096 (b + 1) shared rows.  Workers 0, 3 and 7 are checked."""
    wl = WORKLOADS["dense_8x4096"]
    inp = make_inputs(wl, device=DEV, gen_device=DEV, decode_steps=3)
    rows = [0, 1, 127, 128, 4095, 4096, 4097, 20000, 32766, 32767]
    check_prefix_layer(inp, 3, workers=[0, 3, 7], pre_rows=rows)


def test_prefix_aware_dense_24x4096_operating_point():
    """The paper's own operating point (Sec. V, threshold x block size: a 96 k history in 4 k
    blocks, 24 workers): one 98304-token prefill, then three steps of all 24 workers, six column
    groups of the cascade kernel at prefixes of up to 98304 rows.  Workers 0, 11 and 23 and a
    few prefill rows are checked against the fp64 checker, which recomputes the whole shared cache."""
    wl = WORKLOADS["dense_24x4096"]
    inp = make_inputs(wl, device=DEV, gen_device=DEV, decode_steps=3)
    assert inp.cu_seqlens[-1] == 98304 and len(inp.block_lens) == 24
    rows = [0, 4095, 4096, 49151, 98302, 98303]
    check_prefix_layer(inp, 3, workers=[0, 11, 23], pre_rows=rows)


def test_prefix_aware_moe_layer():
    layer = LayerConfig(d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=64, ffn_dim=320, n_experts=16, top_k=4,
                        rope_theta=500000.0)
    wl = Workload("small_moe", layer, [130, 40, 77], 3, 2)
    inp = make_inputs(wl)
    g = run_prefix_layer(inp, 2)
    ref = O.Layer(layer.as_dict(), {k: to_numpy_f64(v) for k, v in inp.weights.items()})
    pre, yd, Kt, Vt = ref.forward_prefix(to_numpy_f64(inp.x_prefill), inp.cu_seqlens, to_numpy_f64(inp.x_decode))
    log, n_close = ErrLog(), 0
    for b in range(3):
        log.cmp("Ktail%d" % b, to_numpy_f64(g["tails"].block_k(b)), Kt[b])
        log.cmp("Vtail%d" % b, to_numpy_f64(g["tails"].block_v(b)), Vt[b])
    # every step's routing table against the checker's logits, every row's output for the experts the GPU chose
    Kc = [np.zeros((0, ref.Hkv, ref.hd)) for _ in range(3)]
    Vc = [np.zeros((0, ref.Hkv, ref.hd)) for _ in range(3)]
    xd = to_numpy_f64(inp.x_decode)
    for s in range(2):
        gi, gg = g["idx"][s].cpu().numpy(), g["gate"][s].cpu().numpy()
        for b in range(3):
            st = ref.decode_block_prefix(xd[s, b], pre["K"], pre["V"], int(inp.cu_seqlens[b + 1]), Kc[b], Vc[b])
            Kc[b], Vc[b] = st["Kt"], st["Vt"]
            n_close += H.check_routing(gi[b:b + 1], st["logits"][None], layer.top_k, 2e-2, gg[b:b + 1])
            log.cmp("y_dec%d_%d" % (s, b), to_numpy_f64(g["y_dec"][s, b:b + 1]), ref.ffn(st["h"][None], forced_idx=gi[b:b + 1])[0])
            assert np.array_equal(st["y"], yd[s, b])
    log.check("rows with a close call: %d of 6 (all compared) |" % n_close)
