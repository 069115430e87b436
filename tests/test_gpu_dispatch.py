"""GPU parity at the sizes where the choices between kernels and work splits change (against the fp64 oracle)."""
import numpy as np
import pytest
import torch

import paper_2510_09608_amd as sv
import sv_inputs as si
from oracle import sv_oracle as orc
from oracle import sv_step
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
PLAIN, TERMS = sv.SV_CHUNK_F32_PLAIN, sv.SV_CHUNK_F32_TERMS


def attn_case(dtype, hq, hkv, d, n_kv, n_q, causal, seed, splits=0):
    """One sv_attn_chunk against the oracle; returns the cache with its inputs for further calls."""
    print(f"attn_chunk {dtype} {hq}/{hkv} x {d} n_kv={n_kv} n_q={n_q} causal={causal} splits={splits}", flush=True)
    w = si.Workload("d", 1, hq, hkv, d, dtype, 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, seed)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4,
                     (0, 0, 0), 1, n_kv + 8, max(n_q, 1))
    cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
    q, k, v = w.qkv(0, np.arange(n_kv))
    q = q[n_kv - n_q:]
    cache.append(0, 0, np.zeros(n_kv, dtype=np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    qd = gu.dev(q, w)
    od = torch.empty_like(qd)
    cache.attn_chunk(0, 0, qd, od, causal)
    ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64),
                            np.arange(n_kv - n_q, n_kv), causal)
    err = gu.max_err(gu.host(od), ref)
    assert err <= gu.TOL[dtype], err
    return cache, w, q, k, v


@pytest.mark.parametrize("hq,hkv,n", [(32, 8, 2305), (28, 4, 1203), (6, 3, 900), (5, 5, 70)])
def test_whole_window_prefill_longest_rows_first(hq, hkv, n):
    """Causal prefill of a whole window in one key range: row tiles go out longest first, heads in turn (more and
    fewer workgroups than CUs, head counts that do and do not divide 8, a ragged last row tile)."""
    attn_case("bf16", hq, hkv, 128, n, n, True, 4000 + n, splits=1)
    attn_case("bf16", hq, hkv, 128, n, n, True, 4000 + n)


@pytest.mark.parametrize("dtype,mode", [("bf16", sv.SV_ROPE_3D), ("f32", sv.SV_ROPE_1D)])
def test_tokens_of_a_batch_registered_together(dtype, mode):
    """Ids, positions and stored K of the decode steps of several streams, listed out of order, one of them evicted
    (the other half of its ping-pong store is live) and one left out of some steps."""
    hq, hkv, d = (28, 4, 128) if dtype == "bf16" else (2, 1, 64)
    sec = ((16, 24, 24) if d == 128 else (8, 12, 12)) if mode == sv.SV_ROPE_3D else (0, 0, 0)
    w = si.Workload("b", 1, hq, hkv, d, dtype, mode, 1e4, sec, 0, 0, 0, 0, 0, 0, None, 0, 91)
    n_streams, vis = 3, (2, 3, 4)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, mode, 1e4, sec, n_streams, 96, 32)
    text0 = (5, 9, 17)
    for s in range(n_streams):
        _, k, v = w.qkv(0, np.arange(text0[s]))
        cache.append(s, 0, np.zeros(text0[s], np.uint8), None, gu.dev(k, w), gu.dev(v, w))
        _, k, v = w.qkv(0, np.arange(24))
        cache.append(s, 0, np.ones(24, np.uint8), vis, gu.dev(k, w), gu.dev(v, w))
    cache.evict(1, 3, 24, 2)
    kept, new_k = {0: 5 + 24, 1: 5 + 24, 2: 17 + 24}, {0: [], 1: [], 2: []}
    for step, ids in enumerate(([2, 0, 1], [1, 2], [0, 1, 2])):
        q, k, v = w.qkv(0, np.arange(1000 + 10 * step, 1000 + 10 * step + len(ids)))
        for s, row in zip(ids, k):
            new_k[s].append(row)
        q, k, v = gu.dev(q, w), gu.dev(k, w), gu.dev(v, w)
        cache.decode_step(0, ids, q, k, v, torch.empty_like(q))
        print(f"step {step} {ids}", flush=True)
    n_dec = {0: 2, 1: 3, 2: 3}
    for s in range(n_streams):
        ids, pos = cache.retained(s)
        n0, n = kept[s], n_dec[s]
        assert len(ids) == n0 + n
        first = text0[s] + 24
        assert list(ids[n0:]) == list(range(first, first + n))
        base = n0 if mode == sv.SV_ROPE_1D else n0 - 24 + max(vis)   # a vision block advances by its extent
        assert pos[n0:].tolist() == [[base + i] * 3 for i in range(n)]
        want = orc.rope(np.stack(new_k[s]), np.asarray(pos[n0:]), mode, 1e4, sec)
        assert gu.max_err(cache.read_kv(s, 0, 0, n0, n), want) <= (4e-2 if dtype == "bf16" else 1e-5)


# ---- head_dim 64 / single precision on the matrix cores ------------------------------------------------------------

@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 16, 2, 64), ("bf16", 5, 5, 64), ("bf16", 21, 3, 64),
                                           ("f32", 8, 2, 128), ("f32", 2, 1, 64), ("f32", 12, 2, 64), ("f32", 21, 3, 128)])
@pytest.mark.parametrize("n_kv,n_q,causal,splits", [
    (1, 1, True, 0), (64, 64, True, 0), (65, 33, True, 0), (1333, 300, True, 3), (777, 100, False, 2), (2500, 257, True, 0)])
def test_chunk_and_decode_of_every_matrix_core_layout(dtype, hq, hkv, d, n_kv, n_q, causal, splits):
    """Chunk prefill and, on the same cache, one decode token: ragged rows, keys and ranges of each instantiation."""
    cache, w, q, k, v = attn_case(dtype, hq, hkv, d, n_kv, n_q, causal, 5000 + n_kv + hq, splits)
    qd = gu.dev(q[-1:], w)
    od = torch.empty_like(qd)
    cache.attn_decode(0, [0], qd, od)
    ref = orc.gqa_attention(q[-1:].astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.array([n_kv - 1]), True)
    assert gu.max_err(gu.host(od), ref) <= gu.TOL[dtype]


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (16, 2, 64), (12, 12, 128)])
@pytest.mark.parametrize("n_kv,n_q,causal", [(128, 16, True), (129, 128, True), (193, 7, False), (257, 64, True),
                                             (700, 64, True), (640, 640, True)])
def test_chunk_on_ranges_of_two_tiles(hq, hkv, d, n_kv, n_q, causal):
    """Chunks on few keys, cut into ranges of two key tiles: ranges the mask leaves nothing of, a last one of one key."""
    attn_case("bf16", hq, hkv, d, n_kv, n_q, causal, 8000 + n_kv + hq)


@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 14, 2, 64), ("f32", 8, 2, 128), ("f32", 2, 1, 64)])
@pytest.mark.parametrize("mode,grid,n_text,preamble,budgets,store", [
    (1, (1, 16, 16), 4, 48, (32, 600, 40), 0), (1, (1, 7, 5), 3, 51, (9, 100, 11), 2), (0, (2, 3, 3), 5, 13, (4, 50, 9), 1),
    (1, (1, 17, 16), 5, 77, (50, 1000, 21), 2)])
def test_stream_seconds_of_every_matrix_core_layout(dtype, hq, hkv, d, mode, grid, n_text, preamble, budgets, store):
    """Six seconds through sv_stream_step on a two-layer cache: outputs, ids, positions and the stored K and V rows
    against the oracle (blocks of V that evictions cut, runs that start inside a block, both ways to store a chunk)."""
    sec = ((16, 24, 24) if d == 128 else (8, 12, 12)) if mode == 1 else (0, 0, 0)
    n_sink, vw, tw = budgets
    nv = grid[0] * grid[1] * grid[2]
    w = si.Workload("t", 2, hq, hkv, d, dtype, mode, 1.0e4, sec, n_sink, vw, tw, preamble, nv, n_text,
                    grid if mode == 1 else None, 6, 6000 + nv)
    bf, layers, tol = dtype == "bf16", [0, 1], gu.TOL[dtype]
    cache = gu.make_cache(w, n_layers=2, capacity=w.capacity() + 64)
    cache.set_option(sv.SV_OPT_CHUNK_STORE, store)
    o = sv_step.new_stream(w, layers)
    sv_step.append_preamble(o, w, layers)
    stack = lambda which, g, heads: torch.stack([gu.dev(si.normal(w.seed, which, l, g, heads, d, bf), w) for l in layers])
    gids = np.arange(preamble)
    gu.StreamRunner(cache, *budgets).preamble(list(stack(si.TENSOR_K, gids, hkv)), list(stack(si.TENSOR_V, gids, hkv)))
    for c in range(w.n_chunks):
        print(f"{dtype} d{d} mode {mode} grid {grid} chunk {c}", flush=True)
        ro = sv_step.step_chunk(o, w, c, layers)
        ch = w.chunk(c)
        gv, gt = np.arange(ch.vision.gid0, ch.vision.gid0 + nv), np.arange(ch.text_gid0, ch.text_gid0 + n_text)
        qv, kv, vv = (stack(x, gv, h) for x, h in ((si.TENSOR_Q, hq), (si.TENSOR_K, hkv), (si.TENSOR_V, hkv)))
        qt, kt, vt = (stack(x, gt, h).transpose(0, 1).contiguous()
                      for x, h in ((si.TENSOR_Q, hq), (si.TENSOR_K, hkv), (si.TENSOR_V, hkv)))
        ov, ot = torch.empty_like(qv), torch.empty_like(qt)
        n_ret = cache.stream_step(0, *budgets, q_vision=qv, k_vision=kv, v_vision=vv, o_vision=ov,
                                  grid_thw=ch.vision.grid_thw, q_text=qt, k_text=kt, v_text=vt, o_text=ot)
        assert n_ret == ro["n_retained"]
        n, pos = len(o), o.positions()
        for j in layers:
            assert gu.max_err(gu.host(ov[j]), ro["prefill"][j]) <= tol, (c, j)
            for t in range(n_text):
                assert gu.max_err(gu.host(ot[t, j]), ro["decode"][t][j][0]) <= tol, (c, j, t)
            K, V = np.stack(o.k[j]), np.stack(o.v[j])
            assert np.array_equal(cache.read_kv(0, j, 1, 0, n).astype(np.float64), V), (c, j)
            e = gu.max_err(cache.read_kv(0, j, 0, 0, n), orc.rope(K, pos, mode, w.rope_theta, sec))
            assert e <= (4e-2 if bf else 1e-5) * (1 + c), (c, j, e)
        ids, p2 = cache.retained(0)
        assert np.array_equal(ids, np.asarray(ro["gids_end"])) and np.array_equal(p2, ro["pos_end"])


# ---- batches: one list of blocks cut into equal runs ----------------------------------------------------------------

def batch_ref(q, kv, lens, g):
    """fp64 attention of one query row per stream over the first lens[b] keys of its K and V [n, Hkv, d]."""
    out = []
    for b, n in enumerate(lens):
        out.append(orc.gqa_attention(q[b:b + 1].astype(np.float64), kv[b][0][:n].astype(np.float64),
                                     kv[b][1][:n].astype(np.float64), np.array([n - 1]), True)[0])
    return np.stack(out)


@pytest.mark.parametrize("hq,hkv,d,lens", [
    (28, 4, 128, [1, 127, 128, 129, 2000, 640]),                      # fewer blocks than CUs, groups of one block
    (28, 4, 128, [9000, 300, 4097, 128, 5000, 1, 2500]),              # long runs, whole groups inside a run
    (16, 2, 128, [4096] * 16),                                        # groups and runs end together
    (12, 12, 128, [700, 1500]), (8, 8, 64, [3000, 100, 1]), (14, 2, 64, [2300, 5000, 64]),
    (7, 1, 128, [150 + 37 * i for i in range(40)]),                   # more rows than the small table holds
    (3, 1, 128, [20000, 20000])])
def test_decode_batch_runs(hq, hkv, d, lens):
    """sv_attn_decode (arena and static scratch), then a fused sv_decode_step, of a batch; shorter and longer batches of
    the same cache in between, so that the slots of one launch are not those of the next."""
    w = si.Workload("r", 1, hq, hkv, d, "bf16", 0, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 7000 + hq + len(lens))
    n_s = len(lens)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_1D, 1e4, (0, 0, 0), n_s, max(lens) + 8, 16)
    base = w.qkv(0, np.arange(max(lens)))
    kv = []
    for b, n in enumerate(lens):
        k, v = np.roll(base[1], 13 * b, axis=0)[:n], np.roll(base[2], 29 * b, axis=0)[:n]
        kv.append((orc.rope(k, np.repeat(np.arange(n)[:, None], 3, 1), 0, 1e4, (0, 0, 0)), v))
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    q = w.qkv(0, np.arange(50000, 50000 + n_s))[0]
    qd = gu.dev(q, w)
    want = batch_ref(q, kv, lens, hq // hkv)
    for fn in (cache.attn_decode, cache.attn_decode_static):
        for ids in (list(range(n_s)), [0, n_s - 1], list(range(n_s))[::-1], [n_s - 1] * 3, list(range(n_s))):
            print(f"decode batch {hq}/{hkv} x {d} rows {len(ids)} {fn.__name__}", flush=True)
            qi = qd[torch.tensor(ids, device=qd.device)].contiguous()
            od = torch.full_like(qi, float("nan"))
            fn(0, ids, qi, od)
            assert gu.max_err(gu.host(od), want[ids]) <= gu.TOL["bf16"]
    qn, kn, vn = w.qkv(0, np.arange(60000, 60000 + n_s))
    od = torch.full_like(qd, float("nan"))
    cache.decode_step(0, list(range(n_s)), gu.dev(qn, w), gu.dev(kn, w), gu.dev(vn, w), od)
    kv2, qr = [], []
    for b, n in enumerate(lens):
        pos = np.full((1, 3), n)
        kv2.append((np.concatenate([kv[b][0], orc.rope(kn[b:b + 1], pos, 0, 1e4, (0, 0, 0))]), np.concatenate([kv[b][1], vn[b:b + 1]])))
        qr.append(orc.rope(qn[b:b + 1], pos, 0, 1e4, (0, 0, 0))[0])
    assert gu.max_err(gu.host(od), batch_ref(np.stack(qr), kv2, [n + 1 for n in lens], hq // hkv)) <= gu.TOL["bf16"]


def test_decode_batch_more_groups_than_static_slots():
    """60 rows of 64 kv heads in the static array, which has slots for 492 pieces: every group is one workgroup's."""
    w = si.Workload("r", 1, 64, 64, 128, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 7100)
    lens = [3 + 5 * i for i in range(60)]
    cache = sv.Cache(1, 64, 64, 128, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 60, max(lens) + 8, 16)
    kv = []
    for b, n in enumerate(lens):
        _, k, v = w.qkv(0, np.arange(400 * b, 400 * b + n))
        kv.append((k, v))
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    q = w.qkv(0, np.arange(50000, 50060))[0]
    want = batch_ref(q, kv, lens, 1)
    for fn in (cache.attn_decode_static, cache.attn_decode, cache.attn_decode_static):
        print(fn.__name__, flush=True)
        od = torch.full((60, 64, 128), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        fn(0, list(range(60)), gu.dev(q, w), od)
        assert gu.max_err(gu.host(od), want) <= gu.TOL["bf16"]


@pytest.mark.parametrize("hkv,d,sink", [(2, 64, 0), (4, 128, 3)])
def test_values_behind_a_removed_run_of_any_length(hkv, d, sink):
    """V rows, bit for bit, after evictions that remove runs of 1 .. 9 and 35 tokens behind the sink: their new blocks of
    8 are shifted out of two old ones (every shift), a copy of one, or gathered across the run's end; ragged last block."""
    n = 150
    w = si.Workload("c", 1, hkv, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 93)
    cache = sv.Cache(1, hkv, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, 256, n)
    _, k, v = w.qkv(0, np.arange(n))
    cache.append(0, 0, np.zeros(n, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    kept = np.arange(n)
    for run in (1, 2, 3, 4, 5, 6, 7, 8, 9, 35):
        print(f"evict a run of {run} of {kept.size}", flush=True)
        kept = np.concatenate([kept[:sink], kept[sink + run:]])
        assert cache.evict(0, sink, 0, kept.size - sink) == kept.size
        assert np.array_equal(cache.read_kv(0, 0, 1, 0, kept.size), v[kept]) and \
            np.array_equal(cache.read_kv(0, 0, 0, 0, kept.size), k[kept]), run


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (16, 2, 64)])
@pytest.mark.parametrize("n_old,grid,splits", [
    (20, (1, 5, 9), 0), (64, (1, 1, 1), 2), (127, (1, 13, 19), 2), (700, (1, 13, 19), 5), (1981, (2, 16, 16), 3),
    (3000, (1, 13, 19), 0), (2048, (1, 16, 16), 7)])
def test_last_range_of_the_new_keys(hq, hkv, d, n_old, grid, splits):
    """A second whose attention launch stores the chunk (the last key range begins at the new keys, at, just below or a
    tile below the retained ones' end) against the same second with a store launch of its own and ranges all alike."""
    w = si.Workload("s", 1, hq, hkv, d, "bf16", 1, 1e6, (16, 24, 24) if d == 128 else (8, 12, 12), 0, 0, 0, 0, 0, 0, None, 0, 97)
    n = grid[0] * grid[1] * grid[2]
    _, k0, v0 = w.qkv(0, np.arange(n_old))
    q, k, v = w.qkv(0, np.arange(n_old, n_old + n))
    got = []
    for store in (1, 2):
        cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, 1, 1e6, w.mrope_sections, 1, n_old + n + 8, n)
        cache.set_option(sv.SV_OPT_CHUNK_STORE, store)
        cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
        cache.append(0, 0, np.zeros(n_old, np.uint8), None, gu.dev(k0, w), gu.dev(v0, w))
        qd, kd, vd = (gu.dev(x, w).unsqueeze(0).contiguous() for x in (q, k, v))
        o = torch.full_like(qd, float("nan"))
        print(f"store={store} {hq}/{hkv}x{d} {n_old}+{n} splits={splits}", flush=True)
        cache.stream_step(0, 0, sv.SV_WINDOW_INF, sv.SV_WINDOW_INF, q_vision=qd, k_vision=kd, v_vision=vd, o_vision=o, grid_thw=grid)
        got.append((gu.host(o), cache.read_kv(0, 0, 0, 0, n_old + n), cache.read_kv(0, 0, 1, 0, n_old + n)))
    assert gu.max_err(got[1][0], got[0][0]) <= gu.TOL["bf16"]
    assert gu.max_err(got[1][1], got[0][1]) <= 4e-2 and np.array_equal(got[1][2], got[0][2])


@pytest.mark.parametrize("hq,hkv,d,n_kv,n_q,causal,splits", [
    (2, 1, 64, 72, 16, True, 0), (2, 1, 64, 40, 32, True, 1), (2, 1, 64, 200, 33, True, 0), (8, 2, 128, 1333, 8, True, 0),
    (8, 2, 128, 500, 16, True, 3), (8, 2, 128, 129, 16, False, 1), (5, 5, 128, 3000, 64, True, 0), (5, 5, 64, 31, 1, True, 0),
    (5, 5, 64, 777, 65, True, 0), (12, 2, 64, 2500, 10, False, 0), (28, 4, 128, 5000, 4, True, 0), (28, 4, 128, 97, 9, True, 2)])
def test_fp32_chunk_of_few_rows(hq, hkv, d, n_kv, n_q, causal, splits):
    """fp32 chunk prefill with up to 64 rows per kv head (the wavefronts share them and deal out the tiles) and just above:
    one to all wavefronts with a tile, rows that see nothing of a range, ragged last rows and tiles."""
    attn_case("f32", hq, hkv, d, n_kv, n_q, causal, 7000 + n_kv, splits)


# ---- merges inside a decode launch that do not wait for each other ---------------------------------------------------

@pytest.mark.parametrize("dtype,hq,hkv,d,lens", [
    ("bf16", 28, 4, 128, [5392]), ("bf16", 28, 4, 128, [300]), ("bf16", 16, 2, 64, [5392]), ("bf16", 64, 64, 128, [300]),
    ("bf16", 3, 1, 128, [20000]), ("f32", 8, 2, 128, [5392]), ("f32", 2, 1, 64, [130]), ("bf16", 8, 8, 64, [9000]),
    ("bf16", 28, 4, 128, [9000, 300, 4097, 128, 5000, 1, 2500]), ("bf16", 7, 1, 128, [150 + 37 * i for i in range(40)]),
    ("bf16", 3, 1, 128, [20000, 20000]), ("bf16", 14, 2, 64, [2300, 5000, 64])])
def test_decode_merge_left_to_late_workgroups(dtype, hq, hkv, d, lens):
    """Workgroups that look for the others' results once and then leave their share of the merge to whoever publishes later:
    bit for bit the result of those that wait, launch after launch (a header that ran ahead, or words taken for those of the
    launch before, would show in the next), on shorter rows in between, and beside another stream's work."""
    w = si.Workload("l", 1, hq, hkv, d, dtype, 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9400 + len(lens))
    n_s = len(lens)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0),
                     n_s + 1, max(lens) + 8, 16)
    _, k, v = w.qkv(0, np.arange(max(lens)))
    for b, n in enumerate(lens + [max(1, min(lens) // 2)]):
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k[:n], w), gu.dev(v[:n], w))
    ids, short = list(range(n_s)), [n_s]
    q = [gu.dev(x, w) for x in w.qkv(0, np.arange(60000, 60000 + 6 * (n_s + 1)))[0].reshape(6, n_s + 1, hq, d)]

    def launches(fn, looks, beside):
        cache.set_option(sv.SV_OPT_DECODE_TILES_PER_WAVE, looks)
        out = []
        for i in range(24):
            if beside and i % 4 == 0:
                other.wait_stream(torch.cuda.current_stream())
                with torch.cuda.stream(other):
                    a @ a
            x = q[i % 6]
            o = torch.full_like(x, float("nan"))
            fn(0, ids, x[:n_s], o[:n_s])
            if i % 3 == 0:
                fn(0, short, x[n_s:], o[n_s:])
            out.append(o)
        torch.cuda.synchronize()
        return out
    other, a = torch.cuda.Stream(), torch.randn(2048, 2048, device="cuda:0")
    fns = [cache.attn_decode] + ([cache.attn_decode_static] if dtype == "bf16" else [])
    for fn in fns:
        print(f"{dtype} {hq}/{hkv} x {d} {lens[:3]} {fn.__name__}", flush=True)
        want = launches(fn, 0, False)
        assert not torch.isnan(want[1][:n_s]).any()
        for beside in (False, True, False):
            got = launches(fn, sv.SV_MERGE_ONE_LOOK, beside)
            for i, (x, y) in enumerate(zip(got, want)):
                assert torch.equal(x[:n_s], y[:n_s]) and (i % 3 or torch.equal(x[n_s:], y[n_s:])), (fn.__name__, beside, i)


@pytest.mark.parametrize("hq,hkv,d,n_s,layers", [(28, 4, 128, 1, 1), (16, 2, 64, 2, 1), (8, 8, 128, 1, 3)])
def test_decode_lists_longer_than_the_arena_has_rows_for(hq, hkv, d, n_s, layers):
    """Lists that name a stream more than once, longer than the number of streams and of layers: several launches."""
    lens = [900, 333][:n_s]
    w = si.Workload("a", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9600)
    cache = sv.Cache(layers, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), n_s, 1000, 16)
    _, k, v = w.qkv(0, np.arange(900))
    for b, n in enumerate(lens):
        for layer in range(layers):
            cache.append(b, layer, np.zeros(n, np.uint8) if layer == 0 else None, None, gu.dev(k[:n], w), gu.dev(v[:n], w))
    ids = [(3 * i) % n_s for i in range(7)]
    q = w.qkv(0, np.arange(60000, 60007))[0]
    o = torch.full((7, hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
    print(f"{hq}/{hkv} x {d}: {ids} of {n_s} streams, {layers} layers", flush=True)
    cache.attn_decode(0, ids, gu.dev(q, w), o)
    want = batch_ref(q, [(k, v)] * 7, [lens[i] for i in ids], hq // hkv)
    assert gu.max_err(gu.host(o), want) <= gu.TOL["bf16"]


# ---- values of kernels that other tests reach by shape only -----------------------------------------------------------

@pytest.mark.parametrize("hq,hkv,d,lens", [
    (8, 2, 128, [1, 15, 16, 17, 64, 65, 500]), (2, 1, 64, [700, 3]), (21, 3, 128, [1500, 129, 128]),
    (7, 1, 64, [40 + 13 * i for i in range(70)]),                      # more rows than one launch takes
    # 101 MB of K and V and more: non-temporal loads, one to four and more heads per kv head
    (8, 8, 128, [7000, 6000]), (56, 8, 128, [7000, 6000]), (16, 8, 64, [13000, 11800]), (40, 8, 64, [13000, 11800])])
def test_fp32_decode_batch_values(hq, hkv, d, lens):
    """Several fp32 rows in a launch: sv_attn_decode, then a fused sv_decode_step with the K and V it stores (rows of one
    tile, of one key range, of many, and their merge)."""
    w = si.Workload("f", 1, hq, hkv, d, "f32", 0, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9700 + len(lens))
    n_s = len(lens)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32, sv.SV_ROPE_1D, 1e4, (0, 0, 0), n_s, max(lens) + 2, 16)
    base, kv = w.qkv(0, np.arange(max(lens))), []
    for b, n in enumerate(lens):
        k, v = np.roll(base[1], 13 * b, axis=0)[:n], np.roll(base[2], 29 * b, axis=0)[:n]
        kv.append((orc.rope(k, np.repeat(np.arange(n)[:, None], 3, 1), 0, 1e4, (0, 0, 0)), v))
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    q = w.qkv(0, np.arange(50000, 50000 + n_s))[0]
    print(f"fp32 decode batch {hq}/{hkv} x {d} rows {n_s}", flush=True)
    ids = list(range(n_s))
    od = torch.full((n_s, hq, d), float("nan"), device="cuda:0")
    cache.attn_decode(0, ids, gu.dev(q, w), od)
    assert gu.max_err(gu.host(od), batch_ref(q, kv, lens, hq // hkv)) <= gu.TOL["f32"]
    qn, kn, vn = w.qkv(0, np.arange(60000, 60000 + n_s))
    od = torch.full((n_s, hq, d), float("nan"), device="cuda:0")
    cache.decode_step(0, ids, gu.dev(qn, w), gu.dev(kn, w), gu.dev(vn, w), od)
    kv2, qr = [], []
    for b, n in enumerate(lens):
        pos = np.full((1, 3), n)
        kr = orc.rope(kn[b:b + 1], pos, 0, 1e4, (0, 0, 0))
        kv2.append((np.concatenate([kv[b][0], kr]), np.concatenate([kv[b][1], vn[b:b + 1]])))
        qr.append(orc.rope(qn[b:b + 1], pos, 0, 1e4, (0, 0, 0))[0])
        assert gu.max_err(cache.read_kv(b, 0, 0, n, 1), kr) <= 1e-5 and np.array_equal(cache.read_kv(b, 0, 1, n, 1), vn[b:b + 1])
    assert gu.max_err(gu.host(od), batch_ref(np.stack(qr), kv2, [n + 1 for n in lens], hq // hkv)) <= gu.TOL["f32"]


@pytest.mark.parametrize("hq,d,n", [(8, 128, 12400), (56, 128, 12400), (16, 64, 24700), (40, 64, 24700)])
def test_fp32_decode_of_one_long_stream(hq, d, n):
    """101 MB of 8 kv heads: the single-stream kernels (one to four heads per kv head, and more) with non-temporal loads."""
    cache, w, q, k, v = attn_case("f32", hq, 8, d, n, 1, True, 9800)
    qd = gu.dev(q, w)
    od = torch.empty_like(qd)
    cache.attn_decode(0, [0], qd, od)
    ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.array([n - 1]), True)
    assert gu.max_err(gu.host(od), ref) <= gu.TOL["f32"]


@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 16, 2, 64), ("f32", 8, 2, 128), ("f32", 8, 8, 64), ("f32", 2, 1, 64)])
@pytest.mark.parametrize("n_q", [200, 5])
def test_wide_score_range_of_every_matrix_core_layout(dtype, hq, hkv, d, n_q):
    """Row maxima that jump by tens to hundreds of binary orders between key tiles, as in test_attn_chunk_wide_score_range:
    chunk prefill (with 5 queries in fp32 the kernel for few rows; in fp32 also the other two kernels, asked for) and decode of one and
    of two rows.

    fp32: a score s is off by up to 4 x 1.6 times 2^-24 of its size (see test_gpu_precision) and its weight by as much of
    itself.  What that does to a row's output: the largest weight p multiplies a value within (1 - p) x 9 of the output (values
    are up to 4.5), the others, 1 - p together, values within 9 of it."""
    n_kv = 1100
    w = si.Workload("a", 1, hq, hkv, d, dtype, 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9900)
    q, k, v = w.qkv(0, np.arange(n_kv))
    q, k = q[n_kv - n_q:], k.copy()
    k[0:64] *= 1.0 / 64
    k[192:256] *= 16
    k[640:704] *= 32
    k[901] *= 128
    k[n_kv - 100:n_kv - 90] *= 8
    q64, k64, v64 = (x.astype(np.float64) for x in (q, k, v))
    scores = np.einsum("qhd,khd->qhk", q64, np.repeat(k64, hq // hkv, 1)) / np.sqrt(d)

    def check(o, at, causal):
        """o: the outputs of the last len(at) queries, at: their slots"""
        ref = orc.gqa_attention(q64[-len(at):], k64, v64, at, causal)
        if dtype == "bf16":
            assert gu.max_err(gu.host(o), ref) <= gu.TOL["bf16"]
            return
        s = scores[-len(at):]
        if causal:
            s = np.where(np.arange(n_kv) <= at[:, None, None], s, -np.inf)
        p = np.exp(s - s.max(-1, keepdims=True))
        rest = 1 - 1 / p.sum(-1)
        size = np.abs(np.where(np.isfinite(s), s, 0)).max(-1)
        tol = gu.TOL["f32"] + 4 * 1.6 * 2.0 ** -24 * size * rest * 18
        gu.max_err(gu.host(o), ref)
        assert (np.abs(gu.host(o) - ref).max(-1) <= tol).all()
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 2,
                     n_kv + 8, n_q)
    for s in range(2):
        cache.append(s, 0, np.zeros(n_kv, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    qd = gu.dev(q, w)
    for causal in (True, False):
        for splits in (0, 1, 4) + ((1 | PLAIN, 4 | PLAIN, 1 | TERMS, 4 | TERMS) if dtype == "f32" else ()):
            print(f"wide scores {dtype} {hq}/{hkv} x {d} n_q={n_q} causal={causal} splits={splits}", flush=True)
            cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
            od = torch.full_like(qd, float("nan"))
            cache.attn_chunk(0, 0, qd, od, causal)
            check(od, np.arange(n_kv - n_q, n_kv), causal)
    for ids in ([0], [0, 1]):
        x = qd[-len(ids):].contiguous()
        od = torch.full_like(x, float("nan"))
        cache.attn_decode(0, ids, x, od)
        check(od, np.full(len(ids), n_kv - 1), True)


@pytest.mark.parametrize("dtype,hq,hkv,d", [("f32", 2, 2, 64), ("f32", 4, 2, 128), ("f32", 16, 4, 64), ("f32", 7, 1, 128),
                                           ("f32", 16, 2, 128), ("bf16", 3, 3, 64), ("bf16", 8, 2, 64), ("bf16", 14, 2, 64),
                                           ("bf16", 16, 2, 64), ("bf16", 4, 2, 64)])
def test_generic_row_kernels_of_every_layout(dtype, hq, hkv, d):
    """SV_FLAG_GENERIC_KERNELS on the types and sizes that the matrix-core kernels normally take: chunk prefill, decode of one
    and of three rows, a fused decode step, one and several key ranges."""
    tol, rope = gu.TOL[dtype], (sv.SV_ROPE_1D, 1e4, (0, 0, 0))
    w = si.Workload("g", 1, hq, hkv, d, dtype, 0, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9950 + hq)
    lens, n_q = [333, 70, 1], 41
    base = w.qkv(0, np.arange(max(lens)))
    for splits in (0, 1, 5):
        print(f"generic {dtype} {hq}/{hkv} x {d} splits={splits}", flush=True)
        cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, *rope, 3, max(lens) + 8, n_q,
                         flags=sv.SV_FLAG_GENERIC_KERNELS)
        cache.set_option(sv.SV_OPT_DECODE_SPLITS, splits)
        kv = []
        for b, n in enumerate(lens):
            k, v = base[1][:n], base[2][:n]
            cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
            kv.append((cache.read_kv(b, 0, 0, 0, n).astype(np.float64), v))
        q = base[0][:n_q]
        qd = gu.dev(q, w)
        od = torch.full_like(qd, float("nan"))
        cache.attn_chunk(0, 0, qd, od, True)
        ref = orc.gqa_attention(q.astype(np.float64), kv[0][0], kv[0][1].astype(np.float64), np.arange(333 - n_q, 333), True)
        assert gu.max_err(gu.host(od), ref) <= tol
        for ids in ([0], [2, 0, 1]):
            x = qd[:len(ids)].contiguous()
            od = torch.full_like(x, float("nan"))
            cache.attn_decode(0, ids, x, od)
            assert gu.max_err(gu.host(od), batch_ref(q[:len(ids)], [kv[i] for i in ids], [lens[i] for i in ids], hq // hkv)) <= tol
        qn, kn, vn = w.qkv(0, np.arange(60000, 60003))
        od = torch.full((3, hq, d), float("nan"), device="cuda:0", dtype=qd.dtype)
        cache.decode_step(0, [0, 1, 2], gu.dev(qn, w), gu.dev(kn, w), gu.dev(vn, w), od)
        kv2, qr = [], []
        for b, n in enumerate(lens):
            pos = np.full((1, 3), n)
            kv2.append((np.concatenate([kv[b][0], cache.read_kv(b, 0, 0, n, 1).astype(np.float64)]), np.concatenate([kv[b][1], vn[b:b + 1]])))
            assert gu.max_err(cache.read_kv(b, 0, 0, n, 1), orc.rope(kn[b:b + 1], pos, 0, 1e4, (0, 0, 0))) <= (4e-2 if dtype == "bf16" else 1e-5)
            assert np.array_equal(cache.read_kv(b, 0, 1, n, 1), vn[b:b + 1])
            qr.append(orc.rope(qn[b:b + 1], pos, 0, 1e4, (0, 0, 0))[0])
        assert gu.max_err(gu.host(od), batch_ref(np.stack(qr), kv2, [n + 1 for n in lens], hq // hkv)) <= tol


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (16, 2, 64)])
@pytest.mark.parametrize("step", [0.9, 6.6, 7.4, 8.2, 9.5])
def test_chunk_row_maxima_that_rise_by_about_the_allowed_step(hq, hkv, d, step):
    """Scores that rise from key tile to key tile by about the 8 binary orders for which a row keeps its reference (and by one, so
    that they add up to it): rows of one tile lie below, at and above the step.  Tile 6 falls back, 200 orders below."""
    n_kv, n_q = 1100, 150
    w = si.Workload("r", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9950)
    q, k, v = w.qkv(0, np.arange(n_kv))
    bf16 = lambda x: torch.from_numpy(x).to(torch.bfloat16).float().numpy()   # what the cache holds is what the oracle reads
    level = np.arange(n_kv) // 64 * step
    level[6 * 64:7 * 64] -= 200
    q = bf16(1 + 0.1 * q[n_kv - n_q:])
    k = bf16((level / (np.sqrt(d) * 1.4427))[:, None, None] + 0.5 * k)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n_kv + 8, n_q)
    cache.append(0, 0, np.zeros(n_kv, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    qd = gu.dev(q, w)
    for causal in (True, False):
        ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.arange(n_kv - n_q, n_kv), causal)
        for splits in (1, 3):
            print(f"rising maxima {hq}/{hkv} x {d} step={step} causal={causal} splits={splits}", flush=True)
            cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
            od = torch.full_like(qd, float("nan"))
            cache.attn_chunk(0, 0, qd, od, causal)
            assert gu.max_err(gu.host(od), ref) <= gu.TOL["bf16"]


@pytest.mark.parametrize("dtype,hq,hkv,d,n", [
    ("bf16", 8, 2, 128, 33 * 128 - 5), ("bf16", 2, 2, 128, 65 * 128 + 3), ("bf16", 4, 2, 64, 66 * 128), ("bf16", 1, 1, 128, 128 * 128),
    ("bf16", 5, 1, 64, 32 * 128 + 1), ("f32", 8, 2, 128, 34 * 64), ("f32", 2, 1, 64, 66 * 64 + 1), ("f32", 1, 1, 64, 127 * 64)])
def test_decode_outputs_shared_out_in_finer_units(dtype, hq, hkv, d, n):
    """Merges of more than 32 and of more than 64 key ranges, whose workgroups take 16 and 8 outputs at a time where there are
    enough of them: the result, and the same from workgroups that are late."""
    cache, w, q, k, v = attn_case(dtype, hq, hkv, d, n, 1, True, 9970)
    ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.array([n - 1]), True)
    for _ in range(2):
        od = torch.full((1, hq, d), float("nan"), device="cuda:0", dtype=gu.tdtype(w))
        cache.attn_decode(0, [0], gu.dev(q, w), od)
        assert gu.max_err(gu.host(od), ref) <= gu.TOL[dtype]
    test_decode_merge_left_to_late_workgroups(dtype, hq, hkv, d, [n])


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (28, 4, 128), (16, 2, 64), (2, 2, 64), (1, 1, 128)])
def test_decode_merges_of_up_to_64_key_ranges_and_of_more(hq, hkv, d):
    """Streams that grow from 64 key ranges to 65 (28 / 4 heads: one tile per wavefront is forced), and 127 and 128 ranges: 32, 16 and
    8 outputs at a time, by a wavefront each or by all of them, waiting and late."""
    w = si.Workload("m", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9971)
    f64 = lambda x: x.astype(np.float64)
    lens = [64 * 128 - 1, 126 * 128 + 1, 127 * 128] if hkv < 4 else [64 * 128 - 1]
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), len(lens), max(lens) + 8, 16)
    q, k, v = w.qkv(0, np.arange(max(lens) + 2))
    for b, n in enumerate(lens):
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k[:n], w), gu.dev(v[:n], w))
        for m in (n + 1, n + 2):
            print(f"{hq}/{hkv} x {d} {m} tokens", flush=True)
            x, out = slice(m - 1, m), []
            for option in (1 if hkv == 4 else 0, sv.SV_MERGE_ONE_LOOK + (1 if hkv == 4 else 0)):
                cache.set_option(sv.SV_OPT_DECODE_TILES_PER_WAVE, option)
                out.append(torch.full((1, hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16))
                if option < sv.SV_MERGE_ONE_LOOK:
                    cache.decode_step(0, [b], gu.dev(q[x], w), gu.dev(k[x], w), gu.dev(v[x], w), out[-1])
                else:
                    cache.attn_decode(0, [b], gu.dev(q[x], w), out[-1])
            ref = orc.gqa_attention(f64(q[x]), f64(k[:m]), f64(v[:m]), np.array([m - 1]), True)
            assert gu.max_err(gu.host(out[0]), ref) <= gu.TOL["bf16"] and torch.equal(out[0], out[1])


@pytest.mark.parametrize("hq,hkv,d,n", [
    (12, 12, 128, 2688), (12, 12, 128, 2689), (12, 12, 128, 3040), (12, 12, 128, 3041), (12, 12, 128, 3700), (12, 12, 128, 4300),
    (12, 12, 128, 4865), (16, 4, 64, 8225), (8, 1, 128, 8193), (8, 1, 128, 10300)])
def test_decode_key_ranges_between_one_tile_per_wavefront_and_two(hq, hkv, d, n):
    """Lengths at which a single stream's ranges become 160, 192, 224 and 256 keys long and where that ends (with more than 256 MB in all
    layers, see test_decode_key_ranges_of_layers_within_the_infinity_cache_and_beyond; a single layer, as here, has ranges of 256 keys
    at those of more than one kv head): attention alone, then two fused steps, whose token is the last of a range, or one of its own."""
    cache, w, q, k, v = attn_case("bf16", hq, hkv, d, n, 1, True, 9980)
    new = [w.qkv(0, np.arange(60000 + i, 60001 + i)) for i in range(2)]
    for i in range(3):
        od = torch.full((1, hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        if i == 0:
            cache.attn_decode(0, [0], gu.dev(q, w), od)
        else:
            q, kn, vn = new[i - 1]
            cache.decode_step(0, [0], gu.dev(q, w), gu.dev(kn, w), gu.dev(vn, w), od)
            k, v = np.concatenate([k, kn]), np.concatenate([v, vn])
        ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.array([n + i - 1]), True)
        assert gu.max_err(gu.host(od), ref) <= gu.TOL["bf16"]
    test_decode_merge_left_to_late_workgroups("bf16", hq, hkv, d, [n])


@pytest.mark.parametrize("dtype,hq,hkv,d,mode", [
    ("bf16", 4, 2, 128, sv.SV_ROPE_3D), ("bf16", 4, 4, 64, sv.SV_ROPE_1D), ("f32", 2, 1, 64, sv.SV_ROPE_3D),
    ("f32", 4, 2, 128, sv.SV_ROPE_1D), ("bf16", 4, 2, 64, sv.SV_ROPE_NONE)])
@pytest.mark.parametrize("budgets", [(5, 30, 9), (0, 0, 0), (70, 300, 0), (3, 1000, 1000)])
def test_runs_registered_by_the_eviction(dtype, hq, hkv, d, mode, budgets):
    """Seconds through sv_stream_step, whose eviction registers both runs, against the calls one by one: ids, positions, every
    stored row, outputs, and the rotation of the newest run's queries afterwards.  Text runs of none, one, as many as are registered
    that way and one more; grids of all extents and none; evictions that leave nothing and that do nothing."""
    sec = ((16, 24, 24) if d == 128 else (8, 12, 12)) if mode == sv.SV_ROPE_3D else (0, 0, 0)
    dt, code = (torch.float32, sv.SV_DTYPE_F32) if dtype == "f32" else (torch.bfloat16, sv.SV_DTYPE_BF16)
    a, b = (sv.Cache(2, hq, hkv, d, code, mode, 1e4, sec, 1, 1400, 256) for _ in range(2))
    g = torch.Generator(device="cuda:0").manual_seed(77)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g).to(dt)
    run = gu.StreamRunner(b, *budgets)
    pre = rnd(2, 2, 80, hkv, d)
    for c in (a, b):
        gu.StreamRunner(c, *budgets).preamble(list(pre[0]), list(pre[1]))
    tol = gu.TOL[dtype]
    for grid, t in (((1, 4, 4), 4), ((2, 3, 5), 1), ((1, 1, 7), 0), ((3, 2, 2), 64), ((1, 16, 16), 65), ((4, 1, 1), 3), ((1, 5, 3), 2)):
        print(f"{dtype} d{d} mode {mode} {budgets} grid {grid} text {t}", flush=True)
        n = grid[0] * grid[1] * grid[2]
        thw = None if mode == sv.SV_ROPE_NONE and t == 1 else grid
        q, k, v = rnd(2, n, hq, d), rnd(2, n, hkv, d), rnd(2, n, hkv, d)
        qt, kt, vt = rnd(t, 2, 1, hq, d), rnd(t, 2, 1, hkv, d), rnd(t, 2, 1, hkv, d)
        o, ot, o2, ot2 = torch.empty_like(q), torch.empty_like(qt), torch.empty_like(q), torch.empty_like(qt)
        text = dict(q_text=qt, k_text=kt, v_text=vt, o_text=ot) if t else {}
        kept = a.stream_step(0, *budgets, q_vision=q.clone(), k_vision=k, v_vision=v, o_vision=o, grid_thw=thw, **text)
        assert kept == run.evict()
        run.prefill(list(q.clone()), list(k), list(v), list(o2), thw)
        for i in range(t):
            run.decode(list(qt[i]), list(kt[i]), list(vt[i]), list(ot2[i]))
        total = a.len(0)
        assert total == b.len(0)
        for x, y in zip(a.retained(0), b.retained(0)):
            assert np.array_equal(x, y)
        for layer in range(2):
            for which in range(2):
                assert np.array_equal(a.read_kv(0, layer, which, 0, total), b.read_kv(0, layer, which, 0, total)), (layer, which)
        # (both are within the tolerance of the exact result, but for a rounding of the rotated queries)
        assert gu.max_err(gu.host(o), gu.host(o2)) <= 2 * tol and (t == 0 or gu.max_err(gu.host(ot), gu.host(ot2)) <= 2 * tol)
        m = t if t else n
        x = rnd(m, hq, d)
        y = x.clone()
        a.rope_apply(0, total - m, m, x, None)
        b.rope_apply(0, total - m, m, y, None)
        assert torch.equal(x, y)


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 128), (8, 8, 64)])
@pytest.mark.parametrize("lens", [(33000, 32100, 1), (66000, 66100, 77), (70111, 31, 92161, 129)])
def test_decode_batches_of_few_and_of_many_blocks_per_workgroup(hq, hkv, d, lens):
    """Batches of more K and V than the caches hold, with runs of 8, of 16 and 17 and of 19 and 20 blocks per workgroup, against
    float32.  The outputs of these lengths are small: the tolerance is the rounding of the result and six standard deviations of the
    sum of the weights' roundings (2^-8 of a weight at most, independent of each other)."""
    g = torch.Generator(device="cuda:0").manual_seed(91)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g).to(torch.bfloat16)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), len(lens), max(lens) + 8, 1)
    q, ref, tol = rnd(len(lens), hq, d), [], []
    for b, n in enumerate(lens):
        k, v = rnd(n, hkv, d), rnd(n, hkv, d)
        for i in range(0, n, 16384):
            cache.append(b, 0, np.zeros(min(16384, n - i), np.uint8), None, k[i:i + 16384].contiguous(), v[i:i + 16384].contiguous())
        pv = torch.softmax((k.float() * q[b].float()).sum(2) / d ** 0.5, 0)[:, :, None] * v.float()
        ref.append(pv.sum(0))
        tol.append(2 ** -8 * ref[b].abs() + 6 * 2 ** -8 / 3 ** 0.5 * (pv * pv).sum(0).sqrt() + 1e-5)
    out = torch.full_like(q, float("nan"))
    cache.attn_decode(0, list(range(len(lens))), q, out)
    err = (out.float() - torch.stack(ref)).abs()
    assert bool((err <= torch.stack(tol)).all()), float((err / torch.stack(tol)).max())


@pytest.mark.parametrize("hq,hkv,d", [(1, 1, 128), (3, 1, 128), (5, 1, 64), (12, 2, 128), (7, 1, 64), (8, 1, 128)])
@pytest.mark.parametrize("n_q,n_kv", [(1, 200), (13, 205), (37, 300), (90, 400), (257, 1000)])
def test_chunk_rows_of_every_group_size(hq, hkv, d, n_q, n_kv):
    """The (token, head) rows of a wavefront, for groups that do and do not divide 32, chunks that end inside a wavefront's rows and a
    workgroup's, as final results and as partial ones; queries and outputs at an offset of one element from 16 bytes."""
    w = si.Workload("g", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9990)
    q, k, v = w.qkv(0, np.arange(n_kv))
    q = q[n_kv - n_q:]
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n_kv + 8, n_q)
    cache.append(0, 0, np.zeros(n_kv, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.arange(n_kv - n_q, n_kv), True)
    for splits in (1, 3):
        for off in (0, 1):
            buf = torch.full((2, q.size + 8), float("nan"), device="cuda:0", dtype=torch.bfloat16)
            qd, od = (x[off:off + q.size].view(n_q, hq, d) for x in buf)
            qd.copy_(gu.dev(q, w))
            cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
            cache.attn_chunk(0, 0, qd, od, True)
            assert gu.max_err(gu.host(od), ref) <= gu.TOL["bf16"], (splits, off)
            assert bool(torch.isnan(buf[1, :off]).all()) and bool(torch.isnan(buf[1, off + q.size:]).all())


@pytest.mark.parametrize("hq,hkv,d,mode", [(2, 1, 64, sv.SV_ROPE_1D), (3, 3, 64, sv.SV_ROPE_3D), (4, 2, 128, sv.SV_ROPE_3D), (5, 1, 128, sv.SV_ROPE_1D)])
@pytest.mark.parametrize("n,kept", [(1, 1), (4, 28), (5, 28), (12, 20), (12, 21), (9, 90), (12, 116), (12, 117), (6, 122)])
def test_f32_chunk_of_few_rows_that_stores_its_tokens(hq, hkv, d, mode, n, kept):
    """A short fp32 chunk on up to 128 keys, one more, and where new keys begin inside a tile, whose attention launch (head_dim 64) rotates and
    stores: the rows that a launch of its own would have stored, its outputs, and those of the oracle."""
    sec = ((16, 24, 24) if d == 128 else (8, 12, 12)) if mode == sv.SV_ROPE_3D else (0, 0, 0)
    a, b = (sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32, mode, 1e4, sec, 1, 256, 64) for _ in range(2))
    b.set_option(sv.SV_OPT_CHUNK_STORE, 1)
    g = torch.Generator(device="cuda:0").manual_seed(78)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g)
    pre, q, k, v = rnd(2, 1, kept, hkv, d), rnd(1, n, hq, d), rnd(1, n, hkv, d), rnd(1, n, hkv, d)
    out = []
    for c in (a, b):
        gu.StreamRunner(c, 999, 999, 999).preamble(list(pre[0]), list(pre[1]))
        o = torch.full_like(q, float("nan"))
        c.stream_step(0, 999, 999, 999, q_vision=q.clone(), k_vision=k, v_vision=v, o_vision=o, grid_thw=(1, 1, n))
        out.append(gu.host(o))
    total = a.len(0)
    assert total == kept + n == b.len(0)
    rows = [[c.read_kv(0, 0, which, 0, total) for which in range(2)] for c in (a, b)]
    assert all(np.array_equal(x, y) for x, y in zip(*rows))
    x = q[0].clone()
    a.rope_apply(0, kept, n, x, None)
    ref = orc.gqa_attention(gu.host(x).astype(np.float64), rows[0][0].astype(np.float64), rows[0][1].astype(np.float64), np.arange(kept, total), True)
    assert gu.max_err(out[0][0], ref) <= gu.TOL["f32"] and gu.max_err(out[1][0], ref) <= gu.TOL["f32"]


def layers_case(hq, hkv, d, n, layers, seed):
    """A cache whose layers all hold the same n tokens: attention alone of the first and the last layer, then two fused steps through
    all of them, whose tokens are the last of a key range or one of their own; every layer's result and row against the oracle."""
    print(f"decode {hq}/{hkv} x {d} n={n} layers={layers}", flush=True)
    w = si.Workload("y", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, seed)
    cache = sv.Cache(layers, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n + 8, 1)
    q, k, v = w.qkv(0, np.arange(n))
    kd, vd = gu.dev(k, w), gu.dev(v, w)
    for layer in range(layers):
        cache.append(0, layer, np.zeros(n, np.uint8) if layer == 0 else None, None, kd, vd)
    for i in range(3):
        o = torch.full((layers, 1, hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        if i == 0:
            qn, calls = q[n - 1:], (0, layers - 1)
            for layer in calls:
                cache.attn_decode(layer, [0], gu.dev(qn, w), o[layer])
        else:
            qn, kn, vn = w.qkv(0, np.arange(60000 + i, 60001 + i))
            calls = range(layers)
            for layer in calls:
                cache.decode_step(layer, [0], gu.dev(qn, w), gu.dev(kn, w), gu.dev(vn, w), o[layer])
            k, v = np.concatenate([k, kn]), np.concatenate([v, vn])
        ref = orc.gqa_attention(qn.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.array([n + i - 1]), True)
        for layer in calls:
            assert gu.max_err(gu.host(o[layer]), ref) <= gu.TOL["bf16"], (i, layer)
    for layer in (0, layers - 1):
        assert np.array_equal(cache.read_kv(0, layer, 0, n - 2, 4), k[n - 2:]) and np.array_equal(cache.read_kv(0, layer, 1, n - 2, 4), v[n - 2:])


@pytest.mark.parametrize("hq,hkv,d,n,layers", [
    (12, 12, 128, 1108, 6), (12, 12, 128, 1110, 6), (12, 12, 128, 1227, 5), (12, 12, 128, 1229, 5), (12, 12, 128, 2686, 16),
    (12, 12, 128, 2686, 17), (28, 4, 128, 3585, 5), (8, 8, 64, 3327, 6), (8, 8, 64, 3330, 6), (1, 1, 128, 13313, 6)])
def test_decode_k_tiles_through_lds_and_into_registers(hq, hkv, d, n, layers):
    """One tile per wavefront, on both sides of what sends K through LDS: 6.5 MB in the launch, 36 MB in all layers, and 256 MB."""
    layers_case(hq, hkv, d, n, layers, 9995)


@pytest.mark.parametrize("hq,hkv,d,n,layers", [
    (12, 12, 128, 2688, 17), (12, 12, 128, 2689, 17), (12, 12, 128, 3041, 15), (12, 12, 128, 3700, 11), (12, 12, 128, 3700, 12),
    (12, 12, 128, 4300, 11), (12, 12, 128, 4865, 9), (28, 4, 128, 8225, 15), (28, 4, 128, 8225, 16)])
def test_decode_key_ranges_of_layers_within_the_infinity_cache_and_beyond(hq, hkv, d, n, layers):
    """More key ranges of 128 keys than CUs: ranges of 256 keys up to 256 MB in all layers, of 160, 192, 224 and 256 beyond."""
    layers_case(hq, hkv, d, n, layers, 9996)


@pytest.mark.parametrize("lens", [(131072, 98000, 31), (131072, 102400, 31)])
def test_decode_batches_on_both_sides_of_56_blocks_per_workgroup(lens):
    """Runs of 56 blocks, whose K goes through LDS, and of 57, whose does not (non-temporal loads)."""
    test_decode_batches_of_few_and_of_many_blocks_per_workgroup(8, 8, 64, lens)


@pytest.mark.parametrize("n", [28600, 29200])
def test_layers_as_rows_on_both_sides_of_56_blocks_per_workgroup(n):
    """The same with plain loads: 64 layers of one stream in one launch, after a fused step and one more, whose token the first one
    stored; tolerance as for the batches."""
    layers, d = 64, 64
    g = torch.Generator(device="cuda:0").manual_seed(92)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g).to(torch.bfloat16)
    cache = sv.Cache(layers, 1, 1, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n + 8, 1)
    k, v = rnd(n, 1, d), rnd(n, 1, d)
    for layer in range(layers):
        cache.append(0, layer, np.zeros(n, np.uint8) if layer == 0 else None, None, k, v)
    k, v = (x.expand(layers, n, d) for x in (k[:, 0], v[:, 0]))
    for step in range(2):
        q, kn, vn = rnd(layers, 1, d), rnd(layers, 1, d), rnd(layers, 1, d)
        out = torch.full_like(q, float("nan"))
        cache.decode_step_layers(0, q, kn, vn, out)
        k, v = torch.cat([k, kn], 1), torch.cat([v, vn], 1)
        pv = torch.softmax((k.float() * q.float()).sum(2) / d ** 0.5, 1)[:, :, None] * v.float()
        ref = pv.sum(1)
        tol = 2 ** -8 * ref.abs() + 6 * 2 ** -8 / 3 ** 0.5 * (pv * pv).sum(1).sqrt() + 1e-5
        err = (out[:, 0].float() - ref).abs()
        assert bool((err <= tol).all()), (step, float((err / tol).max()))


@pytest.mark.parametrize("total", [30000, 40000, 70000])
def test_runs_registered_by_scans_of_several_passes(total):
    """Seconds behind evictions whose scan has up to 128 workgroups of tokens, one or several passes each, and as many registering ones
    as there can be (their words lie behind the others'), then behind shorter ones, which clear what they do not use: retained ids and
    positions as the oracle has them, the second's stored K as rotated at those positions, V as given."""
    print(f"long-cache second: {total} tokens", flush=True)
    d, sec, grid, nv, nt = 64, (8, 12, 12), (2, 24, 30), 1440, 37
    cache = sv.Cache(1, 1, 1, d, sv.SV_DTYPE_F32, sv.SV_ROPE_3D, 1e4, sec, 1, total + 4096, 2048)
    o = orc.OracleStream(1, 1, 1, 2, orc.ROPE_3D, 1e4, (1, 0, 0))
    z, zt = (lambda n: np.zeros((n, 1, 2))), torch.zeros(1024, 1, d, device="cuda:0")
    g = torch.Generator(device="cuda:0").manual_seed(79)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g)
    n = 0
    while n < total:
        for ty, cnt, thw in ((orc.VISION, 2 * 12 * 16, (2, 12, 16)), (orc.TEXT, 37, None)):
            cache.append(0, 0, np.full(cnt, 1 if ty == orc.VISION else 0, dtype=np.uint8), thw, zt[:cnt], zt[:cnt])
            o.append_meta([ty] * cnt, thw)
            o.append_kv(0, z(cnt), z(cnt))
            n += cnt
    for budgets in [(100, total - 6000, total // 20), (64, total // 3, 333), (64, 3000, 333), (0, 100, 0), (64, 5000, 333)]:
        k, v, kt, vt = rnd(1, nv, 1, d), rnd(1, nv, 1, d), rnd(nt, 1, 1, 1, d), rnd(nt, 1, 1, 1, d)
        q, qt = rnd(1, nv, 1, d), rnd(nt, 1, 1, 1, d)
        kept = cache.stream_step(0, *budgets, q_vision=q, k_vision=k, v_vision=v, o_vision=torch.empty_like(q), grid_thw=grid,
                                 q_text=qt, k_text=kt, v_text=vt, o_text=torch.empty_like(qt))
        assert kept == o.evict(*budgets)
        for ty, cnt, thw in ((orc.VISION, nv, grid), (orc.TEXT, nt, None)):
            o.append_meta([ty] * cnt, thw)
            o.append_kv(0, z(cnt), z(cnt))
        ids, pos = cache.retained(0)
        assert np.array_equal(ids, np.asarray(o.gid, dtype=np.int64))
        assert np.array_equal(pos.astype(np.int64), o.positions())
        kn = np.concatenate([gu.host(k)[0], gu.host(kt)[:, 0, 0]])
        vn = np.concatenate([gu.host(v)[0], gu.host(vt)[:, 0, 0]])
        assert gu.max_err(cache.read_kv(0, 0, 0, kept, nv + nt), orc.rope(kn, o.positions()[kept:], orc.ROPE_3D, 1e4, sec)) <= gu.TOL["f32"]
        assert np.array_equal(cache.read_kv(0, 0, 1, kept, nv + nt), vn.astype(np.float32))


@pytest.mark.parametrize("hq,hkv,d,lens,layers", [
    (12, 12, 128, (1280, 1270), 6), (12, 12, 128, (1280, 1270), 2), (28, 4, 128, (2048, 1983, 2040), 5), (8, 8, 64, (2046, 2000), 5)])
def test_decode_batches_of_one_block_per_workgroup(hq, hkv, d, lens, layers):
    """Batches of one key block per workgroup, K into registers where the layers together are 36 to 256 MB: attention alone, then two
    fused steps through all layers, the second of which reads what the first one stored."""
    w = si.Workload("o", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9997)
    cache = sv.Cache(layers, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), len(lens), max(lens) + 8, 1)
    ids, kv = list(range(len(lens))), []
    for b, n in enumerate(lens):
        _, k, v = w.qkv(b, np.arange(n))
        kv.append((k, v))
        for layer in range(layers):
            cache.append(b, layer, np.zeros(n, np.uint8) if layer == 0 else None, None, gu.dev(k, w), gu.dev(v, w))
    for i in range(3):
        q, kn, vn = w.qkv(0, np.arange(60000 + 10 * i, 60000 + 10 * i + len(lens)))
        o = torch.full((layers, len(lens), hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        for layer in range(layers):
            if i == 0:
                cache.attn_decode(layer, ids, gu.dev(q, w), o[layer])
            else:
                cache.decode_step(layer, ids, gu.dev(q, w), gu.dev(kn, w), gu.dev(vn, w), o[layer])
        if i > 0:
            kv = [(np.concatenate([k, kn[b:b + 1]]), np.concatenate([v, vn[b:b + 1]])) for b, (k, v) in enumerate(kv)]
        ref = batch_ref(q, kv, [len(k) for k, _ in kv], hq // hkv)
        for layer in range(layers):
            assert gu.max_err(gu.host(o[layer]), ref) <= gu.TOL["bf16"], (i, layer)


@pytest.mark.parametrize("hq,hkv,d,lens", [(12, 12, 128, (1500,)), (28, 4, 128, (3650,)), (8, 8, 64, (3400,)), (12, 12, 128, (1280, 1265))])
@pytest.mark.parametrize("mode", [sv.SV_ROPE_1D, sv.SV_ROPE_3D])
def test_decode_is_bit_for_bit_the_same_however_k_travels(hq, hkv, d, lens, mode):
    """The same tokens in a cache of one layer, whose K goes through LDS, and in one of six, whose K goes into registers: fused steps with
    rotation, attention alone and with static scratch, and what the steps stored."""
    sec = ((16, 24, 24) if d == 128 else (8, 12, 12)) if mode == sv.SV_ROPE_3D else (0, 0, 0)
    caches = [sv.Cache(layers, hq, hkv, d, sv.SV_DTYPE_BF16, mode, 1e4, sec, len(lens), max(lens) + 8, 16) for layers in (1, 6)]
    g = torch.Generator(device="cuda:0").manual_seed(93)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g).to(torch.bfloat16)
    ids = list(range(len(lens)))
    for b, n in enumerate(lens):
        k, v = rnd(n, hkv, d), rnd(n, hkv, d)
        for c in caches:
            for layer in range(c.cfg.n_layers):
                c.append(b, layer, np.zeros(n, np.uint8) if layer == 0 else None, None, k, v)
    for step in range(3):
        print(f"decode {hq}/{hkv} x {d} {lens} mode {mode} step {step}", flush=True)
        q, kn, vn = rnd(len(lens), hq, d), rnd(len(lens), hkv, d), rnd(len(lens), hkv, d)
        out = []
        for c in caches:
            for layer in range(c.cfg.n_layers):
                o = torch.full((3, len(lens), hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
                c.attn_decode(layer, ids, q, o[0])
                c.attn_decode_static(layer, ids, q, o[1])
                out.append(o)
            for layer in range(c.cfg.n_layers):
                c.decode_step(layer, ids, q, kn, vn, out[layer - c.cfg.n_layers][2])
        assert not torch.isnan(out[0]).any() and torch.equal(out[0][0], out[0][1])
        assert all(torch.equal(out[0], o) for o in out[1:])
    for b, n in enumerate(lens):
        for which in range(2):
            rows = [c.read_kv(b, layer, which, n - 4, 7) for c in caches for layer in (0, c.cfg.n_layers - 1)]
            assert all(np.array_equal(rows[0], x) for x in rows[1:])


@pytest.mark.parametrize("dtype,hq,hkv,d,step", [
    ("bf16", 28, 4, 128, 128), ("bf16", 16, 2, 64, 128), ("bf16", 3, 3, 128, 128), ("f32", 8, 2, 128, 64), ("f32", 2, 1, 64, 64)])
def test_decode_ranges_whose_wavefronts_have_one_tile_or_none(dtype, hq, hkv, d, step):
    """One to four key ranges of one tile per wavefront, the last of them with one to four tiles, whole or a key more or less: attention
    alone and a fused step, whose token is in the last tile or is a tile of its own."""
    lens = [step * n + m for n in range(4) for m in (1, step // 4 - 1, step // 4, step // 4 + 1, step // 2, step - 1)] + [4 * step]
    w = si.Workload("o", 1, hq, hkv, d, dtype, 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9997)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0),
                     len(lens), max(lens) + 8, 16)
    q, k, v = w.qkv(0, np.arange(max(lens) + 1))
    f64 = lambda x: x.astype(np.float64)
    for b, n in enumerate(lens):
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k[:n], w), gu.dev(v[:n], w))
        for new in (False, True):
            m = n + new
            print(f"{dtype} {hq}/{hkv} x {d} n={n} new={new}", flush=True)
            od = torch.full((1, hq, d), float("nan"), device="cuda:0", dtype=gu.tdtype(w))
            if new:
                cache.decode_step(0, [b], gu.dev(q[n:m], w), gu.dev(k[n:m], w), gu.dev(v[n:m], w), od)
            else:
                cache.attn_decode(0, [b], gu.dev(q[n - 1:n], w), od)
            ref = orc.gqa_attention(f64(q[m - 1:m]), f64(k[:m]), f64(v[:m]), np.array([m - 1]), True)
            assert gu.max_err(gu.host(od), ref) <= gu.TOL[dtype]
        assert np.array_equal(cache.read_kv(b, 0, 0, n, 1), k[n:n + 1]) and np.array_equal(cache.read_kv(b, 0, 1, n, 1), v[n:n + 1])


@pytest.mark.parametrize("dtype,hq,hkv,d,mode,flags", [
    ("bf16", 4, 2, 128, sv.SV_ROPE_3D, 0), ("bf16", 4, 4, 64, sv.SV_ROPE_1D, 0), ("f32", 2, 1, 64, sv.SV_ROPE_3D, 0),
    ("bf16", 4, 2, 128, sv.SV_ROPE_3D, sv.SV_FLAG_GENERIC_KERNELS), ("f32", 4, 2, 128, sv.SV_ROPE_1D, sv.SV_FLAG_GENERIC_KERNELS)])
def test_decoded_tokens_registered_ahead(dtype, hq, hkv, d, mode, flags):
    """Decode steps of three streams that fall out of step with each other, past one registration's tokens and up to the end of the
    capacity, with appends, evictions (one that does nothing) and seconds in between, against append, rope_apply and attn_decode:
    ids, positions (of the device's own count), stored rows and outputs."""
    sec = ((16, 24, 24) if d == 128 else (8, 12, 12)) if mode == sv.SV_ROPE_3D else (0, 0, 0)
    dt, code = (torch.float32, sv.SV_DTYPE_F32) if dtype == "f32" else (torch.bfloat16, sv.SV_DTYPE_BF16)
    cap = 70
    a, b = (sv.Cache(2, hq, hkv, d, code, mode, 1e4, sec, 3, cap, 24, flags=flags) for _ in range(2))
    g = torch.Generator(device="cuda:0").manual_seed(78)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g).to(dt)

    def append(s, n, thw=None):
        types = np.full(n, sv.SV_TEXT if thw is None else sv.SV_VISION, np.uint8)
        k, v = rnd(2, n, hkv, d), rnd(2, n, hkv, d)
        for c in (a, b):
            for layer in range(2):
                c.append(s, layer, types if layer == 0 else None, thw if layer == 0 else None, k[layer], v[layer])

    def step(ids):
        q, k, v = rnd(2, len(ids), hq, d), rnd(2, len(ids), hkv, d), rnd(2, len(ids), hkv, d)
        oa, ob = torch.empty_like(q), torch.empty_like(q)
        for layer in range(2):
            a.decode_step(layer, ids, q[layer], k[layer], v[layer], oa[layer])
            for i, s in enumerate(ids):
                b.append(s, layer, np.zeros(1, np.uint8) if layer == 0 else None, None, k[layer, i:i + 1], v[layer, i:i + 1])
            for i, s in enumerate(ids):
                b.rope_apply(s, b.len(s) - 1, 1, q[layer, i:i + 1], None)
            b.attn_decode(layer, ids, q[layer], ob[layer])
        # (each is within the tolerance of the exact result)
        assert gu.max_err(gu.host(oa), gu.host(ob)) <= 2 * gu.TOL[dtype]

    def second(s):
        n, t = 6, 2
        q, k, v = rnd(2, n, hq, d), rnd(2, n, hkv, d), rnd(2, n, hkv, d)
        qt, kt, vt = rnd(t, 2, 1, hq, d), rnd(t, 2, 1, hkv, d), rnd(t, 2, 1, hkv, d)
        for c in (a, b):
            c.stream_step(s, 4, 12, 9, q_vision=q.clone(), k_vision=k, v_vision=v, o_vision=torch.empty_like(q), grid_thw=(1, 2, 3),
                          q_text=qt, k_text=kt, v_text=vt, o_text=torch.empty_like(qt))

    def check(what):
        print(f"{dtype} d{d} mode {mode} flags {flags}: {what}", flush=True)
        for s in range(3):
            n = a.len(s)
            assert n == b.len(s)
            for x, y in zip(a.retained(s), b.retained(s)):
                assert np.array_equal(x, y)
            for layer in range(2):
                for which in range(2):
                    # (K: one rounding of the rotation where the two kernels order it differently)
                    x, y = a.read_kv(s, layer, which, 0, n), b.read_kv(s, layer, which, 0, n)
                    assert np.allclose(x, y, rtol=0 if which else (2.0 ** -7 if dtype == "bf16" else 1e-5), atol=0 if which else 1e-6)

    for s, n in enumerate((5, 9, 1)):
        append(s, n)
        append(s, 12, (2, 2, 3))
    for ids in ([0], [1, 0], [2, 0, 1], [2]):
        step(ids)
    check("out of step")
    append(0, 3)
    append(1, 6, (1, 3, 2))
    step([0, 1, 2])
    check("appended to")
    assert [c.evict(2, 100, 100, 100) for c in (a, b)] == [a.len(2)] * 2   # nothing leaves
    assert a.evict(1, 2, 7, 3) == b.evict(1, 2, 7, 3)
    step([2, 1])
    check("evicted")
    second(0)
    step([0])
    step([1, 0])
    check("a second")
    for _ in range(18):
        step([2, 1])
    check("past one registration")
    for s in (2, 0):
        while a.len(s) < cap:
            step([s])
    check("full")
    with pytest.raises(sv.SvError):
        step([0, 1])
    check("refused")


@pytest.mark.parametrize("dtype,hq,hkv,d,flags", [
    ("bf16", 4, 2, 128, 0), ("bf16", 4, 4, 64, 0), ("f32", 2, 1, 64, 0), ("bf16", 4, 2, 128, sv.SV_FLAG_GENERIC_KERNELS)])
@pytest.mark.parametrize("ids", [[0], [1, 0]])
def test_captured_decode_steps_replayed_after_later_registrations(dtype, hq, hkv, d, flags, ids):
    """Decode steps (1-D positions) in graphs that hold no registration and that hold two in their middle, replayed again after the
    steps behind them and with eager work in between: bit for bit what another cache gives that takes the steps one by one."""
    dt, code = (torch.float32, sv.SV_DTYPE_F32) if dtype == "f32" else (torch.bfloat16, sv.SV_DTYPE_BF16)
    a, b = (sv.Cache(2, hq, hkv, d, code, sv.SV_ROPE_1D, 1e4, (0, 0, 0), 2, 400, 16, flags=flags) for _ in range(2))
    g = torch.Generator(device="cuda:0").manual_seed(79)
    rnd = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g).to(dt)
    for s in range(2):
        for layer in range(2):
            k, v = rnd(300 + s, hkv, d), rnd(300 + s, hkv, d)
            for c in (a, b):
                c.append(s, layer, np.zeros(300 + s, np.uint8) if layer == 0 else None, None, k, v)
    steps, n = 41, len(ids)
    q, k, v = rnd(steps, 2, n, hq, d), rnd(steps, 2, n, hkv, d), rnd(steps, 2, n, hkv, d)
    oa, ob = torch.empty_like(q), torch.empty_like(q)

    def run(c, o, t0, t1):
        for t in range(t0, t1):
            for layer in range(2):
                c.decode_step(layer, ids, q[t, layer], k[t, layer], v[t, layer], o[t, layer])

    def captured(t0, t1):
        torch.cuda.synchronize()
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=side):
            run(a, oa, t0, t1)
        graph.replay()
        torch.cuda.synchronize()
        return graph

    run(b, ob, 0, steps)
    run(a, oa, 0, 3)
    graphs = [captured(3, 6)]
    run(a, oa, 6, 15)
    graphs.append(captured(15, steps))
    assert torch.equal(oa, ob)
    for graph, t0, t1 in ((graphs[0], 3, 6), (graphs[1], 15, steps), (graphs[1], 15, steps), (graphs[0], 3, 6)):
        print(f"{dtype} {hq}/{hkv} x {d} flags {flags} rows {ids}: steps {t0} to {t1} again", flush=True)
        oa[t0:t1] = float("nan")
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(oa, ob)
    for s in ids:
        assert a.len(s) == b.len(s) == 300 + s + steps
        for x, y in zip(a.retained(s), b.retained(s)):
            assert np.array_equal(x, y)
        for which in range(2):
            assert all(np.array_equal(a.read_kv(s, layer, which, 0, a.len(s)), b.read_kv(s, layer, which, 0, a.len(s))) for layer in range(2))


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (16, 2, 64), (3, 3, 128), (8, 1, 64)])
@pytest.mark.parametrize("n_q,n_kv", [(1, 2100), (5, 4200), (37, 4300), (73, 2200), (200, 1100), (300, 700)])
def test_chunk_merge_of_few_and_of_many_ranges(hq, hkv, d, n_q, n_kv):
    """Chunks in 2 to 34 key ranges of several tiles (as many as the keys and the scratch memory allow of those asked for), one, two and
    four groups of lanes to a row, heads that fill a workgroup's groups and that do not, and causal rows that see only some of the ranges,
    against the oracle."""
    w = si.Workload("m", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 771)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n_kv, n_q)
    q, k, v = w.qkv(0, np.arange(n_kv))
    q = q[n_kv - n_q:]
    cache.append(0, 0, np.zeros(n_kv, dtype=np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    qd = gu.dev(q, w)
    for causal in (True, False):
        ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.arange(n_kv - n_q, n_kv), causal)
        for splits in (2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 17, 22, 24, 25, 31, 33, 34, 47, 52, 64):
            print(f"{hq}/{hkv} x {d} n_q={n_q} n_kv={n_kv} causal={causal} splits={splits}", flush=True)
            cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
            od = torch.full_like(qd, float("nan"))
            cache.attn_chunk(0, 0, qd, od, causal)
            assert gu.max_err(gu.host(od), ref) <= gu.TOL["bf16"]


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (16, 2, 64), (3, 3, 128), (8, 1, 64)])
def test_chunk_merge_of_every_number_of_ranges_per_lane(hq, hkv, d):
    """A stream that grows tile by tile to 64 key ranges of one tile each: every number of ranges that a lane of the merge takes with one,
    two and four groups of lanes to a row, with and without one less for the last groups, full and with a last tile of one key, which
    not all rows see, against the oracle."""
    w = si.Workload("m", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 773)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, 64 * 64, 37)
    cache.set_option(sv.SV_OPT_CHUNK_SPLITS, 64)
    q, k, v = w.qkv(0, np.arange(64 * 64))
    f64 = lambda x: x.astype(np.float64)
    ranges = list(range(2, 25)) + [n for n in range(25, 65) if n % 4 in (0, 1)]
    seen, had = set(), 0
    for n in ranges:
        groups = 1 if n <= 12 else 2 if n <= 24 else 4
        seen.add((groups, -(-n // groups), n % groups == 0))
        for n_kv, n_q in ((64 * n - 63, 5), (64 * n, 5 if n % 5 else 37)):
            print(f"{hq}/{hkv} x {d} {n} ranges n_kv={n_kv} n_q={n_q}", flush=True)
            cache.append(0, 0, np.zeros(n_kv - had, np.uint8), None, gu.dev(k[had:n_kv], w), gu.dev(v[had:n_kv], w))
            had = n_kv
            x = q[n_kv - n_q:n_kv]
            ref = orc.gqa_attention(f64(x), f64(k[:n_kv]), f64(v[:n_kv]), np.arange(n_kv - n_q, n_kv), True)
            od = torch.full((n_q, hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
            cache.attn_chunk(0, 0, gu.dev(x, w), od, True)
            assert gu.max_err(gu.host(od), ref) <= gu.TOL["bf16"]
    assert seen == {(1, i, True) for i in range(2, 13)} | {(2, i, e) for i in range(7, 13) for e in (True, False)} | {
        (4, i, e) for i in range(7, 17) for e in (True, False)}


# (28 and 30 heads of 3500 tokens, 7 of 15000 and 3 of 34200 take four heads to a thread in every layout, 5 of 21000 and 2 of 51300 two,
# 1 of 102500 one)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("hq,n", [(28, 1843), (30, 700), (7, 2750), (1, 33), (28, 3700), (30, 3501), (7, 15001), (3, 34201), (5, 21001),
                                  (2, 51301), (1, 102501)])
def test_rotation_of_long_runs(dtype, d, hq, n):
    """Rows rotated one, two and four heads to a thread, with and without the run's table, heads that fill the last share and that do
    not: bit for bit what pieces of 31 tokens give, whose heads go one by one."""
    dt, code = (torch.float32, sv.SV_DTYPE_F32) if dtype == "f32" else (torch.bfloat16, sv.SV_DTYPE_BF16)
    g = torch.Generator(device="cuda:0").manual_seed(hq)
    q, k = (torch.randn(n, h, d, device="cuda:0", generator=g).to(dt) for h in (hq, 1))
    for max_q in (n, 8):
        print(f"{dtype} d{d} {hq} heads n={n} max_q={max_q}", flush=True)
        cache = sv.Cache(1, hq, 1, d, code, sv.SV_ROPE_3D, 1e6, (16, 24, 24) if d == 128 else (8, 12, 12), 1, n, max_q)
        cache.append(0, 0, np.zeros(n, np.uint8), None, k, k)
        x, y, kx, ky = q.clone(), q.clone(), k.clone(), k.clone()
        cache.rope_apply(0, 0, n, x, kx)
        for j in range(0, n, 31):
            m = min(31, n - j)
            cache.rope_apply(0, j, m, y[j:j + m], ky[j:j + m])
        assert torch.equal(x, y) and torch.equal(kx, ky) and not torch.equal(x, q)


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (2, 1, 64), (9, 3, 64), (5, 5, 128)])
@pytest.mark.parametrize("n_q,n_kv", [(1, 1100), (9, 2100), (70, 2200), (200, 300), (9, 2048), (40, 2019)])
def test_fp32_chunk_merge_of_few_and_of_many_ranges(hq, hkv, d, n_q, n_kv):
    """fp32 chunks in 2 to 64 key ranges, one, two and four groups of lanes to a row, whole passes and not, heads that fill a workgroup
    and that do not, causal rows that see only some of the ranges, against the oracle."""
    w = si.Workload("m", 1, hq, hkv, d, "f32", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 772)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n_kv, n_q)
    q, k, v = w.qkv(0, np.arange(n_kv))
    q = q[n_kv - n_q:]
    cache.append(0, 0, np.zeros(n_kv, dtype=np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    qd = gu.dev(q, w)
    for causal in (True, False):
        ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.arange(n_kv - n_q, n_kv), causal)
        for splits in (0, 2, 7, 8, 9, 15, 16, 17, 31, 34, 64, 1 | PLAIN, 3 | PLAIN, 17 | PLAIN, 1 | TERMS, 3 | TERMS, 17 | TERMS, 64 | TERMS):
            print(f"f32 {hq}/{hkv} x {d} n_q={n_q} n_kv={n_kv} causal={causal} splits={splits}", flush=True)
            cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
            od = torch.full_like(qd, float("nan"))
            cache.attn_chunk(0, 0, qd, od, causal)
            assert gu.max_err(gu.host(od), ref) <= gu.TOL["f32"]


@pytest.mark.parametrize("hq,hkv,d", [(28, 4, 128), (16, 2, 64), (3, 3, 128), (4, 1, 64)])
@pytest.mark.parametrize("layers", [1, 24])
def test_decode_batches_whose_wavefronts_have_one_tile_or_none(hq, hkv, d, layers):
    """Batches of one block of 128 keys per workgroup, rows of one to four of them, the last with one to four tiles, whole or a key more or
    less: attention alone and fused steps, whose token is in the last tile or is a tile or a block of its own.  With few layers K goes
    through LDS; with many it comes straight into registers where a launch reads more than 6.5 MB (head_dim 128)."""
    lens = [128 * a + m for a in range(4) for m in (1, 31, 32, 33, 127, 128)] if layers == 1 else [504] * 3 + [1633, 1600, 127]
    w = si.Workload("o", 1, hq, hkv, d, "bf16", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9998)
    cache = sv.Cache(layers, hq, hkv, d, sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), len(lens), max(lens) + 8, 16)
    q, k, v = w.qkv(0, np.arange(max(lens) + 1))
    f64 = lambda x: x.astype(np.float64)
    ids = list(range(len(lens)))
    kd, vd = gu.dev(k, w), gu.dev(v, w)
    for b, n in enumerate(lens):
        for layer in range(layers):
            cache.append(b, layer, np.zeros(n, np.uint8) if layer == 0 else None, None, kd[:n], vd[:n])
    for new in (False, True):
        print(f"{hq}/{hkv} x {d} layers={layers} new={new}", flush=True)
        at = [n - 1 + new for n in lens]
        for layer in range(layers):
            od = torch.full((len(lens), hq, d), float("nan"), device="cuda:0", dtype=torch.bfloat16)
            if new:
                cache.decode_step(layer, ids, gu.dev(q[at], w), gu.dev(k[at], w), gu.dev(v[at], w), od)
            else:
                cache.attn_decode(layer, ids, gu.dev(q[at], w), od)
            if layer in (0, layers - 1):
                for b, p in enumerate(at):
                    ref = orc.gqa_attention(f64(q[p:p + 1]), f64(k[:p + 1]), f64(v[:p + 1]), np.array([p]), True)
                    assert gu.max_err(gu.host(od[b:b + 1]), ref) <= gu.TOL["bf16"]
    for b, n in enumerate(lens):
        for which, x in ((0, k), (1, v)):
            assert np.array_equal(cache.read_kv(b, layers - 1, which, n, 1), x[n:n + 1])
