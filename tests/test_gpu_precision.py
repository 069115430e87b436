"""How far attention is from 64-bit arithmetic, in the root mean square of the result: what the data types give and no less.

Bound for fp32, in units u = 2^-24 (a rounding is u / sqrt(3) in the mean): a score of head_dim D in chains of L products that
meet pairwise is off by sqrt(L / 2 + log2(D / L)) roundings (one less where the last one is kept), 1.6 u at most (D = 128, L = 8), and its weight by as much; the
weight itself by half a u; a tile's share of the output (chains of up to 8 keys, pairwise) and up to 20 tiles added one by one
by sqrt(4 + 2 + 20 / 2) roundings, 2.3 u; key ranges, sums and quotient by another u.  Together 3.0 u; the bound is 3.6."""
import numpy as np
import pytest
import torch

import paper_2510_09608_amd as sv
import sv_inputs as si
from oracle import sv_oracle as orc
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
PLAIN, TERMS = sv.SV_CHUNK_F32_PLAIN, sv.SV_CHUNK_F32_TERMS


def cache_of(dtype, hq, hkv, d, lens, max_q, seed):
    """A cache whose stream b holds lens[b] tokens, every one the beginning of the same rows; and those rows."""
    w = si.Workload("p", 1, hq, hkv, d, dtype, 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, seed)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32 if dtype == "f32" else sv.SV_DTYPE_BF16, sv.SV_ROPE_NONE, 1e4, (0, 0, 0),
                     len(lens), max(lens) + 8, max_q)
    _, k, v = w.qkv(0, np.arange(max(lens)))
    for b, n in enumerate(lens):
        cache.append(b, 0, np.zeros(n, np.uint8), None, gu.dev(k[:n], w), gu.dev(v[:n], w))
    return cache, w, k.astype(np.float64), v.astype(np.float64)


def rms_error(o, ref):
    return float(np.sqrt(np.mean((gu.host(o) - ref) ** 2) / np.mean(ref ** 2)))


def one_chunk(q, k, v, causal, splits):
    """sv_attn_chunk of fp32 queries on fp32 keys and values, [tokens][heads][head_dim], without a rotary mode."""
    (n_q, hq, d), (n_kv, hkv, _) = q.shape, k.shape
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n_kv + 8, n_q)
    cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
    q, k, v = (torch.from_numpy(np.ascontiguousarray(x, np.float32)).to("cuda:0") for x in (q, k, v))
    cache.append(0, 0, np.zeros(n_kv, np.uint8), None, k, v)
    o = torch.empty_like(q)
    cache.attn_chunk(0, 0, q, o, causal)
    return o


def exact_chunk(q, k, v, causal):
    n_q, n_kv = len(q), len(k)
    return orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.arange(n_kv - n_q, n_kv), causal)


def chunk_error(*case):
    return chunk_case(*case)[:2]


def chunk_case(dtype, hq, hkv, d, n_kv, n_q, causal, splits=0):
    print(f"chunk {dtype} {hq}/{hkv} x {d}: {n_q} queries, {n_kv} keys, {splits} ranges", flush=True)
    cache, w, k, v = cache_of(dtype, hq, hkv, d, [n_kv], n_q, 9000 + n_kv)
    cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
    q = w.qkv(0, np.arange(60000, 60000 + n_q))[0]
    qd = gu.dev(q, w)
    o = torch.empty_like(qd)
    cache.attn_chunk(0, 0, qd, o, causal)
    ref = orc.gqa_attention(q.astype(np.float64), k, v, np.arange(n_kv - n_q, n_kv), causal)
    return rms_error(o, ref), ref, o


@pytest.mark.parametrize("hq,hkv,d,n_kv,n_q,causal", [
    (28, 4, 128, 400, 64, True), (8, 2, 128, 72, 16, True), (8, 2, 128, 2600, 300, True), (28, 4, 128, 1500, 9, False),
    (2, 1, 64, 400, 16, True), (8, 8, 64, 400, 130, True), (8, 8, 64, 2600, 500, True)])
def test_fp32_chunk_is_as_exact_as_its_sums(hq, hkv, d, n_kv, n_q, causal):
    """Chunk prefill as the library chooses kernel and key ranges, and their merge."""
    assert chunk_error("f32", hq, hkv, d, n_kv, n_q, causal)[0] <= 3.6 * U


@pytest.mark.parametrize("hq,hkv,d,n_kv,n_q,causal,splits", [
    (28, 4, 128, 586, 586, True, 0), (32, 8, 128, 587, 287, True, 0), (8, 8, 128, 821, 521, True, 0), (8, 2, 128, 1156, 456, True, 0),
    (8, 2, 128, 2600, 300, True, 1), (28, 4, 128, 1500, 200, False, 2), (14, 2, 64, 2000, 90, True, 2), (8, 8, 64, 2600, 500, True, 4)])
def test_fp32_chunk_by_fp32_instructions_is_as_exact_as_its_sums(hq, hkv, d, n_kv, n_q, causal, splits):
    """Ranges of 4 to 82 tiles of 32 keys through the kernel that has 32 rows to a wavefront: tiles that take turns in LDS, sums
    rescaled on the way."""
    assert chunk_error("f32", hq, hkv, d, n_kv, n_q, causal, splits | PLAIN)[0] <= 3.6 * U


def decode_error(dtype, hq, hkv, d, lens, steps=12, tiles=0):
    print(f"decode {dtype} {hq}/{hkv} x {d}: {lens} keys, {tiles} tiles", flush=True)
    cache, w, k, v = cache_of(dtype, hq, hkv, d, lens, 16, 9100 + sum(lens))
    cache.set_option(sv.SV_OPT_DECODE_TILES_PER_WAVE, tiles)
    q = w.qkv(0, np.arange(60000, 60000 + steps * len(lens)))[0].reshape(steps, len(lens), hq, d)
    o = torch.stack([gu.dev(x, w) for x in q])
    for i in range(steps):
        cache.attn_decode(0, list(range(len(lens))), gu.dev(q[i], w), o[i])
    at = np.tile(np.array(lens) - 1, steps)
    ref = orc.gqa_attention(q.reshape(-1, hq, d).astype(np.float64), k, v, at, True)
    ref = ref.reshape(q.shape)
    return rms_error(o, ref), ref


@pytest.mark.parametrize("hq,hkv,d,lens", [
    (8, 2, 128, [400]), (28, 4, 128, [72]), (28, 4, 128, [3000]), (2, 1, 64, [72]), (8, 8, 64, [1500]),
    (8, 2, 128, [400, 311, 1700]), (8, 8, 64, [300, 20, 900, 1500, 64])])
def test_fp32_decode_is_as_exact_as_its_sums(hq, hkv, d, lens):
    """Decode of one stream (key ranges merged in the launch) and of several (merged by a launch of its own)."""
    assert decode_error("f32", hq, hkv, d, lens)[0] <= 3.6 * U


@pytest.mark.parametrize("tiles", [0, 3])
@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (4, 2, 128), (3, 1, 128), (8, 2, 128), (8, 8, 64), (2, 1, 64), (6, 2, 64), (16, 4, 64)])
def test_fp32_decode_of_up_to_four_heads_per_kv_head(hq, hkv, d, tiles):
    """The 4 x 4 matrix instructions: the first and last key of a tile, wavefronts with one tile, three or none, one stream and
    several (0: the number of tiles a wavefront is given by itself)."""
    for lens in ([1], [15], [16], [17], [65], [129], [407], [33, 200, 1, 64]):
        assert decode_error("f32", hq, hkv, d, lens, steps=4, tiles=tiles)[0] <= 3.6 * U


def rounded_to_bf16(ref):
    """Root mean square error of the exact result once it is rounded to bf16."""
    return rms_error(torch.from_numpy(ref).to(torch.bfloat16), ref)


@pytest.mark.parametrize("hq,hkv,lens", [(16, 2, [400]), (14, 2, [5392]), (4, 4, [33]), (16, 2, [1500, 31, 640]), (4, 4, [2300, 2300])])
def test_bf16_decode_of_head_dim_64_rounds_its_result_alone(hq, hkv, lens):
    """Probabilities keep their 24 bits: what is left is the result's rounding.  (fp32 sums of some thousand products are off
    by about 1e-6, in quadrature with 1.7e-3; with probabilities rounded to bf16 it would be 1.2 times as much.)"""
    err, ref = decode_error("bf16", hq, hkv, 64, lens)
    assert err <= 1.002 * rounded_to_bf16(ref)


@pytest.mark.parametrize("hq,hkv,n_kv,n_q,causal,splits", [
    (16, 2, 400, 64, True, 1), (14, 2, 1500, 130, False, 1), (4, 4, 33, 33, True, 1), (16, 2, 700, 700, True, 1),
    (16, 2, 5392, 256, True, 0), (4, 4, 1500, 300, True, 0), (14, 2, 900, 20, False, 9)])
def test_bf16_chunk_of_head_dim_64_rounds_its_result_alone(hq, hkv, n_kv, n_q, causal, splits):
    """Probabilities to 16 bits and more (2^-17 in quadrature with 2^-9.2), sums and partial results in fp32."""
    err, ref = chunk_error("bf16", hq, hkv, 64, n_kv, n_q, causal, splits)
    assert err <= 1.002 * rounded_to_bf16(ref)


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (2, 1, 64)])
def test_fp32_infinite_value_stays_infinite(hq, hkv, d):
    """One value of V is infinite: so is the output in that head dim, and no other (one key range and several, few rows and
    many, one decode row and two)."""
    lens = [300, 300]
    w = si.Workload("i", 1, hq, hkv, d, "f32", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9990)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 2, 308, 100)
    q, k, v = w.qkv(0, np.arange(300))
    v = v.copy()
    v[123, 0, 5] = np.inf
    for s in range(2):
        cache.append(s, 0, np.zeros(300, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    want = np.zeros((hq, d), bool)
    want[:hq // hkv, 5] = True
    outs = []
    for n_q in (100, 3):
        for splits in (1, 3, 1 | PLAIN, 3 | PLAIN, 1 | TERMS, 3 | TERMS):
            print(f"infinite value {hq}/{hkv} x {d} n_q={n_q} splits={splits}", flush=True)
            cache.set_option(sv.SV_OPT_CHUNK_SPLITS, splits)
            o = torch.empty(n_q, hq, d, device="cuda:0")
            cache.attn_chunk(0, 0, gu.dev(q[:n_q], w), o, False)
            outs.append(o)
    for ids in ([0], [0, 1]):
        o = torch.empty(len(ids), hq, d, device="cuda:0")
        cache.attn_decode(0, ids, gu.dev(q[:len(ids)], w), o)
        outs.append(o)
    for o in outs:
        x = gu.host(o)
        assert (np.isposinf(x) == want).all() and np.isfinite(x[:, ~want]).all()


@pytest.mark.parametrize("hq,hkv,d,n_kv,n_q,causal,splits", [
    (8, 2, 128, 403, 403, True, 1),     # row tiles that see 1 to 13 tiles of keys: halves with a tile more than the other, or none
    (8, 2, 128, 416, 33, False, 1), (8, 2, 128, 1031, 65, True, 2), (6, 6, 128, 700, 129, True, 1), (28, 4, 128, 1500, 200, True, 3),
    (2, 1, 64, 320, 320, True, 1), (8, 8, 64, 353, 161, False, 1), (14, 2, 64, 2000, 90, True, 4)])
def test_fp32_chunk_from_bf16_terms_is_as_exact_as_its_sums(hq, hkv, d, n_kv, n_q, causal, splits):
    """The kernel whose products are made of bf16 terms, on ranges of 10 to 22 tiles of 32 keys: the bound of the fp32
    instructions (what the six products leave out and the matrix cores' rounding are in what is measured below it), and other
    bits than theirs."""
    err, _, o = chunk_case("f32", hq, hkv, d, n_kv, n_q, causal, splits | TERMS)
    assert err <= 3.6 * U
    assert not torch.equal(chunk_case("f32", hq, hkv, d, n_kv, n_q, causal, splits | PLAIN)[2], o)


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("q_exp,k_exp,v_exp,ignored", [
    (70, -70, 0, False), (115, -115, 0, False), (-110, 110, 0, False), (-118, 118, 0, False), (0, 0, -115, False), (0, 0, 100, False), (0, 0, 0, True)])
def test_fp32_chunk_of_numbers_that_terms_do_not_hold(hq, hkv, d, q_exp, k_exp, v_exp, ignored):
    """Queries, keys and values scaled by powers of two, at which bf16 terms still hold them (70, -110, 100) and would lose bits
    (115, -118, -115: 17 to 140 times 2^-24 with three terms, as computed in 64 bits), and a key whose scores are minus infinity:
    results as exact as ever."""
    print(f"terms {hq}/{hkv} x {d}: 2^{q_exp} 2^{k_exp} 2^{v_exp} ignored={ignored}", flush=True)
    n_kv, n_q = 330, 140
    w = si.Workload("t", 1, hq, hkv, d, "f32", 2, 1e4, (0, 0, 0), 0, 0, 0, 0, 0, 0, None, 0, 9991)
    cache = sv.Cache(1, hq, hkv, d, sv.SV_DTYPE_F32, sv.SV_ROPE_NONE, 1e4, (0, 0, 0), 1, n_kv + 8, n_q)
    q, k, v = (x.copy() for x in w.qkv(0, np.arange(n_kv)))
    q = q[:n_q]
    if ignored:
        q[:, :, 3] = np.abs(q[:, :, 3]) + 0.5
        k[77, :, 3] = -np.inf
    q, k, v = q * np.float32(2.0 ** q_exp), k * np.float32(2.0 ** k_exp), v * np.float32(2.0 ** v_exp)
    cache.append(0, 0, np.zeros(n_kv, np.uint8), None, gu.dev(k, w), gu.dev(v, w))
    cache.set_option(sv.SV_OPT_CHUNK_SPLITS, 1 | TERMS)
    o = torch.empty(n_q, hq, d, device="cuda:0")
    cache.attn_chunk(0, 0, gu.dev(q, w), o, False)
    if ignored:   # (the same with that key left out)
        k, v = np.delete(k, 77, 0), np.delete(v, 77, 0)
    ref = orc.gqa_attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), np.full(n_q, len(k) - 1), True)
    s = 2.0 ** -v_exp
    assert rms_error(torch.from_numpy(gu.host(o).astype(np.float64) * s), ref * s) <= 3.6 * U


def normal(seed, *shape):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


def one_hot(seed, n, heads, d, dims):
    """Rows that have one number only, in one of dims."""
    rng = np.random.default_rng(seed)
    x = np.zeros((n, heads, d), np.float32)
    np.put_along_axis(x, rng.choice(dims, (n, heads, 1)), rng.standard_normal((n, heads, 1)).astype(np.float32), 2)
    return x


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("what", ["queries", "keys", 0, 1, 2, 3])
def test_fp32_chunk_scores_that_are_one_product(hq, hkv, d, what):
    """Queries (anywhere, in the i-th quarter of the head dims) or keys of a single number: a score is one product, which an fp32
    instruction rounds (2^-25.2 of it in the mean) and of which the six products of bf16 terms leave out 2^-27.4.  With nothing
    else lost on the way the error, which such scores dominate, is no larger than by fp32 instructions."""
    n, n_q = 1024, 256
    k, v, q = normal(1, n, hkv, d), normal(2, n, hkv, d), normal(3, n_q, hq, d) * np.float32(16)   # scores of N(0, 16^2)
    if what == "keys":
        k = one_hot(4, n, hkv, d, np.arange(d)) * np.float32(np.sqrt(d))
    else:
        dims = np.arange(d) if what == "queries" else np.arange(d // 4) + d // 4 * what
        q = one_hot(5, n_q, hq, d, dims) * np.float32(16 * np.sqrt(d))
    ref = exact_chunk(q, k, v, False)
    plain, terms = (rms_error(one_chunk(q, k, v, False, 1 | kind), ref) for kind in (PLAIN, TERMS))
    print(f"single numbers {what} {hq}/{hkv} x {d}: {plain / U:.2f} and {terms / U:.2f} u", flush=True)
    assert terms <= plain


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 8, 64)])
def test_fp32_chunk_of_one_visible_key_is_its_value(hq, hkv, d):
    """The first query of a causal prefill, and queries of which every weight but one underflows: the value, but for the last place
    (its weight is 1 and what the score's last addition left: the product is rounded, and the quotient).  By bf16 terms the product is
    the sum of one exact large product and of small ones that are known to 2^-8 of a last place and off by as much, 2^-27.4 and more, as
    they leave out: one in 32 may round the other way."""
    off = {}
    for kind in (PLAIN, TERMS):
        n_off = 0
        for seed in range(8):
            q, k, v = normal(1 + 10 * seed, 160, hq, d), normal(2 + 10 * seed, 160, hkv, d), normal(3 + 10 * seed, 160, hkv, d)
            far = -np.abs(k)
            far[133] *= -100
            one = gu.host(one_chunk(q, k, v, True, 1 | kind))[0], np.repeat(v[0], hq // hkv, 0)
            sole = gu.host(one_chunk(np.abs(q), far, v, False, 2 | kind)), np.repeat(v[133], hq // hkv, 0)[None]
            for o, x in (one, sole):
                assert (np.abs(o - x) <= np.spacing(np.abs(x))).all()
            n_off += np.mean(one[0] != one[1]) / 8
        off[kind] = n_off
    print(f"one visible key {hq}/{hkv} x {d}: {off[PLAIN]:.4f} and {off[TERMS]:.4f} of the numbers are off", flush=True)
    assert off[TERMS] <= off[PLAIN] + 1 / 32


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("kind", [PLAIN, TERMS])
@pytest.mark.parametrize("v_exp", [40, 60, 100])
def test_fp32_chunk_of_weights_that_terms_would_not_hold(hq, hkv, d, kind, v_exp):
    """Head dims whose only values lie behind weights of 2^-97 to 2^-124 of the largest, and are large enough to matter: the weights keep
    their 24 bits, as the others do (a bf16 term ends at 2^-133: a weight of 2^-117 would be off by 8e-6 of itself, one of 2^-125 by
    2e-3).  The scores are one product of few bits, and exact."""
    n, n_q, far = 330, 140, np.arange(20, 330, 10)
    rng = np.random.default_rng(d + v_exp)
    unit = 16 if d == 128 else 8
    q, k, v = np.zeros((n_q, hq, d), np.float32), normal(2, n, hkv, d), normal(3, n, hkv, d)
    q[:, :, 7] = unit * (1 + rng.integers(0, 9, (n_q, hq)) / 64)
    k[:, :, 7] = rng.integers(-8, 9, (n, hkv)) / 8
    k[12, :, 7] = 2
    k[far, :, 7] = 2 - np.round(8 * np.linspace(67, 76, len(far)) * np.sqrt(d) / unit)[:, None] / 8   # at most 76.2 x 9 / 8 = 85.8 nats
    v[:, :, d // 2:] = 0
    for i, t in enumerate(far):   # every such key has head dims of its own
        own = np.arange(d // 2 + i, d, len(far))
        v[t, :, own] = normal(100 + i, len(own), hkv) * np.float32(2.0 ** v_exp)
    ref = exact_chunk(q, k, v, False)
    o = gu.host(one_chunk(q, k, v, False, 1 | kind)).astype(np.float64)
    err = np.sqrt(np.mean((o[..., d // 2:] / ref[..., d // 2:] - 1) ** 2, (0, 1)))   # (a number is one product)
    print(f"small weights {hq}/{hkv} x {d} 2^{v_exp} terms={kind == TERMS}: {err.max() / U:.2f} u", flush=True)
    assert err.max() <= 3.6 * U


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("kind", [PLAIN, TERMS])
@pytest.mark.parametrize("v_exp", [-104, -109, -112, -120, -127, -134, -140])
@pytest.mark.parametrize("dims", [4, 8, 0])
def test_fp32_chunk_of_values_that_terms_would_not_hold(hq, hkv, d, kind, v_exp, dims):
    """Values around 2^-109, below which three bf16 terms lose bits, in the head dims that have a bit (0: in all): as exact as ever, in
    the first rows of a causal prefill, too, which see few keys.  Results below 2^-126 are multiples of 2^-149."""
    n = 400
    q, k, v = normal(1, n, hq, d), normal(2, n, hkv, d), normal(3, n, hkv, d)
    if v_exp == -109:   # just as large as terms hold
        v = np.sign(v) * (1 + np.random.default_rng(4).random(v.shape, np.float32))
    small = (np.arange(d) & dims) != 0 if dims else np.ones(d, bool)
    v[:, :, small] *= np.float32(2.0 ** v_exp)
    ref = exact_chunk(q, k, v, True)
    o = gu.host(one_chunk(q, k, v, True, 1 | kind)).astype(np.float64)
    e, r = (o - ref)[..., small], ref[..., small]
    for rows in (8, n):
        err, size = np.sqrt(np.mean(e[:rows] ** 2)), np.sqrt(np.mean(r[:rows] ** 2))
        print(f"small values {hq}/{hkv} x {d} 2^{v_exp} bit {dims} terms={kind == TERMS} rows={rows}: {err / size / U:.2f} u", flush=True)
        assert err <= 3.6 * U * size + 2.0 ** -149
