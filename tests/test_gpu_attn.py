"""GPU parity of the attention path (tm_attn.h) against the oracle: the quantise-and-store kernel bit for bit, the decode
attention within  |O - Oref| <= 2e-3 + 5e-3*|Oref|  and relative Frobenius error <= 2e-3  (the probabilities enter the
second matrix product as fp16, and O is rounded to fp16 once)."""
import sys

import numpy as np
import pytest

from oracle import oracle_attn as oa
from workloads import attn as wa

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2508_15601_amd as tm
    tm.load_library()
    return tm


def _say(msg):
    print(msg, file=sys.stderr, flush=True)


def _close(O, Oref):
    o, r = O.astype(np.float64), Oref.astype(np.float64)
    worst = float((np.abs(o - r) / (2e-3 + 5e-3 * np.abs(r))).max())
    fro = float(np.linalg.norm(o - r) / max(np.linalg.norm(r), 1e-30))
    return worst <= 1.0 and fro <= 2e-3, worst, fro


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("B,Hkv,T,chunks", [(1, 1, 32, [32]), (2, 3, 70, [40, 1, 1, 28]), (3, 2, 97, [97]), (2, 1, 33, [1] * 33),
                                             (2, 2, 300, [5, 200, 15, 80])])
@pytest.mark.parametrize("bits", [8, 4])
def test_kv_append_bit_exact(tm, B, Hkv, T, chunks, bits):
    """Keys and values appended in chunks land in the cache layout with exactly the oracle's codes and pairs."""
    import torch
    _say(f"kv append B={B} Hkv={Hkv} T={T} chunks={chunks[:4]} bits={bits}")
    cbytes = 128 * bits // 8
    _, K, V, _ = wa.draw(B, Hkv, Hkv, T, seed=T)
    K[0, 0, 0, :] = 1.5                                   # a constant row: scale falls back to 1
    V[-1, -1, -1, :64] = 0.0
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    cap = cache.capacity
    tm.tm_kv_upload(cache, np.zeros(B * Hkv * cap * cbytes, np.uint8), np.zeros(B * Hkv * cap * cbytes, np.uint8),
                    np.zeros(B * Hkv * cap * 2, np.uint32))
    pos = 0
    for n in chunks:
        Kn = np.ascontiguousarray(K[:, :, pos:pos + n].transpose(0, 2, 1, 3))      # [B, n, Hkv, 128]
        Vn = np.ascontiguousarray(V[:, :, pos:pos + n].transpose(0, 2, 1, 3))
        tm.tm_kv_append(cache, _dev(Kn), _dev(Vn), torch.full((B,), pos, dtype=torch.int32, device="cuda"))
        pos += n
    kbuf, vbuf, szbuf = tm.tm_kv_download(cache)
    Kq, Ks, Kz, Vq, Vs, Vz = oa.kv_cache_unpack(kbuf, vbuf, szbuf, B, Hkv, cap, bits)
    for got, want in zip((Kq, Ks, Kz), oa.kv_quantise(K, bits)):
        g, w = got[:, :, :T], want
        assert np.array_equal(g.view(np.uint16) if g.dtype == np.float16 else g, w.view(np.uint16) if w.dtype == np.float16 else w)
    for got, want in zip((Vq, Vs, Vz), oa.kv_quantise(V, bits)):
        g, w = got[:, :, :T], want
        assert np.array_equal(g.view(np.uint16) if g.dtype == np.float16 else g, w.view(np.uint16) if w.dtype == np.float16 else w)
    assert not Kq[:, :, T:].any() and not Vq[:, :, T:].any()                       # nothing written past the tokens
    # tokens that would fall outside the cache are dropped
    tm.tm_kv_append(cache, _dev(Kn), _dev(Vn), torch.full((B,), cap, dtype=torch.int32, device="cuda"))
    k2, v2, s2 = tm.tm_kv_download(cache)
    assert np.array_equal(k2, kbuf) and np.array_equal(v2, vbuf) and np.array_equal(s2, szbuf)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("n", [1, 40])                       # the kernels of a decoding step and of a prompt
def test_kv_append_extreme_values(tm, n, bits):
    """Codes are those of the division, bit for bit, over the whole range of fp16: values of every exponent, vectors of subnormal
    numbers only (a scale that rounds to a subnormal one, or to zero), infinities, a constant, the largest range."""
    import torch
    B, Hkv = 8, 3
    _say(f"kv append extreme values n={n} bits={bits}")
    rng = np.random.default_rng(n + bits)
    x = rng.integers(0, 1 << 16, (2, B, n, Hkv, 128), np.uint16).view(np.float16)
    x = np.where(np.isfinite(x), x, np.float16(0))           # every finite bit pattern
    x[:, 1] = (x[:, 1].view(np.uint16) & 0x83ff).view(np.float16)            # subnormal
    x[:, 2] = (x[:, 2].view(np.uint16) & 0x8007).view(np.float16)            # a range below half the smallest scale
    x[:, 3, ..., 5] = np.inf
    x[:, 4, ..., 9] = -np.inf
    x[:, 5] = np.float16(0.37)
    x[:, 6, ..., 0], x[:, 6, ..., 1] = np.float16(65504), np.float16(-65504)
    cache = tm.tm_kv_create(B, Hkv, 64, bits)
    tm.tm_kv_append(cache, _dev(x[0]), _dev(x[1]), torch.zeros(B, dtype=torch.int32, device="cuda"))
    got = oa.kv_cache_unpack(*tm.tm_kv_download(cache), B, Hkv, cache.capacity, bits)
    with np.errstate(all="ignore"):
        want = [w for v in x for w in oa.kv_quantise(v.transpose(0, 2, 1, 3), bits)]
    for g, w in zip(got, want):
        assert np.array_equal(g[:, :, :n].astype(np.float32), w.astype(np.float32))
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
def test_kv_append_ragged_positions(tm, bits):
    """Sequences at different positions, runs that start and end inside a 32-token block (the block-wise kernel merges with
    what the cache holds), a run cut off by the capacity, and a run that starts before position 0."""
    import torch
    B, Hkv, cap = 3, 2, 192
    _say(f"kv append ragged positions bits={bits}")
    cbytes = 128 * bits // 8
    _, K, V, _ = wa.draw(B, Hkv, Hkv, cap, seed=11)
    cache = tm.tm_kv_create(B, Hkv, cap, bits)
    assert cache.capacity == cap
    tm.tm_kv_upload(cache, np.zeros(B * Hkv * cap * cbytes, np.uint8), np.zeros(B * Hkv * cap * cbytes, np.uint8),
                    np.zeros(B * Hkv * cap * 2, np.uint32))
    filled = np.zeros((B, cap), bool)
    # (count, positions per sequence): first lays single tokens and short runs, then long runs over and between them
    for n, pos in [(3, [0, 30, 189]), (20, [5, 40, 100]), (70, [25, 64, 150]), (33, [-7, 129, 10]), (17, [95, 0, 175])]:
        Kn = np.zeros((B, n, Hkv, 128), np.float16)
        Vn = np.zeros((B, n, Hkv, 128), np.float16)
        for b in range(B):
            for j in range(n):
                t = pos[b] + j
                if 0 <= t < cap:
                    Kn[b, j], Vn[b, j] = K[b, :, t], V[b, :, t]
                    filled[b, t] = True
                else:
                    Kn[b, j], Vn[b, j] = 7.0, -3.0              # must never reach the cache
        tm.tm_kv_append(cache, _dev(Kn), _dev(Vn), torch.tensor(pos, dtype=torch.int32, device="cuda"))
    kbuf, vbuf, szbuf = tm.tm_kv_download(cache)
    got = oa.kv_cache_unpack(kbuf, vbuf, szbuf, B, Hkv, cap, bits)
    want = oa.kv_quantise(K, bits) + oa.kv_quantise(V, bits)
    m = filled[:, None, :]
    assert filled.any() and not filled.all()
    for g, w in zip(got, want):
        g = g.view(np.uint16) if g.dtype == np.float16 else g
        w = w.view(np.uint16) if w.dtype == np.float16 else w
        mm = np.broadcast_to(m[..., None] if g.ndim == 4 else m, g.shape)
        assert np.array_equal(g[mm], w[mm])
        assert not g[~mm].any()                                  # untouched tokens still hold the zeros uploaded
    cache.close()


ATTN_CASES = [
    # B, Hq, Hkv, T, lens (None: drawn)
    (1, 1, 1, 1, [1]),
    (2, 4, 4, 31, None),
    (2, 8, 2, 32, [32, 17]),
    (3, 8, 1, 33, None),
    (2, 16, 1, 100, None),
    (1, 32, 8, 257, None),
    (4, 12, 3, 1000, None),                # several blocks per wave
    (1, 8, 2, 5000, [5000]),               # split context, merged by the second kernel
    (2, 8, 8, 4100, [4100, 1300]),         # splits of which some are empty for the short sequence
    (1, 64, 8, 640, None),
    (2, 4, 2, 64, [33, 64]),               # a 4-bit block whose second half holds one token / is full
    (1, 8, 2, 8200, [8161]),               # split context ending in the first half of a 64-token block
    # more than sixteen query heads per KV head: one pass per sixteen heads (a last pass of 16, of 4, of 8 heads)
    (2, 32, 1, 300, None),
    (1, 40, 2, 5000, [5000]),              # 20 per KV head, split context merged by the second kernel
    (2, 48, 2, 700, [700, 90]),            # 24 per KV head, split context merged in the kernel
]


@pytest.mark.parametrize("B,Hq,Hkv,T,lens", ATTN_CASES)
@pytest.mark.parametrize("bits", [8, 4])
def test_attn_decode_against_oracle(tm, B, Hq, Hkv, T, lens, bits):
    import torch
    _say(f"attn decode B={B} Hq={Hq} Hkv={Hkv} T={T} lens={lens} bits={bits}")
    Q, K, V, drawn = wa.draw(B, Hq, Hkv, T, seed=B * 100 + Hq + T)
    lens = np.array(lens, np.int32) if lens is not None else drawn
    Kq, Ks, Kz = oa.kv_quantise(K, bits)
    Vq, Vs, Vz = oa.kv_quantise(V, bits)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    cap = cache.capacity
    # the cache is filled by the library's own kernel; positions past T keep whatever the allocation held
    tm.tm_kv_append(cache, _dev(np.ascontiguousarray(K.transpose(0, 2, 1, 3))), _dev(np.ascontiguousarray(V.transpose(0, 2, 1, 3))),
                    torch.zeros(B, dtype=torch.int32, device="cuda"))
    scale = 1.0 / np.sqrt(128.0)
    outs = []
    for _ in range(2):
        O = torch.full((B, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
        tm.tm_attn_decode(_dev(Q), cache, _dev(lens), O, scale, max_len=int(lens.max()))
        torch.cuda.synchronize()
        outs.append(O.cpu().numpy())
    assert np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))        # run-to-run identical
    Oref = oa.attn_decode(Q, Kq, Ks, Kz, Vq, Vs, Vz, lens, scale)
    ok, worst, fro = _close(outs[0], Oref)
    assert ok, (worst, fro)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
def test_attn_decode_special_cases(tm, bits):
    """Sharp softmax (one token takes all the weight), a sequence without tokens, cache bytes past the context that hold
    NaN pairs, and max_len left at 0."""
    import torch
    _say(f"attn special cases bits={bits}")
    B, Hq, Hkv, T = 2, 8, 2, 128
    Q, K, V, _ = wa.draw(B, Hq, Hkv, T, seed=5)
    Kq, Ks, Kz = oa.kv_quantise(K, bits)
    Vq, Vs, Vz = oa.kv_quantise(V, bits)
    Kd = oa.kv_dequant(Kq, Ks, Kz)
    Q[0, :4] = (Kd[0, 0, 70] * 1.0).astype(np.float16)     # heads 0..3 (KV head 0) point at token 70
    lens = np.array([80, 0], np.int32)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    cap = cache.capacity
    assert cap == T
    kbuf, vbuf, szbuf = wa.encode_cache(*[np.ascontiguousarray(a) for a in (Kq, Ks, Kz, Vq, Vs, Vz)], bits=bits)
    sz = szbuf.reshape(B, Hkv, cap, 2).copy()
    sz[:, :, 80:] = 0x7E007E00                              # NaN scale and zero-point past the context
    tm.tm_kv_upload(cache, kbuf, vbuf, sz.reshape(-1))
    O = torch.full((B, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
    tm.tm_attn_decode(_dev(Q), cache, _dev(lens), O, 4.0)   # max_len = 0: the capacity
    torch.cuda.synchronize()
    O = O.cpu().numpy()
    assert not O[1].any()                                   # no tokens: zeros
    Oref = oa.attn_decode(Q[:1], Kq[:1], Ks[:1], Kz[:1], Vq[:1], Vs[:1], Vz[:1], lens[:1], 4.0)
    ok, worst, fro = _close(O[:1], Oref)
    assert ok, (worst, fro)
    assert np.allclose(O[0, 0].astype(np.float64), oa.kv_dequant(Vq, Vs, Vz)[0, 0, 70], rtol=1e-2, atol=2e-3)
    # a max_len below the sequence's length cuts the context at a block boundary instead of dropping blocks in the middle
    tm.tm_kv_upload(cache, kbuf, vbuf, szbuf)
    lens2 = np.array([128, 100], np.int32)
    O2 = torch.full((B, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
    tm.tm_attn_decode(_dev(Q), cache, _dev(lens2), O2, 0.1, max_len=64)
    torch.cuda.synchronize()
    Oref2 = oa.attn_decode(Q, Kq, Ks, Kz, Vq, Vs, Vz, np.array([64, 64], np.int32), 0.1)
    ok, worst, fro = _close(O2.cpu().numpy(), Oref2)
    assert ok, (worst, fro)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
def test_attn_decode_full_size_sampled(tm, bits):
    """The benchmark's largest shape in its own launch configuration (batch 128 x context 2048, 32 query / 8 KV heads, the
    prompt stored by one block-wise append, one decode launch without splits); the oracle recomputes a sample of the
    sequences from the same keys and values."""
    import torch
    B, Hq, Hkv, T = 128, 32, 8, 2048
    _say(f"attn full size B={B} T={T} bits={bits}")
    g = torch.Generator(device="cuda").manual_seed(1234 + bits)
    K = torch.randn((B, T, Hkv, 128), generator=g, device="cuda").to(torch.float16)
    V = torch.randn((B, T, Hkv, 128), generator=g, device="cuda").to(torch.float16)
    Q = torch.randn((B, Hq, 128), generator=g, device="cuda").to(torch.float16)
    lens = torch.randint(1, T + 1, (B,), generator=g, device="cuda").to(torch.int32)
    lens[0] = T
    lens[5] = 1
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    tm.tm_kv_append(cache, K, V, torch.zeros(B, dtype=torch.int32, device="cuda"))
    O = torch.full((B, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
    scale = 1.0 / np.sqrt(128.0)
    tm.tm_attn_decode(Q, cache, lens, O, scale, max_len=T)
    torch.cuda.synchronize()
    assert not torch.isnan(O).any()
    sample = [0, 5, 17, 64, 127]
    Ks = K[sample].permute(0, 2, 1, 3).contiguous().cpu().numpy()           # [n, Hkv, T, 128]
    Vs = V[sample].permute(0, 2, 1, 3).contiguous().cpu().numpy()
    Oref = oa.attn_decode(Q[sample].cpu().numpy(), *oa.kv_quantise(Ks, bits), *oa.kv_quantise(Vs, bits),
                          lens[sample].cpu().numpy(), scale)
    ok, worst, fro = _close(O[sample].cpu().numpy(), Oref)
    assert ok, (worst, fro)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hkv,G,T,bound", [
    (2, 14, 4, 4800, 0),       # 28 (sequence, head) pairs: nine splits, merged by the last CTA in two batches (4-bit: eight or fewer)
    (1, 16, 2, 16384, 0),      # sixteen splits (4-bit: the same)
    (1, 3, 2, 16384, 0),       # more than sixteen: the merge kernel
    (2, 66, 1, 8192, 0),       # 132 pairs over a long context: two CTAs per CU
    (5, 60, 9, 700, 300),      # more pairs than CUs: no split; a bound below the lengths
])
def test_attn_decode_splits(tm, B, Hkv, G, T, bound, bits):
    """Every way a context is split and merged, with scores that grow along the context (the running reference has to move
    again and again, the merge has to weigh splits far apart), a sequence of one token and one without any."""
    import torch
    _say(f"attn decode splits B={B} Hkv={Hkv} G={G} T={T} bits={bits}")
    rng = np.random.default_rng(T + Hkv + bits)
    g = torch.Generator(device="cuda").manual_seed(T + bits)
    K, V = (torch.randn((B, T, Hkv, 128), generator=g, device="cuda").to(torch.float16) for _ in range(2))
    Q = torch.randn((B, Hkv * G, 128), generator=g, device="cuda").to(torch.float16)
    direction = Q.view(B, 1, Hkv, G, 128)[:, :, :, 0].float()
    K = (K.float() + torch.linspace(-1.0, 1.0, T, device="cuda").view(1, T, 1, 1) * direction).to(torch.float16)
    lens = np.array([T] + [0, 1, T // 2, T - 1][:B - 1], np.int32)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    for t in range(0, T, 2048):
        tm.tm_kv_append(cache, K[:, t:t + 2048].contiguous(), V[:, t:t + 2048].contiguous(), torch.full((B,), t, dtype=torch.int32, device="cuda"))
    outs = []
    for _ in range(3):
        O = torch.full((B, Hkv * G, 128), float("nan"), dtype=torch.float16, device="cuda")
        tm.tm_attn_decode(Q, cache, _dev(lens), O, 128 ** -0.5, max_len=bound)
        torch.cuda.synchronize()
        outs.append(O.cpu().numpy())
    assert all(np.array_equal(outs[0].view(np.uint16), o.view(np.uint16)) for o in outs[1:])
    seen = lens if not bound else np.minimum(lens, -(-bound // (256 // bits)) * (256 // bits))
    for b in range(B):
        if seen[b] == 0:
            assert not outs[0][b].any()
            continue
        hk = int(rng.integers(Hkv))
        k, v = (x[b:b + 1, :, hk:hk + 1].permute(0, 2, 1, 3).contiguous().cpu().numpy() for x in (K, V))
        ref = oa.attn_decode(Q[b:b + 1, hk * G:(hk + 1) * G].cpu().numpy(), *oa.kv_quantise(k, bits), *oa.kv_quantise(v, bits), seen[b:b + 1], 128 ** -0.5)
        ok, worst, fro = _close(outs[0][b:b + 1, hk * G:(hk + 1) * G], ref)
        assert ok, (b, worst, fro)
    cache.close()


@pytest.mark.parametrize("G", [4, 16])                       # both forms of the kernel: up to eight query heads per KV head, more
@pytest.mark.parametrize("bits", [8, 4])
def test_attn_decode_sums_of_a_long_context(tm, bits, G):
    """Unsplit contexts of 32768 tokens (256 (sequence, head) pairs, one CTA each) with a zero query: every probability is
    exactly one, so that the result is the mean of the dequantised values, up to the fp32 sums and the final rounding.  In units of
    a value's scale: a wave adds up 8192 codes of 127 on average, so its sums end near 2^20, where an fp32 ulp is 1/16 (0.036 rms on the
    way there).  256 products with, at four values a step, eight roundings of 0.29 ulp each make 0.47, the four waves 0.94; the
    result before the division is 42 * sqrt(32768) = 7600: 1.2e-4 of it (4-bit codes: sums and result are both 17 times smaller).
    (The bias of 1024 per code stays for 128 tokens at most, a seventh of those sums.)
    Twice that is allowed.  Sums that carry a conversion bias of 1024 per token to the end are eight times as long: 1e-3."""
    import torch
    B, Hkv, T = 64, 4, 32768
    _say(f"attn decode long sums bits={bits} G={G}")
    g = torch.Generator(device="cuda")
    g.manual_seed(bits + G)
    V = torch.randn((T, Hkv, 128), generator=g, device="cuda").half()
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    for t in range(0, T, 2048):
        v = V[t:t + 2048].expand(B, 2048, Hkv, 128).contiguous()
        tm.tm_kv_append(cache, v, v, torch.full((B,), t, dtype=torch.int32, device="cuda"))
    Q = torch.zeros((B, Hkv * G, 128), dtype=torch.float16, device="cuda")
    O = torch.full_like(Q, float("nan"))
    tm.tm_attn_decode(Q, cache, torch.full((B,), T, dtype=torch.int32, device="cuda"), O, 128 ** -0.5, max_len=T)
    torch.cuda.synchronize()
    q, s, z = oa.kv_quantise(V.cpu().numpy().transpose(1, 0, 2)[None], bits)
    ref = ((q[0].astype(np.float64) - z[0].astype(np.float64)[..., None]) * s[0].astype(np.float64)[..., None]).mean(1)     # [Hkv][128]
    got = O.cpu().numpy().reshape(B, Hkv, G, 128).astype(np.float64)
    rms = np.sqrt((ref ** 2).mean())
    floor = np.sqrt(((ref.astype(np.float16).astype(np.float64) - ref) ** 2).mean())
    err = np.sqrt(((got - ref[None, :, None]) ** 2).mean())
    _say(f"  error {err / rms:.3e} of the result, fp16 rounding alone {floor / rms:.3e}")
    assert err <= np.hypot(floor, 2.5e-4 * rms), (err / rms, floor / rms)
    cache.close()


@pytest.mark.parametrize("n,past", [(1, 4095), (1, 2047), (32, 2000), (512, 1500)])      # two decoding steps, both prompt kernels
@pytest.mark.parametrize("bits", [8, 4])
def test_attn_error_is_that_of_probabilities_and_result(tm, bits, n, past):
    """Gaussian queries, keys and values.  Two roundings to fp16 belong to the path: of the result (computed here) and of every
    probability times its scale.  The latter is 2^-10 / sqrt(12) of a power of two, over mantissas spread evenly in the
    logarithm 2.1e-4 of the value, independent from token to token, hence 2.1e-4 of the result.  A query rounded after its
    scaling would add as much again (the scores' spread is one): 3.6e-4 in all.  8 % above the two is allowed."""
    import torch
    Hkv, G, T = 8, 4, past + n
    _say(f"attn error bits={bits} n={n} past={past}")
    rng = np.random.default_rng(bits * 1000 + past)
    K, V = (rng.standard_normal((1, Hkv, T, 128)).astype(np.float16) for _ in range(2))
    Q = rng.standard_normal((1, n, Hkv * G, 128)).astype(np.float16)
    cache = tm.tm_kv_create(1, Hkv, T, bits)
    tm.tm_kv_append(cache, _dev(K.transpose(0, 2, 1, 3)), _dev(V.transpose(0, 2, 1, 3)), torch.zeros(1, dtype=torch.int32, device="cuda"))
    O = torch.full((1, n, Hkv * G, 128), float("nan"), dtype=torch.float16, device="cuda")
    if n == 1:
        tm.tm_attn_decode(_dev(Q[:, 0]), cache, torch.full((1,), T, dtype=torch.int32, device="cuda"), O[:, 0], 128 ** -0.5)
    else:
        tm.tm_attn_prefill(_dev(Q), cache, torch.full((1,), past, dtype=torch.int32, device="cuda"), O, 128 ** -0.5)
    torch.cuda.synchronize()
    k, v = (oa.kv_dequant(*oa.kv_quantise(x, bits))[0] for x in (K, V))                            # [Hkv][T][128]
    future = np.arange(T)[None] > past + np.arange(n)[:, None]
    ref = np.empty((n, Hkv * G, 128))
    for h in range(Hkv * G):
        s = np.where(future, -np.inf, Q[0, :, h].astype(np.float64) @ k[h // G].T * 128 ** -0.5)
        e = np.exp(s - s.max(1, keepdims=True))
        ref[:, h] = (e / e.sum(1, keepdims=True)) @ v[h // G]
    rms = np.sqrt((ref ** 2).mean())
    result = np.sqrt(((ref.astype(np.float16) - ref) ** 2).mean()) / rms
    err = np.sqrt(((O.cpu().numpy()[0] - ref) ** 2).mean()) / rms
    _say(f"  error {err:.3e}, rounding of the result {result:.3e}")
    assert err <= 1.08 * np.hypot(result, 2.1e-4), (err, result)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hkv,G,T,bound,splits", [
    (2, 72, 1, 8192, 8192, 4),       # just over half as many pairs as CUs, long contexts: two CTAs per CU
    (4, 72, 1, 8192, 8192, 2),       # a few pairs more than CUs
    (2, 80, 1, 8192, 8192, 1),       # between the two, and far above: one CTA per pair
    (5, 66, 9, 2048, 2048, 1),
    (4, 8, 2, 8192, 0, 8),           # fewer: cut into as many pieces as give one CTA per CU
    (1, 16, 2, 16384, 16384, 16),
])
def test_attn_decode_split_rule(tm, B, Hkv, G, T, bound, splits, bits):
    """How many pieces a context is cut into on 256 CUs, and that launches with as many are right."""
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    assert tm.tm_get_attn_plan(cache, Hkv * G, max_len=bound) == (splits, 0)
    cache.close()
    test_attn_decode_splits(tm, B, Hkv, G, T, bound, bits)


def _random_cases(n, seed):
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(n):
        Hkv = int(rng.choice([1, 2, 3, 8]))
        G = int(rng.choice([1, 2, 4, 5, 8, 9, 16]))
        B = int(rng.choice([1, 2, 5, 9]))
        T = int(rng.choice([1, 40, 64, 65, 130, 700, 2100, 6000]))
        cases.append((i, B, Hkv * G, Hkv, T, int(rng.choice([4, 8]))))
    return cases


@pytest.mark.parametrize("i,B,Hq,Hkv,T,bits", _random_cases(24, 2024))
def test_attn_decode_random_shapes(tm, i, B, Hq, Hkv, T, bits):
    """Seeded random shapes: group sizes on both sides of the shared-pass limit (8), odd batch and head counts, contexts
    from one token to several splits, ragged lengths (some sequences empty), both code widths."""
    import torch
    _say(f"attn random {i}: B={B} Hq={Hq} Hkv={Hkv} T={T} bits={bits}")
    Q, K, V, lens = wa.draw(B, Hq, Hkv, T, seed=1000 + i, min_len=0)
    if B > 2:
        lens[1] = 0
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    tm.tm_kv_append(cache, _dev(np.ascontiguousarray(K.transpose(0, 2, 1, 3))), _dev(np.ascontiguousarray(V.transpose(0, 2, 1, 3))),
                    torch.zeros(B, dtype=torch.int32, device="cuda"))
    O = torch.full((B, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
    scale = 1.0 / np.sqrt(128.0)
    tm.tm_attn_decode(_dev(Q), cache, _dev(lens), O, scale, max_len=int(max(lens.max(), 1)))
    torch.cuda.synchronize()
    O = O.cpu().numpy()
    some = lens > 0                                          # the oracle defines attention over at least one token
    assert not O[~some].any()                                # an empty sequence gets zeros
    kq, vq = oa.kv_quantise(K[some], bits), oa.kv_quantise(V[some], bits)
    Oref = oa.attn_decode(Q[some], *kq, *vq, lens[some], scale)
    ok, worst, fro = _close(O[some], Oref)
    assert ok, (worst, fro)
    cache.close()


@pytest.mark.parametrize("bits,T", [(8, 3000), (4, 3000), (8, 40000)])
def test_attn_hip_graph_replay_matches_eager(tm, bits, T):
    """A decoding step - append of the newest token, then attention over split contexts (merged in the kernel through
    the arrival counters at 3000 tokens, by the merge kernel at 40000) - allocates nothing and leaves its counters at
    zero, so it can be captured into a HIP graph; every replay, with eager work between, reproduces the eager bits."""
    import torch
    B, Hq, Hkv = 2, 8, 2
    _say(f"attn graph replay bits={bits} T={T}")
    g = torch.Generator(device="cuda").manual_seed(7)
    K = torch.randn((B, T, Hkv, 128), generator=g, device="cuda").to(torch.float16)
    V = torch.randn((B, T, Hkv, 128), generator=g, device="cuda").to(torch.float16)
    Q = torch.randn((B, Hq, 128), generator=g, device="cuda").to(torch.float16)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    zero = torch.zeros(B, dtype=torch.int32, device="cuda")
    tm.tm_kv_append(cache, K[:, :T - 1].contiguous(), V[:, :T - 1].contiguous(), zero)
    last_k, last_v = K[:, T - 1:].contiguous(), V[:, T - 1:].contiguous()
    pos = torch.full((B,), T - 1, dtype=torch.int32, device="cuda")
    lens = torch.tensor([T, T - 700], dtype=torch.int32, device="cuda")

    def step(out):
        tm.tm_kv_append(cache, last_k, last_v, pos)
        tm.tm_attn_decode(Q, cache, lens, out, 0.09, max_len=T)

    O_eager = torch.empty((B, Hq, 128), dtype=torch.float16, device="cuda")
    step(O_eager)
    torch.cuda.synchronize()
    O_graph = torch.empty_like(O_eager)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            step(O_graph)
            step(O_graph)
    for rep in range(3):
        O_graph.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O_graph.view(torch.int16), O_eager.view(torch.int16)), f"replay {rep}"
        O2 = torch.empty_like(O_eager)
        step(O2)                                             # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(O2.view(torch.int16), O_eager.view(torch.int16))
    # and the eager result is the right one (sampled against the oracle on the first sequence)
    Ks = K[:1].permute(0, 2, 1, 3).contiguous().cpu().numpy()
    Vs = V[:1].permute(0, 2, 1, 3).contiguous().cpu().numpy()
    Oref = oa.attn_decode(Q[:1].cpu().numpy(), *oa.kv_quantise(Ks, bits), *oa.kv_quantise(Vs, bits), np.array([T]), 0.09)
    ok, worst, fro = _close(O_eager[:1].cpu().numpy(), Oref)
    assert ok, (worst, fro)
    cache.close()


# ------------------------------------------------------------------ a chunk of prompt tokens (prefill)

PREFILL_CASES = [
    # B, Hq, Hkv, cached tokens T, positions, counts (None: all), query rows n
    (1, 4, 1, 40, [0], None, 40),                         # whole prompt, G = 4
    (3, 8, 2, 96, [0, 0, 0], [70, 1, 33], 70),            # ragged prompt lengths in one call
    (2, 4, 4, 50, [0, 0], [50, 17], 50),                  # G = 1: sixteen tokens per CTA
    (2, 16, 1, 45, [0, 0], None, 45),                     # G = 16: one token per CTA
    (2, 6, 2, 37, [0, 0], [37, 20], 37),                  # G = 3: five tokens per CTA, one column idle
    (2, 8, 1, 64, [0, 0], None, 64),                      # G = 8
    (3, 8, 2, 130, [40, 0, 100], [20, 5, 17], 20),        # later chunks of longer prompts (chunked prefill)
    (2, 8, 2, 300, [0, 150], [300, 150], 300),            # several blocks per wave, ragged tail
    (2, 40, 2, 90, [0, 30], [60, 33], 60),                # G = 20: a pass of sixteen heads and one of four
]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hq,Hkv,T,positions,counts,n", PREFILL_CASES)
def test_attn_prefill_against_oracle(tm, B, Hq, Hkv, T, positions, counts, n, bits):
    import torch
    _say(f"attn prefill B={B} Hq={Hq} Hkv={Hkv} T={T} positions={positions} counts={counts} n={n} bits={bits}")
    rng = np.random.default_rng(B * 1000 + Hq * 10 + T + bits)
    _, K, V, _ = wa.draw(B, Hq, Hkv, T, seed=T + Hq)
    Q = rng.standard_normal((B, n, Hq, 128)).astype(np.float16)
    kq, vq = oa.kv_quantise(K, bits), oa.kv_quantise(V, bits)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    tm.tm_kv_append(cache, _dev(np.ascontiguousarray(K.transpose(0, 2, 1, 3))), _dev(np.ascontiguousarray(V.transpose(0, 2, 1, 3))),
                    torch.zeros(B, dtype=torch.int32, device="cuda"))
    pos = np.array(positions, np.int32)
    cnt = np.full(B, n, np.int32) if counts is None else np.array(counts, np.int32)
    scale = 1.0 / np.sqrt(128.0)
    outs = []
    for _ in range(2):
        O = torch.full((B, n, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
        tm.tm_attn_prefill(_dev(Q), cache, _dev(pos), O, scale, counts=None if counts is None else _dev(cnt))
        torch.cuda.synchronize()
        outs.append(O.cpu().numpy())
    assert np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))        # run-to-run identical
    Oref = oa.attn_prefill(Q, *kq, *vq, pos, cnt, scale)
    for b in range(B):
        assert np.isnan(outs[0][b, cnt[b]:]).all()                                 # rows past the count are left alone
        ok, worst, fro = _close(outs[0][b, :cnt[b]], Oref[b, :cnt[b]])
        assert ok, (b, worst, fro)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
def test_attn_prefill_long_prompt_sampled(tm, bits):
    """A 2048-token prompt in the benchmark's head geometry (32 query / 8 KV heads), as bench.py launches it; the oracle
    checks sampled query rows, the first and last of them included."""
    import torch
    _say(f"attn prefill long prompt bits={bits}")
    B, Hq, Hkv, T = 1, 32, 8, 2048
    rng = np.random.default_rng(bits)
    _, K, V, _ = wa.draw(B, Hq, Hkv, T, seed=3)
    Q = rng.standard_normal((B, T, Hq, 128)).astype(np.float16)
    kq, vq = oa.kv_quantise(K, bits), oa.kv_quantise(V, bits)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    tm.tm_kv_append(cache, _dev(np.ascontiguousarray(K.transpose(0, 2, 1, 3))), _dev(np.ascontiguousarray(V.transpose(0, 2, 1, 3))),
                    torch.zeros(B, dtype=torch.int32, device="cuda"))
    O = torch.full((B, T, Hq, 128), float("nan"), dtype=torch.float16, device="cuda")
    tm.tm_attn_prefill(_dev(Q), cache, torch.zeros(B, dtype=torch.int32, device="cuda"), O, 128 ** -0.5)
    torch.cuda.synchronize()
    O = O.cpu().numpy()
    assert not np.isnan(O).any()
    rows = np.unique(np.concatenate([[0, 1, 31, 32, 33, 63, 64, T - 1], rng.integers(0, T, 24)]))
    for i in rows:                                          # row i as a one-token chunk at position i
        ref = oa.attn_prefill(Q[:, i:i + 1], *kq, *vq, np.array([i], np.int32), np.array([1], np.int32), 128 ** -0.5)
        ok, worst, fro = _close(O[:, i:i + 1], ref)
        assert ok, (int(i), worst, fro)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hkv,G,cap,positions,n", [
    (32, 16, 3, 128, [0, 5, 58, -20, 100], 70),      # 256-row CTAs: two stages, ragged rows, positions outside the cache
    (8, 16, 3, 128, [0, 5, 58, -20, 100], 70),       # 128-row CTAs (two wave groups along the context)
    (4, 16, 20, 96, [0, 31, 32, 64], 32),            # more than sixteen query heads per KV head
    (16, 32, 1, 128, [0, 1, 8], 120),                # one row per token
    (1, 8, 4, 1344, [331], 1000),                    # many stages after a past that ends inside one, 128 rows
    (2, 8, 8, 960, [331, 0], 600),                   # the same, 256 rows
])
def test_attn_prefill_row_tiles(tm, B, Hkv, G, cap, positions, n, bits):
    """Chunks with enough rows for 128- and 256-row CTAs: ragged counts, masked edges of runs and stages, tokens of the cache
    that were never stored (their bytes are set to all ones: not-a-number scales).  Sampled heads against the oracle, within
    the bounds of the module."""
    import torch
    _say(f"attn prefill row tiles B={B} Hkv={Hkv} G={G} cap={cap} n={n} bits={bits}")
    rng = np.random.default_rng(B * 100 + Hkv + G + bits)
    pos = np.array([positions[b % len(positions)] for b in range(B)], np.int32)
    cnt = np.array([n - (7 * b) % n for b in range(B)], np.int32)
    cache = tm.tm_kv_create(B, Hkv, cap, bits)
    cbytes = B * Hkv * cache.capacity * 128 * bits // 8
    tm.tm_kv_upload(cache, np.full(cbytes, 255, np.uint8), np.full(cbytes, 255, np.uint8),
                    np.full(B * Hkv * cache.capacity * 2, 0xFFFFFFFF, np.uint32))
    K, V = (rng.standard_normal((B, Hkv, cap, 128)).astype(np.float16) for _ in range(2))
    live = np.minimum(np.maximum(pos + cnt, 0), cap)
    for b0 in range(0, B, 8):                            # sequence by sequence: only the tokens up to its last query row
        for b in range(b0, min(b0 + 8, B)):
            at = torch.full((B,), cache.capacity, dtype=torch.int32, device="cuda")      # the others' tokens are dropped
            at[b] = 0
            if live[b]:
                Kn, Vn = (np.zeros((B, live[b], Hkv, 128), np.float16) for _ in range(2))
                Kn[b], Vn[b] = K[b, :, :live[b]].transpose(1, 0, 2), V[b, :, :live[b]].transpose(1, 0, 2)
                tm.tm_kv_append(cache, _dev(Kn), _dev(Vn), at)
    Q = rng.standard_normal((B, n, Hkv * G, 128)).astype(np.float16)
    outs = []
    for _ in range(2):
        O = torch.full((B, n, Hkv * G, 128), float("nan"), dtype=torch.float16, device="cuda")
        tm.tm_attn_prefill(_dev(Q), cache, _dev(pos), O, 128 ** -0.5, counts=_dev(cnt))
        torch.cuda.synchronize()
        outs.append(O.cpu().numpy())
    assert np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))
    for b in sorted({0, 1, B // 2, B - 2, B - 1} & set(range(B))):
        hk = int(rng.integers(Hkv))
        heads = slice(hk * G, (hk + 1) * G)
        kq, vq = oa.kv_quantise(K[b:b + 1, hk:hk + 1], bits), oa.kv_quantise(V[b:b + 1, hk:hk + 1], bits)
        rows = [i for i in range(cnt[b]) if 0 <= pos[b] + i < cap]
        for i in {*rows[:3], *rows[-3:], *rows[len(rows) // 2:len(rows) // 2 + 2]}:
            ref = oa.attn_prefill(Q[b:b + 1, i:i + 1, heads], *kq, *vq, pos[b:b + 1] + i, np.array([1], np.int32), 128 ** -0.5)
            ok, worst, fro = _close(outs[0][b:b + 1, i:i + 1, heads], ref)
            assert ok, (b, i, worst, fro)
        dead = [i for i in range(n) if i not in rows]
        assert np.isnan(outs[0][b, dead]).all()          # rows past the count or outside the cache are left alone
        assert not np.isnan(outs[0][b, rows]).any()
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hkv,G,cap,n,rows", [(32, 16, 3, 128, 70, 256), (8, 16, 3, 128, 70, 128), (4, 16, 20, 96, 32, 256),
                                                (16, 32, 1, 128, 120, 128), (1, 8, 4, 1344, 1000, 128), (2, 8, 8, 960, 600, 256),
                                                (1, 1, 8, 2048, 40, 0)])
def test_attn_prefill_rows_of_a_cta(tm, B, Hkv, G, cap, n, rows, bits):
    """The cases of test_attn_prefill_row_tiles run on CTAs of as many rows as they are written for (0: the 16-column kernel)."""
    cache = tm.tm_kv_create(B, Hkv, cap, bits)
    assert tm.tm_get_attn_plan(cache, Hkv * G, count=n) == (1, rows)
    cache.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,Hkv,G,past,n,rows", [(1, 8, 4, 331, 1000, 128), (2, 8, 8, 331, 600, 256), (1, 1, 8, 331, 40, 0)])
def test_attn_prefill_moving_references(tm, B, Hkv, G, past, n, rows, bits):
    """Scores that climb along the context by 2^58 in all, or fall, and that change by 2^35 from one run of 32 tokens to the next:
    real rows have to move their softmax reference again and again, and the two wave groups of a 128-row CTA, which take the runs
    in turn, meet with references that far apart."""
    import torch
    T = past + n
    _say(f"attn prefill moving references B={B} Hkv={Hkv} G={G} n={n} bits={bits}")
    rng = np.random.default_rng(n + bits)
    u = rng.standard_normal(128)
    u /= np.linalg.norm(u)
    t = np.arange(T)
    climb = 40.0 * t / T - 20.0 + np.where(t // 32 % 2, 12.0, -12.0)              # the score, natural logarithm
    K = (0.5 * rng.standard_normal((B, Hkv, T, 128)) + (climb * 128 ** 0.5 / 8)[:, None] * u).astype(np.float16)
    V = rng.standard_normal((B, Hkv, T, 128)).astype(np.float16)
    sign = np.where(np.arange(Hkv * G) % 2, -1.0, 1.0)                            # every second head sees them fall
    Q = (8 * sign[:, None] * u + 0.2 * rng.standard_normal((B, n, Hkv * G, 128))).astype(np.float16)
    cache = tm.tm_kv_create(B, Hkv, T, bits)
    assert tm.tm_get_attn_plan(cache, Hkv * G, count=n) == (1, rows)
    zero, at = (torch.full((B,), x, dtype=torch.int32, device="cuda") for x in (0, past))
    tm.tm_kv_append(cache, _dev(K.transpose(0, 2, 1, 3)), _dev(V.transpose(0, 2, 1, 3)), zero)
    O = torch.full((B, n, Hkv * G, 128), float("nan"), dtype=torch.float16, device="cuda")
    tm.tm_attn_prefill(_dev(Q), cache, at, O, 128 ** -0.5)
    torch.cuda.synchronize()
    O = O.cpu().numpy()
    assert not np.isnan(O).any()
    kq, vq = oa.kv_quantise(K, bits), oa.kv_quantise(V, bits)
    for i in sorted({0, 1, n // 3, n // 2, n - 2, n - 1, *rng.integers(0, n, 6).tolist()}):
        ref = oa.attn_prefill(Q[:, i:i + 1], *kq, *vq, np.full(B, past + i, np.int32), np.ones(B, np.int32), 128 ** -0.5)
        ok, worst, fro = _close(O[:, i:i + 1], ref)
        assert ok, (i, worst, fro)
    cache.close()


def test_attn_prefill_argument_checks(tm):
    import torch
    cache = tm.tm_kv_create(1, 2, 64, 8)
    Q = torch.zeros((1, 4, 8, 128), dtype=torch.float16, device="cuda")
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    with pytest.raises(tm.TmError):
        tm.tm_attn_prefill(Q, cache, pos, torch.empty_like(Q), 0.0)               # scale
    with pytest.raises(tm.TmError):
        tm.tm_attn_prefill(torch.zeros((1, 4, 7, 128), dtype=torch.float16, device="cuda"), cache, pos,
                           torch.zeros((1, 4, 7, 128), dtype=torch.float16, device="cuda"), 0.1)   # heads not a multiple
    # positions outside the cache: nothing is written, nothing faults
    O = torch.full((1, 4, 8, 128), float("nan"), dtype=torch.float16, device="cuda")
    tm.tm_attn_prefill(Q, cache, torch.full((1,), 64, dtype=torch.int32, device="cuda"), O, 0.1)
    tm.tm_attn_prefill(Q, cache, torch.full((1,), -9, dtype=torch.int32, device="cuda"), O, 0.1)
    torch.cuda.synchronize()
    assert torch.isnan(O).all()
    cache.close()
