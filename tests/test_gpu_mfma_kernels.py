"""GPU tests of the kernels that stream tiles straight into shared memory: the voice-hits screen with the
rows it leaves to the double kernel, and both passes of the prefill scores, at the sizes where they
change path and where tiles end.  Every test prints the case it runs before touching the GPU."""
import numpy as np
import pytest

from synth import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle as O
    O.build()


HITS = [  # (L, H_q, H_kv, T_a, n_tok, K, what)
    (32, 16, 8, 1031, 33, 4, ""),           # 128 rows a work-group, a sample of the keys, ragged ends
    (32, 16, 8, 1024, 40, 8, "dup"),        # the same with keys that tie
    (32, 16, 8, 70, 33, 8, ""),             # the sample is all keys
    (32, 16, 8, 63, 33, 8, ""),             # the double kernel alone, and just not (many rows)
    (32, 16, 8, 64, 33, 8, "dup"),
    (2, 8, 8, 127, 3, 4, "dup"),            # the same with few rows
    (2, 8, 8, 128, 3, 4, ""),
    (1, 8, 2, 5, 1, 4, ""),
    (32, 16, 8, 2051, 17, 4, ""),           # 64 rows a work-group
    (2, 8, 8, 4096, 3, 4, ""),              # 32 rows, eight shares of the keys, a sample
    (1, 24, 8, 4111, 1, 8, "dup"),
    (1, 8, 2, 129, 1, 1, ""),
    (1, 8, 2, 1300, 9, 4, "zero"),          # zero queries: every key ties, the list overflows
    (1, 8, 2, 5000, 9, 8, "same"),          # 200 equal best keys: the list overflows after a sample too
    (1, 8, 2, 1300, 9, 4, "big"),           # products beyond fp32
    (1, 8, 2, 1300, 9, 4, "tiny"),          # products below fp32's normal range
    (1, 8, 2, 1300, 9, 4, "low"),           # products near fp32's normal range, just below the screen's range
    (1, 8, 2, 1300, 9, 4, "lowest"),        # the smallest values that it takes
    (1, 8, 2, 1300, 9, 4, "cancel"),        # logits far below their products
    (1, 8, 2, 1300, 9, 4, "inf"),           # one infinite key element
    (32, 16, 8, 1031, 33, 4, "offset"),     # a large constant in two channels
    (2, 8, 8, 4111, 3, 8, "offset"),
    (32, 16, 8, 1031, 33, 4, "late"),       # large and first non-zero elements outside the sample: both sweeps again
    (2, 8, 8, 4111, 3, 8, "late"),
    (2, 8, 8, 4111, 3, 4, "late"),
    (32, 16, 8, 1031, 33, 4, "edge"),       # channels and keys of zeros and subnormal values, one huge query element
    (2, 8, 8, 4111, 3, 8, "edge"),
    (2, 8, 2, 1300, 9, 4, "nan"),           # a NaN key element, a NaN and an infinite query: the other rows
    (2, 8, 2, 4111, 9, 8, "nan"),
    (2, 8, 2, 1300, 9, 4, "zeros"),         # a head whose keys are all zero
]


@pytest.mark.parametrize("shape", HITS, ids=[f"L{s[0]}_q{s[1]}_kv{s[2]}_Ta{s[3]}_tok{s[4]}_K{s[5]}{s[6]}" for s in HITS])
def test_voice_screen_matches_oracle(shape):
    import torch
    from oracle import oracle as O
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log, to_dev
    L, Hq, Hkv, Ta, n_tok, K, what = shape
    log(f"[case] voice screen {shape}")
    rng = np.random.default_rng(7 + Ta + n_tok)
    kf = rng.standard_normal((L, Hkv, Ta + 3, 128), dtype=np.float32)
    qf = rng.standard_normal((n_tok, L, Hq, 128), dtype=np.float32)
    kf[:, :, Ta:] *= 100                          # text rows take no part
    if what == "dup":
        kf[:, :, 1::5] = kf[:, :, :1]             # a fifth of the keys are one key
    elif what == "zero":
        qf[::2] = 0
    elif what == "same":
        kf[:, :, 100:4900:24] = kf[:, :, :1] = qf[0, 0, 0] * 2
    elif what == "big":
        kf *= np.float32(2e19)
        qf *= np.float32(1e20)
    elif what == "tiny":
        kf *= np.float32(1e-20)
        qf *= np.float32(1e-19)
    elif what in ("low", "lowest"):
        kf *= np.float32(2.0 ** (-57 if what == "low" else -53))
        qf *= np.float32(2.0 ** (-57 if what == "low" else -53))
    elif what == "cancel":
        # q . k = 0 for the bf16 values, up to a small last term
        h = gen.bf16_to_f32(gen.f32_to_bf16(qf))
        qf = np.concatenate([h[..., :64], -h[..., :64]], axis=-1)
        kf[..., 64:] = kf[..., :64]
        kf[..., 127] += np.float32(0.01) * rng.standard_normal(kf.shape[:-1], dtype=np.float32)
    elif what == "offset":
        kf[..., 5] += 400
        kf[..., 77] -= 400
    elif what == "late":
        # positions 101 and 407 are in no sample of every second or third key
        kf[..., 9] = 0
        kf[:, :, 101, 9] = 3
        kf[:, :, 407, 20:40] *= 30
    elif what == "edge":
        kf[..., 3] = 0
        kf[..., 4] *= np.float32(2.0 ** -128)
        kf[:, :, 5:50] = 0
        kf[:, :, 50:60] *= np.float32(2.0 ** -127)
        qf[0, :, :, 3:5] = np.float32(2.0 ** 90)
        qf[1] *= np.float32(2.0 ** -127)
    elif what == "zeros":
        kf[0, 0] = 0
    k, q = gen.f32_to_bf16(kf), gen.f32_to_bf16(qf)
    ok = np.ones((n_tok, L, Hq), bool)
    if what == "inf":
        k[0, 0, 77, 5] = 0x7F80
    elif what == "nan":
        k[0, 0, 77, 5] = 0x7FC0
        q[1, 1, 0, 7] = 0x7FC0
        q[2, 1, 1, 7] = 0xFF80
        ok[:, 0, : Hq // Hkv] = False
        ok[1, 1, 0] = False                          # an infinite query: logits of +-inf tie by position
    a = rng.integers(0, Ta, size=n_tok)
    span = np.stack([a, np.minimum(a + rng.integers(1, 1 + Ta // 3, size=n_tok), Ta)], axis=1).astype(np.int32)
    hits = torch.full((n_tok, L, Hq), -7, dtype=torch.int32, device="cuda")
    W.wnw_voice_hits(to_dev(k), to_dev(q), torch.from_numpy(span).cuda(), K, Ta, hits)
    torch.cuda.synchronize()
    got = hits.cpu().numpy()
    assert ((got >= 0) & (got <= K)).all()
    bad = np.argwhere(ok & (got != O.voice_hits(k, q, span, K, Ta)))
    assert not len(bad), f"{len(bad)} of {hits.numel()} differ, first at (token, layer, q-head) {bad[0].tolist()}"


PREFILL = [  # (L, H_q, H_kv, T_a, T_t, query scale)
    (32, 32, 8, 200, 193, 1.0),      # 256 rows and keys a work-group would suffice: pass 1 with two blocks
    (32, 16, 8, 2049, 9, 1.0),       # pass 2 with four blocks, one key past a work-group
    (1, 8, 2, 31, 33, 1.0),          # every key block holds text
    (2, 6, 2, 64, 1, 1.0),           # one text row, whole tiles
    (1, 8, 1, 161, 64, 1.0),         # audio ends one key into a block of 32
    (1, 4, 4, 1, 130, 1.0),          # one audio key
    (1, 8, 2, 515, 70, 12.0),        # logits of hundreds: the running maximum is raised again and again
]


@pytest.mark.parametrize("shape", PREFILL, ids=[f"L{s[0]}_q{s[1]}_kv{s[2]}_Ta{s[3]}_Tt{s[4]}_x{s[5]:g}" for s in PREFILL])
def test_prefill_scores_match_oracle(shape):
    import torch
    from oracle import oracle as O
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log, to_dev
    L, Hq, Hkv, Ta, Tt, scale = shape
    log(f"[case] prefill scores {shape}")
    rng = np.random.default_rng(Ta * 7 + Tt)
    G, T, D = Hq // Hkv, Ta + Tt, 128
    k = gen.f32_to_bf16(rng.standard_normal((1, L, Hkv, T, D), dtype=np.float32))
    q = gen.f32_to_bf16(np.float32(scale) * rng.standard_normal((1, L, Hq, Tt, D), dtype=np.float32))
    kd = to_dev(k)
    cfg = W.make_config(1, L, Hq, Hkv, Ta, Tt, 32, 2000)
    ctx = W.wnw_init_cache(cfg, kd, kd)
    try:
        sc = torch.full((1, L, Hkv, Ta), -1.0, dtype=torch.float32, device="cuda")
        W.wnw_prefill_scores(ctx, to_dev(q), sc)
        torch.cuda.synchronize()
        got = sc.cpu().numpy()[0]
    finally:
        W.wnw_destroy(ctx)
    heads = [(l, h) for l in range(L) for h in range(Hkv)]
    for l, h in heads if len(heads) <= 4 else [heads[i] for i in (0, len(heads) // 2 + 1, len(heads) - 1)]:
        c1 = O.make_cfg(1, 1, G, 1, D, Ta, Tt, 32, 2000)
        ref = O.prefill_scores(c1, k[:, l:l + 1, h:h + 1], q[:, l:l + 1, h * G:(h + 1) * G])[0, 0, 0]
        # A term's exponent (base 2) is a logit x minus the row's log-sum-exp, about max |x|, plus 32: a few
        # roundings of values up to 32 + 2 max |x| (the products' sums, the scale, the statistic, the FMA)
        x = gen.bf16_to_f32(q[0, l, h * G:(h + 1) * G].reshape(-1, D)) @ gen.bf16_to_f32(k[0, l, h]).T
        top = float(np.abs(x).max()) / np.sqrt(D) * np.log2(np.e)
        tol = 8 * 2.0 ** -24 * (32 + 2 * top)
        rel = np.abs(got[l, h] - ref) / np.maximum(ref, 2.0 ** -100)   # terms below 2^-158 flush
        rms = float(np.linalg.norm(got[l, h] - ref) / np.linalg.norm(ref))
        log(f"[prefill] head ({l},{h}): max rel err {rel.max():.3g} of {tol:.3g}, rms {rms:.3g}")
        assert (rel <= tol).all()
        if scale == 1:
            # exponents stay below 32: at worst half a unit of the last place (2^-20) from a row's statistic, which
            # all its terms share, and as a mean 2^-19 / sqrt(12) from the FMA; ln 2 times that, and a little for sums
            assert rms <= 9e-7


def _at_offset(t, n):
    """The same values n elements past an aligned address."""
    import torch
    u = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    assert u.data_ptr() % 16 == 0
    return u[n: n + t.numel()].view(t.shape).copy_(t)


@pytest.mark.parametrize("off", [(1, 0), (0, 1), (2, 3), (4, 8)], ids=lambda o: f"k{o[0]}_q{o[1]}")
def test_rows_at_any_address(off):
    """Keys and queries that start between multiples of 16 bytes, the size of the loads straight into
    shared memory: the same results as aligned ones."""
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log(f"[case] prefill scores and voice hits, rows {off} elements past 16 bytes")
    g = torch.Generator(device="cuda").manual_seed(3)
    L, Hq, Hkv, Ta, Tt, n_tok, K = 2, 8, 2, 515, 70, 9, 4
    k = torch.randn((1, L, Hkv, Ta + Tt, 128), generator=g, device="cuda").bfloat16()
    q = torch.randn((1, L, Hq, Tt, 128), generator=g, device="cuda").bfloat16()
    qa = torch.randn((n_tok, L, Hq, 128), generator=g, device="cuda").bfloat16()
    span = torch.tensor([[50 * i, 50 * i + 40] for i in range(n_tok)], dtype=torch.int32, device="cuda")
    got = []
    for ko, qo in ((0, 0), off):
        kd, qd, qad = _at_offset(k, ko), _at_offset(q, qo), _at_offset(qa, qo)
        ctx = W.wnw_init_cache(W.make_config(1, L, Hq, Hkv, Ta, Tt, 32, 2000), kd, kd)
        try:
            sc = torch.full((1, L, Hkv, Ta), -1.0, device="cuda")
            W.wnw_prefill_scores(ctx, qd, sc)
            hits = torch.full((n_tok, L, Hq), -7, dtype=torch.int32, device="cuda")
            W.wnw_voice_hits(kd[0], qad, span, K, Ta, hits)
            torch.cuda.synchronize()
            got.append((sc, hits))
        finally:
            W.wnw_destroy(ctx)
    assert bool(torch.isfinite(got[0][0]).all()) and bool((got[0][1] >= 0).all())
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("what", ["text key", "audio key", "query", "infinite text key"])
@pytest.mark.parametrize("Ta,Tt", [(96, 1), (64, 1), (7, 1), (128, 40), (515, 70)])
def test_prefill_nan_stays_nan(Ta, Tt, what):
    """A NaN (or infinite) element that a row sees makes every score of its KV-head NaN; the other heads'
    scores are those of clean inputs."""
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log(f"[case] prefill scores with a bad {what}, Ta {Ta} Tt {Tt}")
    g = torch.Generator(device="cuda").manual_seed(Ta)
    L, Hq, Hkv = 2, 6, 2
    k = torch.randn((1, L, Hkv, Ta + Tt, 128), generator=g, device="cuda").bfloat16()
    q = torch.randn((1, L, Hq, Tt, 128), generator=g, device="cuda").bfloat16()
    got = []
    for bad in (False, True):
        if bad and what == "query":
            q[0, 1, 1, Tt - 1, 9] = float("nan")     # q-head 1 of KV-head 0
        elif bad and what == "infinite text key":
            k[0, 1, 0, Ta, 9] = float("inf")
            q[0, 1, 0, 0, 9] = 1.0
        elif bad:
            k[0, 1, 0, Ta if what == "text key" else Ta - 1, 9] = float("nan")
        ctx = W.wnw_init_cache(W.make_config(1, L, Hq, Hkv, Ta, Tt, 32, 2000), k, k)
        try:
            sc = torch.full((1, L, Hkv, Ta), -1.0, device="cuda")
            W.wnw_prefill_scores(ctx, q, sc)
            torch.cuda.synchronize()
            got.append(sc[0])
        finally:
            W.wnw_destroy(ctx)
    assert bool(torch.isfinite(got[0]).all())
    assert bool(torch.isnan(got[1][1, 0]).all())
    got[1][1, 0] = got[0][1, 0]
    assert torch.equal(got[0], got[1])
