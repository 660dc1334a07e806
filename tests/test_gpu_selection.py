"""GPU test of the selection's ranking and slot assignment at the chunk counts where they change method, in
the three places the selection runs: inside the anchor tiles' launch (several anchor heads and sequences, so
that its arrivals chain), inside the tidal launch, and in kernels of its own.  Each
case checks from the library's trace that the selection ran where it should.  The chunk scores that the step
reports fix the selection exactly; residency and slot bytes follow from it."""
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("mode", ["same", "next", "next_copies"])
@pytest.mark.parametrize("n,size", [(n, size) for n in (3, 64, 128, 129, 160, 161, 256, 257, 420, 421, 768, 769, 1000)
                                    for size in ("small", "large")] + [(257, "wide"), (300, "wide")])
def test_selection_follows_the_scores(n, size, mode, capfd, monkeypatch):
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log(f"[case] selection over {n} chunks, {mode}, {size}")
    # `large`: more anchor tiles than the chip holds at once, so that the selection has its own kernel;
    # `wide`: few anchor tiles beside many static ones, which hide a selection over more than 256 chunks
    big = size == "large"
    B, L, Tt = {"small": (2, 3, 8), "large": (1, 80, 5000), "wide": (1, 160, 8)}[size]
    Hq, Hkv, cl, delta = 8, 4, 2, 3
    Ta, k = n * cl, max(1, n // 5)
    flags = {"same": 0, "next": W.WNW_F_SELECT_NEXT_STEP,
             "next_copies": W.WNW_F_SELECT_NEXT_STEP | W.WNW_F_RECALL_MEMCPY}[mode]
    # the arrays of 420 chunks and more do not fit the tidal launch's shared memory
    where = ("inside the tidal launch" if mode == "next_copies" and n < 420 else
             "inside the anchor launch" if mode != "next_copies" and not big and (n <= 256 or (size, mode) == ("wide", "next"))
             else "before the tidal launch")
    g = torch.Generator(device="cuda").manual_seed(n)
    kv = [torch.randn((B, L, Hkv, Ta + Tt, 128), generator=g, device="cuda").bfloat16() for _ in range(2)]
    roles = np.full((L, Hkv), W.WNW_FIXED, np.uint8)
    roles[: 3 if size == "wide" else L, 0] = W.WNW_ANCHOR
    roles[0, 1:3] = W.WNW_TIDAL
    pf = torch.rand((B, L, Hkv, Ta), generator=g, device="cuda")
    monkeypatch.setenv("WNW_LOG", "1")
    ctx = W.wnw_init_cache(W.make_config(B, L, Hq, Hkv, Ta, Tt, cl, 5000, top_k=k, flags=flags), *kv)
    try:
        W.wnw_set_roles_device(ctx, roles, pf)
        cb = W.wnw_query_geometry(ctx)["chunk_bytes"]
        out = torch.empty((B, L, Hq, 128), device="cuda")
        sc = torch.empty((B, n), device="cuda")
        sel = torch.full((B, k), -5, dtype=torch.int32, device="cuda")
        picked = [[] for _ in range(B)]
        for s in range(6):
            # step 1: zero queries, every chunk ties with its equals and the lowest ids win
            q = torch.randn((B, L, Hq, 128), generator=g, device="cuda") * (0.0 if s == 1 else 1.0)
            W.wnw_decode_step(ctx, q.bfloat16(), out, sc, sel)
            torch.cuda.synchronize()
            for b in range(B):
                v = sc.cpu().numpy()[b]
                want = np.sort(np.lexsort((np.arange(n), -v))[:k])
                assert np.array_equal(sel.cpu().numpy()[b], want), f"step {s}, sequence {b}"
                picked[b].append(set(want.tolist()))
        flags_dev = np.zeros((B, n), np.uint8)
        W.wnw_debug_read_resident(ctx, flags_dev)
        x, y = np.empty(cb, np.uint8), np.empty(cb, np.uint8)
        for b in range(B):
            resident = set().union(*picked[b][-delta:])
            seen = set().union(*picked[b][-delta - 1: -1]) if flags else resident
            assert set(np.nonzero(flags_dev[b])[0].tolist()) == seen, f"sequence {b}"
            for c in sorted(resident)[:: max(1, len(resident) // 16)]:
                W.wnw_debug_read_slot(ctx, b, c, x, cb)
                W.wnw_debug_read_host_chunk(ctx, b, c, y, cb)
                assert np.array_equal(x, y), f"sequence {b}, segment {c}"
        assert W.wnw_get_stats(ctx)["slot_exhausted"] == 0
    finally:
        W.wnw_destroy(ctx)
    ran = re.findall(r"^\[wnw\] step .* selection (.+)$", capfd.readouterr().err, re.M)
    assert ran == [where] * 6, ran
