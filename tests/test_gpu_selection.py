"""GPU test of the selection's ranking and slot assignment at the chunk counts where they change method, in
every place the selection runs (its own kernel, the anchor tiles' launch, the tidal launch).  The chunk
scores that the step reports fix the selection exactly; residency and slot bytes follow from it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("mode", ["same", "next", "next_copies"])
@pytest.mark.parametrize("big", [False, True], ids=["small", "large"])
@pytest.mark.parametrize("n", [3, 64, 160, 161, 256, 257, 420, 421, 768, 769, 1000])
def test_selection_follows_the_scores(n, big, mode):
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log(f"[case] selection over {n} chunks, {mode}, {'many' if big else 'few'} anchor tiles")
    # `large`: more anchor tiles than the chip holds at once, so that the selection has its own kernel
    L, Hq, Hkv, cl, Tt, delta = (80 if big else 1), 8, 4, 2, (5000 if big else 8), 3
    Ta, k = n * cl, max(1, n // 5)
    flags = {"same": 0, "next": W.WNW_F_SELECT_NEXT_STEP,
             "next_copies": W.WNW_F_SELECT_NEXT_STEP | W.WNW_F_RECALL_MEMCPY}[mode]
    g = torch.Generator(device="cuda").manual_seed(n)
    kv = [torch.randn((1, L, Hkv, Ta + Tt, 128), generator=g, device="cuda").bfloat16() for _ in range(2)]
    roles = np.full((L, Hkv), W.WNW_FIXED, np.uint8)
    roles[:, 0] = W.WNW_ANCHOR
    roles[0, 1:3] = W.WNW_TIDAL
    pf = torch.rand((1, L, Hkv, Ta), generator=g, device="cuda")
    ctx = W.wnw_init_cache(W.make_config(1, L, Hq, Hkv, Ta, Tt, cl, 5000, top_k=k, flags=flags), *kv)
    try:
        W.wnw_set_roles_device(ctx, roles, pf)
        cb = W.wnw_query_geometry(ctx)["chunk_bytes"]
        out = torch.empty((1, L, Hq, 128), device="cuda")
        sc = torch.empty((1, n), device="cuda")
        sel = torch.full((1, k), -5, dtype=torch.int32, device="cuda")
        picked = []
        for s in range(6):
            # step 1: zero queries, every chunk ties with its equals and the lowest ids win
            q = torch.randn((1, L, Hq, 128), generator=g, device="cuda") * (0.0 if s == 1 else 1.0)
            W.wnw_decode_step(ctx, q.bfloat16(), out, sc, sel)
            torch.cuda.synchronize()
            v = sc.cpu().numpy()[0]
            want = np.sort(np.lexsort((np.arange(n), -v))[:k])
            assert np.array_equal(sel.cpu().numpy()[0], want), f"step {s}"
            picked.append(set(want.tolist()))
        resident = set().union(*picked[-delta:])
        flags_dev = np.zeros((1, n), np.uint8)
        W.wnw_debug_read_resident(ctx, flags_dev)
        seen = set().union(*picked[-delta - 1: -1]) if flags else resident
        assert set(np.nonzero(flags_dev[0])[0].tolist()) == seen
        a, b = np.empty(cb, np.uint8), np.empty(cb, np.uint8)
        for c in sorted(resident)[:: max(1, len(resident) // 16)]:
            W.wnw_debug_read_slot(ctx, 0, c, a, cb)
            W.wnw_debug_read_host_chunk(ctx, 0, c, b, cb)
            assert np.array_equal(a, b), f"segment {c}"
        assert W.wnw_get_stats(ctx)["slot_exhausted"] == 0
    finally:
        W.wnw_destroy(ctx)
