"""GPU test of key sensitivity where rows are split over work-groups: ragged lengths around the split's
bounds, many calls in flight on several streams and threads, and a captured call."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# squares of 128 values summed in fp32 through a tree of depth 10, halved by the root, and one rounding
RTOL = 10 * 2.0 ** -24 / 2 + 2.0 ** -23


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _case(seed, n_tok, L, Hkv, Ta):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    grad = torch.randn((n_tok, L, Hkv, Ta, 128), generator=g, device="cuda")
    grad *= torch.exp(2 * torch.randn((n_tok, L, Hkv, Ta, 1), generator=g, device="cuda"))
    return grad, grad.double().norm(dim=-1).mean(dim=-1)


# unsplit: the ends of rounds of 128 positions and of pairs of them; split: from 1536 positions (few rows), 1250
# (36 rows), 1024 (72), 1152 (144) and 2560 (160 and 191) on
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 300, 1, 128), (1, 300, 1, 129), (1, 30, 10, 256), (1, 1, 5, 257),
                                   (1, 1, 2, 513), (1, 1, 3, 1535), (1, 1, 3, 1536), (2, 3, 2, 1537), (1, 36, 1, 1249),
                                   (1, 36, 1, 1250), (1, 72, 1, 1023), (1, 72, 1, 1024), (1, 24, 8, 1100), (2, 36, 2, 1151),
                                   (2, 36, 2, 1152), (1, 160, 1, 2559), (1, 160, 1, 2560), (1, 191, 1, 3001), (1, 1, 1, 9001)],
                         ids=lambda s: f"tok{s[0]}_L{s[1]}_kv{s[2]}_Ta{s[3]}")
def test_split_rows(shape):
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log(f"[case] key sensitivity {shape}")
    grad, want = _case(sum(shape), *shape)
    sens = torch.full(shape[:3], -1.0, device="cuda")
    for _ in range(3):
        W.wnw_key_sensitivity(grad, sens)
    torch.cuda.synchronize()
    assert float(((sens - want) / want).abs().max()) <= RTOL


def test_split_rows_on_streams_and_threads_and_captured():
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log("[case] key sensitivity, 3 threads with 2 streams each, 40 calls a stream; then a captured call")
    work = [_case(100 + i, 1, 4 + i, 3, 3000 + 501 * i) for i in range(6)]
    torch.cuda.synchronize()
    got, failed = [None] * 6, []

    def run(i):
        try:
            streams = [torch.cuda.Stream() for _ in range(2)]
            outs = []
            for _ in range(40):
                for j, st in enumerate(streams):
                    with torch.cuda.stream(st):
                        o = torch.full(work[2 * i + j][0].shape[:3], -1.0, device="cuda")
                        W.wnw_key_sensitivity(work[2 * i + j][0], o, st)
                        outs.append((2 * i + j, o))
            for st in streams:
                st.synchronize()
            for j in range(2):
                got[2 * i + j] = torch.stack([o for k, o in outs if k == 2 * i + j])
        except Exception as e:   # reported by the main thread
            failed.append(e)

    th = [threading.Thread(target=run, args=(i,)) for i in range(3)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not failed, failed
    for i, (_, want) in enumerate(work):
        assert float(((got[i] - want) / want).abs().max()) <= RTOL, i
        assert bool((got[i] == got[i][:1]).all()), i      # the parts are added in a fixed order
    grad, want = work[0]
    sens = torch.full(grad.shape[:3], -1.0, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        W.wnw_key_sensitivity(grad, sens)
    for _ in range(3):
        sens.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert float(((sens - want) / want).abs().max()) <= RTOL


def test_split_rows_depend_on_no_other_stream():
    """A stream is held back by a sleeping kernel with a call queued behind it; calls on another stream
    end meanwhile."""
    import time
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log("[case] key sensitivity on one stream while another with a queued call is held back")
    grad, want = _case(5, 1, 4, 3, 3000)
    outs = [torch.full(grad.shape[:3], -1.0, device="cuda") for _ in range(25)]
    W.wnw_key_sensitivity(grad, outs[0])
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.cuda._sleep(1_000_000)
    torch.cuda.synchronize()
    per_ms = 1_000_000 / (1e3 * (time.perf_counter() - t0))   # what the sleeping kernel counts in a millisecond

    def hold(st, ms):
        awake = torch.cuda.Event()
        with torch.cuda.stream(st):
            torch.cuda._sleep(int(per_ms * ms))
            awake.record()
        return awake

    # two streams may share a hardware queue, where one's work runs behind the other's whatever the library
    # does: take one that does not
    held, other = torch.cuda.Stream(), None
    for st in [torch.cuda.Stream() for _ in range(6)]:
        awake = hold(held, 100)
        with torch.cuda.stream(st):
            outs[0].fill_(-1.0)
        st.synchronize()
        free = not awake.query()
        torch.cuda.synchronize()
        if free:
            other = st
            break
    if other is None:
        pytest.skip("no stream with a hardware queue of its own")
    awake = hold(held, 300)
    W.wnw_key_sensitivity(grad, outs[0], held)
    for o in outs[1:]:
        W.wnw_key_sensitivity(grad, o, other)
    other.synchronize()
    asleep = not awake.query()
    torch.cuda.synchronize()
    assert asleep, "calls on one stream waited for another"
    for o in outs:
        assert float(((o - want) / want).abs().max()) <= RTOL


def test_split_rows_while_another_thread_captures():
    import torch
    from paper_2608_22704_amd import wnw as W
    from tests.wnw_harness import log
    log("[case] key sensitivity, eager calls of a thread while another captures")
    grad, want = _case(6, 1, 4, 3, 3000)
    outs = [torch.full(grad.shape[:3], -1.0, device="cuda") for _ in range(5)]
    st, failed = torch.cuda.Stream(), []
    W.wnw_key_sensitivity(grad, outs[4], st)

    def run():
        try:
            for o in outs[1:4]:
                W.wnw_key_sensitivity(grad, o, st)
        except Exception as e:   # reported by the main thread
            failed.append(e)

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        W.wnw_key_sensitivity(grad, outs[0])
        t = threading.Thread(target=run)
        t.start()
        t.join()
        W.wnw_key_sensitivity(grad, outs[4])
    assert not failed, failed
    outs[4].fill_(-1.0)
    graph.replay()
    torch.cuda.synchronize()
    for o in outs:
        assert float(((o - want) / want).abs().max()) <= RTOL
