"""The bounded plan cache on the GPU: many distinct masks keep it at its capacity, and
a mask whose plan was evicted (and freed once its kernels finished) is planned again
and still matches the oracle."""
import ctypes

import numpy as np
import pytest

import workloads
from oracle import attention as oa
from tests.gpu_helpers import assert_parity, from_dev, hip_library, to_dev, widen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2502_06155_amd as ta  # noqa: E402

CAP = 256  # TA_PLAN_CACHE_ENTRIES


def test_many_masks_stay_within_the_cache_and_evicted_plans_still_work():
    B, H, F, T, d = 1, 2, 6, 40, 64
    qb, kb, vb = workloads.make_qkv(B, H, F, T, d, seed=140)
    q, k, v = (to_dev(x) for x in (qb, kb, vb))
    scale = d ** -0.5
    s = torch.cuda.current_stream()
    rng = np.random.default_rng(141)
    first = (rng.random((F, F)) < 0.5).astype(np.uint8)
    first[0, :] = 1  # a split heavy row: merge kernel and workspace too
    out0 = torch.empty_like(q)
    ta.tile_attn_fwd(q, k, v, out0, B, H, F, T, d, first, scale, s)
    torch.cuda.synchronize()
    ref0 = from_dev(out0)
    assert_parity(ref0, oa.attention(qb, kb, vb, first, T, scale), "cache-first")
    # 2^36 masks exist at F = 6: draw distinct ones, all different from `first`
    seen = {first.tobytes()}
    outs = []
    while len(seen) < 3 * CAP:
        m = (rng.random((F, F)) < 0.5).astype(np.uint8)
        if m.tobytes() in seen:
            continue
        seen.add(m.tobytes())
        o = torch.empty_like(q)
        ta.tile_attn_fwd(q, k, v, o, B, H, F, T, d, m, scale, s)  # queued without waits
        if len(outs) < 4 or len(seen) % 97 == 0:
            outs.append((m, o))
        live, retired = ta.tile_attn_plan_cache_stats()
        assert live <= CAP, live
    torch.cuda.synchronize()
    live, retired = ta.tile_attn_plan_cache_stats()
    print(f"[cache] live {live} retired {retired}", flush=True)
    assert live == CAP and retired == 0
    for m, o in outs:
        assert_parity(from_dev(o), oa.attention(qb, kb, vb, m, T, scale), "cache-evicting")
    # `first` was evicted long ago: planned and uploaded again, same result bit for bit
    out1 = torch.empty_like(q)
    ta.tile_attn_fwd(q, k, v, out1, B, H, F, T, d, first, scale, s)
    torch.cuda.synchronize()
    assert np.array_equal(from_dev(out1), ref0)


def test_plans_last_used_on_a_quiet_stream_are_freed():
    # The call that evicts a plan waits for the device and frees it, whichever streams it was
    # last used on and however long ago.
    B, H, F, T, d = 1, 1, 7, 20, 64
    qb, kb, vb = workloads.make_qkv(B, H, F, T, d, seed=150)
    q, k, v = (to_dev(x) for x in (qb, kb, vb))
    scale = d ** -0.5
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    side.wait_stream(main)
    rng = np.random.default_rng(151)

    def masks(n):
        out = {}
        while len(out) < n:
            m = (rng.random((F, F)) < 0.5).astype(np.uint8)
            out[m.tobytes()] = m
        return list(out.values())

    def call(m, s):
        o = torch.empty_like(q)
        o.record_stream(s)
        ta.tile_attn_fwd(q, k, v, o, B, H, F, T, d, m, scale, s)
        return o

    def fill(s):  # CAP new masks: evicts every plan the cache holds
        for m in masks(CAP):
            call(m, s)

    fill(main)
    few = masks(8)
    for m in few:
        call(m, side)  # planned
    for m in few:
        call(m, side)  # hits
    fill(main)
    torch.cuda.synchronize()
    live, retired = ta.tile_attn_plan_cache_stats()
    print(f"[cache] quiet stream: live {live} retired {retired}", flush=True)
    assert live == CAP and retired == 0
    o = call(few[0], side)  # planned again
    torch.cuda.synchronize()
    live, retired = ta.tile_attn_plan_cache_stats()
    assert live == CAP and retired == 0
    assert_parity(from_dev(o), oa.attention(qb, kb, vb, few[0], T, scale), "cache-quiet")
    # the same on ten streams at once
    streams = [torch.cuda.Stream() for _ in range(10)]
    many = masks(80)
    for m in many:
        call(m, main)
    for i, m in enumerate(many):  # eight hits on each of ten streams
        streams[i // 8].wait_stream(main)
        call(m, streams[i // 8])
    fill(main)
    fill(main)
    torch.cuda.synchronize()
    live, retired = ta.tile_attn_plan_cache_stats()
    print(f"[cache] quiet streams: live {live} retired {retired}", flush=True)
    assert live == CAP and retired == 0


def test_plans_used_on_destroyed_streams_are_freed():
    # Plans last used on streams that are synchronised and destroyed, whose handles later
    # streams may receive: eviction asks nothing of a stream, so they are freed as any others.
    hip = ctypes.CDLL(hip_library())
    B, H, F, T, d = 1, 1, 8, 20, 64
    qb, kb, vb = workloads.make_qkv(B, H, F, T, d, seed=170)
    q, k, v = (to_dev(x) for x in (qb, kb, vb))
    scale = d ** -0.5
    rng = np.random.default_rng(171)
    torch.cuda.synchronize()

    def call(m, s):
        o = torch.full_like(q, float("nan"))
        torch.cuda.synchronize()
        ta.tile_attn_fwd(q, k, v, o, B, H, F, T, d, m, scale, s)
        return o

    def on_own_stream(m):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(s)) == 0
        o = call(m, s.value)
        o = call(m, s.value)  # a hit
        assert hip.hipStreamSynchronize(s) == 0 and hip.hipStreamDestroy(s) == 0
        return o

    few = [(rng.random((F, F)) < 0.5).astype(np.uint8) for _ in range(80)]
    outs = [on_own_stream(m) for m in few]
    for _ in range(CAP):
        call((rng.random((F, F)) < 0.5).astype(np.uint8), torch.cuda.current_stream())
    assert ta.tile_attn_plan_cache_stats() == (CAP, 0)
    again = on_own_stream(few[0])  # planned again, on a handle that may have been used before
    torch.cuda.synchronize()
    assert np.array_equal(from_dev(again), from_dev(outs[0]))
    for m, o in zip(few[::16], outs[::16]):
        assert_parity(from_dev(o), oa.attention(qb, kb, vb, m, T, scale), "cache-destroyed-stream")


def test_gradient_plans_serve_every_launch_shape():
    # The work plan of a gradient pass depends on the masks alone: once a call has planned them,
    # calls of other batch sizes, frame lengths and head dims plan and allocate nothing, so they
    # can be captured without a run of their own. Nine shapes: more than a plan remembers shares
    # for.
    H, F = 3, 9
    rng = np.random.default_rng(160)
    masks = (rng.random((H, F, F)) < 0.3).astype(np.uint8)
    masks[0, 4, :], masks[:, :, 2] = 1, 1  # split on both sides
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    shapes = [(2, 150, 128), (1, 150, 128), (2, 97, 96), (1, 64, 64), (1, 33, 96), (2, 1, 64),
              (1, 130, 128), (1, 65, 64), (2, 96, 96)]
    calls = []
    with torch.cuda.stream(s):
        gen = torch.Generator(device="cuda").manual_seed(161)
        for B, T, d in shapes:
            q, k, v, g = (torch.randn((B, H, F * T, d), generator=gen, device="cuda").to(torch.bfloat16)
                          for _ in range(4))
            out, lse = torch.empty_like(q), torch.empty((B, H, F * T), dtype=torch.float32, device="cuda")
            ta.tile_attn_fwd_heads(q, k, v, out, B, H, F, T, d, masks, d ** -0.5, lse, s)
            grads = [torch.full_like(q, float("nan")) for _ in range(3)]
            calls.append(((q, k, v, out, g, lse, *grads, B, H, F, T, d, masks, d ** -0.5, s), grads))

        def bwd(i):
            ta.tile_attn_bwd(*calls[i][0])

        bwd(0)  # the largest: plans and sizes the workspace
        s.synchronize()
        before = ta.tile_attn_plan_cache_stats()[0]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            for i in range(1, len(calls)):
                bwd(i)
        assert ta.tile_attn_plan_cache_stats()[0] == before
        for i in range(1, len(calls)):
            bwd(i)
        s.synchronize()
        eager = [[from_dev(x) for x in c[1]] for c in calls]
        for rep in range(3):
            for _, grads in calls[1:]:
                for x in grads:
                    x.fill_(float("nan"))
            s.synchronize()
            graph.replay()
            s.synchronize()
            for (_, grads), want in zip(calls[1:], eager[1:]):
                for x, w in zip(grads, want):
                    assert np.array_equal(from_dev(x), w), rep
    assert all(np.isfinite(widen(w)).all() for e in eager for w in e)
