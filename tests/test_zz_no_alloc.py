"""raas_decode_step_static (the step's scratch in the library's fixed device
array, for callers that cannot allocate) against raas_decode_step, through
the C ABI: two pools of one configuration take the same inputs, one through
each entry point; retention must match bit for bit at every step and outputs
within the parity bounds. Runs go from a larger step to smaller ones, so
later calls find the array holding an earlier call's contents. A step whose
scratch would not fit is refused before anything runs."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from harness import ParityReport, compare_outputs, new_pool, record, say, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_11147_amd as raas

    raas.load_library()


def _w(**kw):
    base = dict(name="static", batch=4, n_layers=1, n_q_heads=8, n_kv_heads=2, head_dim=128, dtype="bf16",
                page_size=16, budget=256, prefill_len=100, decode_steps=200, ms_period=16,
                ms_phase_random=True, ms_wmin=8, ms_wmax=64)
    base.update(kw)
    return synth.Workload(**base)


# larger first, then smaller: (workload, splits, pool options)
RUNS = [
    (_w(batch=6), 3, {}),                                                  # split path: partials + scores
    (_w(batch=4, budget=128, prefill_len=300), 2, dict(prompt_tokens=320, prompt_topk=3)),  # + selection lists
    (_w(batch=3, dtype="f32"), None, {}),                                  # fp32: no scratch
    (_w(batch=3, dtype="f32", head_dim=64), None, {}),                     # fp32 fused: no scratch
    (_w(batch=2, n_q_heads=16, n_kv_heads=4), None, dict(scope=1)),        # one page table per sequence
    (_w(batch=2, budget=128, prefill_len=40), 2, dict(aggregation=1)),     # per-head bounds as scratch
    (_w(batch=2), None, {}),                                               # fused: no scratch at all
]


def _step_both(a, b, w, qd, kd, vd, S, dt):
    import torch

    B, Hq, Hkv, d = w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim
    outs, states = [], []
    for pool, static in ((a, False), (b, True)):
        out = torch.full((B, Hq, d), 3.0, dtype=dt, device="cuda")
        pt = torch.full((B, Hkv, S), -9, dtype=torch.int32, device="cuda")
        ts = torch.full((B, Hkv, S), -9, dtype=torch.int32, device="cuda")
        ev = torch.full((B, Hkv), -9, dtype=torch.int32, device="cuda")
        if static:
            pool.decode_step_static(0, qd, kd, vd, out, pt, ts, ev)
        else:
            pool.decode_step(0, qd, kd, vd, out, pt, ts, ev)
        outs.append(out)
        states.append((pt, ts, ev))
    torch.cuda.synchronize()
    return outs, states


def test_static_scratch_matches_decode_step():
    import torch

    for w, splits, opts in RUNS:
        say("case static scratch batch %d dtype %s splits %s %s" % (w.batch, w.dtype, splits, opts))
        a, b = new_pool(w, splits, **opts), new_pool(w, splits, **opts)
        K, V = synth.prefill(w, 3, 0)
        for pool in (a, b):
            pool.prefill(0, to_device(K, w.dtype), to_device(V, w.dtype))
        S = a.slots
        U, G, d = w.batch * w.n_kv_heads, w.group, w.head_dim
        dt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
        rep = ParityReport(units_checked=U)
        q, k, v = synth.steps(w, 3, 0, 0, w.decode_steps)
        qd, kd, vd = to_device(q, w.dtype), to_device(k, w.dtype), to_device(v, w.dtype)
        for t in range(w.decode_steps):
            outs, states = _step_both(a, b, w, qd[t], kd[t], vd[t], S, dt)
            for x, y in zip(*states):
                assert torch.equal(x, y), (w.batch, opts, t)
            rep.evictions += int((states[0][2] >= 0).sum())
            compare_outputs(outs[1].float().cpu().numpy().reshape(U, G, d),
                            outs[0].float().cpu().numpy().reshape(U, G, d), w.dtype, "step %d" % t, rep)
            rep.steps = t + 1
        sa, sb = a.export_state(0), b.export_state(0)
        for key in sa:
            assert np.array_equal(sa[key], sb[key]), key
        a.close()
        b.close()
        record(rep, "static scratch batch %d %s splits %s %s" % (w.batch, w.dtype, splits, opts))
        assert rep.evictions > 0


@pytest.mark.parametrize("kw,splits", [
    (dict(batch=4, budget=1280), None),                              # 8 units of 40 blocks
    (dict(batch=4, budget=1792, page_size=64), None),                # 56 blocks, 28 slots
    (dict(batch=3, budget=512, dtype="f32", head_dim=64), None),     # 32 blocks of 16 tokens
    (dict(batch=3, budget=512, dtype="f32"), 3),                     # forced: scratch in the array
], ids=["bf16", "few-slots", "f32", "f32-array"])
def test_static_rounds_as_decode_step(kw, splits):
    """One plan for both entry points: with the deterministic option a static
    step's outputs equal an ordinary one's bit for bit, also where the plan
    splits units that one workgroup could cover."""
    import torch

    w = _w(prefill_len=kw["budget"] - 100, decode_steps=140, **kw)
    say("case static rounding %s splits %s" % (kw, splits))
    pools = [new_pool(w, splits, deterministic=True) for _ in range(2)]
    K, V = synth.prefill(w, 3, 0)
    for pool in pools:
        pool.prefill(0, to_device(K, w.dtype), to_device(V, w.dtype))
    dt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    qd, kd, vd = (to_device(x, w.dtype) for x in synth.steps(w, 3, 0, 0, w.decode_steps))
    for t in range(w.decode_steps):
        outs, states = _step_both(*pools, w, qd[t], kd[t], vd[t], w.slots, dt)
        assert torch.equal(*outs), t
        for x, y in zip(*states):
            assert torch.equal(x, y), t
    for pool in pools:
        pool.close()


def test_static_scratch_refuses_oversized_step():
    import torch

    import paper_2502_11147_amd as raas

    w = synth.get_workload("llama8b-b32-L2048")
    pool = new_pool(w, 64)  # 64 splits of 256 units over a nearly full pool: 34 MB of partials
    K = torch.zeros((w.batch, w.n_kv_heads, 2000, w.head_dim), dtype=torch.bfloat16, device="cuda")
    pool.prefill(0, K, K)
    q = torch.zeros((w.batch, w.n_q_heads, w.head_dim), dtype=torch.bfloat16, device="cuda")
    kv = torch.zeros((w.batch, w.n_kv_heads, w.head_dim), dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    with pytest.raises(raas.RaasError) as e:
        pool.decode_step_static(0, q, kv, kv, out)
    assert e.value.code == raas.E_INVALID and "scratch" in str(e.value)
    st = pool.export_state(0)
    assert np.all(st["clock"] == 2000)  # nothing ran
    pool.decode_step(0, q, kv, kv, out)  # the pool's own scratch still serves it
    assert np.all(pool.export_state(0)["clock"] == 2001)
    pool.close()


@pytest.mark.parametrize("kw,splits,opt", [(dict(budget=512), 4, {}), (dict(budget=512), 4, dict(scope=1)),
                                           (dict(budget=256, dtype="f32"), 3, {}), (dict(budget=256), None, {})],
                         ids=["split", "sequence", "f32-split", "fused"])
def test_graph_replays(kw, splits, opt):
    """A captured static step replayed with new inputs against eager steps of
    a second pool: the arrival counters of split units and shared decisions
    are back at zero after every replay, with eager work of the program in
    between. Retention bit for bit, outputs within the parity bounds."""
    import torch

    w = _w(batch=3, prefill_len=60, **kw)
    B, Hq, Hkv, d, S = w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, w.slots
    dt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *shape: torch.randn(*shape, generator=g, device="cuda").to(dt)
    pools = [new_pool(w, splits, **opt) for _ in range(2)]
    k0, v0 = rand(B, Hkv, 60, d), rand(B, Hkv, 60, d)
    bufs = [dict(out=torch.zeros(B, Hq, d, dtype=dt, device="cuda"),
                 page_table=torch.zeros(B, Hkv, S, dtype=torch.int32, device="cuda"),
                 timestamps=torch.zeros(B, Hkv, S, dtype=torch.int32, device="cuda"),
                 evicted=torch.zeros(B, Hkv, dtype=torch.int32, device="cuda")) for _ in pools]
    q, k, v = rand(B, Hq, d), rand(B, Hkv, d), rand(B, Hkv, d)
    step = lambda i: pools[i].decode_step_static(0, q, k, v, **bufs[i])

    def new_inputs():
        for x in (q, k, v):
            x.copy_(rand(*x.shape))

    for p in pools:
        p.prefill(0, k0, v0)
    for _ in range(w.budget - 60 + 2 * w.page_size):
        new_inputs()
        step(0)
        step(1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(0)
    for i in range(3 * w.page_size):
        new_inputs()
        graph.replay()
        step(1)
        if i % 5 == 0:
            torch.cuda.synchronize()
        a, b = bufs
        for name in ("page_table", "timestamps", "evicted"):
            assert torch.equal(a[name], b[name]), (i, name)
        tol = 2e-2 if dt == torch.bfloat16 else 2e-5
        assert (a["out"].float() - b["out"].float()).abs().max() <= tol, i
    say("case graph replays %s %s %s" % (kw, splits, opt))
    for p in pools:
        p.close()


def _captured_kernels(step):
    """Host functions of the kernels that a captured call launches."""
    import ctypes

    import torch

    class Params(ctypes.Structure):  # hipKernelNodeParams
        _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                    ("grid", ctypes.c_uint * 3), ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]

    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(x.split()[-1] for x in f if "libamdhip64" in x))
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        step()
    raw, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p = Params()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        out.append((p.func, tuple(p.grid)))
    return out


def test_captured_load_kind_is_the_pool_s_own():
    """What other pools streamed before a capture does not choose the captured
    step's kernel: its replays take the kind that the pool alone would."""
    import torch

    say("case captured load kind")
    w, big = _w(batch=8, budget=256), synth.get_workload("llama8b-b32-L2048")
    pools = [new_pool(w), new_pool(big)]
    steps = []
    for x, pool in zip((w, big), pools):
        kv = torch.zeros(x.batch, x.n_kv_heads, x.budget - 32, x.head_dim, dtype=torch.bfloat16, device="cuda")
        pool.prefill(0, kv, kv)
        q = torch.zeros(x.batch, x.n_q_heads, x.head_dim, dtype=torch.bfloat16, device="cuda")
        new = torch.zeros(x.batch, x.n_kv_heads, x.head_dim, dtype=torch.bfloat16, device="cuda")
        out = torch.empty_like(q)
        steps.append(lambda pool=pool, q=q, new=new, out=out: pool.decode_step_static(0, q, new, new, out))
    steps[0]()
    alone = _captured_kernels(steps[0])
    steps[0]()
    for _ in range(3):  # 0.8 GB between two steps of the small pool
        steps[1]()
    torch.cuda.synchronize()
    assert _captured_kernels(steps[0]) == alone and len(alone) == 1
    for pool in pools:
        pool.close()
