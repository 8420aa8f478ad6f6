"""The launches are asynchronous on the caller's stream and allocate nothing, so they can be
captured into a HIP graph and run on several streams at once.  Replays are checked against
the eager result every time, with eager work and synchronisations between them."""
import ctypes
import re
import sys
import threading
import time

import numpy as np
import pytest
import torch

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf

from gpu_util import TOL, device_inputs, to_device, to_host64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("softmax", [False, True])
def test_graph_replays_match_eager(softmax):
    w = mi.make_problem(4, 300, 64, 264, 64, "f16", softmax, "normal" if softmax else "uniform", seed=4242)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    F = to_device(mi.to_bits(mi.draw(4242, 4, (4, 64, 64), w.dist), "f16"), "f16")
    scale = w.scale if softmax else None

    def run(E, G):
        if softmax:
            mcf.softmax_gemm_chain(A, B, D, w.scale, out=E)
        else:
            mcf.gemm_chain(A, B, D, out=E)
        mcf.gemm_chain3(A, B, D, F, scale=scale, out=G)

    E0, G0 = torch.empty((4, 300, 64), dtype=torch.float16, device="cuda"), torch.empty((4, 300, 64), dtype=torch.float16, device="cuda")
    run(E0, G0)                                  # eager: also sets the kernels' attributes before the capture
    torch.cuda.synchronize()
    ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
    assert np.max(np.abs(to_host64(E0, "f16") - ref)) <= TOL * np.max(np.abs(ref))
    E1, G1 = torch.zeros_like(E0), torch.zeros_like(G0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):                    # the binding launches on torch's current (capturing) stream
        run(E1, G1)
    for rep in range(4):
        print(f"case graph replay {rep} softmax={softmax}", flush=True)
        E1.fill_(-3.0)                           # eager work between the replays
        G1.fill_(-3.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(E1, E0) and torch.equal(G1, G0)     # same kernel, same inputs: bit-identical


def test_concurrent_streams():
    """Different problems on three streams at once; the kernels keep no state outside their
    arguments, so every result equals the one computed alone."""
    cases = []
    for i, (K, L, softmax) in enumerate(((64, 64, False), (128, 128, True), (32, 32, False))):
        w = mi.make_problem(6, 520, K, 400, L, "bf16", softmax, "normal" if softmax else "uniform", seed=4300 + i)
        x = mi.make_inputs(w)
        A, B, D = device_inputs(w, x)
        alone = mcf.softmax_gemm_chain(A, B, D, w.scale) if softmax else mcf.gemm_chain(A, B, D)
        cases.append((w, x, A, B, D, alone))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]          # default priority
    outs = [torch.empty_like(c[5]) for c in cases]
    print("case three streams", flush=True)
    for rep in range(20):
        for s, (w, x, A, B, D, alone), out in zip(streams, cases, outs):
            if w.softmax:
                mcf.softmax_gemm_chain(A, B, D, w.scale, out=out, stream=s)
            else:
                mcf.gemm_chain(A, B, D, out=out, stream=s)
    torch.cuda.synchronize()
    for (w, x, A, B, D, alone), out in zip(cases, outs):
        assert torch.equal(out, alone)
        ref = oracle.chain(x["A"], x["B"], x["D"], softmax=w.softmax, scale=w.scale)
        assert np.max(np.abs(to_host64(out, "bf16") - ref)) <= TOL * np.max(np.abs(ref))


# calls whose n the library splits by itself: a softmax on few blocks, and a k loop
SPLIT = [(4, 64, 64, 4096, 64, True), (1, 128, 1024, 1000, 128, False)]


def _split_call(b, M, K, N, L, softmax):
    w = mi.make_problem(b, M, K, N, L, "f16", softmax, "normal" if softmax else "uniform", seed=4400 + N)
    A, B, D = device_inputs(w, mi.make_inputs(w))
    problem = mcf.binding.make_problem(b, M, K, N, L, "f16", b_stride=(N * K, 1, K) if softmax else None)
    assert mcf.call_tiles(problem, softmax)[1] > 1
    code = 1 if softmax else 0
    return lambda out=None, n_split=0, stream=None: mcf.binding._call(code, w.scale, 0, A, B, D, None, out, None, stream, n_split)


@pytest.mark.parametrize("case", SPLIT, ids=str)
def test_split_calls_captured_by_torch(case):
    """The ranges are captured with a workspace of the graph's own: tensors that come and go between the
    replays do not meet it."""
    call = _split_call(*case)
    split, whole = call(), call(n_split=1)
    torch.cuda.synchronize()
    assert not torch.equal(split, whole)      # two kernels and another order of the sums
    E = torch.zeros_like(split)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(E)
    for rep in range(4):
        print(f"case split capture replay {rep}", case, flush=True)
        E.fill_(-3.0)
        junk = [torch.full((1 << k,), float("nan"), device="cuda") for k in range(10, 22)]
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(E, split)
        del junk


@pytest.mark.parametrize("case", SPLIT, ids=str)
def test_calls_captured_by_others_are_not_split(case):
    """A stream that the HIP runtime captures for someone else: torch's allocator knows nothing of the graph, so the call
    takes no workspace from it and n stays whole, as one kernel."""
    hip = ctypes.CDLL(re.search(r"\S*/libamdhip64\.so\S*", open("/proc/self/maps").read()).group())  # the one torch runs on
    call = _split_call(*case)
    whole = call(n_split=1)                   # eager: also sets the kernel's attributes before the capture
    E, ref = torch.zeros_like(whole), whole.clone()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    handle, graph, exe, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_size_t()
    print("case foreign capture", case, flush=True)
    assert hip.hipStreamBeginCapture(handle, 1) == 0          # thread-local mode
    try:
        call(E, stream=stream)
        with pytest.raises(mcf.McfError) as refused:
            call(E, n_split=2, stream=stream)
    finally:
        assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert refused.value.status == 2
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and n.value == 1
    assert hip.hipGraphInstantiate(ctypes.byref(exe), graph, None, None, ctypes.c_size_t(0)) == 0
    for rep in range(3):
        E.fill_(-3.0)
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(exe, handle) == 0
        torch.cuda.synchronize()
        assert torch.equal(E, ref)
    assert hip.hipGraphExecDestroy(exe) == 0 and hip.hipGraphDestroy(graph) == 0


@pytest.mark.parametrize("case", SPLIT[:1] + [(1, 128, 64, 128, 64, False)], ids=str)
def test_other_threads_run_during_calls(case):
    """A call lets the interpreter lock go: with a switch interval that never ends, another thread only runs
    when the calling one does so."""
    b, M, K, N, L, softmax = case
    w = mi.make_problem(b, M, K, N, L, "f16", softmax, "normal" if softmax else "uniform", seed=4500)
    A, B, D = device_inputs(w, mi.make_inputs(w))
    run = lambda: mcf.softmax_gemm_chain(A, B, D, w.scale) if softmax else mcf.gemm_chain(A, B, D)
    run()
    torch.cuda.synchronize()
    ticks, stop = [0], threading.Event()

    def tick():
        while not stop.is_set():
            ticks[0] += 1
            time.sleep(0)     # gives the lock back

    other, interval = threading.Thread(target=tick), sys.getswitchinterval()
    print("case threads", case, flush=True)
    other.start()
    try:
        time.sleep(0.05)
        sys.setswitchinterval(60.0)
        before = ticks[0]
        for _ in range(300):
            run()
        during = ticks[0] - before
    finally:
        sys.setswitchinterval(interval)
        stop.set()
        other.join()
    torch.cuda.synchronize()
    assert during >= 100
