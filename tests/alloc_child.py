"""One case of the allocation tests, in a process of its own whose HIP allocation calls pass
through tests/hip_shim.cpp: python alloc_child.py SHIM CASE."""

import ctypes
import os
import sys

SHIM = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before anything that uses the runtime
for _name, _res in (("shim_live", ctypes.c_size_t), ("shim_peak", ctypes.c_size_t), ("shim_calls", ctypes.c_long)):
    getattr(SHIM, _name).restype = _res
SHIM.shim_limit.argtypes = SHIM.shim_total.argtypes = [ctypes.c_size_t]
NO_LIMIT = ctypes.c_size_t(-1).value

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import torch  # noqa: E402

from paper_1812_11689_amd import rpf  # noqa: E402


def calls():
    return tuple(SHIM.shim_calls(k) for k in range(4))


def library_peak(fn):
    """fn's result, and the bytes of device memory the library took for it at most."""
    rpf.release_cached_memory()
    torch.cuda.synchronize()
    before = SHIM.shim_live()
    SHIM.shim_peak(1)
    r = fn()
    torch.cuda.synchronize()
    return r, SHIM.shim_peak(1) - before


def case_shim():
    """The library's allocations pass through the shim (else the other cases prove nothing)."""
    before = calls()
    rpf.release_cached_memory()
    x = torch.randn(1000, 8, device="cuda")
    rpf.exact_knn(x, x[:4], 3)
    torch.cuda.synchronize()
    assert calls()[0] > before[0]
    SHIM.shim_limit(0)
    rpf.release_cached_memory()
    try:
        rpf.exact_knn(x, x[:4], 3, None)
        raise SystemExit("an exact search without any memory")
    except rpf.RpfError as e:
        assert e.status == rpf.RPF_ENOMEM, e
    SHIM.shim_limit(NO_LIMIT)


def case_exact_workspace():
    """rpf_exact_knn's workspace stays within what rpf.h states, for a deep result list over
    many points too (the sample, and the bounds to it, grow with K n)."""
    n, d, m, K = 20_000_000, 4, 128, 256
    x = torch.randn(n, d, device="cuda")
    q = x[:m].clone()
    out = (torch.empty(m, K, dtype=torch.int32, device="cuda"), torch.empty(m, K, device="cuda"))
    torch.cuda.synchronize()
    (i, _), peak = library_peak(lambda: rpf.exact_knn(x, q, K))
    del out
    print(f"n={n} m={m} K={K}: {peak / 2**30:.2f} GiB", flush=True)
    assert bool((i[:, 0] == torch.arange(m, device="cuda")).all())
    assert peak <= (9 << 30), f"{peak} bytes"  # the filter's 4.5 GiB and the distance rows' 4


def case_exact_answer_without_distance_rows():
    """A search that the filter answers does not fail for the exhaustive kernels' buffer."""
    n, d, m, K = 1_000_000, 16, 600, 10
    x = torch.randn(n, d, device="cuda")
    q = x[:m].clone()
    want = rpf.exact_knn(x, q, K)
    torch.cuda.synchronize()
    rpf.release_cached_memory()
    SHIM.shim_limit(1 << 30)
    refused = calls()[3]
    got = rpf.exact_knn(x, q, K)
    torch.cuda.synchronize()
    SHIM.shim_limit(NO_LIMIT)
    assert calls()[3] > refused
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    # and queries left to those kernels get theirs from the rows that could be had
    x[: n // 2] = x[0]
    q = x[:m].clone()
    want = rpf.exact_knn(x, q, K)
    torch.cuda.synchronize()
    rpf.release_cached_memory()
    SHIM.shim_limit(200 << 20)
    got = rpf.exact_knn(x, q, K)
    torch.cuda.synchronize()
    SHIM.shim_limit(NO_LIMIT)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def case_noalloc():
    """rpf_query_noalloc allocates nothing: no device block, no host memory, no event, not on a
    process's first call either (leaves above 256 points: their query copies come with the
    build)."""
    import threading
    n, d, T, n0, K = 20_000, 16, 4, 400, 5
    x = torch.randn(n, d, device="cuda")
    R = torch.randn(T, 2 ** rpf.depth(n, n0) - 1, 1, d, device="cuda")
    f = rpf.build(x, T, n0, R, dist_prec="bf16")
    q = [x[i:i + m].contiguous() for i, m in ((0, 1), (5, 20), (40, 700))]  # pair by pair; grouped
    o = [(torch.empty(len(v), K, dtype=torch.int32, device="cuda"), torch.empty(len(v), K, device="cuda")) for v in q]
    torch.cuda.synchronize()
    before = calls()
    for v, w in zip(q, o):
        f.query_noalloc(v, K, w)
    torch.cuda.synchronize()
    after = calls()
    assert after == before, (before, after)
    for v, w in zip(q, o):
        i, dist = f.query(v, K)
        assert torch.equal(i, w[0]) and torch.equal(dist, w[1])
    # beside other threads' queries, which may hold the event
    def other():
        for _ in range(200):
            f.query(q[1], K)
    th = threading.Thread(target=other)
    torch.cuda.synchronize()
    th.start()
    for _ in range(200):
        f.query_noalloc(q[1], K, o[1])
    th.join()
    torch.cuda.synchronize()
    i, dist = f.query(q[1], K)
    assert torch.equal(i, o[1][0]) and torch.equal(dist, o[1][1])


def case_tries():
    """Several tries per node where the device cannot hold the projections of all of them at once,
    or of any: the same forest, from fewer at a time."""
    for n, d, T, n0, n_try, limit in ((200_000, 4, 16, 64, 16, 100 << 20), (3000, 4, 64, 20, 10, 5 << 20)):
        x = torch.randn(n, d, device="cuda")
        R = torch.randn(T, 2 ** rpf.depth(n, n0) - 1, n_try, d, device="cuda")
        dumps = []
        for lim in (NO_LIMIT, limit):
            torch.cuda.synchronize()
            rpf.release_cached_memory()
            SHIM.shim_limit(lim)
            refused = calls()[3]
            f = rpf.build(x, T, n0, R, n_try=n_try)
            torch.cuda.synchronize()
            SHIM.shim_limit(NO_LIMIT)
            assert (calls()[3] > refused) == (lim == limit)
            dumps.append([f.tree_dump(t) for t in range(T)])
            f.free()
        for a, b in zip(*dumps):
            for k in ("perm", "chosen", "split_idx"):
                assert torch.equal(a[k], b[k]), k
        print(f"n={n}: as with all tries at once", flush=True)


def case_plan_tries():
    """The same for the parts of a plan, which keep their temporaries: 4 GiB over all parts."""
    sizes, T, n0, n_try = [60_000, 50_000, 3000], 16, 64, 16
    xs = [torch.randn(n, 4, device="cuda") for n in sizes]
    Rs = [torch.randn(T, 2 ** rpf.depth(n, n0) - 1, n_try, 4, device="cuda") for n in sizes]
    got = []
    for short in (False, True):
        torch.cuda.synchronize()
        rpf.release_cached_memory()
        if short:  # the projections of all tries take 230 MB of `peak`, those of one 15
            SHIM.shim_total(SHIM.shim_live() + peak - (100 << 20))
        refused = calls()[3]
        plan, p = library_peak(lambda: rpf.Plan(sizes, 4, T, n0, 5, n_try=n_try, max_part_points=60_000))
        peak = p
        SHIM.shim_total(NO_LIMIT)
        assert (calls()[3] > refused) == short
        plan.set_inputs(xs, Rs)
        plan.launch()
        plan.check()
        got.append([tuple(v.clone() for v in plan.result(i)) for i in range(len(sizes))])
        plan.close()
    for a, b in zip(*got):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


globals()["case_" + sys.argv[2]]()
print("done", flush=True)
