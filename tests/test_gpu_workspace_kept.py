"""The device buffer the library keeps between calls: bounded, given back, and never in the way of
a result."""
import threading
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.fixture(scope="module")
def M():
    import paper_2503_04424_amd as m
    m.load()
    return m


def spd(n):
    a = torch.eye(n, dtype=torch.float64, device="cuda") * 2.0
    a[1:, :-1].diagonal().fill_(0.5)
    return a


def free(at_least=0):
    """Free bytes of the device.  The driver may count memory that has been given back only some
    milliseconds after the free returned: a moment for what came before, and up to two seconds for
    what is expected."""
    torch.cuda.synchronize()
    time.sleep(0.1)
    end = time.monotonic() + 2.0
    while (now := torch.cuda.mem_get_info()[0]) < at_least and time.monotonic() < end:
        time.sleep(0.01)
    return now


def test_bounded_and_given_back(M):
    small, mid, big = spd(256), spd(5000), spd(9000)     # workspaces of 0.5, 200 and 648 MB
    M.mdet_logdet_device(small, mem_budget=1 << 40)       # with a budget: nothing stays behind
    base = free()
    want = M.mdet_logdet_device(mid).logabsdet
    kept = base - free()
    assert 150 * MIB <= kept <= 512 * MIB
    assert M.mdet_logdet_device(mid).logabsdet == want    # from the same buffer
    assert abs((base - free()) - kept) <= 8 * MIB
    M.mdet_logdet_device(big)                             # over the bound: not kept, the other one gone
    assert base - free(base - 16 * MIB) <= 16 * MIB
    M.mdet_logdet_device(mid)
    assert base - free() >= 150 * MIB
    for _ in range(40):                                   # calls that have no use for 200 MB
        M.mdet_logdet_device(small)
    assert base - free(base - 32 * MIB) <= 32 * MIB
    M.mdet_logdet_device(mid)
    M.mdet_logdet_device(small, mem_budget=1 << 40)
    assert base - free(base - 16 * MIB) <= 16 * MIB


@pytest.mark.parametrize("host", [False, True])
def test_calls_with_their_own_workspace(M, host):
    """A budget frees the buffer whoever owns the call's workspace, and calls with a workspace of
    their own count as calls without a use for it."""
    n, bs = 700, 128
    small, mid = spd(n), spd(5000)
    packed = M.pack_lower_block_columns(small.cpu(), bs)

    def call(budget, expected=0):
        ws, _ = M.mdet_workspace_query(n, torch.float64, bs, budget, overwrite=False, for_device_input=not host)
        buf = torch.empty(ws, dtype=torch.uint8, device="cuda")
        held = free()
        for _ in range(1 if budget else 31):
            if host:
                M.mdet_logdet_host(packed, n, bs, mem_budget=budget, overwrite=False, workspace=buf)
            else:
                M.mdet_logdet_device(small, block_size=bs, mem_budget=budget, overwrite=False, workspace=buf)
        return free(held + expected) - held               # what the calls gave back

    call(1 << 40)
    M.mdet_logdet_device(mid)                             # leaves 200 MB
    assert call(1 << 40, 150 * MIB) >= 150 * MIB
    M.mdet_logdet_device(mid)
    assert abs(call(0)) <= 8 * MIB                        # 31 calls: still there
    assert call(0, 150 * MIB) >= 150 * MIB                # the 32nd


def test_threads_and_leftovers(M):
    # a buffer full of another call's numbers, NaN among them, changes nothing; several threads
    # at once each get the right result
    bad = spd(1500)
    bad[7, 3] = float("nan")
    M.mdet_logdet_device(bad, raise_on_error=False)
    cases = []
    for n, bs in ((1500, 256), (700, 128), (1100, 192), (64, 64)):
        a = W.scaled_down(W.config(1), n, bs).dense()
        cases.append((torch.from_numpy(a).cuda(), bs, oracle.ldlt_logdet(a).logabsdet))
    errs = []

    def work(k):
        a, bs, want = cases[k]
        st = torch.cuda.Stream()
        for _ in range(6):
            r = M.mdet_logdet_device(a, block_size=bs, stream=st)
            if not (r.status == 0 and abs(r.logabsdet - want) <= 1e-10 * abs(want)):
                errs.append((k, r))

    th = [threading.Thread(target=work, args=(k,)) for k in range(len(cases))]
    [t.start() for t in th]
    [t.join() for t in th]
    assert not errs
