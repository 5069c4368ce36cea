"""Eigensolves of two contexts at once, each on its own thread and stream: a team's
workgroups then start late and apart, as the other context's kernels hold compute
units, and every solve still has to give the bits it gives alone."""
import threading

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def matrix(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn(n, n // 4, device="cuda", dtype=torch.float64, generator=g) * 0.3
    return torch.diag(torch.rand(n, device="cuda", dtype=torch.float64, generator=g) * 2500 + 0.1) + X @ X.T


@pytest.mark.parametrize("orders,rounds", [((2048, 1940), 25), ((513, 1100, 300), 20),
                                           ((3072, 2500), 6), ((3300, 1500), 3)])
def test_two_contexts_solve_at_once(orders, rounds):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2210_17093_amd.qsgw as q
    Ms = {n: matrix(n) for n in orders}
    torch.cuda.synchronize()
    c0 = q.Context()
    ref = {n: [x.clone() for x in q.qsgw_rpa_solve(c0, Ms[n].clone())] for n in orders}
    torch.cuda.synchronize()
    bad, done = [], []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                c = q.Context(stream)
                for r in range(rounds):
                    for n in orders[::-1] if k else orders:
                        Z, Om = q.qsgw_rpa_solve(c, Ms[n].clone())
                        stream.synchronize()
                        if not (torch.equal(Z, ref[n][0]) and torch.equal(Om, ref[n][1])):
                            bad.append((k, r, n))
                        done.append(n)
                c.close()
        except Exception as e:  # (the assertion below shows it)
            bad.append((k, repr(e)))

    print("two contexts", orders, flush=True)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    c0.close()
    assert not bad and len(done) == 2 * rounds * len(orders), bad
