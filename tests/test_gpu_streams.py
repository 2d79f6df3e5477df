"""Handles take the second streams of their factorisations from a bounded
pool and give them back: many handles one after the other, several alive at
once and handles of several threads compute what one handle alone computes."""
import threading

import pytest
import torch

import paper_2609_14706_amd as ffe

pytestmark = pytest.mark.gpu


def _fit(G, stream=None):
    f = ffe.FlipFlop(G, stream=stream)
    f.iterate(2)
    A, B = f.factors()
    f.close()
    return A, B


def _samples(gpu, seed):
    g = torch.Generator().manual_seed(seed)
    # 520 and 640 wide: five leaves each, both factors use a second stream
    return torch.randn(8, 520, 640, generator=g).to(gpu)


def test_one_after_the_other_and_many_alive(gpu):
    G = _samples(gpu, 1)
    want = _fit(G)
    for _ in range(4):
        got = _fit(G)
        assert all(torch.equal(x, y) for x, y in zip(got, want))
    alive = [ffe.FlipFlop(G) for _ in range(7)]   # 14 sets, more than the pool keeps
    for f in alive:
        f.iterate(2)
    for f in alive:
        got = f.factors()
        assert all(torch.equal(x, y) for x, y in zip(got, want))
        f.close()
    assert all(torch.equal(x, y) for x, y in zip(_fit(G), want))


def test_handles_of_several_threads(gpu):
    Gs = [_samples(gpu, s) for s in range(4)]
    want = [_fit(G) for G in Gs]
    torch.cuda.synchronize()
    got, errors = [None] * 4, []

    def work(k):
        try:
            stream = torch.cuda.Stream(gpu)
            for _ in range(3):
                got[k] = _fit(Gs[k], stream)
        except Exception as e:  # noqa: BLE001
            errors.append(e)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors and not any(t.is_alive() for t in threads)
    for g, w in zip(got, want):
        assert all(torch.equal(x, y) for x, y in zip(g, w))
