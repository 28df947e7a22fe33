"""A grouped on-chip solve captured into a graph: replayed between eager group
calls of the same first plan (other members, a larger group that outgrows the
first one's work list) and after its integrals changed, against the eager
call."""
import pytest

from paper_2307_10675_amd import ifci, synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("space", [3, 12])
@pytest.mark.parametrize("count", [2, 9])
def test_captured_group(count, space):
    import torch
    kw = dict(max_space=space, r_tol=1e-8, max_iter=500)
    probs = [synthetic.chain(3, seed=811, order=3), synthetic.single(6, 12, 812), synthetic.single(2, 12, 813),
             synthetic.chain(4, seed=814, order=2)]
    probs = [probs[j % len(probs)] for j in range(count)]
    plans = [ifci.Plan(p, **kw).attach(p.h, p.eri) for p in probs]
    others = [ifci.Plan(p, **kw).attach(p.h, p.eri) for p in
              [synthetic.chain(5, seed=820 + j, order=3) for j in range(40)]]
    print(f"[capture] {count} plans max_space {space}", flush=True)
    want = ifci.davidson_group(plans)  # allocates the work list
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = ifci.davidson_group(plans)
    between = [lambda: None,
               lambda: ifci.davidson_group([plans[0], others[0]]),
               lambda: ifci.davidson_group([plans[0]] + others),
               None,
               lambda: ifci.davidson_group(plans[::-1])]
    for step, eager in enumerate(between):
        if step == 3:  # new integrals in the same workspace
            h, eri = plans[1]._ints
            h.mul_(1.01)
            ifci._check(ifci.lib().ifci_set_integrals(plans[1]._h, ifci._ptr(h), ifci._ptr(eri), ifci._stream()))
            want = ifci.davidson_group(plans)
        else:
            eager()
        torch.cuda.synchronize()
        for o in out:
            for t in o:
                t.zero_()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert (a[1] == ifci.INC_DONE).all()
            for x, y in zip(a, b):
                assert torch.equal(x, y), step
