"""GPU parity of the step's tail (one workgroup per logits row, the last to arrive decides) against the
CPU oracle at the ends of its range: one row, the most rows a step has (R = 16), every accepted length,
single draws and tree levels, model shapes with and without the MFMA path; the workspace holds arbitrary
bytes before the weights are loaded."""
import pytest

import synth_inputs as si
from oracle import VerifyParams
from test_gpu_parity import GREEDY, X, _mid_cfg, _report  # noqa: F401  (X is a fixture)

pytestmark = pytest.mark.gpu

TOP8 = VerifyParams(mode=1, top_ka=8, temperature=0.8, sample=1, seed=77)
TREE1 = VerifyParams(mode=1, top_ka=8, temperature=0.05, sample=2, seed=78, top_ks=1, pts_prune=1e-5)
TREE4 = VerifyParams(mode=1, top_ka=8, temperature=0.05, sample=2, seed=79, top_ks=4, pts_prune=1e-5)


@pytest.mark.parametrize("K,vocab,vp,plain", [
    (15, 1024, GREEDY, False), (15, 1000, TREE1, False), (5, 1024, TREE4, False), (1, 1000, TOP8, False),
    (4, 1000, TOP8, True), (4, 1024, GREEDY, True),
])
def test_tail(X, K, vocab, vp, plain):
    cfg = _mid_cfg(n_layers=1, n_draft=K, vocab=vocab, prefix=9)

    def engine(*a, **kw):
        eng = X.pkg.Engine(*a, **kw)
        eng.d_ws.fill_(0x5A)
        return eng

    w, orc, states, eng = X.H.setup_pair(cfg, engine, 3)

    def forced(step, b, st, blk):
        full = X.H.true_continuation(orc, st, blk[0], K, GREEDY)
        j = (step * 5 + b) % (K + 1)
        if j < K:
            full[j + 1] = (full[j + 1] + vocab // 2) % vocab
        return full

    first = [row[:1] for row in si.first_block(cfg, 3)] if plain else si.first_block(cfg, 3)
    tal = X.H.lockstep(cfg, orc, states, eng, X.xsm, vp, 4, first, plain=plain, forced=None if plain else forced)
    _report(tal, f"tail K={K} V={vocab}{' plain' if plain else ''}")
