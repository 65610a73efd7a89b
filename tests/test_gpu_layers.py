"""GPU parity of the persistent layers kernel (passes of more than 16 rows, d = 1024 and 1536)
against the CPU oracle at the sizes where its partitions can go wrong: row tiles that are full, hold
one row or are one too many; as many row groups as fit; attention units shorter and longer than a
task's share, and pieces of a unit merged across tasks; prefill passes of one row more than a tile."""
import pytest

import synth_inputs as si
from oracle import VerifyParams
from test_gpu_parity import GREEDY, X, _c1_small, _report  # noqa: F401  (X is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,lens", [
    (2, [40, 3, 64, 61, 128, 17]),                    # 18 rows; contexts around a chunk's end
    (8, [700, 450]),                                  # 18 rows; every unit spans several tasks
    (3, [260, 1, 65, 33, 900, 47, 129, 20]),          # 32 rows: two full tiles
    (2, [5 + 6 * b for b in range(11)]),              # 33 rows: one more
    (5, [190 - 7 * b for b in range(20)]),            # 120 rows
    (4, [30 + b for b in range(64)]),                 # 320 rows
])
def test_decoding_rows(X, K, lens):
    cfg = _c1_small(n_layers=2, n_draft=K, vocab=1024)
    w, orc, states, eng = X.H.setup_pair(cfg, X.pkg.Engine, len(lens), prefix_lens=lens)
    tal = X.H.lockstep(cfg, orc, states, eng, X.xsm, GREEDY, 2, si.first_block(cfg, len(lens)))
    _report(tal, f"layers kernel {len(lens)} x {K + 1} rows")
    eng.xsm_check_device()


def test_plain_rows_and_a_skipped_sequence(X):
    """17 plain rows, then the same batch with one row's length out of range: skipped, the others unharmed."""
    lens = [20 + 11 * b for b in range(17)]
    cfg = _c1_small(n_layers=2, n_draft=2, vocab=1024)
    w, orc, states, eng = X.H.setup_pair(cfg, X.pkg.Engine, 17, prefix_lens=lens)
    tal = X.H.lockstep(cfg, orc, states, eng, X.xsm, GREEDY, 2, si.first_block(cfg, 17), plain=True)
    _report(tal, "layers kernel 17 plain rows")
    torch = X.torch
    buf = eng.buffers(17, spec=False, debug=True)
    cur = [st.n for st in states]
    buf.kv_len.copy_(torch.tensor(cur)); buf.block.copy_(torch.tensor(si.first_block(cfg, 17)[:, :1]))
    vp = X.H.to_vp_gpu(X.xsm, GREEDY)
    eng.xsm_plain_step(buf, vp, max(cur))
    good = buf.logits.clone()
    buf.kv_len.copy_(torch.tensor(cur)); buf.kv_len[5] = -1
    buf.block.copy_(torch.tensor(si.first_block(cfg, 17)[:, :1]))
    eng.xsm_plain_step(buf, vp, max(cur))
    n = buf.n_accepted.cpu().tolist()
    assert n[5] == 0 and all(v == 1 for b, v in enumerate(n) if b != 5)
    keep = [b for b in range(17) if b != 5]
    assert torch.allclose(buf.logits[keep], good[keep], rtol=0, atol=2e-3 * float(good[keep].abs().max()))


@pytest.mark.parametrize("prefix", [17, 33, 64, 257, 321])
def test_prefill_rows(X, prefix):
    cfg = _c1_small(n_layers=2, n_draft=2, vocab=1024)
    w, orc, states, eng = X.H.setup_pair(cfg, X.pkg.Engine, 2, prefix_lens=[prefix, prefix + 1])
    tal = X.H.lockstep(cfg, orc, states, eng, X.xsm, GREEDY, 2, si.first_block(cfg, 2))
    _report(tal, f"layers kernel prefill {prefix}")


@pytest.mark.parametrize("n_seq,n_cond", [(4, 100), (7, 64), (16, 130)])
def test_cross_attention(X, n_seq, n_cond):
    cfg = si.get_config("c3", n_layers=2, n_cond=n_cond, vocab=1024, max_ctx=512)
    lens = [0 if b == 1 else 18 + 23 * b for b in range(n_seq)]
    w, orc, states, eng = X.H.setup_pair(cfg, X.pkg.Engine, n_seq, prefix_lens=lens)
    vp = VerifyParams(mode=1, top_ka=8, temperature=0.8, sample=1, seed=5)
    tal = X.H.lockstep(cfg, orc, states, eng, X.xsm, vp, 2, si.first_block(cfg, n_seq))
    _report(tal, f"layers kernel cross-attention B{n_seq} n_cond {n_cond}")
    eng.xsm_check_device()


def test_timeout_is_reported_in_band_and_falls_back(X):
    """The failure path, forced from the host (the error word is set as a timed-out wait would set it; no
    wait is made to spin and every kernel exits normally): steps and prefills enqueued before the report
    change nothing and say so, and the passes after it run on the per-stage kernels and match the oracle."""
    cfg = _c1_small(n_layers=2, n_draft=2, vocab=1024)
    torch, lens = X.torch, [40, 3, 64, 61, 128, 17]
    w, orc, states, eng = X.H.setup_pair(cfg, X.pkg.Engine, 6, prefix_lens=lens)
    first = si.first_block(cfg, 6)
    buf = eng.buffers(6, spec=True)
    buf.kv_len.copy_(torch.tensor(lens)); buf.block.copy_(torch.tensor(first))
    buf.out_tokens.fill_(-7)
    eng.xsm_debug_inject_device_error(77)
    for _ in range(2):
        eng.xsm_spec_step(buf, X.H.to_vp_gpu(X.xsm, GREEDY), max(lens))
    eng.xsm_prefill([0, 2], torch.ones(2, 20, cfg["d_model"], dtype=torch.bfloat16, device="cuda:0"))
    eng.xsm_prefill([4], torch.ones(1, 19, cfg["d_model"], dtype=torch.bfloat16, device="cuda:0"))
    torch.cuda.synchronize()
    assert buf.n_accepted.tolist() == [0] * 6
    assert all(int(f) & X.xsm.XSM_FLAG_DEVICE_TIMEOUT for f in buf.flags.tolist())
    assert buf.kv_len.tolist() == lens and buf.block.tolist() == first.tolist()
    assert (buf.out_tokens == -7).all()
    with pytest.raises(X.xsm.XsmError, match="timed out"):
        eng.xsm_check_device()
    eng.xsm_check_device()                               # reported once
    X.xsm.xsm_debug_trace_enable(True); X.xsm.xsm_debug_trace_report()
    tal = X.H.lockstep(cfg, orc, states, eng, X.xsm, GREEDY, 2, first)
    ran = X.xsm.xsm_debug_trace_report(); X.xsm.xsm_debug_trace_enable(False)
    _report(tal, "after the layers kernel's injected timeout: per-stage kernels")
    assert "gemm_ws" in ran, sorted(ran)
