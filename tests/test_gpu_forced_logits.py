"""Teacher forcing with a logits buffer (the projection writes the caller's buffer and per-tile
records; the forced token's log-prob comes from the two) against teacher forcing without one
(stored logits, one scan a row), and the buffer's contents against the oracle.

Every step's logits of every live row are held to the oracle's in fp64, at the parity tests'
bounds.  Rows of finished sentences keep what was in them (with pruning, which takes them off
the live list), and so do the words on either side of the buffer.  A row's log-sum-exp is
summed in another order with the buffer than without, at most V = 2000 rounded terms apart, far
below the 1e-6 relative it is held to."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G
from tests.test_gpu_parity import LOGIT_TOL

pytestmark = pytest.mark.gpu

MARK = -7.0     # around the buffer


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("V,shift,prune", [(101, 0, 1), (517, 1, 1), (2000, 0, 0), (2000, 2, 1)])
def test_forced_scores_with_and_without_a_logits_buffer(V, shift, prune, dtype):
    from paper_2109_08008_amd import nt
    torch = G.torch_cuda()
    shape = synth.ModelShape(128, 4, 512, 2, 2, V)
    blob = synth.make_weights(shape, seed=5, lively=True)
    model = G.new_model(shape, blob, dtype)
    rng = np.random.default_rng(V + shift)
    srcs = [list(rng.integers(4, V, size=n)) for n in (1, 5, 9, 3, 7)]
    T = 6
    forced = rng.integers(4, V, size=(T, 5)).astype(np.int32)
    forced[2, 1] = G.EOS
    forced[3, 0] = V + 7          # out of range: ends the sentence
    forced[4, 2] = -1
    ends = [3, 2, 4, T, T]        # tokens each sentence emits; the last two reach their limit
    want = [[int(w) for w in forced[:n, b]] for b, n in enumerate(ends)]
    om = G.oracle_model(shape, blob, dtype)
    ref = [om.teacher_forced_logits(s, tg) for s, tg in zip(srcs, want)]
    search = synth.SearchSetup(beam=1, max_len_a=0.0, max_len_b=T, token_budget=0, prune=prune)
    runs = []
    for with_logits in (True, False):
        st, keep = G.gpu_encode(model, srcs, search)
        buf = torch.full((5 * V + shift + 8,), MARK, dtype=torch.float32, device="cuda")
        body = buf[shift:shift + 5 * V].view(5, V)
        for t in range(T):
            d = torch.from_numpy(forced[t]).cuda()
            body.fill_(float("nan"))
            alive = nt.nt_decode_step(st, d.data_ptr(), body.data_ptr() if with_logits else None)
            if with_logits:
                got = body.cpu().numpy()
                for b in range(5):
                    if t <= ends[b]:      # live: its end was not reached before this step
                        assert np.abs(got[b] - ref[b][t]).max() <= LOGIT_TOL[dtype], (t, b)
                    elif prune:
                        assert np.isnan(got[b]).all(), (t, b)
                assert bool((buf[:shift] == MARK).all()) and bool((buf[shift + 5 * V:] == MARK).all())
            assert alive == sum(t < n and t + 1 < T for n in ends)
            if alive == 0:
                break
        runs.append(nt.nt_dec_state_read(st))
        nt.nt_free_state(st)
    model.close()
    (ta, sa, la), (tb, sb, lb) = runs
    assert [list(x) for x in ta] == want and [list(x) for x in tb] == want
    np.testing.assert_allclose(sa, sb, rtol=1e-6, atol=1e-6)
    for a, b in zip(la, lb):
        np.testing.assert_allclose(a, b, rtol=1e-6, atol=1e-6)
