"""Teacher forcing with a logits buffer (the projection writes the caller's buffer and per-tile
records; the forced token's log-prob comes from the two) against teacher forcing without one
(stored logits, one scan a row).  The logits are the same bits on both paths; a row's
log-sum-exp is summed in another order, at most V = 2000 rounded terms apart, far below the
1e-6 relative they are held to."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("V,shift,prune", [(101, 0, 1), (517, 1, 1), (2000, 0, 0), (2000, 2, 1)])
def test_forced_scores_with_and_without_a_logits_buffer(V, shift, prune, dtype):
    from paper_2109_08008_amd import nt
    torch = G.torch_cuda()
    shape = synth.ModelShape(128, 4, 512, 2, 2, V)
    model = G.new_model(shape, synth.make_weights(shape, seed=5, lively=True), dtype)
    rng = np.random.default_rng(V + shift)
    srcs = [list(rng.integers(4, V, size=n)) for n in (1, 5, 9, 3, 7)]
    T = 6
    forced = rng.integers(4, V, size=(T, 5)).astype(np.int32)
    forced[2, 1] = G.EOS
    forced[3, 0] = V + 7          # out of range: ends the sentence
    forced[4, 2] = -1
    search = synth.SearchSetup(beam=1, max_len_a=0.0, max_len_b=T, token_budget=0, prune=prune)
    runs = []
    for with_logits in (True, False):
        st, keep = G.gpu_encode(model, srcs, search)
        buf = torch.full((5 * V + shift,), -7.0, dtype=torch.float32, device="cuda")
        for t in range(T):
            d = torch.from_numpy(forced[t]).cuda()
            if nt.nt_decode_step(st, d.data_ptr(), buf.data_ptr() + 4 * shift if with_logits else None) == 0:
                break
        runs.append(nt.nt_dec_state_read(st))
        nt.nt_free_state(st)
        if with_logits:
            assert bool((buf[:shift] == -7.0).all()) and bool(torch.isfinite(buf).all())
    model.close()
    (ta, sa, la), (tb, sb, lb) = runs
    assert [list(x) for x in ta] == [list(x) for x in tb]
    np.testing.assert_allclose(sa, sb, rtol=1e-6, atol=1e-6)
    for a, b in zip(la, lb):
        np.testing.assert_allclose(a, b, rtol=1e-6, atol=1e-6)
