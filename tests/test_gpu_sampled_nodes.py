"""The sampling rule at the vocabularies where its kernel changes (8 and 16
registers of 4 ids per thread, rows that end inside a wave, the one-workgroup
walk above 65536), through the allocation-free entry point: against the oracle
with the margins of test_gpu_sampled.py, wide trees with many rejections, and
masked tokens (logits of -inf)."""
import numpy as np
import pytest

import synth
from oracle import verify as ov

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2412_18934_amd import dv  # noqa: E402
from tests.test_gpu_sampled import _correlated_drafts, _dev, _draft_tree, _judge  # noqa: E402


@pytest.mark.parametrize("vocab,m,depth,noise", [
    (4, 5, 3, 0.5), (260, 33, 2, 3.0), (2052, 64, 9, 0.7), (32768, 20, 4, 1.5), (32772, 20, 4, 1.5),
    (65536, 9, 3, 1.0), (65540, 9, 3, 1.0)])
def test_vocabulary_sizes(vocab, m, depth, noise):
    differ = 0
    for rep in range(3):
        seed = 8000 + 10 * rep + m
        rng = np.random.default_rng(seed)
        logits = synth.normal(seed, 90, m * vocab, 2.5, "f32").reshape(m, vocab)
        if rep == 2:
            logits[:, 1::3] = -np.inf      # masked ids: probability 0
        q = _correlated_drafts(np.where(np.isinf(logits), -30.0, logits), 0.9, noise, rng)
        toks, par = _draft_tree(m, depth, q, seed, vocab)
        ua, ub = synth.sampling_uniforms(seed, m)
        trace = []
        n, path, bonus = ov.accept_sampled(logits, toks, par, q, 0.9, ua, ub, trace=trace)
        lg, qd = _dev(logits), _dev(q)
        acc = [dv.dv_accept_sampled_noalloc(lg.data_ptr(), toks, par, vocab, qd.data_ptr(), 0.9, ua, ub)
               for _ in range(2)]
        assert acc[0].path_list == acc[1].path_list and acc[0].bonus_token == acc[1].bonus_token
        differ += not _judge(acc[0], n, path, bonus, trace, par, vocab)
    assert differ <= 1
