"""Trees of 33 to 64 nodes whose gate/up rows or vocabulary need twice as many
64-row as 128-row workgroup rounds on the chip: those projections run on the
prefill GEMM.  The row counts are the first ones past one round of 64-row
workgroups (the last 128-row workgroup half filled) and the last ones before;
K has more and fewer steps than its K groups share evenly.  Oracle and bars as
in test_gpu_parity.py; logits, argmax and a repeated step also against each
other."""
import numpy as np
import pytest

import synth
from oracle import verify as ov
from tests.helpers import GpuCase, compare_step, small_cfg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)


def _cu():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("d,past_ffn,past_vocab", [(256, True, True), (320, True, False), (64, False, True),
                                                   (192, False, False)])
def test_wide_tree_projections(d, past_ffn, past_vocab):
    # 64-row groups: rows / 64; one round holds _cu() of them
    ffn = 32 * (_cu() + (1 if past_ffn else 0))
    vocab = 64 * (_cu() + (1 if past_vocab else 0))
    cfg = small_cfg(n_layers=2, d_model=d, n_heads=d // 64, head_dim=64, d_ffn=ffn, vocab=vocab,
                    weight_dtype="bf16", init_std=0.09 * np.sqrt(256.0 / d) * np.sqrt(0.25))
    case = GpuCase(cfg, seed=601, capacity=160)
    try:
        om = case.w.oracle()
        kv = case.new_kv()
        kv_o = case.synthetic_context(kv, 602, 45)
        for m in (32, 33, 47, 48, 49, 64):
            toks, par = synth.random_tree(603 + m, m, 6, cfg.vocab)
            ref = ov.verify_step(om, kv_o, toks, par)
            ref["tokens"], ref["parents"] = np.asarray(toks), np.asarray(par)
            acc, lg = case.step(kv, toks, par)
            compare_step(acc, lg, ref, 2e-2)
            assert np.array_equal(np.argmax(lg[:m], axis=1), np.asarray(acc.argmax[:m]))
            acc2, lg2 = case.step(kv, toks, par)
            assert np.array_equal(lg, lg2)
    finally:
        case.close()
