"""Kernels at the sizes where a tile, a remainder or a dispatch rule ends, through the engine, against the oracle.

Every check is teacher-forced on the engine's own tokens (tests.gpu_helpers.compare): 1e-4 for fp32 engines, 2e-2 for
bf16 ones against the oracle with a bf16 K/V cache, the bounds of the other GPU tests."""
import numpy as np
import pytest

from moa_inputs import ModelShape, generate_weights
from moa_inputs.configs import EngineConsts
from tests.gpu_helpers import compare, run_requests

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"


def _check(shape, dtype, lens, G, seed, models=1, consts=None):
    ws = [generate_weights(shape, dtype, seed, 97, m) for m in range(models)]
    rng = np.random.default_rng([seed, 13])
    reqs = [(rng.integers(0, shape.vocab, n).astype(np.int32), i % models, G) for i, n in enumerate(lens)]
    consts = consts or EngineConsts(num_kv_blocks=256, max_num_seqs=max(8, len(lens)), max_prefill_tokens=96,
                                    max_model_len=512)
    toks, logs = run_requests(shape, dtype, consts, ws, reqs)
    for i, (p, m, _) in enumerate(reqs):
        compare(shape, ws[m], p, toks[i], logs[i], dtype == "bf16", 1e-4 if dtype == "f32" else 2e-2,
                what=f"call {i} ({len(p)} tokens)", report_pure=False)


# fp32 GEMM: K = 64 (one 16-k step per wave), 256 and 320; one to 33 rows in a step (16-row chunks and their
# remainders); a vocabulary past 1,024 64-column items takes the four-tile variant
@pytest.mark.parametrize("ffn,vocab,lens", [(64, 64, [1]), (320, 192, [16, 1, 17]), (64, 65600, [33, 5])])
def test_fp32_gemm_edges(ffn, vocab, lens):
    shape = ModelShape(n_layers=1, d_model=256, n_heads=1, n_kv_heads=1, head_dim=64, ffn_dim=ffn, vocab=vocab)
    _check(shape, "f32", lens, 3, seed=ffn + vocab, models=min(2, len(lens)))
