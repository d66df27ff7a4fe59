"""bf16 batches whose tokens and logits are pinned bit for bit.

A greedy chain follows its logits' last bits: where two logits are close, another order of a sum picks another token,
and everything after it differs. A faster kernel therefore keeps the order of every sum of a bf16 step (the k-splits of
each projection, hi before lo in each 32-wide k-step, partial sums added in order to the residual, two score chains in
prefill attention), and these batches say whether it did. The recorded values are the engine's own on an MI355X, from
kernels that the oracle checks in the other GPU tests; they hold tokens whole and the logits' SHA-256.
"""
import hashlib
import json
import os

import numpy as np
import pytest

from moa_inputs import ModelShape, f32_to_bf16_bits, generate_weights
from moa_inputs.configs import EngineConsts
from tests.gpu_helpers import run_requests

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"


GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "bf16_bits.json")


def _batch(lens, shape, G=3, of=None, budget=512, sharp=False):
    """lens: prompt lengths; of: each prompt's model (default: one model); shape: layers, d, heads, KV heads, head_dim,
    ffn, vocab; sharp: W_q times 32, so that scores spread over tens of log2 units."""
    return dict(lens=list(lens), shape=shape, G=G, of=list(of or [0] * len(lens)), budget=budget, sharp=sharp)


def _rows(shape, *rows, G=4):
    """Every step has rows[m] rows of model m: one-token prompts, all of G tokens."""
    return _batch([1] * sum(rows), shape, G=G, of=[m for m, n in enumerate(rows) for _ in range(n)])


_ragged = [1, 31, 32, 33, 63, 64, 65, 97, 127, 128, 129, 161, 7, 12, 13, 45, 200, 300, 5, 82]
BATCHES = {
    # prefill attention: one step of more than 256 rows and 20 prompts, every edge of its tiles of 32 keys and 128 rows
    "prompts hd64": _batch(_ragged, (2, 512, 4, 2, 64, 256, 512), G=1, budget=2048),
    "prompts hd128": _batch(_ragged, (2, 512, 4, 2, 128, 256, 512), G=1, budget=2048),
    "sharp prompts hd64": _batch(_ragged, (1, 512, 4, 2, 64, 256, 512), G=1, budget=2048, sharp=True),
    "sharp prompts hd128": _batch(_ragged, (1, 512, 8, 2, 128, 256, 512), G=1, budget=2048, sharp=True),
    # small-M GEMM: 7 to 16 rows, one model and several; K/32 with few and many twos; prompts whose last rows alone
    # reach the head; a qkv width of whole 128-column tiles only, at any number of rows
    "rows 7": _rows((2, 512, 8, 2, 64, 1408, 1152), 7),
    "rows 8": _rows((1, 2048, 32, 8, 64, 5632, 1152), 8),
    "rows 9": _rows((1, 2048, 16, 2, 128, 8192, 1024), 9),
    "rows 16": _rows((2, 256, 4, 1, 64, 1408, 512), 16),
    "rows 12 5": _rows((1, 1536, 16, 2, 128, 1024, 1152), 12, 5),
    "rows 8 8 8": _rows((1, 4096, 8, 2, 128, 896, 512), 8, 8, 8),
    "chunked prompts hd128": _batch([700, 650, 600], (2, 512, 4, 2, 128, 256, 512), G=1, budget=333),
    "qkv 384": _batch([300, 290], (1, 512, 4, 1, 64, 256, 512), G=1, of=[0, 1], budget=1024),
    # row GEMMs: steps of up to six rows; K of 8 to 448 k-steps, both head widths, one to eight query heads per KV
    # head, prompts of a few tokens prefilled in such steps, several models on two streams, a deep ffn on a narrow d
    # on either side of the rule
    "row 1": _rows((3, 2048, 32, 8, 64, 8192, 1152), 1, G=6),
    "row 6": _rows((2, 512, 2, 2, 128, 1408, 512), 6, G=6),
    "rows 2 3 1": _rows((2, 256, 8, 1, 64, 128, 512), 2, 3, 1, G=6),
    "rows 2 deep": _rows((1, 512, 8, 2, 64, 14336, 512), 2),
    "rows 3 deep": _rows((1, 512, 8, 2, 64, 14336, 512), 3),
    "row 4096": _rows((1, 4096, 32, 8, 128, 14336, 512), 2),
    "short prompts": _batch([3, 1, 2, 5, 1], (2, 1536, 12, 12, 64, 1024, 1152), G=5, of=[0, 1, 0, 1, 1], budget=4),
    # medium rows: k-splits of every projection between 17 rows and the large-row plan, ffn / 128 odd and even
    "rows 17": _rows((1, 2048, 32, 8, 64, 5504, 1024), 17),
    "rows 24": _rows((2, 1536, 8, 2, 128, 8960, 1024), 24),
    "rows 48": _rows((1, 2048, 32, 8, 64, 6528, 1152), 48, G=3),
    "rows 60": _rows((1, 2048, 32, 8, 64, 8192, 1024), 60, G=3),
    "rows 96": _rows((1, 2048, 32, 8, 64, 8192, 512), 96, G=3),
    "rows 90 70 50": _rows((1, 1024, 8, 4, 64, 1792, 512), 90, 70, 50, G=3),
    "rows 130 20": _rows((1, 4096, 8, 2, 64, 1792, 512), 130, 20, G=2),
    "rows 200": _rows((1, 512, 8, 2, 64, 896, 512), 200, G=2),
    # gate-up grids of more than 256 of the widest tiles, 512 and 256 columns
    "rows 150 150 60": _rows((1, 256, 4, 2, 64, 16384, 512), 150, 150, 60, G=2),
    "rows 100 100": _rows((1, 256, 4, 2, 64, 16512, 512), 100, 100, G=2),
}


def _weights(shape, seed, m, sharp):
    w = generate_weights(shape, "bf16", seed, 97, m)
    rng = np.random.default_rng([seed, m, 3])
    for n in w:
        if n.endswith("norm"):
            w[n] = f32_to_bf16_bits(rng.uniform(0.5, 1.5, shape.d_model).astype(np.float32))
        elif sharp and n.endswith("wq"):
            w[n] = np.where(w[n] & 0x7f80, w[n] + np.uint16(5 << 7), w[n]).astype(np.uint16)
    return w


def run_batch(b, **kw):
    layers, d, nh, nkv, hd, ffn, vocab = b["shape"]
    shape = ModelShape(n_layers=layers, d_model=d, n_heads=nh, n_kv_heads=nkv, head_dim=hd, ffn_dim=ffn, vocab=vocab)
    ws = [_weights(shape, d + ffn, m, b["sharp"]) for m in range(max(b["of"]) + 1)]
    rng = np.random.default_rng([len(b["lens"]), d, ffn])
    reqs = [(rng.integers(0, vocab, n).astype(np.int32), b["of"][i], b["G"]) for i, n in enumerate(b["lens"])]
    consts = EngineConsts(num_kv_blocks=sum((n + b["G"]) // 16 + 1 for n in b["lens"]), max_num_seqs=len(b["lens"]),
                          max_prefill_tokens=b["budget"], max_model_len=max(b["lens"]) + b["G"])
    return run_requests(shape, "bf16", consts, ws, reqs, **kw)


def digest(toks, logs):
    h = hashlib.sha256()
    for x in logs:
        h.update(np.ascontiguousarray(x, dtype=np.float32).tobytes())
    return {"tokens": [[int(t) for t in x] for x in toks], "logits": h.hexdigest()}


@pytest.mark.parametrize("name", sorted(BATCHES))
def test_bits(name):
    with open(GOLDEN) as f:
        want = json.load(f)[name]
    got = digest(*run_batch(BATCHES[name]))
    assert got["tokens"] == want["tokens"]
    assert got["logits"] == want["logits"], f"{name}: tokens agree, logits' bits do not"
