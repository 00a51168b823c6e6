"""GPU parity of the projections at the edges of their tiles, through the C ABI.

A prefill of M rows and the decode steps after it run every projection of a
layer on the kernel that M selects: up to 128 rows the streaming GEMM, above it
the tiled one over the packed weights (128 x 128, 128 x 256 and 256 x 256 tiles).
The bar is the bf16 parity bound of the other cases: whatever the tile, the
products are the same and their sums float32; only the order of the sums differs
(the number of K slices depends on M and the grid, the row-major kernel permutes k).
"""
import numpy as np
import pytest

import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def _small(n_prompts, group, prompt_len, vocab=32000, steps=2):
    wl = W.workload("small").replace(gain_jitter=0.05, n_prompts=n_prompts, group=group, prompt_len=prompt_len)
    wl.senior.n_layers, wl.junior.n_layers = 1, 1
    wl.senior.vocab = wl.junior.vocab = vocab
    wl.sample.max_new = steps
    return wl


# (prompts, responses, prompt length, vocabulary, sequences checked): rows of
# the prefill are prompts x (length - 1), of a step prompts x responses
CASES = [
    (1, 1, 130, 32000, None),            # 129 rows: a second tile of one row; steps of one row
    (3, 11, 86, 32000, [0, 20, 32]),     # 255 rows; steps of 33 rows (two 32-row blocks, one row used)
    (2, 1, 130, 32000, None),            # 258 rows
    (2, 1, 1030, 32000, [1]),            # 2058 rows: 256 x 256 tiles with a ragged last row
    (5, 26, 9, 32001, [0, 70, 129]),     # 40 rows; steps of 130 rows, logits of an odd vocabulary in tiles
    (3, 43, 3, 32000, [5, 128]),         # steps of 129 rows, logits of a 128 x 256 tiled head
    (2, 2, 18, 32000, None),             # steps of 4 rows, the most with a row's SwiGLU along a lane's elements
    (5, 1, 18, 32000, None),             # steps of 5 rows
    (3, 32, 3, 31972, [5, 95]),          # steps of 96 rows, a last vocabulary block of 4 entries
]


@pytest.mark.parametrize("n_prompts,group,prompt_len,vocab,rows", CASES)
def test_projection_tile_edges(n_prompts, group, prompt_len, vocab, rows):
    P.log(f"case GEMM shapes: {n_prompts} prompts of {prompt_len} tokens x {group}, V {vocab}")
    p = P.run(_small(n_prompts, group, prompt_len, vocab), logits_at=(1, 2), seq_subset=rows)
    P.check(p, P.TOL_BF16)
    assert np.isfinite(p.out["logprob"]).all()


# gate/up of the tiled GEMM.  An FFN that is not a multiple of 256 has no packed
# down matrix, so its activations stay in split format: 128 x 128 tiles with a short
# and a deep ring, 128 x 256 tiles.  2048 / 4096: K slices and a SwiGLU pass (fp16, and
# split format where the FFN is 4080).
@pytest.mark.parametrize("d,ffn,n_prompts,prompt_len", [
    (256, 272, 2, 66), (512, 272, 1, 130), (256, 4112, 8, 66), (2048, 4096, 2, 66), (2048, 4080, 1, 257)])
def test_gate_up_routes(d, ffn, n_prompts, prompt_len):
    P.log(f"case gate/up: d_model {d}, ffn {ffn}, {n_prompts} prompts of {prompt_len} tokens")
    wl = _small(n_prompts, 1, prompt_len, vocab=512)
    for m in (wl.senior, wl.junior):
        m.d_model, m.ffn_dim, m.n_q_heads, m.n_kv_heads = d, ffn, 4, 2
    p = P.run(wl, logits_at=(1, 2))
    P.check(p, P.TOL_BF16)


# the float32 pair: up to 32 rows on the few-row kernel (4 or 8 rows at a time),
# above it the 32 x 32 tiles; 1023 and 511 are vocabularies with a last odd column
@pytest.mark.parametrize("n_prompts,group,prompt_len,vocab", [
    (1, 1, 2, 512), (1, 4, 6, 511), (1, 5, 9, 512), (3, 3, 4, 1023), (1, 31, 33, 512), (2, 16, 17, 511),
    (3, 11, 12, 512)])
def test_float32_projections_of_few_rows(n_prompts, group, prompt_len, vocab):
    P.log(f"case float32 GEMM shapes: {n_prompts} prompts of {prompt_len} tokens x {group}, V {vocab}")
    wl = W.workload("tiny").replace(gain_jitter=0.1, n_prompts=n_prompts, group=group, prompt_len=prompt_len)
    wl.senior.vocab = wl.junior.vocab = vocab
    wl.sample.max_new = 3
    p = P.run(wl, logits_at=(1, 3))
    P.check(p, P.TOL_F32)
