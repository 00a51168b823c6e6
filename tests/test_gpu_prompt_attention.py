"""GPU parity of the prompt rows' QKV post-processing and attention at the edges
of their row groups (16 rows) and stages (32 positions), for each head size and
group size they have a kernel for, through the C ABI: a few prompts at a time,
and many in one pass (5 rows and more per compute unit).

The first step after the prefill attends to every prompt position, so its logits
see the prompt's K/V of both layers, and the second layer's K/V sees the first
layer's attention output at every prompt row.
"""
import pytest

import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 16, 17, 18, 32, 33, 34, 48, 50, 65, 97]


def _pair(hd, gqa_sen, gqa_jun, lengths, max_new=2):
    wl = W.workload("small").replace(gain_jitter=0.05, n_prompts=len(lengths), group=1, prompt_len=max(lengths))
    for m, gqa, nkv in ((wl.senior, gqa_sen, 2), (wl.junior, gqa_jun, 1)):
        m.n_layers, m.d_model, m.head_dim, m.n_kv_heads, m.n_q_heads = 2, 256, hd, nkv, nkv * gqa
        m.ffn_dim, m.vocab = 512, 512
    wl.sample.max_new = max_new
    return wl


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("gqa_sen,gqa_jun", [(4, 2), (1, 8), (8, 16)])
def test_prompt_attention_edges(hd, gqa_sen, gqa_jun):
    P.log(f"case prompt attention: head_dim {hd}, groups of {gqa_sen} and {gqa_jun} heads, prompt lengths {LENGTHS}")
    wl = _pair(hd, gqa_sen, gqa_jun, LENGTHS)
    ws, wj, _, bnd = W.make_all(wl)
    prompts = [W.make_prompts(wl)[i][:n] for i, n in enumerate(LENGTHS)]
    p = P.run(wl, logits_at=(1, 2), max_prefill_tokens=256, weights=(ws, wj, prompts, bnd))
    P.check(p, P.TOL_BF16)


@pytest.mark.parametrize("hd,gqa_sen,gqa_jun", [(32, 4, 2), (64, 4, 2), (128, 4, 2), (64, 8, 1), (128, 1, 8)])
def test_many_prompt_rows_in_one_pass(hd, gqa_sen, gqa_jun):
    lengths = LENGTHS * 8                               # 3464 rows
    P.log(f"case prompt rows: head_dim {hd}, groups of {gqa_sen} and {gqa_jun} heads, {len(lengths)} prompts")
    wl = _pair(hd, gqa_sen, gqa_jun, lengths)
    wl.junior.n_kv_heads, wl.junior.n_q_heads = 2, 2 * gqa_jun
    ws, wj, _, bnd = W.make_all(wl)
    prompts = [p[:n] for p, n in zip(W.make_prompts(wl), lengths)]
    rows = list(range(0, 96, 7)) + [95]
    p = P.run(wl, logits_at=(1, 2), max_prefill_tokens=4096, weights=(ws, wj, prompts, bnd), seq_subset=rows)
    P.check(p, P.TOL_BF16)


@pytest.mark.parametrize("hd,dtype", [(32, "f32"), (64, "f32"), (128, "f32"), (32, "bf16"), (64, "bf16"),
                                      (128, "bf16")])
def test_plain_attention_of_many_and_few_rows(hd, dtype):
    """Groups of three heads (and float32) take the plain attention: the prompts'
    rows in one pass the form for a full device, the steps' 14 rows the one whose
    value product is in parts; contexts of up to three 128-position blocks."""
    lengths = LENGTHS + [130, 260]
    P.log(f"case plain attention: head_dim {hd}, {dtype}, prompt lengths {lengths}")
    wl = _pair(hd, 3, 3, lengths)
    wl.senior.dtype = wl.junior.dtype = dtype
    ws, wj, _, bnd = W.make_all(wl)
    prompts = [p[:n] for p, n in zip(W.make_prompts(wl), lengths)]
    p = P.run(wl, logits_at=(1, 2), max_prefill_tokens=1024, weights=(ws, wj, prompts, bnd))
    P.check(p, P.TOL_F32 if dtype == "f32" else P.TOL_BF16)
