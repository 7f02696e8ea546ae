"""How the attention of a pass is cut into work items must not show in its results: the same prompt rows come out with the
same bits whether their blocks walk all chunks themselves or leave partial results for the merge."""
import numpy as np
import pytest

import das_inputs as di

pytestmark = pytest.mark.gpu

# two heads per key head at head dim 64 (chunks of 1024 keys), seven at head dim 128 (chunks of 2048)
HEADS = {"d64": di.MODELS["tiny"], "d128": di.ModelShape("narrow7b", 2, 256, 28, 4, 128, 512, 4096, rope_theta=1.0e6)}


def _prefill(shape, prompts, max_rows):
    import paper_2511_13841_amd as das
    lens = [len(p) for p in prompts]
    dm = das.DasModel(das.config_for(shape, max_seqs=len(prompts), max_ctx=max(lens) + 32, max_rows=max_rows, max_draft=0,
                                     num_pages=sum(n // 16 + 1 for n in lens) + 4), None, keep_logits=True, seed=3)
    ids = list(range(len(prompts)))
    nxt = dm.prefill(ids, prompts)
    kv = [dm.kv_export(i, shape.n_layers - 1, 0, n) for i, n in zip(ids, lens)]
    dm.verify_step(ids, lens, [[] for _ in ids])
    logits = dm.debug_logits()
    dm.free()
    return nxt, kv, logits


@pytest.mark.parametrize("heads,lens,many,few", [
    ("d64", [1, 1023, 1025, 2080], 1100, 65),                           # 65 rows: 9 row blocks, the fewest of a many-row block
    ("d64", [2080, 2049, 2048, 2047, 1030, 2080, 2080, 2080], 16384, 65),   # 122 blocks of up to three chunks in one pass
    ("d128", [31, 2047, 2049], 1100, 19), ("d128", [6100], 2400, 19), ("d128", [6100], 2400, 36)])   # 67 blocks, then 67, then 36
def test_prompt_blocks_taken_whole_equal_blocks_cut_at_chunks(heads, lens, many, few):
    """Passes of `many` rows have enough blocks to be taken whole (in part: also single-chunk and cut blocks among them); a pass
    of `few` rows is one block and is cut at every chunk.  The K and V of the last layer (every position's attention output is
    behind them) and the logits after the prompt are equal bit for bit."""
    shape = HEADS[heads]
    prompts = di.prompts(lens, shape.vocab, 5)
    print(heads, lens, "passes of", many, "rows", flush=True)
    n1, kv1, l1 = _prefill(shape, prompts, many)
    print("passes of", few, "rows", flush=True)
    n2, kv2, l2 = _prefill(shape, prompts, few)
    assert list(n1) == list(n2)
    for (k1, v1), (k2, v2) in zip(kv1, kv2):
        np.testing.assert_array_equal(k1, k2)
        np.testing.assert_array_equal(v1, v2)
    np.testing.assert_array_equal(l1, l2)
