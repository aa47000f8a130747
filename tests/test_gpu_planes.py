"""Projections on bf16 hi/lo planes, few-row attention on packed query vectors, packed prefill chunks
and runs of spans in the persistent attention, at the sizes where a tile, a row group or a run
ends, against the CPU oracle.

Tolerance: an activation enters a product as hi + lo with a relative error of at most 2^-17, so a
projected value is off by about 2^-17 of its terms' root sum of squares; over one layer's five
projections and the head that is below 1e-4 of logits of about 0.5 here.  1e-3 leaves room for
the largest of some 10^5 logits and still fails for a lost `lo` plane (2^-9), which would show
as 2e-3 or more."""
import pytest

from sd2_inputs.configs import Dims, Workload

pytestmark = pytest.mark.gpu

TOL = 1e-3
# 3 query heads per KV head and head dim 64 / 4 and head dim 32; 63 vocabulary tiles, so the last
# pair of sub-tiles is half empty; K of 768, 512, 1280: odd numbers of K steps.  Neither model
# suits the persistent path.
VER = Dims(1, 768, 12, 4, 1280, 1008, 5e5)
DRF = Dims(1, 512, 16, 4, 768, 1008, 5e5)


def _run(expect_path=0, **kw):
    from gpu_harness import parity_run
    seqs = kw.pop("seqs", None)
    wl = Workload(**dict(dict(name="planes", verifier=VER, drafter=DRF, dtype="bf16", temperature=1.0), **kw))
    st = parity_run(wl, expect_path=expect_path, seqs=seqs)
    assert st.pinned > 0
    assert max(st.max_err_v, st.max_err_d, st.max_err_s) <= TOL


@pytest.mark.parametrize("batch,k", [(1, 15), (1, 16), (4, 7), (3, 10), (4, 15), (5, 12), (16, 7), (13, 9), (16, 15)])
def test_verify_rows_at_row_group_edges(batch, k):
    # 16, 17, 32, 33, 64, 65, 128, 130 and 256 verify rows; 1 to 32 drafter rows
    _run(batch=batch, k=k, prompt=(1, 40), new_tokens=k + 2, seed=51 + batch * k, seqs=sorted({0, batch // 2, batch - 1}))


@pytest.mark.parametrize("k", [4, 5, 10])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 64, 65, 128, 129, 400])
def test_few_row_attention_at_tile_and_span_edges(n, k):
    # 15, 18 and 33 query vectors per KV head: one column tile not quite full, two, three
    _run(batch=2, k=k, prompt=(n, n), new_tokens=k + 1, seed=70 + n)


# head dim 128 and one query head per KV head in both models
VER128 = Dims(1, 1024, 8, 8, 1280, 1008, 5e5)
DRF128 = Dims(1, 512, 4, 4, 768, 1008, 5e5)


@pytest.mark.parametrize("k", [4, 14])
def test_few_row_attention_head_dim_128_one_head_per_kv_head(k):
    # 5 and 15 verify rows, 1 and 2 drafter rows: column tiles that rows alone leave partly empty
    _run(verifier=VER128, drafter=DRF128, batch=2, k=k, prompt=(250, 300), new_tokens=8, seed=91)


def test_many_row_attention_head_dim_128_verify_rows():
    # 17 verify rows, one more than a row block, over several spans
    _run(verifier=VER128, drafter=DRF128, batch=2, k=16, prompt=(250, 300), new_tokens=8, seed=91)


def test_packed_prefill_ragged():
    # a workspace above the static one: chunks of 2048 rows over five prompts, packed, the last
    # chunk with few rows of few prompts, some prompts shorter than one chunk
    _run(verifier=Dims(1, 1024, 8, 8, 2048, 1008, 5e5), drafter=Dims(1, 512, 8, 8, 1024, 1008, 5e5), batch=5, k=3,
         prompt=(1, 900), new_tokens=5, seed=101)


def test_packed_prefill_one_and_two_token_prompts():
    # no row, or one, of most prompts (16 prompts of 1 or 2 tokens beside the capacity of a long one)
    _run(verifier=Dims(1, 1024, 8, 8, 2048, 1008, 5e5), drafter=Dims(1, 512, 8, 8, 1024, 1008, 5e5), batch=16, k=3,
         prompt=(1, 2), new_tokens=300, seed=103, seqs=[0, 5, 11])


def test_persistent_attention_runs_of_several_spans():
    # 24 (verify) and 16 (drafter) groups over up to 36 spans: runs of 4 and 3 spans, the last one short
    _run(verifier=Dims(1, 2048, 16, 4, 1024, 1024, 5e5), drafter=Dims(1, 1024, 16, 8, 1024, 1024, 5e5), batch=2, k=5,
         prompt=(1500, 2300), new_tokens=12, seed=107, expect_path=1)
