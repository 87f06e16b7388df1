"""GPU parity of bf16 attention plans whose items take more than one round of
workgroups (the planner deals them out, balanced_ring_kernel runs them),
against the fp64 oracle."""

import numpy as np
import pytest
import torch

from oracle.attention import attention_for_batch
from paper_2607_18839_amd import _lib
from workloads.gen import attn_batch_from_structure

from ._gpu import announce, assert_parity, run_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# A shared item's row sums add probabilities rounded to bf16 (relative error at
# most 2^-9 each, all positive), so a log-sum-exp moves by at most ln(1 + 2^-9),
# which short prefixes come near (a long sum averages the roundings out); fp32
# products and sums add less than 1e-5.
LSE_BOUND = 2.0 ** -9 + 1e-5

# pages, longest prefix, branches per page, longest private history, query heads, kv heads
CASES = [(70, 150, 6, 40, 16, 8),      # more items than workgroups, none longer than two pairs of tiles
         (12, 2500, 24, 500, 16, 2),   # pieces of several pairs, several items per workgroup
         (9, 1500, 9, 700, 16, 8),     # G = 2
         (36, 500, 20, 130, 12, 2),    # G = 6: tokens cross row groups
         (6, 700, 60, 900, 4, 4),      # G = 1, mostly private items
         (1, 900, 120, 200, 64, 8)]    # one page


def structure(case, fork):
    pages, prefix_hi, branches, past_hi, _, _ = case
    rng = np.random.default_rng(17)
    prefix = rng.integers(1, prefix_hi + 1, pages)
    prefix[0] = prefix_hi
    if pages > 2:
        prefix[1] = 0
    page = np.repeat(np.arange(pages), rng.integers(1, branches + 1, pages) if pages > 1 else [branches])
    st = dict(prefix_len=prefix.astype(np.int32), branch_page=page.astype(np.int32),
              num_new=rng.integers(1, 6, len(page)).astype(np.int32),
              past_len=rng.integers(0, past_hi + 1, len(page)).astype(np.int32))
    if fork:
        st["fork_len"] = np.array([rng.integers(0, prefix[p] + 1) for p in page], np.int32)
    return st


@pytest.mark.parametrize("fork", [False, True], ids=["whole", "fork"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_more_than_one_round(case, fork):
    announce(f"rounds {case} fork {fork}")
    st = structure(case, fork)
    b = attn_batch_from_structure(st, *case[4:], 64, "bf16", 5)
    O, lse = run_batch(b, fork_len=st.get("fork_len"))
    Oref, lref = attention_for_batch(b)
    assert_parity(O, Oref, "bf16", f"rounds {case}")
    assert np.abs(lse - lref).max() <= LSE_BOUND


@pytest.mark.parametrize("fork", [False, True], ids=["whole", "fork"])
def test_phases_on_their_own(fork):
    """Phase isolation runs the same lists, each launch one kind of item: the same bits."""
    announce(f"rounds, phases on their own, fork {fork}")
    st = structure(CASES[1], fork)
    b = attn_batch_from_structure(st, *CASES[1][4:], 64, "bf16", 5)
    got = []
    try:
        for isolated in (False, True):
            _lib.hpd_attn_phase_isolation(isolated)
            got.append(run_batch(b, fork_len=st.get("fork_len")))
    finally:
        _lib.hpd_attn_phase_isolation(False)
    assert all(np.array_equal(x, y) for x, y in zip(*got))
