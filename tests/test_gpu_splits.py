"""Rounds of ragged batches whose attention shares fewer workgroups than whole splits per
sequence, uses more of them than one pass of the chip holds, or writes one-split sequences
without a merge; of batches on either side of the page-wise q|k|v post-processing; and fp32
prompts in two passes of at most 32 rows."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import OracleModel, OracleRunner
from paper_2608_29748_amd import binding as B
from workloads import get, make_weights

from gpu_parity import compare_prefill, engine_for, log, run_teacher_forced
from test_gpu_prefill import check_first

pytestmark = pytest.mark.gpu


def teacher_forced(eng, wl, W, prompts, prefill=False):
    tol = {"f32": 1e-4, "bf16": 2e-2}[wl.dtype]
    R = OracleRunner(OracleModel(wl, W))
    first = eng.prefill(prompts, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in prompts]
    check_first(first, R, prompts, states, tol)
    if prefill:
        compare_prefill(eng, R, wl, prompts, states, tol)
    for f, st in zip(first, states):   # (at a near-tie both go on from the GPU's token)
        st.anchor, st.generated = int(f), [int(f)]
    rep = run_teacher_forced(eng, R, wl, states, 3, tol, stages={})
    log(f"[{wl.name} {wl.batch} x {wl.block_size}] rounds max err {rep.max_err}")
    eng.close()


# one long context among short ones: 32 of 40 slots hold it at 20 sequences, 62 are shared out
# at 31 (32 would leave two for it); 25 slots of three sequences, 3 x 9 in whole splits
@pytest.mark.parametrize("batch,block,kv_heads,head_dim,slots", [
    (20, 3, 8, 128, 40), (31, 2, 8, 128, 62), (3, 16, 10, 128, 25), (20, 3, 8, 64, 40), (31, 2, 8, 64, 62)])
def test_ragged_rounds_with_shared_slots_match_oracle(batch, block, kv_heads, head_dim, slots):
    lens = [1150] + [5 + 3 * i for i in range(batch - 1)]
    wl = get("mini-bf16", norm_init="perturbed", batch=batch, block_size=block, prompt_len=(5, 1150), new_tokens=30)
    wl = wl.with_(target=replace(wl.target, n_layers=2, n_q_heads=2 * kv_heads, n_kv_heads=kv_heads,
                                 head_dim=head_dim), cond_layers=(0, 1), draft_layers=1)
    W = make_weights(wl)
    rng = np.random.default_rng(9)
    prompts = [rng.integers(0, wl.target.vocab // 2, size=n).astype(np.int32) for n in lens]
    eng = engine_for(wl, W)
    assert B.rt_debug_choice(eng.cfg, B.RT_C_ATTN_SLOTS, batch, block) == slots
    teacher_forced(eng, wl, W, prompts)


# by row: too few rows of a page in use, or too few rows; by page: 5 rows (pages crossed), 16
@pytest.mark.parametrize("name,batch,block,by_page", [
    ("mini-bf16", 50, 2, 0), ("mini-bf16", 20, 5, 1), ("tiny-f32", 11, 16, 0), ("tiny-f32", 12, 16, 1)])
def test_rounds_by_row_and_by_page_match_oracle(name, batch, block, by_page):
    wl = get(name, norm_init="perturbed", batch=batch, block_size=block, prompt_len=(5, 60), new_tokens=30)
    W = make_weights(wl)
    rng = np.random.default_rng(10)
    prompts = [rng.integers(0, wl.target.vocab // 2, size=5 + i % 40).astype(np.int32) for i in range(batch)]
    eng = engine_for(wl, W)
    assert B.rt_debug_choice(eng.cfg, B.RT_C_PAGE_POST, batch, block) == by_page
    teacher_forced(eng, wl, W, prompts)


# passes cut inside a sequence and a page; on a sequence's end; one prompt of both passes
@pytest.mark.parametrize("lens", [(30, 30), (20, 12, 13), (33,), (64,), (1, 40, 2)])
def test_fp32_prompts_of_two_small_passes_match_oracle(lens):
    wl = get("tiny-f32", norm_init="perturbed", batch=len(lens), prompt_len=(min(lens), max(lens)), new_tokens=30)
    W = make_weights(wl)
    rng = np.random.default_rng(11)
    prompts = [rng.integers(0, wl.target.vocab // 2, size=n).astype(np.int32) for n in lens]
    eng = engine_for(wl, W)
    assert B.rt_debug_choice(eng.cfg, B.RT_C_PROMPT_ROWS, sum(lens)) == 32
    teacher_forced(eng, wl, W, prompts, prefill=True)
