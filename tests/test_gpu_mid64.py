"""Rounds of 33..64 rows on the mid-size GEMM's 64-row tiles: 96-column gate|up tiles and
128-column LM-head tiles with a remainder, o / down k slabs, fp32-operand conditioning; and
rounds of more than 512 rows, on the tiles of the prompt passes."""
from dataclasses import replace

import pytest

from oracle import OracleModel, OracleRunner
from workloads import get, make_prompts, make_weights

from gpu_parity import engine_for, log, run_teacher_forced
from test_gpu_prefill import check_first

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,block,ffn,vocab", [
    (3, 16, 6176, 20496),     # 48 rows; 12352 gate|up columns (128.7 tiles of 96), 160.1 tiles of 128
    (4, 16, 6144, 2048),      # 64 rows; exactly 128 tiles of 96 columns, 64-column LM-head tiles
    (3, 11, 6128, 20480),     # 33 rows; 12256 columns stay on the 32-column kernel
    (33, 16, 512, 2048),      # 528 rows: three 256-row tiles, the last of 16 rows
])
def test_rounds_by_row_count_match_oracle(batch, block, ffn, vocab):
    wl = get("mini-bf16", norm_init="perturbed", batch=batch, block_size=block, prompt_len=(30, 70), new_tokens=40)
    wl = wl.with_(target=replace(wl.target, ffn=ffn, vocab=vocab, n_layers=2), cond_layers=(0, 1), draft_layers=1)
    W = make_weights(wl)
    prompts = make_prompts(wl)
    eng = engine_for(wl, W)
    R = OracleRunner(OracleModel(wl, W))
    first = eng.prefill(prompts, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in prompts]
    check_first(first, R, prompts, states, 2e-2)
    for f, st in zip(first, states):   # (at a near-tie both go on from the GPU's token)
        st.anchor, st.generated = int(f), [int(f)]
    rep = run_teacher_forced(eng, R, wl, states, 3, 2e-2, stages={})
    log(f"[{batch} x {block}] rounds max err {rep.max_err}")
    eng.close()
