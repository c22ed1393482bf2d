"""Rounds of 33..64 rows on the mid-size GEMM's 64-row tiles: 96-column gate|up tiles and
128-column LM-head tiles with a remainder, o / down k slabs, fp32-operand conditioning; rounds
of more than 512 rows; and the wide tiles of prompt passes and large LM heads over several row
tiles, every row compared."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import OracleModel, OracleRunner
from paper_2608_29748_amd import binding as B
from workloads import get, make_prompts, make_weights

from gpu_parity import compare_prefill, engine_for, log, run_teacher_forced
from test_gpu_prefill import check_first
from test_gpu_round import _exact

pytestmark = pytest.mark.gpu


# (rows, ffn, vocab): columns per workgroup of the gate|up GEMM and of the LM head
GEMM_COLS = {(48, 8224, 20496): (96, 128), (64, 8208, 2048): (96, 64), (48, 6176, 20496): (64, 128),
             (64, 6144, 2048): (64, 64), (33, 6128, 20480): (0, 128),
             (528, 512, 2048): (64, 64), (528, 9744, 2048): (256, 64), (528, 8000, 2048): (192, 64),
             (528, 6704, 2048): (160, 64), (528, 512, 40976): (64, 256)}


@pytest.mark.parametrize("batch,block,ffn,vocab", [
    (3, 16, 8224, 20496),     # 48 rows; 16448 gate|up columns (171.3 tiles of 96), 160.1 tiles of 128
    (4, 16, 8208, 2048),      # 64 rows; exactly 171 tiles of 96 columns, 64-column LM-head tiles
    (3, 16, 6176, 20496),     # 12352 columns: 193 tiles of 64
    (4, 16, 6144, 2048),      # 12288 columns, the fewest on this kernel
    (3, 11, 6128, 20480),     # 33 rows; 12256 columns stay on the 32-column kernel
    (33, 16, 512, 2048),      # 528 rows: three 256-row tiles of 64 columns, the last of 16 rows
    # the same rows on wide tiles, with a column remainder: gate|up of 256 (76.1 tiles), 192
    # (83.3) and 160 columns (83.8); a vocabulary of 160.1 tiles of 256 over three row tiles
    (33, 16, 9744, 2048), (33, 16, 8000, 2048), (33, 16, 6704, 2048), (33, 16, 512, 40976),
])
def test_rounds_by_row_count_match_oracle(batch, block, ffn, vocab):
    rows = batch * block
    gate_up, lm_head = GEMM_COLS[rows, ffn, vocab]
    wl = get("mini-bf16", norm_init="perturbed", batch=batch, block_size=block, prompt_len=(30, 70), new_tokens=40)
    # The wide tiles' cases are 512 wide: every step of a layer, their SwiGLU rows among them, is
    # held to 2e-2 from the GPU's own operands, and the final states, whose rounding noise after
    # 8000 FFN columns reaches 2e-2 (0.0244 measured at 256 wide), to the bound that `_exact` gives
    # from that width on: twice the mixed-precision oracle's own distance from 64 bits.
    hidden = 512 if rows > 512 and (ffn > 512 or vocab > 2048) else 256
    wl = wl.with_(target=replace(wl.target, hidden=hidden, ffn=ffn, vocab=vocab, n_layers=2), cond_layers=(0, 1),
                  draft_layers=1)
    W = make_weights(wl)
    prompts = make_prompts(wl)
    eng = engine_for(wl, W)
    assert B.rt_debug_choice(eng.cfg, B.RT_C_GEMM_COLS, rows, B.RT_K_GEMM_GATE_UP) == gate_up
    assert B.rt_debug_choice(eng.cfg, B.RT_C_GEMM_COLS, rows, B.RT_K_LM_HEAD) == lm_head
    R = OracleRunner(OracleModel(wl, W))
    first = eng.prefill(prompts, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in prompts]
    check_first(first, R, prompts, states, 2e-2)
    for f, st in zip(first, states):   # (at a near-tie both go on from the GPU's token)
        st.anchor, st.generated = int(f), [int(f)]
    rep = run_teacher_forced(eng, R, wl, states, 3, 2e-2, exact=_exact(wl, W, R), stages={})
    log(f"[{batch} x {block}] rounds max err {rep.max_err}")
    eng.close()


def test_wide_prompt_tiles_match_oracle():
    """A pass of 4000 rows (the last row tile of 160 rows) at the 4B attention widths: q|k|v on
    192-column tiles, o and down added to the residual from 160-column tiles, whose error the
    next layer's cached keys and values show for every row."""
    wl = get("mini-bf16", norm_init="perturbed", batch=20, prompt_len=(150, 250), new_tokens=12)
    wl = wl.with_(target=replace(wl.target, hidden=2560, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn=512,
                                 vocab=2048, n_layers=2), cond_layers=(0, 1), draft_layers=1)
    W = make_weights(wl)
    rng = np.random.default_rng(12)
    lens = [153 + 5 * i for i in range(20)]
    lens[-1] += 4000 - sum(lens)
    prompts = [rng.integers(0, wl.target.vocab // 2, size=n).astype(np.int32) for n in lens]
    eng = engine_for(wl, W)
    cols = {k: B.rt_debug_choice(eng.cfg, B.RT_C_GEMM_COLS, 4000, k)
            for k in (B.RT_K_GEMM_QKV, B.RT_K_GEMM_O, B.RT_K_GEMM_DOWN)}
    assert cols == {B.RT_K_GEMM_QKV: 192, B.RT_K_GEMM_O: 160, B.RT_K_GEMM_DOWN: 160}
    R = OracleRunner(OracleModel(wl, W))
    first = eng.prefill(prompts, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in prompts]
    check_first(first, R, prompts, states, 2e-2)
    rep = compare_prefill(eng, R, wl, prompts, states, 2e-2)
    log(f"[wide prompt tiles] max err {rep.max_err}")
    eng.close()
