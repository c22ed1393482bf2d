"""Prompt passes over several sequences: prompts laid end to end, passes of equal rows that
start and end inside sequences and inside KV pages, and the first tokens of every pass."""
import numpy as np
import pytest

from oracle import OracleModel, OracleRunner
from workloads import get, make_weights

from gpu_parity import compare_prefill, engine_for, log

pytestmark = pytest.mark.gpu


def check_first(first, R, prompts, states, tol):
    """First tokens: the oracle's, or at a near-tie one whose oracle logit is within 2 tol of
    the largest (each logit may be off by tol)."""
    for f, p, st in zip(first, prompts, states):
        if int(f) != st.anchor:
            z = R.m.target_forward(R.m.new_state(p, 4), p, 0).logits[-1]
            assert z[int(f)] >= z[st.anchor] - 2 * tol, (int(f), st.anchor)


@pytest.mark.parametrize("name,lens,cond", [
    ("mini-bf16", (1, 15, 16, 17, 255, 1500, 130, 2300, 33), None),    # two passes, cut inside a page
    ("mini-bf16-gqa5", (700, 3500, 20), None),                          # hd 128, blocks of 12.8 tokens
    ("mini-bf16-odd", (40, 21, 500, 80), None),                         # 641 rows: k slabs above 512 rows
    ("mini-bf16-b4", (600, 2, 1, 900), None),                           # slabs folded by the norm, 1503 rows
    ("tiny-f32", (3, 2000, 2100, 40), None),                            # fp32 kernels, two passes
    # the drafter does not read the last layer: it runs for the ending sequences' last rows
    ("mini-bf16", (1, 15, 16, 17, 255, 1500, 130, 2300, 33), (0, 1)),   # its input norm captures layer 1
    ("mini-bf16-gqa5", (4500, 20, 51), (0,)),                           # a first pass in which none ends
    ("mini-bf16-b4", tuple(range(5, 45)), (0,)),                        # forty ending rows
    ("tiny-f32", (3, 2000, 2100, 40), (0,)),
])
def test_ragged_prompts_in_shared_passes_match_oracle(name, lens, cond):
    wl = get(name, norm_init="perturbed", batch=len(lens), prompt_len=(min(lens), max(lens)), new_tokens=12)
    if cond is not None:
        wl = wl.with_(cond_layers=cond)
    W = make_weights(wl)
    rng = np.random.default_rng(5)
    prompts = [rng.integers(0, wl.target.vocab // 2, size=n).astype(np.int32) for n in lens]
    eng = engine_for(wl, W)
    R = OracleRunner(OracleModel(wl, W))
    tol = {"f32": 1e-4, "bf16": 2e-2}[wl.dtype]
    first = eng.prefill(prompts, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in prompts]
    check_first(first, R, prompts, states, tol)
    rep = compare_prefill(eng, R, wl, prompts, states, tol)
    log(f"[{name} {len(lens)} prompts] prefill max err {rep.max_err}")
    # a second, shorter prefill on the same handle: stale rows of the first stay unseen
    short = [p[: max(1, len(p) // 3)] for p in prompts[::-1]]
    first = eng.prefill(short, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in short]
    check_first(first, R, short, states, tol)
    compare_prefill(eng, R, wl, short, states, tol)
    eng.close()


def test_captured_round_serves_later_prefills():
    """The captured round and target-only step are kept from one prefill to the next of the
    same batch: results equal a fresh handle's, also after batches of other sizes."""
    wl = get("mini-bf16-ragged", norm_init="perturbed")
    W = make_weights(wl)
    rng = np.random.default_rng(6)
    sets = [[rng.integers(0, wl.target.vocab // 2, size=n).astype(np.int32) for n in lens]
            for lens in ((17, 70, 40), (66, 9, 21), (30, 31), (5, 60, 64))]
    eng = engine_for(wl, W)
    for prompts in sets:
        for steps in (False, True):
            ref = engine_for(wl, W)
            assert list(eng.prefill(prompts, 30)) == list(ref.prefill(prompts, 30))
            for _ in range(2):
                got, want = (eng.ar_steps(3), ref.ar_steps(3)) if steps else (eng.spec_round(), ref.spec_round())
                for a, b in zip(got, want):
                    assert np.array_equal(a, b)
            ref.close()
    eng.close()
