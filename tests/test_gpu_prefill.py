"""Prompt passes over several sequences: prompts laid end to end, passes of equal rows that
start and end inside sequences and inside KV pages, and the first tokens of every pass."""
import numpy as np
import pytest

from oracle import OracleModel, OracleRunner
from workloads import get, make_weights

from gpu_parity import compare_prefill, engine_for, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,lens", [
    ("mini-bf16", (1, 15, 16, 17, 255, 1500, 130, 2300, 33)),    # two passes, cut inside a page
    ("mini-bf16-gqa5", (700, 3500, 20)),                          # hd 128, 128-row blocks of 25.6 tokens
    ("mini-bf16-odd", (40, 21, 500, 80)),                         # 641 rows: k slabs above 512 rows
    ("mini-bf16-b4", (600, 2, 1, 900)),                           # slabs folded by the norm, 1503 rows
    ("tiny-f32", (3, 2000, 2100, 40)),                            # fp32 kernels, two passes
])
def test_ragged_prompts_in_shared_passes_match_oracle(name, lens):
    wl = get(name, norm_init="perturbed", batch=len(lens), prompt_len=(min(lens), max(lens)), new_tokens=12)
    W = make_weights(wl)
    rng = np.random.default_rng(5)
    prompts = [rng.integers(0, wl.target.vocab // 2, size=n).astype(np.int32) for n in lens]
    eng = engine_for(wl, W)
    R = OracleRunner(OracleModel(wl, W))
    first = eng.prefill(prompts, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in prompts]
    assert list(first) == [st.anchor for st in states]
    tol = {"f32": 1e-4, "bf16": 2e-2}[wl.dtype]
    rep = compare_prefill(eng, R, wl, prompts, states, tol)
    log(f"[{name} {lens}] prefill max err {rep.max_err}")
    # a second, shorter prefill on the same handle: stale rows of the first stay unseen
    short = [p[: max(1, len(p) // 3)] for p in prompts[::-1]]
    first = eng.prefill(short, wl.new_tokens)
    states = [R.prefill(p, wl.new_tokens) for p in short]
    assert list(first) == [st.anchor for st in states]
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
