"""Top-k selection of the sampling path over tied and partial chunks: the filtered
distributions of both LM heads against the definition applied to the GPU's own logits."""
from dataclasses import replace

import numpy as np
import pytest

import oracle.sampling as smp
from paper_2608_29748_amd import binding as B
from workloads import get, make_prompts, make_weights

from gpu_parity import engine_for
from test_gpu_sampling import check_dist, gpu_dist

pytestmark = pytest.mark.gpu


CAND_MAX = 2048   # logits that the selection of a chunk collects before it folds the whole chunk


def collected(z, top_k):
    """Logits of each 8192-logit chunk that reach the chunk's bound: every wave's bound is the
    top_k-th of its 64 lanes' largest keys (a larger logit, then a lower index, ranks first)."""
    rank = np.empty(len(z), np.int64)
    rank[np.lexsort((np.arange(len(z)), -z))] = np.arange(len(z))
    out = []
    for i0 in range(0, len(z), 8192):
        r = np.full(8192, len(z))                              # places past the end rank last
        r[: len(z[i0:i0 + 8192])] = rank[i0:i0 + 8192]
        lanes = np.sort(r.reshape(-1, 256).min(axis=0).reshape(4, 64), axis=1)
        out.append(int((rank[i0:i0 + 8192] <= lanes[:, top_k - 1].min()).sum()))
    return out


# vocab: part of one 8192-logit chunk, one chunk exactly, three with a 16-logit last one;
# same: every token's logit equals that of token (id % same), so each value occurs
# vocab / same times (0: all different)
@pytest.mark.parametrize("vocab,same,top_k", [(2048, 0, 20), (8192, 0, 64), (16400, 0, 20), (16400, 1, 20),
                                              (16400, 9, 64), (16400, 40, 20), (16400, 40, 1), (48, 0, 20),
                                              (16400, 4, 40)])   # the last: always more than CAND_MAX reach it
def test_filtered_distributions_with_ties(vocab, same, top_k):
    wl = get("mini-bf16", temperature=1.0, top_k=top_k, top_p=1.0, norm_init="perturbed")
    wl = wl.with_(target=replace(wl.target, vocab=vocab))
    W = make_weights(wl)
    if same:
        head = W["lm_head"]
        W["lm_head"] = np.ascontiguousarray(head[np.arange(vocab) % same])
    eng = engine_for(wl, W)
    eng.set_debug(3)
    eng.prefill(make_prompts(wl), wl.new_tokens)
    eng.spec_round()
    bk = wl.block_size
    for what, tl, ti, tp, rows in (("draft", B.RT_T_DRAFT_LOGITS, B.RT_T_DRAFT_DIST_IDS, B.RT_T_DRAFT_DIST_P, range(1, bk)),
                                   ("verify", B.RT_T_VERIFY_LOGITS, B.RT_T_VERIFY_DIST_IDS, B.RT_T_VERIFY_DIST_P, range(bk))):
        z = eng.read(tl, 0, (bk, vocab), np.float32)
        ids = eng.read(ti, 0, (bk, B.RT_MAX_TOP_K), np.int32)
        prb = eng.read(tp, 0, (bk, B.RT_MAX_TOP_K), np.float32)
        if same == 4:                                          # both full chunks overflow in every row
            assert all(n > CAND_MAX for i in rows for n in collected(z[i], top_k)[:2])
        if same == 0:                                          # none does, up to the largest top_k
            assert all(n <= CAND_MAX for i in rows for n in collected(z[i], top_k))
        for i in rows:
            g = gpu_dist(ids[i], prb[i])
            check_dist(g, z[i].astype(np.float64), wl, f"{what} row {i}")
            order = np.lexsort((np.arange(vocab), -z[i]))[:top_k]
            if len(g.ids) == top_k:      # top_p = 1 may drop a tail of fp32-zero weight only
                assert list(g.ids) == list(order), f"{what} row {i}"
    eng.close()
