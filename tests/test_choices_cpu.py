"""Launch choices that follow from a configuration alone, through rt_debug_choice (no GPU)."""
import pytest

from paper_2608_29748_amd import binding as B


def cfg(**over):
    """The Qwen3-4B layer widths."""
    base = dict(vocab=2048, hidden=2560, n_layers=2, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn=9728,
                rope_theta=1e6, rms_eps=1e-6, draft_layers=1, cond_layer_ids=[0, 1], block_size=16,
                mask_token_id=2047, beta=1.0, cond_mode=B.RT_COND_RETRACE, dtype=B.RT_BF16, max_batch=1,
                max_seq_len=8400, page_size=16)
    base.update(over)
    return B.make_config(**base)


def test_choice_arguments_are_checked():
    c = cfg(max_batch=2)
    for args in ((99, 1, 16), (B.RT_C_ATTN_SLOTS, 0, 16), (B.RT_C_ATTN_SLOTS, 3, 16), (B.RT_C_ATTN_SLOTS, 1, 5)):
        with pytest.raises(B.RetraceError):
            B.rt_debug_choice(c, *args)


# bf16 handles of at most 64 round rows: 129..255 (sequence, KV head) pairs keep two slots a
# sequence, so that a long context among short ones can be shared out; with two slots or more
# per sequence in one pass of 256 workgroups, no more than that
@pytest.mark.parametrize("batch,block,head_dim,slots", [
    (20, 3, 128, 40), (17, 3, 128, 34), (31, 2, 128, 62), (32, 2, 128, 32), (20, 3, 64, 40),
    (3, 16, 128, 32), (11, 5, 128, 32), (1, 16, 128, 32), (3, 16, 64, 32), (3, 20, 128, 32),
    (10, 16, 128, 40),                                        # 160 rows: whole splits
])
def test_attention_slots(batch, block, head_dim, slots):
    c = cfg(max_batch=batch, block_size=block, head_dim=head_dim)
    assert B.rt_debug_choice(c, B.RT_C_ATTN_SLOTS, batch, block) == slots
    # target-only steps of the same handle
    assert B.rt_debug_choice(c, B.RT_C_ATTN_SLOTS, batch, 1) == slots
    # fp32 storage keeps whole splits; so does one sequence, at most one pass of them
    units = batch * -(-4 * block // 64)
    assert B.rt_debug_choice(cfg(max_batch=batch, block_size=block, dtype=B.RT_F32), B.RT_C_ATTN_SLOTS, batch,
                             block) == units * -(-256 // (8 * units))
    one = cfg(max_batch=1, n_q_heads=24, n_kv_heads=24)
    assert B.rt_debug_choice(one, B.RT_C_ATTN_SLOTS, 1, 16) == 10


# pages of five rows or more in use, and enough rows: 96 in bf16, 192 in fp32
@pytest.mark.parametrize("dtype,batch,block,by_page", [
    (B.RT_BF16, 6, 16, 1), (B.RT_BF16, 5, 16, 0), (B.RT_BF16, 20, 5, 1), (B.RT_BF16, 24, 4, 0),
    (B.RT_BF16, 128, 2, 0), (B.RT_F32, 12, 16, 1), (B.RT_F32, 11, 16, 0), (B.RT_F32, 64, 4, 0)])
def test_qkv_post_by_page(dtype, batch, block, by_page):
    c = cfg(dtype=dtype, max_batch=256, block_size=block)
    assert B.rt_debug_choice(c, B.RT_C_PAGE_POST, batch, block) == by_page
    for n in (1, 96, 256):                                    # target-only steps: one row a page
        assert B.rt_debug_choice(c, B.RT_C_PAGE_POST, n, 1) == 0


@pytest.mark.parametrize("dtype,total,rows", [
    (B.RT_F32, 32, 256), (B.RT_F32, 33, 32), (B.RT_F32, 60, 32), (B.RT_F32, 64, 32), (B.RT_F32, 65, 256),
    (B.RT_BF16, 60, 256), (B.RT_BF16, 4096, 4096), (B.RT_BF16, 4097, 2304), (B.RT_BF16, 9000, 3072)])
def test_prompt_rows_per_pass(dtype, total, rows):
    c = cfg(dtype=dtype, max_batch=4)
    assert B.rt_debug_choice(c, B.RT_C_PROMPT_ROWS, total) == rows
    for bad in (0, 4 * 8400 + 1):
        with pytest.raises(B.RetraceError):
            B.rt_debug_choice(c, B.RT_C_PROMPT_ROWS, bad)


# columns per workgroup over the rows of a prompt pass (LM head: a round); 0: not the mid-size kernel
@pytest.mark.parametrize("kind,rows,cols", [
    (B.RT_K_GEMM_QKV, 32, 0), (B.RT_K_GEMM_QKV, 64, 0), (B.RT_K_GEMM_QKV, 4096, 192),
    (B.RT_K_GEMM_GATE_UP, 32, 0), (B.RT_K_GEMM_GATE_UP, 48, 96), (B.RT_K_GEMM_GATE_UP, 128, 96),
    (B.RT_K_GEMM_GATE_UP, 512, 160), (B.RT_K_GEMM_GATE_UP, 4096, 256), (B.RT_K_GEMM_O, 4096, 160),
    (B.RT_K_GEMM_DOWN, 48, 64), (B.RT_K_GEMM_DOWN, 4096, 160), (B.RT_K_LM_HEAD, 32, 0), (B.RT_K_LM_HEAD, 33, 128),
    (B.RT_K_LM_HEAD, 129, 256)])
def test_gemm_columns(kind, rows, cols):
    c = cfg(vocab=151936, mask_token_id=151935, max_batch=32)
    assert B.rt_debug_choice(c, B.RT_C_GEMM_COLS, rows, kind) == cols
    assert B.rt_debug_choice(cfg(dtype=B.RT_F32), B.RT_C_GEMM_COLS, min(rows, 4096), kind) == 0
    for bad in ((0, kind), (4097, kind), (rows, B.RT_K_ATTENTION)):
        with pytest.raises(B.RetraceError):
            B.rt_debug_choice(c, B.RT_C_GEMM_COLS, *bad)
