"""The GEMM over many token rows (prompt passes) at the edges of its tiles: 256 matrix rows x 32, 64 or 128 token rows
per work-group, with and without split k ranges, against the same library's 16-row passes (other kernels)."""
import numpy as np
import pytest

from synthdata import gen_prompt, get_config

pytestmark = pytest.mark.gpu

LENGTHS = [1, 16, 17, 31, 33, 64, 65, 127, 129, 200]


@pytest.mark.parametrize("form", ["0", "1"])       # 1: no k range is split
@pytest.mark.parametrize("name", ["mini_gqa", "mini_mha", "wide_d4096"])
def test_every_prompt_length_gives_the_rows_of_the_short_passes(name, form, monkeypatch):
    from gpu_harness import gpu_context
    cfg = get_config(name)
    monkeypatch.setenv("DEL_WIDE_FORM", form)
    wide, _ = gpu_context(cfg, max_context=max(LENGTHS) + 2)
    monkeypatch.setenv("DEL_PREFILL_ROWS", "0")
    short, _ = gpu_context(cfg, max_context=max(LENGTHS) + 2)
    for plen in LENGTHS:
        prompt = gen_prompt(cfg, length=plen).tolist()
        wide.prefill(prompt)
        short.prefill(prompt)
        for l in range(1, cfg.n_layers + 1):
            for i in range(min(plen, short.last_rows())):
                a, b = wide.hidden(l, wide.last_rows() - 1 - i), short.hidden(l, short.last_rows() - 1 - i)
                # Both sides multiply 16-bit weights by activations kept to 16 mantissa bits.  They differ in the order
                # of sums, and where that moves a key or value across a rounding boundary of the 16-bit cache (2^-9 of
                # that value, a few per row out of thousands): 1e-3 of the row's 2-norm, as for the other passes
                # (measured against the 64-bit result: up to 6e-4).
                assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b), (name, form, plen, l, i)
    wide.close()
    short.close()


@pytest.mark.parametrize("rows,plen", [(32, 131), (48, 203), (144, 431), (1024, 300)])
@pytest.mark.parametrize("name", ["mini_gqa", "mini_mha", "mini_g8"])
def test_prompt_attention_on_a_filled_cache(name, rows, plen, monkeypatch):
    """Passes of `rows` token rows that start at cache lengths off the 64-row stages and 128-row blocks of the prompt
    attention, one, four and eight query heads per kv head, head widths 64 and 128."""
    from gpu_harness import gpu_context
    cfg = get_config(name)
    monkeypatch.setenv("DEL_PREFILL_ROWS", str(rows))
    wide, _ = gpu_context(cfg, max_context=plen + 2)
    monkeypatch.setenv("DEL_PREFILL_ROWS", "0")
    short, _ = gpu_context(cfg, max_context=plen + 2)
    prompt = gen_prompt(cfg, length=plen).tolist()
    wide.prefill(prompt)
    short.prefill(prompt)
    for l in range(1, cfg.n_layers + 1):
        for i in range(short.last_rows()):
            a, b = wide.hidden(l, wide.last_rows() - 1 - i), short.hidden(l, short.last_rows() - 1 - i)
            assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b), (name, rows, plen, l, i)   # as above
    wide.close()
    short.close()
