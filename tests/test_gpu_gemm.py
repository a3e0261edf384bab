"""GPU parity of the bf16 GEMM's tiles (gl_linear) against the CPU oracle, at
the sizes where each can go wrong: one row or column past a tile, a partial or
a single K stage, rows of the output or residual that are not 16-byte aligned,
the residual updated in place."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import check_close, from_dev, require_gpu, to_dev
from paper_2604_21290_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [
    # label, R, K, Cout, act_out, residual, bias, offset of out and residual in elements
    ("128x128_one_row_past", 128 * 191 + 1, 72, 250, 1, True, True, 0),
    ("128x128_whole_stage", 128 * 192, 64, 256, 0, True, False, 0),
    ("128x128_short_last_tile", 128 * 400 - 3, 136, 80, 0, True, True, 0),
    ("128x64_padding_rule", 128 * 200 + 5, 80, 160, 0, True, True, 0),
    ("128x64_three_column_tiles", 128 * 127 + 65, 200, 136, 1, False, True, 0),
    ("128x64_residual", 128 * 383 + 1, 8, 64, 0, True, True, 0),
    ("64x64_ragged", 641, 136, 776, 1, True, True, 0),
    ("64x64_unaligned_out", 1300, 192, 448, 0, True, True, 1),
    ("64x64_aligned_8_bytes", 1300, 64, 456, 0, True, False, 4),
    ("64x64_long_k", 1999, 520, 257, 0, True, True, 0),
    ("64x64_long_k_gelu", 2208, 976, 264, 1, False, True, 0),
    ("64x64_long_k_two_per_cu", 64 * 32 - 3, 520, 64 * 16 - 8, 0, True, True, 0),
    ("64x64_past_two_per_cu", 64 * 32 + 1, 520, 64 * 16, 0, False, True, 0),
    ("128x64_padded_second_round", 128 * 171 + 1, 40, 320, 0, True, True, 0),
    ("128x64_gelu_second_round", 128 * 257, 24, 256, 1, False, True, 0),
    ("128x128_second_round", 128 * 257, 24, 256, 0, True, True, 0),
    # layers that are staged through registers, and their neighbours that are not
    ("registers_16_rows_gelu", 16, 640, 200, 1, False, True, 0),
    ("17_rows_gelu", 17, 640, 200, 1, False, True, 0),
    ("16_rows_gelu_long_k", 16, 648, 200, 1, False, True, 0),
    ("registers_odd_residual", 1000, 256, 157, 0, True, True, 1),
    ("odd_residual_long_k", 1000, 264, 157, 0, True, True, 1),
    ("registers_odd_many_rows", 20000, 128, 20, 0, False, True, 0),
    ("odd_many_rows_long_k", 20000, 136, 20, 0, False, True, 0),
    ("registers_few_columns", 32768, 96, 56, 0, True, True, 0),
    ("registers_half_stage_gelu", 20000, 88, 128, 1, False, True, 0),
    ("whole_stage_gelu", 20000, 64, 128, 1, False, True, 0),
    ("32x64_ragged", 33, 264, 65, 0, True, True, 0),
    ("32x64_two_k_stages", 65, 128 + 8, 72, 1, False, True, 0),
    ("32x64_one_element", 1, 8, 1, 0, True, True, 0),
    # rows of every alignment: 2, 4 and 8 bytes, out and residual at an odd element
    ("128x128_odd_rows_unaligned", 128 * 192 + 7, 40, 255, 0, True, True, 3),
    ("128x128_even_rows", 128 * 192 - 9, 104, 250, 1, False, True, 2),
    ("128x64_odd_rows_unaligned", 128 * 200 + 5, 80, 157, 0, True, True, 5),
    ("64x64_odd_rows_unaligned", 1300, 192, 443, 1, True, True, 7),
    ("64x64_whole_rows_unaligned", 1300, 192, 448, 0, True, True, 5),
    ("32x64_odd_rows", 333, 200, 61, 0, True, True, 1),
    ("32x64_seven_columns", 40, 64, 7, 0, True, False, 3),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_bf16_tiles(case):
    require_gpu()
    from paper_2604_21290_amd import api
    label, R, K, Co, act, with_res, with_bias, off = case
    g = np.random.default_rng(R + 3 * K + Co)
    x = I.store(g.standard_normal((R, K)), I.BF16)
    W = I.store(g.uniform(-1, 1, (Co, K)) / np.sqrt(K), I.BF16)
    b = I.store(g.uniform(-0.5, 0.5, Co), I.BF16) if with_bias else None
    r = I.store(g.standard_normal((R, Co)), I.BF16) if with_res else None
    print("[gpu-test] gemm", label, flush=True)
    guard = torch.full((R * Co + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = guard[off:off + R * Co].view(R, Co)
    if with_res:
        out.copy_(to_dev(r))  # the residual, updated in place
    api.linear(to_dev(x), to_dev(W), None if b is None else to_dev(b), 0, act,
               out if with_res else None, out=out)
    torch.cuda.synchronize()
    lin = O.linear_ref(x.value, W.value, None if b is None else b.value)
    ref = O.gelu_ref(lin) if act else lin
    mag = np.abs(x.value) @ np.abs(W.value).T + (np.abs(b.value) if b is not None else 0.0)
    if r is not None:
        ref, mag = ref + r.value, mag + np.abs(r.value)
    # one rounding of the output and a K-term fp32 sum (GELU's slope is below 1.13)
    check_close(from_dev(out).value, ref, I.BF16, label, mag=1.13 * mag, n_terms=K)
    rest = torch.cat([guard[:off], guard[off + R * Co:]])
    assert bool((rest == 7.0).all()), (label, "wrote past the output")


def _at_end(t):
    """t's values at the end of a device allocation of its own (whole 2 MiB, so that
    nothing is mapped by it past the tensor)."""
    n = t.numel() * t.element_size()
    buf = torch.empty((n // (32 << 20) + 1) * (32 << 20), dtype=torch.uint8, device="cuda")
    v = buf[buf.numel() - n:].view(t.dtype).view(t.shape)
    assert v.data_ptr() % 16 == 0
    v.copy_(t)
    return v


@pytest.mark.parametrize("dt", [I.BF16, I.F32])
@pytest.mark.parametrize("K", [8, 40, 72, 96, 104, 136, 192, 200, 264, 520])
def test_reads_end_with_the_operands(K, dt):
    """A and W at the end of their allocations, contractions shorter than a stage and
    with a partial last one: with and without a GELU on A, many rows and few."""
    require_gpu()
    from paper_2604_21290_amd import api
    for R, Co in ((1, 40), (70, 136), (20000, 20)):
        g = np.random.default_rng(R + K)
        x = I.store(g.standard_normal((R, K)), dt)
        W = I.store(g.uniform(-1, 1, (Co, K)) / np.sqrt(K), dt)
        xd, Wd = _at_end(to_dev(x)), _at_end(to_dev(W))
        for act_in, act_out in ((0, 0), (1, 0), (0, 1)):
            print("[gpu-test] operands' ends", R, K, Co, dt, act_in, act_out, flush=True)
            out = api.linear(xd, Wd, None, act_in, act_out)
            torch.cuda.synchronize()
            ref = O.linear_ref(O.gelu_ref(x.value) if act_in else x.value, W.value)
            check_close(from_dev(out).value, O.gelu_ref(ref) if act_out else ref, dt,
                        f"{R} x {K} -> {Co} {act_in}{act_out}")
