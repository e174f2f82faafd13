"""The GPU tests of the forward's forms and of fp32 in two parts run the kernels that they are there for (no GPU needed)."""
import itertools

import pytest

import launch_choice
import test_gpu_column_shares as columns
import test_gpu_f32_two_parts as two_parts
import test_gpu_forward_forms as forms
import test_gpu_rows512 as rows512


@pytest.mark.parametrize("partial", [False, True])
@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp8qk_bf16v"])
@pytest.mark.parametrize("d", [64, 128])
def test_every_form_has_a_shape(d, dtype, counts, partial):
    """Whatever a launch may take, over a grid of sizes, one of the tested shapes takes too."""
    reached = {launch_choice.launched(h, h, nq, nk, d, dtype, counts, partial)
               for h, nq, nk in itertools.product((1, 2, 4, 8, 12, 20, 40, 64, 100, 200), (33, 64, 100, 300, 500, 999, 2000, 4000),
                                                  (60, 150, 300, 500, 700, 1000, 1300, 2000, 3000, 4600, 7000))}
    shapes = forms.SHAPES + [s[:5] for s in columns.SHAPES if dtype != "fp8qk_bf16v"]
    shapes += [(*s, 64) for s, t, c in rows512.CASES if (t, c) == (dtype, counts)]
    tested = {launch_choice.launched(H, H_kv, Nq, Nk, d, dtype, counts, partial) for H, H_kv, Nq, Nk, dd in shapes if dd == d}
    reached.discard(("Rows256", False))            # (fwd_pipelined_kernel has tests of its own)
    assert len(reached) >= (2 if dtype == "fp8qk_bf16v" and d == 128 else 4)
    assert reached <= tested, reached - tested


@pytest.mark.parametrize("H,N,d,name", [(8, 6000, 64, "Rows256"), (12, 5000, 64, "Rows256"), (20, 3000, 64, "Rows256"), (3, 20000, 64, "Rows256"),
                                        (32, 2048, 64, "Narrow"), (4, 8192, 64, "Narrow"), (4, 1999, 128, "Narrow"), (40, 4096, 64, "Rows256")])
def test_one_key_order_takes_the_faster_of_two(H, N, d, name):
    """Two workgroups of 128 rows on a CU lose 6 to 8 % against one of 256 on long key axes."""
    assert launch_choice.bf16_form_in_one_key_order(H, N, d) == name


@pytest.mark.parametrize("H,N,counts,name", [(80, 500, True, "Rows256"), (100, 500, True, "Rows256"), (128, 500, True, "Rows256"), (128, 500, False, "Rows256"),
                                             (50, 700, False, "Rows256"), (24, 2000, True, "Rows256Wide"), (12, 3000, False, "Rows256Wide")])
def test_fp8_short_key_axes_keep_256_rows(H, N, counts, name):
    """Two key groups pay there from 16 (with counts 25) key tiles on; below, 3 to 5 % were lost."""
    assert launch_choice.form(H, H, N, N, 64, "fp8qk_bf16v", counts)[0] == name


@pytest.mark.parametrize("H,N,name", [(2, 411, "Rows64"), (4, 831, "Rows64"), (9, 502, "Rows64"), (4, 1999, "Rows64Own")])
def test_counts_on_short_key_axes_keep_four_waves(H, N, name):
    """Four waves of d = 128 with counts start soonest: eight took 4 % longer on 7 to 13 key tiles."""
    assert launch_choice.form(H, H, N, N, 128, "bf16", True)[0] == name


@pytest.mark.parametrize("H,Nq,Nk,dtype,counts,taken", [
    (8, 32768, 32768, "bf16", False, True), (16, 16384, 16384, "f16", False, True), (9, 8192, 8192, "bf16", False, True),
    (32, 8192, 8192, "bf16", False, True), (20, 8192, 8192, "f16", True, True), (20, 8192, 8192, "fp8qk_bf16v", False, True),
    (22, 3432, 7940, "bf16", True, True), (229, 270, 72, "f16", False, True), (25, 2717, 200, "f16", True, True),
    (10, 7647, 21574, "f16", False, True), (35, 2036, 4845, "fp8qk_bf16v", False, True), (145, 313, 700, "bf16", True, True),
    (16, 11180, 11180, "fp8qk_bf16v", False, False), (10, 12127, 12127, "fp8qk_bf16v", False, False),   # past 128 key tiles: 3 to 6 % were lost
    (9, 11994, 11994, "fp8qk_bf16v", False, False), (20, 10795, 10795, "bf16", True, False), (171, 476, 8463, "f16", True, False),
    (48, 1333, 29898, "f16", False, False), (114, 693, 16268, "f16", False, False), (286, 420, 7777, "fp8qk_bf16v", False, False),   # past the last-level cache: 3 to 7 %
    (14, 9470, 8100, "f16", True, False), (260, 341, 3124, "bf16", True, False), (258, 324, 1896, "fp8qk_bf16v", False, False),   # a few workgroups behind a round: 12 to 30 %
    (216, 3519, 581, "f16", False, False), (731, 1457, 625, "f16", False, False), (976, 467, 868, "bf16", True, False),   # short key axes: 3 to 5 %
    (57, 1765, 59, "bf16", True, False), (57, 2028, 27, "f16", True, False), (42, 2717, 70, "f16", False, False)])
def test_512_rows_where_they_are_not_slower(H, Nq, Nk, dtype, counts, taken):
    assert launch_choice.rows512(H, H, Nq, Nk, dtype, counts) is taken


def _shapes(test):
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0].startswith("H,Nq,Nk,d"))


@pytest.mark.parametrize("test", [two_parts.test_columns_against_64_bits, two_parts.test_columns_without_the_largest_key,
                                  two_parts.test_ordinary_values_take_two_parts])
def test_fp32_shapes_take_two_parts(test):
    """128 rows and 256 rows at both head dims, ragged in the second half of 256; and at d = 128 an axis with the early check (1024 keys)."""
    shapes = _shapes(test)
    taken = {(d, launch_choice.f32_rows(H, Nq, Nk, d)) for H, Nq, Nk, d in shapes}
    assert taken == {(d, (rows, True)) for d in (64, 128) for rows in (128, 256)}
    for H, Nq, Nk, d in shapes:
        if launch_choice.f32_rows(H, Nq, Nk, d)[0] == 256:
            assert Nq % 256 > 128
    assert any(d == 128 and Nk >= 1024 for H, Nq, Nk, d in shapes)
