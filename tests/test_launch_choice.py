"""The GPU tests of the forward's forms and of fp32 in two parts run the kernels that they are there for (no GPU needed)."""
import itertools

import pytest

import launch_choice
import test_gpu_f32_two_parts as two_parts
import test_gpu_forward_forms as forms


@pytest.mark.parametrize("partial", [False, True])
@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp8qk_bf16v"])
@pytest.mark.parametrize("d", [64, 128])
def test_every_form_has_a_shape(d, dtype, counts, partial):
    """Whatever a launch may take, over a grid of sizes, one of the tested shapes takes too."""
    reached = {launch_choice.form(h, h, nq, nk, d, dtype, counts, partial)
               for h, nq, nk in itertools.product((1, 2, 4, 8, 12, 20, 40, 64, 100, 200), (33, 64, 100, 300, 500, 999, 2000, 4000),
                                                  (60, 150, 300, 500, 700, 1000, 1300, 2000, 3000, 4600, 7000))}
    tested = {launch_choice.form(H, H_kv, Nq, Nk, d, dtype, counts, partial) for H, H_kv, Nq, Nk, dd in forms.SHAPES if dd == d}
    reached.discard(("Rows256", False))            # (fwd_pipelined_kernel has tests of its own)
    assert len(reached) >= (2 if dtype == "fp8qk_bf16v" and d == 128 else 3)
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
