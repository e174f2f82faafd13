"""csrc/sphattn_choice.hpp, the code that picks a launch's kernel, compiled for the host: which form a call takes on a device of
256 compute units."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2505_09326_amd._build import CSRC

FORMS = ("Rows64", "Rows64Wide", "Rows64Own", "Rows128", "Rows128Wide", "Narrow", "Rows256Wide", "Rows256")
ROWS = (64, 64, 64, 128, 128, 128, 256, 256)
CUS = 256

SOURCE = """
#include "sphattn_choice.hpp"
using namespace sphattn;
extern "C" int form(long long slices, long long Nq, long long Nk, int d, int bf16, int fp8, int counts)
{
    return choose_form(slices, Nq, (Nk + kChoiceTile - 1) / kChoiceTile, d, Storage{bf16 != 0, fp8 != 0, counts != 0}, %d).form;
}
extern "C" int form_in_one_order(int form, long long Nk) { return in_one_key_order((Form)form, (Nk + kChoiceTile - 1) / kChoiceTile, true); }
extern "C" int f32_rows(long long heads, long long Nq, long long Nk, int d) { return choose_f32(heads, Nq, Nk, 1, d, %d).rows; }
extern "C" int two_parts(long long Nk, int d) { return f32_two_parts(Nk, d); }
extern "C" int f32_shares(long long slices, long long Nq) { return f32_small_column_shares(slices, Nq, %d); }
extern "C" int column_share(long long slices, long long Nq, long long Nk, int d, int bf16, int fp8, int counts)
{
    const long long tiles = (Nk + kChoiceTile - 1) / kChoiceTile;
    const Storage st{bf16 != 0, fp8 != 0, counts != 0};
    FormChoice c = choose_form(slices, Nq, tiles, d, st, %d);
    return column_shares(c, slices, Nq, tiles, d, st, %d);
}
extern "C" int rows512(long long slices, long long Nq, long long Nk, int bf16, int fp8, int counts, int whole)
{
    return rows512_pay(slices, Nq, (Nk + kChoiceTile - 1) / kChoiceTile, Storage{bf16 != 0, fp8 != 0, counts != 0}, whole != 0, %d);
}
extern "C" int fp8_shape(long long heads, long long N, int d, int counts)
{
    const Fp8Shape s = choose_fp8(heads, N, d, counts != 0, %d);
    return s.nq * 16 + s.waves;
}
""" % ((CUS,) * 7)


@functools.lru_cache(maxsize=None)
def _library():
    with tempfile.TemporaryDirectory() as tmp:
        src, out = os.path.join(tmp, "choice.cpp"), os.path.join(tmp, "choice.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", out, src], check=True)
        lib = ctypes.CDLL(out)
    lib.form.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 4
    lib.form_in_one_order.argtypes = [ctypes.c_int, ctypes.c_longlong]
    lib.f32_rows.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int]
    lib.two_parts.argtypes = [ctypes.c_longlong, ctypes.c_int]
    lib.f32_shares.argtypes = [ctypes.c_longlong] * 2
    lib.column_share.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 4
    lib.rows512.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 4
    lib.fp8_shape.argtypes = [ctypes.c_longlong] * 2 + [ctypes.c_int] * 2
    return lib


def form(H, H_kv, Nq, Nk, d, dtype, counts, partial=False):
    """The form's name, and whether two of its workgroups share a CU.  Query heads of one K/V head are one block of rows."""
    rows = Nq * (H // H_kv)
    f = _library().form(H_kv, rows, Nk, d, dtype == "bf16" and not partial, dtype == "fp8qk_bf16v", counts)
    return FORMS[f], f != len(FORMS) - 1 and H_kv * -(-rows // ROWS[f]) > CUS


def bf16_form_in_one_key_order(H, N, d):
    """The form of a bf16 self-attention launch without counts that keeps the 256-row kernel's order of a row's terms."""
    return FORMS[_library().form_in_one_order(FORMS.index(form(H, H, N, N, d, "bf16", False)[0]), N)]


def f32_rows(H, Nq, Nk, d):
    """Query rows per workgroup of an fp32 launch, and whether it works in two parts."""
    lib = _library()
    rows = lib.f32_rows(H, Nq, Nk, d)
    return rows, rows >= 128 and bool(lib.two_parts(Nk, d))


def fp8_shape(H, N, d, counts):
    """(query blocks of 16 rows per wave, waves) of an all-E4M3 launch of one batch entry."""
    return divmod(_library().fp8_shape(H, N, d, counts), 16)


def rows512(H, H_kv, Nq, Nk, dtype, counts, whole=True):
    """Whether a launch of d = 64 takes 512 rows in eight waves."""
    return bool(_library().rows512(H_kv, Nq * (H // H_kv), Nk, dtype == "bf16", dtype == "fp8qk_bf16v", counts, whole))


def column_shares(H, H_kv, Nq, Nk, d, dtype, counts, partial=False):
    """Workgroups that share the columns of V of a launch's row tile."""
    return _library().column_share(H_kv, Nq * (H // H_kv), Nk, d, dtype == "bf16" and not partial, dtype == "fp8qk_bf16v", counts)


def launched(H, H_kv, Nq, Nk, d, dtype, counts, partial=False):
    """What runs: the form's name with the workgroups that share its columns ("Shared2", whichever 64-row form had the launch),
    or "Rows512"; and whether two of its workgroups share a CU."""
    name, two = form(H, H_kv, Nq, Nk, d, dtype, counts, partial)
    shares = column_shares(H, H_kv, Nq, Nk, d, dtype, counts, partial)
    if shares > 1:
        return f"Shared{shares}", False
    if name == "Rows256" and d == 64 and rows512(H, H_kv, Nq, Nk, dtype, counts, not partial):
        return "Rows512", False
    return name, two


def f32_shares(H, Nq):
    """Workgroups that share the columns of 16 rows of an fp32 launch."""
    return _library().f32_shares(H, Nq)
