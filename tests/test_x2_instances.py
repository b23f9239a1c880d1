"""Which instances of the compiled-length X2 kernels the built library holds: one kernel per row length and nodewise
form (X2N_FP64 = 0, X2N_D32 = 1, X2N_ALT = 2, X2N_HESS = 3, X2N_HESS_ALT = 4).  FP32-mixed evaluations form dPhi/dn
from FP32 differences in the ten lengths of include/dft.h and no other."""
import re

from paper_0910_1531_amd import _abi

FP32_NODES = {16, 24, 32, 48, 64, 96, 128, 192, 256, 384}
FP64_NODES = {8, 9, 12, 18, 27, 36, 54, 72, 81, 108, 144, 162, 216, 243, 288, 324, 432, 486, 512}


def test_fp32_differences_only_where_documented():
    with open(_abi.LIB_PATH, "rb") as f:
        lib = f.read()
    for kernel in (b"k_x2w", b"k_x2h"):   # one wave per field, two waves per row pair
        forms = {(int(n), int(k)) for n, k in re.findall(kernel + rb"IfLi(\d+)ELi(\d+)E", lib)}
        assert {n for n, k in forms if k == 1} == FP32_NODES
        assert {n for n, k in forms if k == 0} == FP64_NODES


def test_no_hessian_kernels_past_the_longest_rows():
    # dft_adjoint and dft_newton refuse n_x > 384
    with open(_abi.LIB_PATH, "rb") as f:
        lib = f.read()
    for kernel in (b"k_x2w", b"k_x2h"):
        hess = {int(n) for n, k in re.findall(kernel + rb"IdLi(\d+)ELi(\d+)E", lib) if int(k) >= 3}
        assert max(hess) == 384
