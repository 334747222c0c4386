"""Argument checks of the entry points that take a dtype for dH (no GPU: fake addresses, every
call returns before any launch)."""
import paper_2606_07574_amd as b4
from tests.test_abi_host import A, Bp, C, D, E, ERR_ALIGN, ERR_CHANNELS, ERR_DTYPE, ERR_NULL, ERR_OVERLAP, ERR_SIZE, F, OK


def test_backward_with_dh_dtype():
    lib = b4.lib()
    for f, per in ((lib.birkhoff4_bwd_ex2, 16), (lib.birkhoff8_bwd_ex, 64)):  # (P, dP, dp_dtype, dH, dh_dtype, B, stream)
        assert f(A, Bp, 0, C, 1, 0, None) == OK
        assert f(A, Bp, 0, C, 1, -1, None) == ERR_SIZE
        assert f(A, Bp, 0, C, 2, 10, None) == ERR_DTYPE
        assert f(A, Bp, 2, C, 0, 10, None) == ERR_DTYPE
        assert f(A, Bp, 0, None, 1, 10, None) == ERR_NULL
        assert f(A, Bp, 0, C + 2, 1, 10, None) == ERR_ALIGN
        # bf16 dH takes half the bytes: its last 16 reach into P here, an fp32 dP's end below it
        assert f(A, Bp, 0, A - 2 * per * 10 + 16, 1, 10, None) == ERR_OVERLAP
        assert f(A, Bp, 0, Bp + 4 * per * 10 - 16, 1, 10, None) == ERR_OVERLAP


def test_mixing_backward_with_dh_dtype():
    lib = b4.lib()
    g = lib.birkhoff4_mix_bwd_ex  # (P, X, dY, x_dtype, dX, dH, dh_dtype, B, C, stream)
    assert g(A, Bp, C, 1, D, E, 1, 0, 64, None) == OK
    assert g(A, Bp, C, 1, D, E, 3, 10, 64, None) == ERR_DTYPE
    assert g(A, Bp, C, 1, D, E, 1, 10, 63, None) == ERR_CHANNELS
    assert g(A, Bp, C, 1, D, A, 1, 10, 64, None) == ERR_OVERLAP
    h = lib.birkhoff8_mix_bwd_ex  # (P, X, dY, x_dtype, dX, dP, dH, dh_dtype, B, C, stream)
    assert h(A, Bp, C, 1, D, E, F, 1, 0, 64, None) == OK
    assert h(A, Bp, C, 1, D, None, F, 1, 10, 64, None) == ERR_NULL
    assert h(A, Bp, C, 1, D, E, E, 1, 10, 64, None) == ERR_OVERLAP        # bf16 dH in dP's memory
    assert h(A, Bp, C, 1, D, E, E + 256, 0, 10, 64, None) == ERR_OVERLAP  # fp32 dH part-way into dP
    assert h(A, Bp, C, 1, D, Bp, F, 0, 10, 64, None) == ERR_OVERLAP       # dP in X
