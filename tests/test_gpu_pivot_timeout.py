"""The pivoting path after an expired wait.

Every device-side wait is bounded: one that expires raises a flag, the queued
launches drain and the call returns N3P_E_TIMEOUT.  A leaf that finds the flag
leaves at once, so whatever the launches behind it index by must not be what
an earlier leaf, or nobody, left in the workspace.  Here the flag is set
before the leaf runs and the workspace is filled with row numbers past the
matrix (all inside buffers of this test), so any use of them shows as a change
of the matrix, of L transposed or of the interchanges.
"""
import ctypes
import os

import pytest

pytestmark = pytest.mark.gpu

PANELS = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libpanels.so")


@pytest.fixture(scope="module")
def env():
    import torch
    if not os.path.exists(PANELS):
        pytest.fail("libpanels.so not built; run __graft_entry__.build()")
    lib = ctypes.CDLL(PANELS)
    lib.panels_xch_bytes.restype = ctypes.c_size_t
    lib.panels_xch_bytes.argtypes = [ctypes.c_int, ctypes.c_int64]
    i64, vp = ctypes.c_int64, ctypes.c_void_p
    lib.panels_leaf.argtypes = [ctypes.c_int, i64, i64, i64, i64, vp, i64, vp, vp, vp, vp, vp]
    lib.panels_block.argtypes = [ctypes.c_int, i64, i64, i64, vp, i64, vp, vp]
    return lib, torch


class Panel:
    """Buffers of one factorisation in progress, the flag of an expired wait set."""

    def __init__(self, lib, torch, prec, Np, row):
        self.lib, self.torch, self.prec, self.Np = lib, torch, prec, Np
        dt = [torch.float16, torch.bfloat16, torch.float32, torch.float64][prec]
        g = torch.Generator(device="cuda").manual_seed(Np)
        # room behind every column and behind the last one
        self.lda = Np + 64
        self.A = torch.randn(Np + 2, self.lda, generator=g, device="cuda").to(dt)
        self.LT = torch.randn(2 * Np + 64, lib.panels_block_columns(), generator=g, device="cuda").to(dt)
        self.ipiv = torch.full((Np,), -7, dtype=torch.int32, device="cuda")
        self.flags = torch.zeros(lib.panels_nflags(), dtype=torch.int32, device="cuda")
        self.flags[lib.panels_flag_timeout()] = 1
        self.xch = torch.full((lib.panels_xch_bytes(prec, Np) // 4,), row, dtype=torch.int32, device="cuda")
        self.before = [t.clone() for t in self.state()]

    def state(self):
        return [self.A, self.LT, self.ipiv, self.flags]

    def leaf(self, c0, k0, kend):
        e = self.lib.panels_leaf(self.prec, self.Np, c0, k0, kend, self.A.data_ptr(), self.lda,
                                 self.ipiv.data_ptr(), self.LT.data_ptr(), self.xch.data_ptr(),
                                 self.flags.data_ptr(), self.torch.cuda.current_stream().cuda_stream)
        assert e == 0

    def block(self, k0, kend):
        e = self.lib.panels_block(self.prec, self.Np, k0, kend, self.A.data_ptr(), self.lda,
                                  self.xch.data_ptr(), self.torch.cuda.current_stream().cuda_stream)
        assert e == 0

    def assert_untouched(self):
        self.torch.cuda.synchronize()
        for name, a, b in zip(("A", "LT", "ipiv", "flags"), self.before, self.state()):
            assert self.torch.equal(a, b), name


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("Np,c0,k0", [(64, 0, 0), (192, 64, 0), (640, 0, 0), (1088, 1024, 1024),
                                      (2112, 1088, 1024)])
def test_one_workgroup_leaf_after_an_expired_wait(env, prec, Np, c0, k0):
    lib, torch = env
    print("case abandoned leaf prec %d Np=%d c0=%d" % (prec, Np, c0), flush=True)
    p = Panel(lib, torch, prec, Np, Np + 8)
    p.leaf(c0, k0, min(k0 + lib.panels_block_columns(), Np))
    p.assert_untouched()


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_cooperative_leaf_after_an_expired_wait(env, prec):
    """More than 4096 rows below the leaf: a panel over several workgroups,
    with the interchanges of an earlier outer block still in its list."""
    lib, torch = env
    Np, c0 = 5248, 1024
    print("case abandoned cooperative leaf prec %d" % prec, flush=True)
    p = Panel(lib, torch, prec, Np, c0 - 8)
    p.leaf(c0, c0, c0 + lib.panels_block_columns())
    p.assert_untouched()


@pytest.mark.parametrize("Np", [2112, 5248])
def test_block_interchanges_after_an_expired_wait(env, Np):
    """The lists of an outer block whose leaves were all abandoned hold the
    rows of the block before, above its own: none of them may be applied."""
    lib, torch = env
    k0 = lib.panels_block_columns()
    kend = 2 * k0
    print("case abandoned block Np=%d" % Np, flush=True)
    p = Panel(lib, torch, 0, Np, k0 - 8)
    for c0 in range(k0, kend, 64):
        p.leaf(c0, k0, kend)
    p.block(k0, kend)
    p.assert_untouched()
