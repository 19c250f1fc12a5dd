"""Launch choices of the operator: whatever kernel and split of the lattice a
launch takes, every site gets the same bits, and they match the oracle."""

import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_1901_07294_amd.wilson as w
from paper_1901_07294_amd.buffers import DeviceGauge

from gpu_util import PRECS, TOL, rel

pytestmark = pytest.mark.gpu

HEADER = "# wilson dslash launch tuning v2: X Y Z T prec c12 nrhs tb gw group rb\n"


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)


@pytest.fixture(autouse=True)
def _clean():
    w.wd_tune_reset()
    yield
    w.wd_tune_reset()


def apply_with(line, tmp_path, g, masses, src):
    """The operator on src with the launch `line` (tb gw group rb) registered, or the default."""
    w.wd_tune_reset()
    n = len(masses)
    if line is not None:
        f = tmp_path / "tune.txt"
        key = " ".join(str(v) for v in (*g.dims, g.prec, int(g.compress12), n))
        f.write_text(f"{HEADER}{key} {line}\n")
        w.wd_tune_load(str(f))
    out = g.spinor(n).zero_()
    w.dslash_apply_multi(g.handle, masses, n, src, out, g.prec, flags=w.WD_FLAG_GAMMA5)
    return out


@pytest.mark.parametrize("prec,c12,nrhs", [("fp64", False, 1), ("fp64", True, 3), ("fp32", False, 2),
                                           ("fp32", True, 5), ("fp16", False, 4), ("fp16", True, 1)])
@pytest.mark.parametrize("dims", [
    (28, 15, 3, 7),   # 140 of 192 lanes, 3 y tiles: the workgroups do not divide by the 8 XCDs
    (9, 33, 3, 5),    # 99 of 128 lanes
    (64, 3, 5, 2),    # whole waves, a tile of 3 rows
    (32, 32, 4, 11),  # 256 lanes, a prime number of t slices
    (16, 16, 1, 1),   # one workgroup per field
], ids=lambda d: "x".join(map(str, d)))
def test_launch_choices_keep_bits(dims, prec, c12, nrhs, tmp_path):
    """The default launch against marches of one slice in hardware order, of
    all slices with every XCD's workgroups contiguous, and a run length far
    beyond the number of workgroups."""
    print(f"case launch dims={dims} prec={prec} c12={c12} nrhs={nrhs}", flush=True)
    U = li.random_gauge(dims, 71)
    psis = li.gaussian_spinors(dims, [72 + k for k in range(nrhs)])
    masses = [0.05 + 0.1 * k for k in range(nrhs)]
    g = DeviceGauge(U, PRECS[prec], c12)
    src = g.pack(psis, nrhs=nrhs)
    default = apply_with(None, tmp_path, g, masses, src)
    for line in ("1 1 0 1", f"{dims[3]} 1 1 1", f"{dims[3]} 1 2147483647 1"):
        other = apply_with(line, tmp_path, g, masses, src)
        torch.cuda.synchronize()
        assert torch.equal(default, other), line
    got = g.unpack(default, nrhs=nrhs)
    got = got if nrhs > 1 else got[None]
    ref = oracle.gamma5_apply(oracle.dslash(U, psis[-1], masses[-1]))
    assert rel(got[-1], ref) <= TOL[PRECS[prec]]
