"""Branches of the face kernels and their launch rules at the sizes and states where they can go wrong,
against the FP64 CPU oracle (bars as in test_gpu_parity: FP64 1e-12, FP32 1e-5, max norm per variable)."""
import pytest
import torch

from gpu_util import oracle_dev, print_case, rel_errors, run_gpu, run_oracle
from synth import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [5, 2])
@pytest.mark.parametrize("ma", [0.34, 0.6])
def test_kinetic_average_on_both_sides_of_its_series_range(ma, order):
    # |U| up to 1 and c = 1 / ma: sqrt(lambda) |U_n| reaches ma / sqrt(2) = 0.24, inside the series' range of
    # 1/4, and 0.42, where the field has Gauss points on both sides of it
    cfg = make_case("tgv", grid=(18, 14, 17)).with_(ma=ma, order=order)
    o, _ = run_oracle(cfg, 2)
    ref = oracle_dev(o.Q, cfg.rho_ref)
    for precision, bar in (("fp64", 1e-12), ("fp32", 1e-5)):
        print_case("kinetic", ma=ma, order=order, precision=precision)
        s, _ = run_gpu(cfg, precision, 2)
        err = rel_errors(s.interior(), ref)
        assert max(err) < bar, (precision, err)
        assert bool(torch.isfinite(s.interior()).all())
