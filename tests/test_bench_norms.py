"""Error figures of bench.py are formed on the host: tensors that refuse any reduction stand for
device tensors (no GPU)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

torch = pytest.importorskip("torch")


class Device(torch.Tensor):
    @classmethod
    def __torch_function__(cls, func, types, args=(), kwargs=None):
        if func.__name__ == "cpu":
            return args[0].as_subclass(torch.Tensor)
        assert func.__name__ not in ("sum", "linalg_vector_norm", "linalg_norm", "norm", "vector_norm"), func
        return super().__torch_function__(func, types, args, kwargs or {})


def test_error_figures_reduce_on_the_host():
    g = torch.Generator().manual_seed(3)
    b = torch.randn(12 * 5 * 27, dtype=torch.float64, generator=g)
    a = b + 1e-3
    da, db = a.as_subclass(Device), b.as_subclass(Device)
    with pytest.raises(AssertionError):
        torch.linalg.norm(da)
    assert bench._rel_l2(da - db, db, torch) == pytest.approx(1e-3 * len(b) ** 0.5 / float(torch.linalg.norm(b)), rel=1e-9)
    pv = bench._per_var_err(da, db, {"hex": (12, 27, 54)}, torch)
    bb = b.view(12, 5, 27)
    assert pv == pytest.approx([1e-3 * (12 * 27) ** 0.5 / float(bb[:, v].norm()) for v in range(5)], rel=1e-9)
