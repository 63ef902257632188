"""The rows of ``smooth_porosity``'s boxes and cylinders: every form whose
values float() takes gives the same array, and nothing else is accepted.
Host code only; exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2204_01117_amd.voxelize import _smooth_objects  # noqa: E402

ROWS = [[0.1, 1.5, 2.0, 3.0, 0.0, 4.0, 0.25], [1, 2, 3, 4, 5, 6, 0]]
FORMS = {
    "lists": lambda r: r,
    "tuples": lambda r: tuple(tuple(x) for x in r),
    "array": lambda r: np.array(r),
    "arrays": lambda r: [np.array(x) for x in r],
    "values of a dict": lambda r: dict(enumerate(r)).values(),
    "tensor": lambda r: torch.tensor(r, dtype=torch.float64),
    "tensor with grad": lambda r: torch.tensor(r, dtype=torch.float64, requires_grad=True),
    "tensors with grad": lambda r: [torch.tensor(x, dtype=torch.float64, requires_grad=True) for x in r],
    "single values with grad": lambda r: [[torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in x] for x in r],
    "unequal lengths": lambda r: [r[0] + r[1][:1], r[1][1:]],
    "a generator in a row": lambda r: [(v for v in x) for x in r],
}
GPU = [pytest.param(f, marks=[pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")])
       for f in ("tensor", "tensors with grad")]


def check(rows):
    want = [float(v) for row in ROWS for v in row]
    o, keep = _smooth_objects((4, 4, 4), (1.0, 1.0, 1.0), rows, [], 0.5)
    assert (o.nboxes, o.ncyls) == (2, 0)
    assert [o.boxes[q] for q in range(14)] == want
    del keep


@pytest.mark.parametrize("form", list(FORMS))
def test_forms_that_float_takes(form):
    check(FORMS[form](ROWS))


@pytest.mark.parametrize("form", GPU)
def test_rows_on_the_gpu(form):
    rows = FORMS[form](ROWS)
    check(rows.cuda() if torch.is_tensor(rows) else [r.cuda() for r in rows])


@pytest.mark.parametrize("rows", [[[[0.1, 1.5], [2.0, 3.0]]], [["x"] * 7], [1.0, 2.0]])
def test_refused(rows):
    with pytest.raises((TypeError, ValueError)):
        _smooth_objects((4, 4, 4), (1.0, 1.0, 1.0), rows, [], 0.5)
