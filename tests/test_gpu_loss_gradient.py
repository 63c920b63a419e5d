"""Every form of a loss gradient that the photometric adjoint takes gives what
its value gives, wherever the value lies."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
api = pytest.importorskip("paper_1904_06017_amd.api")

W, H = 70, 19
F64 = torch.float64
FORMS = {
    "zero": lambda v: torch._efficientzerotensor((), dtype=F64, device="cuda"),
    "sparse": lambda v: torch.tensor([v], dtype=F64, device="cuda").to_sparse(),
}


def _check(form, value):
    """value: what the form holds; the same FP64 quotient, so the same bits."""
    g = torch.Generator(device="cuda").manual_seed(3)
    ref, tar = (255 * torch.rand(H, W, device="cuda", generator=g) for _ in range(2))
    disp = 4 * torch.rand(H, W, device="cuda", generator=g)
    plan = api.Plan(api.make_params(W, H, 8, dtype="f32", delta_p=3.0, plane=(3.0, 0.0, 0.0),
                                    ncc_radius=2, bil_radius=2))
    want = api.photometric_l1_bwd(plan, ref, tar, disp, value)
    got = api.photometric_l1_bwd(plan, ref, tar, disp, form)
    for a, b in zip(got, want):
        assert torch.equal(a.nan_to_num(9.0), b.nan_to_num(9.0))


@pytest.mark.parametrize("name", list(FORMS))
def test_forms_without_a_value_in_memory(name):
    value = 0.0 if name == "zero" else -0.37
    _check(FORMS[name](value), value)


OTHERS = {
    "float32 on the device": lambda v: torch.tensor(v, dtype=torch.float32, device="cuda"),
    "float16 on the device": lambda v: torch.tensor([v], dtype=torch.float16, device="cuda"),
    "float64 on the host": lambda v: torch.tensor([[v]], dtype=F64),
    "float32 on the host": lambda v: torch.tensor(v, dtype=torch.float32),
    "int on the device": lambda v: torch.tensor(3, device="cuda"),
    "negated view": lambda v: torch._neg_view(torch.tensor(-v, dtype=F64, device="cuda")),
    "column of a matrix": lambda v: torch.full((3, 2), v, dtype=F64, device="cuda")[1:2, 1:],
    "requires grad": lambda v: torch.tensor(v, dtype=F64, device="cuda", requires_grad=True).clone(),
    "numpy": lambda v: np.float64(v),
}


@pytest.mark.parametrize("value", [1.0, -0.37, 1e-30, float("inf")])
@pytest.mark.parametrize("name", list(OTHERS))
def test_forms_with_a_value_in_memory(name, value):
    """Of other types than float64 the value read is the type's: a float32 must
    not be taken for half of a double."""
    form = OTHERS[name](value)
    _check(form, float(form.detach() if isinstance(form, torch.Tensor) else form))
