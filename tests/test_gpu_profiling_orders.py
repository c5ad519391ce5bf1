"""The profiled work orders run as they are listed, the orders 2 and 3 among them."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1010_5636_amd as ndq  # noqa: E402
from paper_1010_5636_amd import profiling  # noqa: E402


def test_orders_are_set_as_listed(monkeypatch):
    dims, orders = (4, 4, 4, 8), [(6, 3, 0), (0, 0, -1), (3, 2, 0), (4, 1, -1)]
    g = ndq.Geometry(dims)
    dflt = ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, 18, 12, 2)
    seen = []

    def log(text):
        got = ndq.ndq.get_mrhs_launch(g, ndq.F32, ndq.F32, 18, 12, 2)
        seen.append((got["rg"], got["group_major"], got["chunk"]))

    monkeypatch.setattr(profiling, "ORDERS32", orders)
    monkeypatch.setattr(profiling, "ORDERS32_DIMS", dims, raising=False)
    monkeypatch.setattr(profiling, "_log", log)
    try:
        profiling._orders32(1)
    finally:
        ndq.ndq.set_mrhs_launch(g, ndq.F32, ndq.F32, 18, 12, 2, **dflt)
    assert seen == orders
