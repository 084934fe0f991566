"""Shapes and types that the binding refuses before the library sees a pointer (CPU: the library's entry point is replaced by one that must not be reached)."""
import pytest
import torch


@pytest.fixture
def product(monkeypatch):
    import paper_2602_04929_amd as tb

    class Reached(Exception):
        pass

    class Stub:
        def tboa_gemm_f64_residues(self, *args):
            raise Reached

    def dev(t, dtype=None):      # the checks of the binding's own but for the device
        assert t.is_contiguous() and (dtype is None or t.dtype == dtype)
        return t
    monkeypatch.setattr(tb.binding, "_lib", Stub())
    monkeypatch.setattr(tb.binding, "_dev", dev)
    ctx = object.__new__(tb.Context)
    ctx._h = None
    return ctx.gemm_f64_residues, Reached


def test_product_of_residues(product):
    gemm, reached = product
    z = lambda *s, dtype=torch.float64: torch.zeros(*s, dtype=dtype)  # noqa: E731
    for b, trans in ((z(6, 5), False), (z(5, 6), True)):
        for c in (None, z(4, 5)):
            with pytest.raises(reached):
                gemm(z(4, 6), b, c, transB=trans)
        for c in (z(4, 5, dtype=torch.float32), z(4, 4), z(3, 5), z(5, 4), z(20), z(5, 4).t(), z(4, 10)[:, ::2]):
            with pytest.raises(AssertionError):
                gemm(z(4, 6), b, c, transB=trans)
    for b, trans in ((z(5, 6), False), (z(6, 5), True), (z(7, 5), False)):
        with pytest.raises(AssertionError):
            gemm(z(4, 6), b, transB=trans)
