"""The Python binding without a GPU: what coda_gemm hands to the library is alive while the library runs."""
import weakref

import torch

from paper_2605_19269_amd import coda


class _Library:
    """Stands in for libcoda.so: notes which of the tensors behind the ops exist at the call."""

    def __init__(self, refs):
        self.refs, self.alive = refs, None

    def coda_gemm(self, *args):
        self.alive = [r() is not None for r in self.refs]
        return coda.CODA_OK


def test_tensors_of_a_generator_of_ops_outlive_the_call(monkeypatch):
    refs = []

    def ops():
        for make in (lambda t: coda.row_scale(t), lambda t: coda.store(t.view(4, 8))):
            t = torch.zeros(32)
            refs.append(weakref.ref(t.untyped_storage()))
            op = make(t)
            del t
            yield op
            del op

    A, B = torch.zeros(4, 8, dtype=torch.bfloat16), torch.zeros(8, 8, dtype=torch.bfloat16)
    lib = _Library(refs)
    monkeypatch.setattr(coda, "_lib", lib)
    coda.coda_gemm(A, B, ops(), stream=0)
    assert lib.alive == [True, True]
