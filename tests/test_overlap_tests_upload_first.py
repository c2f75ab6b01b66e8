"""The GPU tests in which steps of one context overlap, on the CPU with a stand-in for the context: the pointer table is uploaded by the first
step with new pointers, on that step's stream, so no step on another stream may be issued before the GPU has been waited for (it
could read a table that is not there yet).  Only the kernels of steps with the same pointers may overlap."""
import types

import pytest
import torch

import test_gpu_layouts as L


@pytest.mark.parametrize("name", ["test_steps_that_overlap_leave_nothing_behind", "test_single_launches_that_overlap_leave_nothing_behind"])
def test_nothing_overlaps_an_upload(name, monkeypatch):
    overlapping, contexts = [], []

    class Context:
        def __init__(self, *args, **kw):
            self.pointers = self.pending = None
            contexts.append(self)

        def step(self, p, g, m, v, gamma, hp, step, stream=None):
            pointers = tuple(x.data_ptr() if torch.is_tensor(x) else x for arrays in (p, g, m, v) for x in arrays)
            if pointers != self.pointers:
                self.pointers, self.pending = pointers, stream
            elif self.pending != "nothing":
                assert stream == self.pending, "a step on another stream than that of the upload, before it has been waited for"
            if stream is not None:
                overlapping.append(stream)

        def get_norms(self):
            raise StopIteration            # a stand-in has no results: the overlapping steps lie behind

        def close(self):
            pass

    def synchronize():
        for c in contexts:
            c.pending = "nothing"

    monkeypatch.setattr(L, "DEV", "cpu")
    monkeypatch.setattr(L.B, "AdaGC", Context)
    numbers = iter(range(1, 9))
    monkeypatch.setattr(torch.cuda, "Stream", lambda: types.SimpleNamespace(cuda_stream=next(numbers)))
    monkeypatch.setattr(torch.cuda, "synchronize", synchronize)
    try:
        getattr(L, name)()
    except StopIteration:
        pass
    assert len(set(overlapping)) == 2
