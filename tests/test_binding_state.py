"""What the binding keeps between calls, without a GPU: stand-ins take the places of the allocator and the C call."""
import threading
import types

import torch

import paper_1907_10134_amd.binding as binding


def test_two_threads_make_their_first_builder_call_together(monkeypatch):
    """Both threads are held where each makes its report word, then inside their C calls at the same time:
    each must read the number of entries its own call left."""
    here = threading.local()
    making, inside, errors = threading.Barrier(2), threading.Barrier(2), []

    def empty(shape, dtype=None, device=None, pin_memory=False):
        if pin_memory and not getattr(here, "made", False):
            here.made = True
            making.wait(10)
        return torch.empty(shape, dtype=dtype)

    monkeypatch.setattr(binding, "torch", types.SimpleNamespace(empty=empty, int32=torch.int32, float32=torch.float32))
    out = [None, None]

    def work(which):
        def indptr(ptr, word, nnz):
            inside.wait(10)
            nnz._obj.value = 100 + which
            inside.wait(10)

        try:
            out[which] = binding._two_call(3, 4, "cpu", indptr, lambda ip, ix, d: None).nnz
        except Exception as e:                                   # noqa: BLE001 (reported by the assertion below)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(30)
    assert not errors and out == [100, 101], (errors, out)


def test_a_thread_keeps_its_report_word(monkeypatch):
    made = []

    def empty(shape, dtype=None, device=None, pin_memory=False):
        made.append(pin_memory)
        return torch.empty(shape, dtype=dtype)

    monkeypatch.setattr(binding, "torch", types.SimpleNamespace(empty=empty, int32=torch.int32, float32=torch.float32))
    counts = []

    def indptr(ptr, word, nnz):
        counts.append(word)
        nnz._obj.value = len(counts)

    def work():
        for k in range(3):
            assert binding._two_call(3, 4, "cpu", indptr, lambda ip, ix, d: None).nnz == k + 1

    t = threading.Thread(target=work)
    t.start()
    t.join(30)
    assert len(set(counts)) == 1 and len(counts) == 3 and made.count(True) == 1
