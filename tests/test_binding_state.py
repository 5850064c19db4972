"""What the binding keeps between calls.  Without a GPU stand-ins take the places of the allocator and the C call."""
import threading
import types

import pytest
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


def _changes(m):
    """Changes of one matrix after its struct was asked for, with what desc() has to do about each: None (refuse) or
    the fields that must have followed.  Addresses and the number of entries stay the same throughout."""
    was = (m.rows, m.cols, m.indptr, m.indices, m.data)

    def restore():
        m.rows, m.cols, m.indptr, m.indices, m.data = was

    m.rows, m.cols = 2, 9
    yield {"rows": 2, "cols": 9}
    restore()
    m.data = m.data.view(torch.int32)
    yield None
    restore()
    m.indices = m.indices.view(torch.float32)
    yield None
    restore()
    m.indptr = m.indptr.view(torch.int16)
    yield None
    restore()
    m.data = torch.as_strided(m.data, (m.nnz,), (2,))
    yield None
    restore()
    m.data.as_strided_((m.nnz // 2,), (2,))              # in place: the tensor object stays the same one
    yield None
    m.data.as_strided_((m.nnz,), (1,))
    yield {"rows": was[0], "cols": was[1]}
    m.data = None
    yield {"data": None}
    restore()


def _check_desc_follows(device):
    m = binding.CsrMatrix(3, 8, torch.tensor([0, 2, 4, 6], dtype=torch.int32, device=device),
                          torch.arange(6, dtype=torch.int32, device=device), torch.arange(12.0, device=device)[:6])
    first = m.desc()
    assert (first.rows, first.cols, first.nnz, first.data) == (3, 8, 6, m.data.data_ptr())
    for want in _changes(m):
        if want is None:
            with pytest.raises(ValueError):
                m.desc()
        else:
            got = m.desc()
            assert all(getattr(got, k) == v for k, v in want.items()), want
    assert (first.rows, first.cols) == (3, 8)            # a struct handed out before is not written to


def test_matrix_descriptor_follows_its_arrays(monkeypatch):
    def ptr(t, dtype=torch.float32, name="tensor"):      # the binding's checks but for the place
        if t is None:
            return None
        if t.dtype != dtype or not t.is_contiguous():
            raise ValueError(name)
        return t.data_ptr()

    monkeypatch.setattr(binding, "_ptr", ptr)
    _check_desc_follows("cpu")


@pytest.mark.gpu
def test_matrix_descriptor_follows_its_arrays_on_the_gpu():
    assert torch.cuda.is_available()
    _check_desc_follows("cuda")
    with pytest.raises(ValueError):                      # nothing checked it before: it must not pass as checked
        binding.CsrMatrix(1, 1, torch.zeros(2, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32),
                          torch.zeros(1, device="cuda")).desc()


@pytest.mark.gpu
def test_builders_from_two_threads():
    """Matrices of different sizes built by two threads at once, each on a stream of its own, the first calls
    included: the threads are new ones every time."""
    import paper_1907_10134_amd as bp

    def work(which, start, out):
        with torch.cuda.stream(torch.cuda.Stream()):
            start.wait(30)
            for k in range(6):
                ci, co, n = 2 + which, 3 + k, 6 + 5 * which
                m = bp.csr_conv3x3(torch.ones((co, ci, 3, 3), device="cuda"), None, n, n)
                f = bp.csr_linear(torch.ones((4 + k, 9 + which), device="cuda"), None)
                out.append((m.nnz == ci * co * (3 * n - 2) ** 2, f.nnz == (4 + k) * (9 + which),
                            int(m.indptr[-1]) == m.nnz, float(m.data.sum()) == m.nnz, float(f.data.sum()) == f.nnz))

    for _ in range(5):
        start, outs = threading.Barrier(2), ([], [])
        threads = [threading.Thread(target=work, args=(k, start, outs[k])) for k in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join(60)
        assert all(len(o) == 6 and all(map(all, o)) for o in outs), outs
