"""Creation under a memory limit: an invalid mask is refused as an invalid mask,
with its own status and text, also where the level arrays could not be
allocated; a valid one then gives the allocation error.  Whatever was allocated
is given back."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    from paper_1104_1703_amd import mg as m
    m.load_library()
    return m


def box(n=32):
    m = np.full((n, n, n), -1, np.int8)
    m[1:-1, 1:-1, 1:-1] = 1
    return m


def cases(mg):
    ok, value, frame, empty = box(), box(), box(), np.full((32, 32, 32), -1, np.int8)
    value[3, 4, 5] = 0
    frame[0, 7, 7] = 1
    return [("valid", ok, mg.MG_ERR_ALLOC, "bytes failed"), ("value", value, mg.MG_ERR_ARG, "1 values other than"),
            ("frame", frame, mg.MG_ERR_ARG, "1 active cells in the outermost layer"),
            ("empty", empty, mg.MG_ERR_NO_ACTIVE, "no active cell")]


@pytest.mark.parametrize("limit", [512, 4096])  # bytes an allocation may have
@pytest.mark.parametrize("which", range(4), ids=["valid", "value", "frame", "empty"])
def test_invalid_mask_is_refused_as_such(mg, which, limit):
    name, mask, status, text = cases(mg)[which]
    print("create", name, limit, flush=True)
    lib = mg.load_library()
    held, stream = set(), torch.cuda.Stream()

    def alloc(n, ctx):
        if n > limit:
            return None
        p = int(torch.cuda.caching_allocator_alloc(int(n), torch.device("cuda", 0), stream))
        held.add(p)
        return p

    def free(p, ctx):
        held.remove(int(p))
        torch.cuda.caching_allocator_delete(int(p))

    a, f = mg._ALLOC_FN(alloc), mg._FREE_FN(free)
    o = mg.default_options()
    o.allocator.alloc, o.allocator.free, o.allocator.ctx = a, f, None
    m = torch.from_numpy(mask).cuda()
    torch.cuda.synchronize()
    out = C.c_void_p()
    st = lib.mg_create_hierarchy(C.c_void_p(m.data_ptr()), 32, 32, 32, 1.0 / 32, C.byref(o),
                                 C.c_void_p(stream.cuda_stream), C.byref(out))
    assert (st, out.value) == (status, None)
    assert text in lib.mg_last_error().decode()
    assert not held
