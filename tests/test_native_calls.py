"""The native marshalling of the binding (CPU): every form of argument the calls take."""
import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import paper_2412_12488_amd as mc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def in_child(code, cwd=ROOT, env=None):
    """Runs code in a process of its own (what it tests used to end the process); its output."""
    res = subprocess.run([sys.executable, "-c", "import paper_2412_12488_amd as mc\n" + code], cwd=cwd,
                         capture_output=True, text=True, timeout=120, env=env)
    assert res.returncode == 0, (res.returncode, res.stderr[-2000:])
    return res.stdout


@pytest.mark.parametrize("form", [list, tuple, lambda v: np.array(v, dtype=np.int32),
                                  lambda v: np.array(v, dtype=np.int64),
                                  lambda v: [np.int32(x) for x in v], lambda v: [float(x) for x in v],
                                  lambda v: np.repeat(np.array(v, dtype=np.int32), 2)[::2]])
def test_lists_of_numbers_in_every_form(form):
    pages = [7, 8, 9, 3, 0, 1]
    assert mc.mc_addr_compress(form(pages)) == [(7, 3), (3, 1), (0, 2)]
    assert mc.mc_kv_check_page_table(form(pages), 10) == mc.MC_OK
    ix = mc.mc_prefix_index_create()
    tokens = list(range(40))
    mc.mc_prefix_index_insert(ix, form(tokens), form([5, 6]))
    assert mc.mc_prefix_index_match(ix, form(tokens[:33])) == (32, [5, 6])
    mc.mc_prefix_index_destroy(ix)


def test_runs_in_every_form_and_capacity():
    assert mc.mc_addr_expand([[2, 2], (9, 1)]) == [2, 3, 9]
    assert mc.mc_addr_expand(np.array([[2, 2], [9, 1]], dtype=np.int32)) == [2, 3, 9]
    assert mc.mc_addr_expand([(2, 2)], 5) == [2, 3]
    with pytest.raises(mc.McError) as e:
        mc.mc_addr_expand([(2, 2), (9, 1)], capacity=2)
    assert e.value.status == mc.MC_ERR_RANGE


def test_wrong_arguments_raise_and_do_not_crash():
    with pytest.raises(TypeError):
        mc.mc_addr_compress(5)
    with pytest.raises((TypeError, ValueError)):
        mc.mc_addr_compress(["x"])
    with pytest.raises(TypeError):
        mc.mc_kv_alloc_pages(b"four", 1)                    # not a handle
    with pytest.raises(TypeError):
        mc.mc_kv_pack_range(ctypes.c_int32(1), 0, 1, 16, 1, 0, 1, 16, stream=0)
    with pytest.raises(mc.McError) as e:
        mc.mc_kv_alloc_pages(None, 1)
    assert e.value.status == mc.MC_ERR_INVALID
    ix, al = mc.mc_prefix_index_create(), mc.mc_kv_allocator_create(8)
    with pytest.raises(IndexError):
        mc.mc_prep_recv(ix, al, [1, 2, 3], 17)              # reaches past the prompt
    assert mc.mc_kv_allocator_num_free(al) == 8
    mc.mc_prefix_index_destroy(ix)
    mc.mc_kv_allocator_destroy(al)


@pytest.mark.parametrize("runs", [[(3,), (9,)], [(1, 1, 5), (1, 2)], [(3, 1, 9, 1), (50, 4)],
                                  [(1, 1, 5), (1,)], [()], np.zeros((2, 3), dtype=np.int32)])
@pytest.mark.parametrize("capacity", [None, 64])
def test_runs_that_are_not_pairs_are_refused(runs, capacity):
    # never re-cut into other pairs: their pages would be another sequence's
    with pytest.raises(ValueError):
        mc.mc_addr_expand(runs, capacity)


def test_lists_that_change_while_they_are_read():
    # __int__ is the caller's code: it may empty the very list that is being converted
    out = in_child("""
class Clears:
    def __int__(self):
        pages.clear()
        return 1
pages = [Clears() for _ in range(1000)]
print(mc.mc_addr_compress(pages) == [(1, 1)] * 1000, pages)
pages = [Clears() for _ in range(1000)]
print(mc.mc_addr_expand([(7, 1), pages[:2], (9, 1)]) == [7, 1, 9], pages)
runs = pages = [[Clears(), 1] for _ in range(1000)]
print(mc.mc_addr_expand(runs) == [1] * 1000, runs)
pages = [1, 2, Clears(), 4, 5]
print(mc.mc_addr_compress(pages) == [(1, 2), (1, 1), (4, 2)], pages)
""")
    assert out.split() == ["True", "[]"] * 4


def test_numbers_are_read_as_int_reads_them():
    class Nine(int):
        def __int__(self):
            return 9
    assert mc.mc_addr_compress([4, Nine(5), True, np.int64(2)]) == [(4, 1), (9, 1), (1, 2)]
    assert mc.mc_addr_expand([(Nine(5), 1)]) == [9]
    assert mc.mc_addr_compress([2**32 + 3, -2**32 + 4]) == [(3, 2)]       # wraps as a C int does


def test_no_memory_is_an_exception_not_the_end_of_the_process():
    # 1 GiB is left; the sizes asked for take 2 GiB and more
    out = in_child("""
import resource
alloc = mc.mc_kv_allocator_create(8)
now = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (now + (1 << 30), -1))
def tried(f):
    try:
        return f()
    except MemoryError:
        return "MemoryError"
    except mc.McError as e:
        return mc.status_string(e.status)
most = 2**31 - 1
print(tried(lambda: mc.mc_addr_expand([(0, most)])))
print(tried(lambda: mc.mc_addr_expand([(0, most)], capacity=8)))
print(tried(lambda: mc.mc_addr_expand([(0, 2)] * 3, capacity=most)))
print(tried(lambda: mc.mc_addr_expand([(0, most)] * 3)))
print(tried(lambda: mc.mc_kv_alloc_pages(alloc, most)))
print(tried(lambda: mc.mc_kv_check_page_table([0], most)))
print(tried(lambda: mc.mc_kv_alloc_pages(alloc, 8)))
""")
    assert out.splitlines() == ["MemoryError", "MC_ERR_RANGE", "[0, 1, 0, 1, 0, 1]", "MC_ERR_RANGE",
                                "MC_ERR_NO_PAGES", "MemoryError", "[0, 1, 2, 3, 4, 5, 6, 7]"]


def test_iterators_are_refused():
    for numbers in (iter([1, 2]), (x for x in [1, 2]), map(int, "12")):
        with pytest.raises(TypeError):
            mc.mc_addr_compress(numbers)
    with pytest.raises(TypeError):
        mc.mc_addr_expand(iter([(1, 2)]))
    assert mc.mc_addr_compress({4: 0, 5: 0}) == [(4, 2)]        # what has a length is a list of numbers
    assert mc.mc_addr_compress("12") == [(1, 2)]
    assert mc.mc_addr_compress(range(3)) == [(0, 3)]


@pytest.mark.parametrize("scale", [0.5, 1, "0.5", np.float32(0.5), np.float64(0.5), True])
def test_scales_are_read_as_float_reads_them(scale):
    pool = mc.pool_desc(4096, 1, 1, 1, mc.MC_BF16)
    with pytest.raises(mc.McError) as e:        # read; then refused for the workspace of no bytes
        mc.mc_prefix_prefill_attn(pool, 0, 16, 1, 1, 1, 16, 16, 16, 16, scale, 16, 16, 16, 0, stream=0)
    assert e.value.status == mc.MC_ERR_INVALID
    for bad, error in ((None, TypeError), ("half", ValueError)):
        with pytest.raises(error):
            mc.mc_prefix_prefill_attn(pool, 0, 16, 1, 1, 1, 16, 16, 16, 16, bad, 16, 16, 16, 0, stream=0)


class Stands:
    def __init__(self, for_what):
        self._as_parameter_ = for_what


class Holds:
    def __init__(self, address):
        self.address = self.cuda_stream = address

    def data_ptr(self):
        return self.address


@pytest.mark.parametrize("one", [1, True, np.int64(1), ctypes.c_int32(1), Stands(1),
                                 Stands(Stands(ctypes.c_int32(1)))])
def test_counts_that_c_int32_takes(one):
    assert mc.mc_plan_remote_send(one, 0, 0, 5) == {"copy": (0, 1), "prefill": (1, 5), "send": (1, 5)}
    pool = mc.pool_desc(4096, 1, 1, 1, mc.MC_BF16)
    with pytest.raises(mc.McError) as e:        # the range reaches past the one layer
        mc.mc_kv_pack_range(pool, one, 2, 16, 1, 0, 1, 16, stream=0)
    assert e.value.status == mc.MC_ERR_RANGE


def test_arguments_of_other_types_never_reach_the_library():
    pool = mc.pool_desc(4096, 1, 1, 1, mc.MC_BF16)
    other = (ctypes.c_int32 * (ctypes.sizeof(pool) // 4))()
    for bad in (bytes(ctypes.sizeof(pool)), bytearray(ctypes.sizeof(pool)), other,
                np.zeros(ctypes.sizeof(pool), dtype=np.uint8), ctypes.pointer(pool), None, 4096):
        with pytest.raises(TypeError):
            mc.mc_kv_pack_range(bad, 0, 1, 16, 1, 0, 1, 16, stream=0)
    alloc = mc.mc_kv_allocator_create(8)
    for bad in (np.array([0, 0], dtype=np.int32), np.int64(16), b"8 bytes.", (ctypes.c_int32 * 2)(),
                ctypes.c_int64(16), 1.0, "x"):
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            mc.mc_kv_alloc_pages(bad, 1)
    for bad in (1.0, "1", None, ctypes.c_int64(1), ctypes.c_float(1), Stands("1")):
        with pytest.raises(ctypes.ArgumentError):
            mc.mc_plan_remote_send(bad, 0, 0, 5)
    own = Stands(None)
    own._as_parameter_ = own
    with pytest.raises(RecursionError):
        mc.mc_plan_remote_send(own, 0, 0, 5)
    for bad in (1.0, np.int64(16), b"x"):       # of data_ptr() and cuda_stream
        with pytest.raises(ctypes.ArgumentError):
            mc.mc_kv_pack_range(pool, 0, 1, Holds(bad), 1, 0, 1, 16, stream=0)
        with pytest.raises(ctypes.ArgumentError):
            mc.mc_kv_pack_range(pool, 0, 1, 16, 1, 0, 1, 16, stream=Holds(bad))
    for bad in (ctypes.c_int32(1), 1.0):        # counts that size a result: integers
        with pytest.raises(TypeError):
            mc.mc_kv_alloc_pages(alloc, bad)
        with pytest.raises(TypeError):
            mc.mc_addr_expand([(1, 1)], capacity=bad)
    mc.mc_kv_allocator_destroy(alloc)


def test_handles_and_addresses_in_every_form():
    alloc = mc.mc_kv_allocator_create(4)
    assert mc.mc_kv_alloc_pages(alloc.value, 1) == [0]
    assert mc.mc_kv_alloc_pages(Stands(alloc), np.int64(1)) == [1]
    assert mc.mc_kv_alloc_pages(ctypes.c_void_p(alloc.value), 2) == [2, 3]
    for null in (None, ctypes.c_void_p(None), 0):
        with pytest.raises(mc.McError) as e:
            mc.mc_kv_alloc_pages(null, 1)
        assert e.value.status == mc.MC_ERR_INVALID
    mc.mc_kv_allocator_destroy(alloc)
    pool = mc.pool_desc(4096, 1, 1, 1, mc.MC_BF16)
    for null in (None, 0, Holds(None), Holds(ctypes.c_void_p(None))):
        with pytest.raises(mc.McError) as e:
            mc.mc_kv_pack_range(pool, 0, 1, null, 1, 0, 1, 16, stream=Holds(None))
        assert e.value.status == mc.MC_ERR_INVALID


def test_the_library_alone_serves_the_calls_of_pools_and_plans(tmp_path):
    # a copy without the native module and without compilers: what goes through ctypes works, the rest
    # says what is missing
    src = os.path.join(ROOT, "paper_2412_12488_amd")
    shutil.copytree(src, tmp_path / "paper_2412_12488_amd",
                    ignore=shutil.ignore_patterns("_calls.so", "__pycache__"))
    out = in_child("""
alloc = mc.mc_kv_allocator_create(8)
print(mc.mc_abi_version(), mc.mc_kv_allocator_num_free(alloc), mc.mc_attn_workspace_size(1, 1, 32, 8) > 0)
try:
    mc.mc_kv_alloc_pages(alloc, 1)
except (RuntimeError, OSError):
    print("not built")
""", cwd=tmp_path, env=dict(os.environ, HIPCC="/nonexistent/hipcc", CXX="/nonexistent/g++"))
    assert out.split() == ["2", "8", "True", "not", "built"]
