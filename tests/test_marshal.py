"""The binding's host module agrees with the Python code it stands in for, and leaves it what it does not know."""
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2402_01798_amd import binding as B

M = B._tq_marshal
BIG = B._ANY_SIZE


def test_built():
    assert M is not None


@pytest.mark.parametrize("built", [True, False])
def test_a_module_that_does_not_load_is_told(built, tmp_path):
    pkg = tmp_path / "paper_2402_01798_amd"
    pkg.mkdir()
    for name in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(B.HERE, name), pkg)
    if built:
        (pkg / "_tq_marshal.so").write_bytes(b"not a library")
    run = subprocess.run([sys.executable, "-c", "from paper_2402_01798_amd import binding as b; assert b._tq_marshal is None"],
                         cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr
    assert ("_tq_marshal.so does not load" in run.stderr) == built


@pytest.mark.parametrize("functions", ["", "pointers = sized = lambda *a: None", "interface = 2"])
def test_a_module_of_other_sources_is_not_used(functions, tmp_path):
    """One that loads but was built before (or after) the functions the binding calls: told, and the calls go the Python way."""
    pkg = tmp_path / "paper_2402_01798_amd"
    (pkg / "_tq_marshal").mkdir(parents=True)
    for name in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(B.HERE, name), pkg)
    (pkg / "_tq_marshal" / "__init__.py").write_text(functions)
    (pkg / "_tq_marshal.so").write_bytes(b"the package above it is found first")
    program = """if True:
        import torch
        from paper_2402_01798_amd import binding as b
        t = torch.zeros(4)
        for call in (lambda: b.tq_stats(t, t, t), lambda: b.tq_params_multi([t], [t], 3, 0), lambda: b.tq_compress(t, t, t, 3, 0, 0, 0)):
            try:
                call()
            except (ValueError, b.TqError):
                continue
            raise AssertionError("not refused")
    """
    run = subprocess.run([sys.executable, "-c", program], cwd=tmp_path, capture_output=True, text=True, timeout=300,
                         env={**os.environ, "TQ_LIBRARY_PATH": B.LIB_PATH})
    assert run.returncode == 0, run.stderr
    assert "_tq_marshal.so does not load" in run.stderr


def test_sized():
    ts = [torch.zeros(8), torch.nn.Parameter(torch.zeros(8)), torch.zeros(2, 4)]
    for seq in (ts, tuple(ts)):
        assert M.sized(seq, 3, 8, 8, None) and M.sized(seq, 3, 8, 8, torch.float32) and M.sized(seq, 3, 0, BIG, None)
        assert not M.sized(seq, 2, 8, 8, None) and not M.sized(seq, 3, 8, 8, torch.bfloat16)
        assert not M.sized(seq, 3, 9, BIG, None) and not M.sized(seq, 3, 0, 7, None)
    assert M.sized([], 0, 1, 1, None)
    # not a list, not a tensor, no dtype: the Python code's business
    assert not M.sized(iter(ts), 3, 8, 8, None) and not M.sized([1, 2], 2, 0, BIG, None) and not M.sized(ts, 3, 8, 8, "f32")
    with pytest.raises(TypeError):
        M.sized(ts, 3)


class Reversed(list):
    """A list whose elements are not what it stores."""

    def __iter__(self):
        return reversed(list(super().__iter__()))


class Pair(tuple):
    def __len__(self):
        return 1


def test_lists_of_their_own_kind_are_left_to_python():
    small = torch.zeros(4)
    assert not M.sized(Reversed([small, small]), 2, 4, 4, None) and M.pointers(Reversed()) is None
    assert not M.sized(Pair((small, small)), 2, 4, 4, None) and M.pointers(Pair()) is None


def test_pointers_are_left_to_python_off_the_device():
    assert M.pointers([torch.zeros(8)]) is None and M.pointers([None]) is None and M.pointers(iter([])) is None
    assert M.pointers([torch.zeros(8, device="meta")]) is None and M.pointers([]) == b""
    with pytest.raises(ValueError, match="g must be a contiguous device tensor"):
        B._ptr_array([torch.zeros(8)], "g")
    assert M.pointers([], 0, 1, 1, None) == b"" and M.pointers([], 1, 0, BIG, None) is None
    with pytest.raises(TypeError):
        M.pointers([], 0)
    with pytest.raises(TypeError):
        M.pointers([], "0", 0, 0, None)


def test_sizes_are_still_refused():
    d = 1024
    g, q, p = torch.zeros(d), torch.zeros(B.PARAMS_BYTES, dtype=torch.uint8), torch.zeros(B.payload_bytes(d, 3), dtype=torch.uint8)
    with pytest.raises(ValueError, match="share shape and dtype"):
        B.tq_compress_multi([g, g.bfloat16()], [q, q], [p, p], 3, 1, 0, 0)
    with pytest.raises(ValueError, match="does not match d"):
        B.tq_compress_multi([g, g], [q, q], [p, p[:-1]], 3, 1, 0, 0)
    with pytest.raises(ValueError, match="does not match d"):
        B.tq_decompress_aggregate([p, p], [q, q[:-1]], g, 3)


@pytest.mark.gpu
def test_pointers_on_the_device():
    a, b = torch.zeros(64, device="cuda"), torch.zeros(8, 8, device="cuda")
    assert M.pointers([a, b]) == b"".join(t.data_ptr().to_bytes(8, "little") for t in (a, b))
    assert M.pointers([a, b.t()]) is None and M.pointers([a, a.cpu()]) is None
    # with the sizes and the type that are wanted
    assert M.pointers((a, b), 2, 64, 64, torch.float32) == M.pointers([a, b], 2, 0, BIG, None) == M.pointers([a, b])
    for wanted in ((1, 64, 64, None), (3, 64, 64, None), (2, 65, BIG, None), (2, 0, 63, None), (2, 64, 64, torch.bfloat16), (2, 64, 64, "f32")):
        assert M.pointers([a, b], *wanted) is None, wanted
    assert M.pointers([a, b[:7]], 2, 64, BIG, None) is None


CALLS = {"stats": 6, "stats_multi": 6, "params": 6, "params_multi": 6, "compress": 10, "compress_multi": 10, "aggregate": 8,
         "update": 11, "simulate": 10, "stats_segments": 8, "stats_segments_multi": 8, "compress_segments": 11,
         "compress_segments_multi": 11, "aggregate_segments": 10}


@pytest.mark.parametrize("name", CALLS)
def test_whole_calls_leave_what_they_do_not_know(name):
    """Host tensors, other objects in every place, too few or too many arguments, no entry point: None, and no exception is
    left behind.  The address is never called: there is no device tensor here."""
    t, call = torch.zeros(4096), getattr(M, name)
    assert sorted(B._NATIVE.values()) == sorted(CALLS)
    for address in (0, 1 << 40, -1, 1 << 70, None):
        for filler in (t, [t], [], (t, t), 1, -1, 1 << 70, 0.5, True, None, "x"):
            for count in (0, CALLS[name] - 2, CALLS[name] - 1, CALLS[name]):
                assert call(address, *[filler] * count) is None
