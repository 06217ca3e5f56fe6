"""The native issue of the per-token calls (csrc/thk_call.cpp): what it takes, what it leaves to the Python
code, and that both ways of issuing a call are the same call."""
import ctypes
import os
import subprocess
import sys

import pytest
import torch

import paper_2407_21018_amd as thk
from paper_2407_21018_amd import binding

D = 128


def _decode_args(device="cpu", dtype=torch.bfloat16):
    t = lambda *d: torch.zeros(*d, dtype=dtype, device=device)
    shape = thk.make_shape(1, 1, 8, 2, D, 40, 1, 64, 0, thk.THK_BF16, 0)
    return dict(shape=shape, q=t(1, 8, D), k_pruned=t(2, 40, 64), idx=torch.arange(64, dtype=torch.int16, device=device).repeat(2, 1),
                v=t(2, 40, D), k_tail=t(2, 16, D), v_tail=t(2, 16, D), s_tail=3, s_tail_cap=16, out=t(1, 8, D),
                ws=torch.zeros(1 << 16, dtype=torch.uint8, device=device), stream=0)


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("name,make", [
    ("q", lambda x: x.data_ptr()), ("q", lambda x: x[:, :7]), ("q", lambda x: None), ("k_pruned", lambda x: x.transpose(0, 1)),
    ("v", lambda x: x.as_subclass(_Sub)), ("out", lambda x: x.to_sparse()), ("k_tail", lambda x: x[:, ::2]), ("k_tail", lambda x: x[:, :2]),
    ("idx", lambda x: [0]), ("s_tail", lambda x: True), ("s_tail", lambda x: 3.0), ("s_tail", lambda x: 1 << 40), ("ws", lambda x: (1, 2)),
    ("stream", lambda x: "0"), ("shape", lambda x: b"short")])
def test_other_forms_are_left_to_the_python_code(name, make):
    thk.load()
    a = _decode_args()
    a["s_tail"] = 17                                  # more than the tail holds: refused in front of any launch
    assert binding._call.decode_attn(*a.values()) == 2   # ... by the library: the plain form is taken
    a[name] = make(a[name])
    assert binding._call.decode_attn(*a.values()) == -1
    assert binding._call.decode_attn(*list(a.values())[:-1]) == -1


def test_a_tensor_without_memory_is_a_null_pointer_both_ways():
    a = _decode_args()
    a["q"] = a["q"].to("meta")
    thk.load()
    assert binding._call.decode_attn(*a.values()) == 1
    a["q"] = 0                                        # the same, as an address
    with pytest.raises(thk.ThkError) as e:
        thk.thk_decode_attn(*a.values())
    assert e.value.status == 1


def test_checks_raise_as_before():
    a = _decode_args()
    for name, bad, what in (("q", lambda x: x[:, :7], "q holds"), ("v", lambda x: x.transpose(0, 1), "v must be contiguous"),
                            ("k_tail", lambda x: x[:, :2].contiguous(), "k_tail holds")):
        b = dict(a)
        b[name] = bad(b[name])
        with pytest.raises(ValueError, match=what):
            thk.thk_decode_attn(*b.values())
    with pytest.raises(thk.ThkError):                              # a status of the library
        thk.thk_tail_append(a["shape"], a["q"], a["q"], a["k_tail"], a["v_tail"], 16, 16, 0)


def _four_calls(shape, device="cpu"):
    """(native function, public function, arguments) of the four calls, every tensor of one size and large enough for _decode_args' shape."""
    t = lambda: torch.zeros(1 << 15, dtype=torch.bfloat16, device=device)
    idx, ws = torch.arange(64, dtype=torch.int16, device=device).repeat(2), torch.zeros(1 << 16, dtype=torch.uint8, device=device)
    thk.load()
    c = binding._call
    return [(c.decode_attn, thk.thk_decode_attn, (shape, t(), t(), idx, t(), t(), t(), 3, 16, t(), ws, 0)),
            (c.decode_attn_kv, thk.thk_decode_attn_kv, (shape, t(), t(), idx, t(), idx, 64, 64, t(), t(), 3, 16, t(), ws, 0)),
            (c.tail_append, thk.thk_tail_append, (shape, t(), t(), t(), t(), 3, 16, 0)),
            (c.prune, thk.thk_prune, (shape, t(), t(), None, idx, t(), ws, 0))]


def _refused(calls):
    """The four calls with a value that the library refuses in front of any launch, and the status it gives."""
    decode, decode_kv, append, prune = [list(args) for _, _, args in calls]
    decode[7] = decode_kv[10] = 17                    # more rows than the tail holds
    append[5] = 16                                    # no room for another one
    prune[6] = None                                   # no workspace
    return [(native, public, args, status) for (native, public, _), args, status in zip(calls, (decode, decode_kv, append, prune), (2, 2, 2, 5))]


@pytest.mark.parametrize("stream", [0, None])
def test_each_call_is_taken(stream):
    """In the plain form every one of the four reaches the library: its status comes back, not -1."""
    calls = _refused(_four_calls(_decode_args()["shape"]))
    asked = []
    binding._forget_runtime()                         # as at the start of a process
    try:
        if stream is None:
            assert calls[0][0](*calls[0][2][:-1], None) == -1     # the current stream is not known before the runtime is up
            binding._call.stream_getters(lambda device: asked.append(device) or 0, lambda: 3)
        for native, public, args, status in calls:
            args[-1] = stream
            assert native(*args) == status
            with pytest.raises(thk.ThkError) as e:
                public(*args)
            assert e.value.status == status
    finally:
        binding._forget_runtime()
    assert asked == ([3] * 8 if stream is None else [])


@pytest.mark.parametrize("fields", [dict(S_cap=1 << 56), dict(S_cap=(1 << 57) + 40), dict(S=1 << 56), dict(S_cap=1 << 62, T=128), dict(L=1 << 30, B=1 << 30, N_kv=8),
                                    dict(S=(1 << 63) - 1, S_recent=-1), dict(L=1 << 30, B=1 << 29, N_q=16, N_kv=16)])
def test_sizes_beyond_64_bits_are_no_small_sizes(fields):
    """A product of sizes that does not fit 64 bits must not pass for a small one: such a call would read and
    store behind its tensors."""
    shape = _decode_args()["shape"]
    for k, v in fields.items():
        setattr(shape, k, v)
    for native, public, args in _four_calls(shape):
        if public is thk.thk_tail_append and not {"L", "B"} & set(fields):
            continue   # its sizes do not depend on the sequence
        assert native(*args) == -1
        with pytest.raises(ValueError, match="the shape needs"):
            public(*args)


class _OtherStruct(ctypes.Structure):
    _fields_ = thk.thk_shape._fields_


@pytest.mark.parametrize("other", [bytes, bytearray, lambda s: memoryview(bytes(s)), _OtherStruct.from_buffer_copy])
def test_only_a_shape_is_a_shape(other):
    """Whatever else holds as many bytes is refused, as ctypes does."""
    bad = other(_decode_args()["shape"])
    for native, public, args in _four_calls(bad):
        assert native(*args) == -1
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            public(*args)


@pytest.mark.parametrize("found", [None, b"no library"])
def test_the_library_works_without_the_native_issue(found, tmp_path):
    """libthk.so needs neither an interpreter nor a torch of one version; what does may be missing or not load."""
    pkg = tmp_path / "paper_2407_21018_amd"
    pkg.mkdir()
    src = os.path.dirname(binding.__file__)
    for f in ("__init__.py", "binding.py", "libthk.so"):
        os.symlink(os.path.join(src, f), pkg / f)
    if found is not None:
        (pkg / "_thk_call.so").write_bytes(found)
    code = """if True:
        import warnings, torch
        import paper_2407_21018_amd as thk
        from paper_2407_21018_amd import binding
        with warnings.catch_warnings(record=True) as w:
            warnings.simplefilter("always")
            assert thk.thk_version() > 0 and thk.thk_version() > 0
        assert [x.category for x in w] == [RuntimeWarning] and "ctypes" in str(w[0].message) and binding._call is None
        t = torch.zeros(2048, dtype=torch.bfloat16)
        try:
            thk.thk_tail_append(thk.make_shape(1, 1, 8, 2, 128, 40, 1, 64), t, t, t, t, 8, 8, 0)   # refused by the library
        except thk.ThkError as e:
            assert e.status == 2
        else:
            raise AssertionError
        binding._forget_runtime()
    """
    subprocess.run([sys.executable, "-c", code], check=True, cwd=tmp_path, env={**os.environ, "PYTHONPATH": str(tmp_path)}, timeout=300)


class _Watched:
    """The native module, and what its calls returned."""

    def __init__(self, module):
        self.module, self.returned = module, []

    def __getattr__(self, name):
        f = getattr(self.module, name)

        def call(*a):
            st = f(*a)
            self.returned.append((name, st))
            return st
        return call


@pytest.mark.gpu
@pytest.mark.parametrize("side_stream", [False, True])
def test_both_ways_of_issuing_a_call_agree(side_stream, monkeypatch):
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    rnd = lambda *d: torch.randn(*d, generator=g, device="cuda").to(torch.bfloat16)
    U, S, T, cap = 6, 700, 76, 32
    kept = lambda: torch.rand(U, D, generator=g, device="cuda").argsort(-1)[:, :T].sort(-1).values.to(torch.int16).contiguous()
    shape = thk.make_shape(1, 2, 12, 3, D, S, 16, T, 0, thk.THK_BF16, 0)
    q, k, v, kn, vn, q_obs = rnd(2, 12, D), rnd(U, S, D), rnd(U, S, D), rnd(U, D), rnd(U, D), rnd(2, 12, 16, D)
    vp, idxv, tail = rnd(U, S, T), kept(), rnd(U, cap, D)
    st = torch.cuda.Stream() if side_stream else torch.cuda.current_stream()
    st.wait_stream(torch.cuda.current_stream())

    def run(arg):
        score, idx = torch.zeros(U, D, device="cuda"), torch.zeros(U, T, dtype=torch.int16, device="cuda")
        kp, kt, vt = torch.zeros(U, S, T, dtype=q.dtype, device="cuda"), tail.clone(), tail.clone()
        out, out_kv = torch.zeros_like(q), torch.zeros_like(q)
        ws = torch.zeros(max(thk.thk_workspace_bytes(shape, o) for o in (thk.THK_OP_DECODE, thk.THK_OP_PRUNE)), dtype=torch.uint8, device="cuda")
        w = ws if arg is None else (ws.data_ptr(), ws.numel())
        p = (lambda x: x) if arg is None else (lambda x: x.data_ptr())
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):
            thk.thk_prune(shape, p(q_obs), p(k), p(score), p(idx), p(kp), w)
            thk.thk_tail_append(shape, p(kn), p(vn), p(kt), p(vt), 4, cap)
            thk.thk_decode_attn(shape, p(q), p(kp), p(idx), p(v), p(kt), p(vt), 5, cap, p(out), w)
            thk.thk_decode_attn_kv(shape, p(q), p(kp), p(idx), p(vp), p(idxv), T, T, p(kt), p(vt), 5, cap, p(out_kv), w)
        torch.cuda.synchronize()
        return score, idx, kp, kt, vt, out, out_kv

    run(None)                                         # the first call of a process sets the stream getters
    watched = _Watched(binding._call)
    monkeypatch.setattr(binding, "_call", watched)
    native = run(None)
    names = ["prune", "tail_append", "decode_attn", "decode_attn_kv"]
    assert watched.returned == [(n, 0) for n in names]            # taken, and issued
    watched.returned.clear()
    for x, y in zip(native, run("addresses")):
        assert torch.equal(x, y)
    assert watched.returned == [(n, -1) for n in names]           # addresses are left to the Python code
    assert native[5].abs().max() > 0
