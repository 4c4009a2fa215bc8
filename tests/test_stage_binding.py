"""The native half of the Python binding (csrc/mbq_torch.cpp): what it refuses, and that buffers left to it give what kept
buffers give."""
import os
import struct
import sys

import pytest
import torch

import paper_2602_20191_amd as pkg

built = pytest.mark.skipif(not os.path.exists(os.path.join(os.path.dirname(pkg.__file__), "_mbq_torch.so")),
                           reason="library not built")


def inputs(device, T=5, K=256, Ns=(40, 16), P=4, seed=3):
    gen = torch.Generator().manual_seed(seed)
    X = torch.randn((T, K), generator=gen).to(torch.bfloat16).to(device)
    Wr = [(torch.randn((P, K), generator=gen) / K ** 0.5).to(device) for _ in Ns]
    br = [torch.zeros(P, device=device) for _ in Ns]
    W = [(0.02 * torch.randn((N, K), generator=gen)).to(device) for N in Ns]
    return X, Wr, br, W, list(Ns)


@built
def test_library_loads_without_the_native_half(monkeypatch):
    monkeypatch.setattr(pkg, "_lib", None)
    monkeypatch.setattr(pkg, "_native", None)
    monkeypatch.delattr(pkg, "_mbq_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2602_20191_amd._mbq_torch", None)  # an import of it fails
    assert pkg.load().mbq_version().startswith(b"mbq")
    X, Wr, br, W, Ns = inputs("cpu")
    with pytest.raises(pkg.MbqError, match="build it"):
        pkg.mbq_routed_linear_group(X, Wr, br, [torch.zeros(1 << 16, dtype=torch.uint8) for _ in Ns], Ns)


@pytest.mark.parametrize("missing", [RuntimeError("no compiler"), ImportError("no torch")])
def test_library_is_linked_without_the_native_half(monkeypatch, missing):
    from paper_2602_20191_amd import build

    commands = []

    def no_binding():
        raise missing

    monkeypatch.setattr(build, "hipcc", lambda: "hipcc")
    monkeypatch.setattr(build, "_run", lambda cmd: commands.append(cmd) or "")
    monkeypatch.setattr(build, "torch_command", no_binding)
    with pytest.raises(type(missing)):  # and is said, after the library is there
        build.build()
    assert len(commands) == len(build.SOURCES) + 1 and commands[-1][-len(build.SOURCES) - 2:][:2] == ["-o", build.LIB]


@built
def test_module_has_no_thread_local_storage():
    """A module with thread-local storage that nothing reads makes every thread-local access of the libraries loaded before it
    slow for the rest of the process (the C library's table of such modules is then never up to date), torch's own
    calls included."""
    with open(os.path.join(os.path.dirname(pkg.__file__), "_mbq_torch.so"), "rb") as f:
        elf = f.read()
    assert elf[:6] == b"\x7fELF\x02\x01"  # 64 bits, little endian
    table, size, count = struct.unpack_from("<Q", elf, 32)[0], *struct.unpack_from("<HH", elf, 54)
    kinds = [struct.unpack_from("<I", elf, table + i * size)[0] for i in range(count)]
    assert 1 in kinds and 7 not in kinds  # PT_LOAD, PT_TLS


@built
def test_stage_refuses_what_it_cannot_use():
    X, Wr, br, W, Ns = inputs("cpu")
    blobs = [torch.zeros(1 << 16, dtype=torch.uint8) for _ in Ns]
    with pytest.raises(pkg.MbqError):  # host memory
        pkg.mbq_routed_linear_group(X, Wr, br, blobs, Ns)
    with pytest.raises(AssertionError):
        pkg.mbq_routed_linear_group(X.float(), Wr, br, blobs, Ns)
    with pytest.raises(AssertionError):
        pkg.mbq_routed_linear_group(X, Wr[:1], br, blobs, Ns)
    with pytest.raises(AssertionError):
        pkg.mbq_routed_linear_group(X, [], [], [], [])
    with pytest.raises(TypeError):
        pkg.mbq_routed_linear_group(X, [1, 2], br, blobs, Ns)
    with pytest.raises(pkg.MbqError):
        pkg.mbq_routed_linear_group(X, Wr * 10, br * 10, blobs * 10, Ns * 10)


@built
@pytest.mark.parametrize("widths", [None, (4, 2, 2), (3, 1, 2, 2)])
@pytest.mark.parametrize("change", [lambda X: X.float(), lambda X: X.half(), lambda X: X.to(torch.uint8), lambda X: X[0],
                                    lambda X: X[None]])
def test_stage_refuses_activations_of_another_type_or_rank(widths, change):
    """Under every slice configuration: X is read as bf16, a type of one byte would be read past its end."""
    X, Wr, br, W, Ns = inputs("cpu", P=4 if widths is None else len(widths))
    blobs = [torch.zeros(1 << 16, dtype=torch.uint8) for _ in Ns]
    with pytest.raises(AssertionError):
        if widths is None:
            pkg.mbq_routed_linear_group(change(X), Wr, br, blobs, Ns)
        else:
            pkg.mbq_routed_linear_group_cfg(change(X), Wr, br, pkg.Config(widths), blobs, Ns)


@pytest.mark.gpu
@pytest.mark.parametrize("widths", [None, (4, 2, 2), (3, 1, 2, 2)])
@pytest.mark.parametrize("T", [0, 1, 5, 40, 130])
def test_stage_buffers_left_to_the_binding(mbq, widths, T):
    P = 4 if widths is None else len(widths)
    X, Wr, br, W, Ns = inputs("cuda", T=T, P=P)
    blobs = [mbq.mbq_encode(w) for w in W]
    cfg = None if widths is None else mbq.Config(widths)

    def call(**kept):
        if cfg is None:
            return mbq.mbq_routed_linear_group(X, Wr, br, blobs, Ns, **kept)
        return mbq.mbq_routed_linear_group_cfg(X, Wr, br, cfg, blobs, Ns, **kept)

    routing, Y = call()
    assert isinstance(routing, list) and isinstance(Y, list) and all(isinstance(r, tuple) and len(r) == 3 for r in routing)
    for r, y, N in zip(routing, Y, Ns):
        assert [t.shape for t in r] == [(T,), (T,), (5,)] and all(t.dtype == torch.int32 for t in r)
        assert y.shape == (T, N) and y.dtype == torch.float32 and y.device == X.device
    i32 = dict(dtype=torch.int32, device="cuda")
    kept = dict(routing=[[torch.empty(T, **i32), torch.empty(T, **i32), torch.empty(5, **i32)] for _ in Ns],
                Y=tuple(torch.full((T, N), float("nan"), device="cuda") for N in Ns),
                ws_route=mbq.route_workspace(T, X.shape[1], "cuda"), ws_linear=mbq.linear_workspace(T, max(Ns), X.shape[1], "cuda"))
    for names in (kept, ("Y",), ("routing", "ws_linear"), ("ws_route",)):
        got, y = call(**{name: kept[name] for name in names})
        for a, b in zip(routing, got):
            assert all(torch.equal(p, q) for p, q in zip(a, b))
        for i in range(len(Ns)):
            assert torch.equal(Y[i], y[i])
            assert "Y" not in names or y[i] is kept["Y"][i]
            assert "routing" not in names or got[i][0] is kept["routing"][i][0]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _, y = call()
    side.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(Y, y))
    with pytest.raises(mbq.MbqError, match="status"):  # the library's own check
        call(ws_linear=torch.empty(256, dtype=torch.uint8, device="cuda")[:255], ws_route=kept["ws_route"][:8])
    with pytest.raises(mbq.MbqError, match="contiguous"):
        call(Y=[torch.empty((N, T + 1), device="cuda").t()[:T] for N in Ns] if T > 1 else [torch.empty((T, N)) for N in Ns])


@pytest.mark.gpu
@pytest.mark.parametrize("widths", [None, (4, 2, 2)])
def test_stage_without_memory_for_its_outputs(mbq, widths):
    """An allocation that fails is torch's own exception, as for a tensor made in Python, and the next call works."""
    X, Wr, br, W, Ns = inputs("cuda", P=4 if widths is None else len(widths))
    blobs = [mbq.mbq_encode(w) for w in W]

    def call(X, Ns):
        if widths is None:
            return mbq.mbq_routed_linear_group(X, Wr, br, blobs, Ns)
        return mbq.mbq_routed_linear_group_cfg(X, Wr, br, mbq.Config(widths), blobs, Ns)

    with pytest.raises(torch.OutOfMemoryError):  # outputs of 4 TiB
        call(torch.zeros((1 << 16, X.shape[1]), dtype=torch.bfloat16, device="cuda"), [1 << 24] * len(Ns))
    _, Y = call(X, Ns)
    assert [y.shape for y in Y] == [(X.shape[0], N) for N in Ns] and all(bool(y.isfinite().all()) for y in Y)
