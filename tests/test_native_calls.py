"""The extension module's plain calls against the same calls through the Python code: same results on the same memory formats,
and everything that is not plain is left to the Python code, whose errors stay what they were."""
import pytest
import torch

from paper_2604_18616_amd import binding


def modes():
    """The binding with the module and without it."""
    for native in (None, False):
        binding._native = native
        yield native
    binding._native = None


@pytest.fixture(autouse=True)
def restore():
    yield
    binding._native = None


def test_module_is_built_and_leaves_cpu_tensors_to_python():
    module = binding._load_native()
    assert module, "the extension module is missing: build() makes it"
    t, m = torch.zeros(1, 2, 3, 64, dtype=torch.bfloat16), torch.zeros(8, 8, dtype=torch.bfloat16)
    assert module.attn(t, t, t, False, None) is None
    assert module.attn(t, t, None, False, None) is None and module.attn(t, t) is None
    assert module.gemm(m, m, True) is None and module.gemm(m, "b", True) is None and module.gemm() is None
    for _ in modes():
        with pytest.raises(ValueError, match="no CPU path"):
            binding.attn_fwd(t, t, t)
        with pytest.raises(ValueError, match="no CPU path"):
            binding.gemm_bf16(m, m)


@pytest.mark.parametrize("fault", ["missing", "no library", "other torch"])
def test_a_module_that_does_not_fit_is_passed_by(tmp_path, monkeypatch, fault):
    if fault == "other torch":
        monkeypatch.setattr(torch, "__version__", "0.0.0")
    else:
        monkeypatch.setattr(binding, "NATIVE_PATH", str(tmp_path / "_native.so"))
        if fault == "no library":
            (tmp_path / "_native.so").write_bytes(b"not one")
    t = torch.zeros(1, 2, 3, 64, dtype=torch.bfloat16)
    binding._native = None
    with pytest.warns(UserWarning, match="extension module"):
        assert binding._load_native() is False
    with pytest.raises(ValueError, match="no CPU path"):     # by the Python code, and no second warning
        binding.attn_fwd(t, t, t)
    assert binding._native is False


def test_cpu_tensors_are_refused_without_the_library(tmp_path, monkeypatch):
    def build(*_):
        raise AssertionError("a library for a call that cannot be made")
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(binding, "build_library", build)
    monkeypatch.setattr(binding, "_lib", None)
    binding._native = None
    t, m = torch.zeros(1, 2, 3, 64, dtype=torch.bfloat16), torch.zeros(8, 8, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="no CPU path"):
        binding.attn_fwd(t, t, t)
    with pytest.raises(ValueError, match="no CPU path"):
        binding.gemm_bf16(m, m)


def rnd(*shape):
    return torch.randn(shape, device="cuda", dtype=torch.bfloat16)


LAYOUTS = {
    "contiguous": lambda B, H, S, D: rnd(B, H, S, D),
    "bshd": lambda B, H, S, D: rnd(B, S, H, D).transpose(1, 2),
    "cache": lambda B, H, S, D: rnd(B, H, S + 37, D)[:, :, :S],
    "wide rows": lambda B, H, S, D: rnd(B, H, S, D + 8)[..., :D],
    "one for all": lambda B, H, S, D: rnd(1, H, S, D).expand(B, H, S, D),
    "parameter": lambda B, H, S, D: torch.nn.Parameter(rnd(B, H, S, D)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,D,causal,scale", [(2, 8, 2, 1, 700, 128, False, None), (1, 4, 4, 5, 100, 64, True, 0.3),
                                                           (2, 4, 1, 200, 600, 128, True, None), (1, 2, 2, 129, 64, 64, False, 1.0)])
def test_attention_both_ways(layout, B, Hq, Hkv, Sq, Sk, D, causal, scale):
    torch.manual_seed(Sk)
    make = LAYOUTS[layout]
    q, k, v = make(B, Hq, Sq, D), make(B, Hkv, Sk, D), make(B, Hkv, Sk, D)
    print("native attn", layout, B, Hq, Hkv, Sq, Sk, D, causal, flush=True)
    got = [binding.attn_fwd(q, k, v, causal=causal, scale=scale) for _ in modes()]
    (o, lse), (o2, lse2) = got
    assert o.stride() == o2.stride() and lse.stride() == lse2.stride() and o.dtype == o2.dtype and lse.dtype == lse2.dtype
    assert not o.requires_grad and torch.equal(o, o2) and torch.equal(lse, lse2)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1, 1024, 4096), (64, 64, 64), (33, 70, 129), (300, 512, 96)])
@pytest.mark.parametrize("nk", [False, True])
@pytest.mark.parametrize("pad,offset", [(0, 0), (8, 0), (3, 1)])
def test_products_both_ways(M, N, K, nk, pad, offset):
    torch.manual_seed(M)

    def matrix(r, c):
        return rnd(r * (c + pad) + offset)[offset:].view(r, c + pad)[:, :c]
    a, b = matrix(M, K), matrix(N, K) if nk else matrix(K, N)
    print("native gemm", M, N, K, nk, pad, offset, flush=True)
    got = [binding.gemm_bf16(a, b, b_is_nk=nk) for _ in modes()]
    assert got[0].stride() == got[1].stride() and torch.equal(*got)


@pytest.mark.gpu
def test_refusals_stay_the_same():
    t, m = rnd(1, 2, 100, 64), rnd(64, 64)

    class Sub(torch.Tensor):
        pass
    calls = [
        lambda: binding.attn_fwd(t.half(), t, t), lambda: binding.attn_fwd(t[..., ::2], t, t), lambda: binding.attn_fwd(t[0], t, t),
        lambda: binding.attn_fwd(t, t, t[:, :, :50]), lambda: binding.attn_fwd(t, t[:, :1], t), lambda: binding.attn_fwd(t[:, :0], t, t),
        lambda: binding.attn_fwd(t[..., :32], t[..., :32], t[..., :32]), lambda: binding.attn_fwd(t, t, t, scale=-1.0),
        lambda: binding.attn_fwd(t, t, t, scale=float("nan")), lambda: binding.attn_fwd(t.cpu(), t, t), lambda: binding.attn_fwd(t, t, t, scale="x"),
        lambda: binding.attn_fwd(rnd(1, 2, 100, 66)[..., 1:65], t, t),
        lambda: binding.attn_fwd(rnd(1, 3, 100, 64), t, t), lambda: binding.gemm_bf16(m, m[:32]), lambda: binding.gemm_bf16(m.float(), m),
        lambda: binding.gemm_bf16(m.t(), m), lambda: binding.gemm_bf16(m[:0], m), lambda: binding.gemm_bf16(m, m.cpu()), lambda: binding.gemm_bf16(m[None], m),
    ]
    for i, call in enumerate(calls):
        said = []
        for _ in modes():
            with pytest.raises(Exception) as e:
                call()
            said.append((type(e.value), str(e.value)))
        assert said[0] == said[1], (i, said)
    # taken, if not as plain calls: a subclass, an integer scale, a number for a truth value
    o, _ = binding.attn_fwd(t, t, t, scale=0.125)
    for q, causal, scale in ((t.as_subclass(Sub), False, 0.125), (t, 0, 0.125)):
        assert torch.equal(binding.attn_fwd(q, t, t, causal=causal, scale=scale)[0].as_subclass(torch.Tensor), o)
    assert torch.equal(binding.attn_fwd(t, t, t, scale=1)[0], binding.attn_fwd(t, t, t, scale=1.0)[0])


@pytest.mark.gpu
def test_other_streams_and_capture():
    q, k, v = rnd(2, 8, 1, 128), rnd(2, 2, 900, 128), rnd(2, 2, 900, 128)
    a, b = rnd(4, 4096), rnd(512, 4096)
    want = binding.attn_fwd(q, k, v)[0], binding.gemm_bf16(a, b, b_is_nk=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = binding.attn_fwd(q, k, v)[0], binding.gemm_bf16(a, b, b_is_nk=True)
    side.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, c = binding.attn_fwd(q, k, v)[0], binding.gemm_bf16(a, b, b_is_nk=True)
    for _ in range(3):
        o.zero_(), c.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want[0]) and torch.equal(c, want[1])


@pytest.mark.gpu
def test_no_memory_for_the_parts_means_no_cut():
    q, k, v = rnd(1, 32, 64, 128), rnd(1, 8, 20000, 128), rnd(1, 8, 20000, 128)
    a, b = rnd(100, 14336), rnd(4096, 14336)
    lib = binding.load_library()
    assert lib.attn_fwd_workspace_bytes(1, 32, 8, 64, 20000, 128) > 4 << 20 and lib.gemm_bf16_workspace_bytes(100, 4096, 14336) > 4 << 20
    o, lse = torch.empty_like(q), torch.empty(1, 32, 64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert binding.attn_fwd_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), 1, 32, 8, 64, 20000, 128, False, 128 ** -0.5, stream) == 0
    c = binding.gemm_bf16(a, b, b_is_nk=True, tile=lib.gemm_bf16_auto_tile(100, 4096))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    spare = [torch.empty_like(x) for x in (o, c)]            # small blocks for the results below
    del spare
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + 1) / torch.cuda.get_device_properties(0).total_memory)
        full = []
        with pytest.raises(torch.cuda.OutOfMemoryError):
            while True:                                      # what is left of large blocks
                full.append(torch.empty(2 << 20, dtype=torch.uint8, device="cuda"))
        uncut = binding.attn_fwd(q, k, v)[0], binding.gemm_bf16(a, b, b_is_nk=True)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(uncut[0], o) and torch.equal(uncut[1], c)
