"""The extension that makes the plain calls (csrc/fastcall.cpp): what it takes it hands to the C ABI unchanged, everything else it
leaves, having done nothing, to the general code of binding.py."""
import os
import sys
import sysconfig

import pytest
import torch

from paper_2510_14719_amd import binding, build

Q, K, V, O, L = 0x10000000, 0x20000000, 0x30000000, 0x40000000, 0x50000000     # validation never dereferences them


@pytest.fixture(scope="module")
def fast():
    return binding._load_fast()


def test_addresses_reach_the_c_abi_in_order(fast):
    # every code of the argument check, none of which launches anything
    ok = [Q, K, V, O, L, 1, 2, 1024, 128, 0.088, False, 0, 0]
    for f in (fast.attn_fwd, fast.attn_fwd_fp8):
        for i in range(5):
            assert f(*ok[:i], 0, *ok[i + 1:]) == -1
            assert f(*ok[:i], ok[i] + 4, *ok[i + 1:]) == -4
        for i in (5, 6, 7, 8):
            assert f(*ok[:i], 0, *ok[i + 1:]) == -2
        assert f(*ok[:9], -0.5, *ok[10:]) == -3 and f(*ok[:9], 0, *ok[10:]) == -3
        assert f(*ok[:12], 2) == -2
        assert f(*ok[:7], 2 ** 23, *ok[8:]) == -5
        assert f(Q, K, V, Q, *ok[4:]) == -7
    for f in (fast.gemm_nt, fast.gemm_nt_fp8):
        ok = [Q, K, V, 256, 512, 128, 0, 1]
        assert f(0, *ok[1:]) == -1 and f(Q, 0, *ok[2:]) == -1 and f(Q, K, 0, *ok[3:]) == -1
        assert f(Q, K, V, 0, *ok[4:]) == -2 and f(Q, K, V, 256, 0, *ok[5:]) == -2 and f(*ok[:5], 48, *ok[6:]) == -2 and f(*ok[:7], 2) == -2
        assert f(Q + 8, *ok[1:]) == -4 and f(Q, K, V + 1, *ok[3:]) == -4
        assert f(Q, K, Q, *ok[3:]) == -7


def test_it_names_the_torch_it_was_built_for(fast, monkeypatch):
    # it reads torch's objects by the layout of the headers it was compiled with: another torch is refused before anything is read
    assert fast.built_for == binding.torch_build() and torch.__version__ in fast.built_for
    assert fast.__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(binding, "_fast", None)
    monkeypatch.setattr(torch.version, "git_version", "0" * 40)
    with pytest.warns(RuntimeWarning, match="built for torch"):
        assert binding._load_fast() is binding._NoExtension


def test_calls_do_without_the_extension(monkeypatch):
    monkeypatch.setattr(binding, "_fast", None)
    monkeypatch.setitem(sys.modules, "paper_2510_14719_amd._fastcall", None)     # (as where it has not been built)
    with pytest.warns(RuntimeWarning, match="general code"), pytest.raises(binding.AttnFwdError) as e:
        binding.attn_fwd(0, K, V, O, L, 1, 1, 64, 64, 0.125, False, stream=0, dtype=0)
    assert e.value.code == -1
    for f, args in ((binding.attn_fwd_fp8, (Q, K, V, O, L, 1, 1, 64, 96, 0.125, False, 0, 0)), (binding.gemm_nt, (Q, K, V, 64, 64, 48, 0, 0)),
                    (binding.gemm_nt_fp8, (Q, K, V, 64, 64, 48, 0, 0))):
        with pytest.raises(RuntimeError) as e:
            f(*args)
        assert e.value.code == -2


def test_the_library_builds_without_the_headers_of_the_extension(monkeypatch, capsys, tmp_path):
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_fastcall() == "" and "not built" in capsys.readouterr().out
    monkeypatch.setitem(sys.modules, "torch", None)
    assert build.build_fastcall() == "" and "no torch" in capsys.readouterr().out


class Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("place,value", [(0, torch.zeros(4)), (0, torch.zeros(4).as_subclass(Sub)), (0, None), (0, 1.0), (0, -1), (0, 2 ** 64), (5, 1.0), (5, True),
                                         (5, 2 ** 32 + 1), (5, torch.tensor(1)), (9, "1"), (9, None), (9, 10 ** 400), (10, None), (10, 1.0), (11, None), (11, 0.0),
                                         (11, "s"), (12, None), (12, 1.0), (12, True)])
def test_what_is_not_taken(fast, place, value):
    args = [0, K, V, O, L, 1, 2, 1024, 128, 0.088, False, 0, 0]                # (NULL: a call that is taken returns -1)
    assert fast.attn_fwd(*args) == -1
    args[place] = value
    assert fast.attn_fwd(*args) is NotImplemented and fast.attn_fwd_fp8(*args) is NotImplemented
    args = [0, K, V, 256, 512, 128, 0, 0]
    where = {0: 0, 5: 4, 11: 6, 12: 7}.get(place)
    if where is not None:
        args[where] = value
        assert fast.gemm_nt(*args) is NotImplemented and fast.gemm_nt_fp8(*args) is NotImplemented
    assert fast.attn_fwd() is NotImplemented and fast.gemm_nt(*args, 0) is NotImplemented


def test_errors_are_those_of_the_general_code():
    x = torch.zeros(1, 1, 64, 64, dtype=torch.float16)
    with pytest.raises(ValueError, match="device tensors"):
        binding.attn_fwd(x, x, x, x, x, 1, 1, 64, 64, 0.125, False, stream=0)
    with pytest.raises(ValueError, match="pass dtype"):
        binding.gemm_nt(x.float(), x, x, 64, 64, 64, stream=0)
    with pytest.raises(binding.AttnFwdError) as e:
        binding.attn_fwd(0, K, V, O, L, 1, 1, 64, 64, 0.125, False, stream=0, dtype=0)
    assert e.value.code == -1
    with pytest.raises(binding.GemmNtError) as e:
        binding.gemm_nt_fp8(Q, K, V, 64, 64, 48, stream=0)
    assert e.value.code == -2


@pytest.mark.skipif(not hasattr(os, "fork"), reason="needs fork")
def test_a_forked_child_takes_the_general_code(fast):
    pid = os.fork()
    if pid == 0:
        os._exit(0 if fast.gemm_nt(0, K, V, 256, 512, 128, 0, 0) is NotImplemented else 1)
    assert os.waitpid(pid, 0)[1] == 0
    assert fast.gemm_nt(0, K, V, 256, 512, 128, 0, 0) == -1


@pytest.mark.gpu
def test_device_tensors_streams_and_modes(fast):
    from torch.overrides import TorchFunctionMode
    print("device tensors, streams, modes", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((1, 2, 130, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))

    def call(stream=None, **kw):
        o, lse = torch.full_like(q, float("nan")), torch.full((1, 2, 130), float("nan"), device="cuda")
        torch.cuda.synchronize()
        binding.attn_fwd(q, k, v, o, lse, 1, 2, 130, 64, 0.125, True, stream, **kw)
        torch.cuda.synchronize()
        return o, lse

    o0, l0 = call(dtype=binding.BF16, stream=torch.cuda.current_stream())      # a stream object: the general code
    assert not o0.isnan().any()
    side = torch.cuda.Stream()

    class Seen(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    results = [call(), call(dtype=binding.BF16), call(stream=side.cuda_stream), call(stream=side)]
    with torch.cuda.stream(side):
        results.append(call())
    with Seen():
        assert fast.attn_fwd(q, k, v, q, l0, 1, 2, 130, 64, 0.125, True, None, None) is NotImplemented
        results.append(call())
    for o, l in results:
        assert torch.equal(o, o0) and torch.equal(l, l0)
    # torch's current stream is the one that is used: a captured call runs at each replay only
    o, lse = torch.zeros_like(q), torch.zeros_like(l0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.attn_fwd(q, k, v, o, lse, 1, 2, 130, 64, 0.125, True)
    torch.cuda.synchronize()
    assert not o.any()
    for _ in range(3):
        o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, o0) and torch.equal(lse, l0)
    # not contiguous: refused, whoever looks
    t = q.transpose(1, 2)
    assert fast.attn_fwd(t, k, v, o, lse, 1, 2, 130, 64, 0.125, True, None, 1) is NotImplemented
    with pytest.raises(ValueError, match="contiguous"):
        binding.attn_fwd(t, k, v, o, lse, 1, 2, 130, 64, 0.125, True)
    # every other address in front of a plain pointer
    a, b = torch.randn((40, 64), generator=gen, device="cuda").half(), torch.randn((24, 64), generator=gen, device="cuda").half()
    c, c2 = torch.empty((40, 24), dtype=torch.float16, device="cuda"), torch.empty((40, 24), dtype=torch.float16, device="cuda")
    binding.gemm_nt(a, b, c, 40, 24, 64)
    binding.gemm_nt(a.data_ptr(), b.data_ptr(), c2.data_ptr(), 40, 24, 64, torch.cuda.current_stream(), binding.FP16)
    torch.cuda.synchronize()
    assert torch.equal(c, c2) and (c.double() - a.double() @ b.double().T).abs().max() < 0.05
