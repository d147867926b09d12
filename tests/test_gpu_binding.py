"""The native checks of the binding (csrc/binding.cpp) against the Python
checks they stand in front of: plain calls give the same results on either
path (an explicit stream takes the Python path), and every argument that the
Python checks refuse is declined natively, so that the reason is raised."""

import ctypes
import weakref

import pytest
import torch

import paper_2402_02082_amd as glide
from paper_2402_02082_amd import _lib
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

B, N, H, L, G, V = 2, 6, 3, 40, 4, 1001
I32, F32, BF = torch.int32, torch.float32, torch.bfloat16


def _rand(shape, dtype=BF):
    return torch.randn(shape, device="cuda").to(dtype)


def _ints(shape):
    return torch.zeros(shape, dtype=I32, device="cuda")


def _probs(shape):
    return torch.softmax(3 * _rand(shape, F32), dim=-1)


def _tree():
    return torch.arange(-1, N - 1, dtype=I32, device="cuda").repeat(B, 1).contiguous()


def _calls():
    """name -> (function, native name, positional arguments, output positions)"""
    lens = torch.tensor([30, 11], dtype=I32, device="cuda")
    caches = [[_rand((B, H, L, 128)) for _ in range(2)] for _ in range(2)]
    attn = [_rand((B, N, H, 128)), *[c[0] for c in caches], lens, _tree(), _rand((B, N, H, 128)), 0.0, 0, None]
    return {
        "attn": (glide.glide_tree_attn, "tree_attn", attn, [5]),
        "cross": (glide.glide_tree_attn, "tree_attn", attn[:4] + [None] + attn[5:7] + [3, None], [5]),
        "commit": (glide.glide_verify_commit, "verify_commit",
                   [_rand((B, N + 1, V), F32), _ints((B, N)), _tree(), *caches, lens, _ints((B,)),
                    _ints((B, N + 1)), _ints((B,)), _ints((B,)), None, _ints((B, N))], [6, 7, 8, 9, 11]),
        "cape": (glide.cape_expand, "cape", [_probs((B, G, V)), 3, 16, _ints((B, 16)), _ints((B, 16)),
                                             _ints((B,)), False, None], [3, 4, 5]),
        "sample": (glide.spec_sample_verify, "spec_sample",
                   [_ints((B, G)), _probs((B, G, V)), _probs((B, G + 1, V)),
                    torch.rand((B, G + 1), device="cuda"), _ints((B,)), _ints((B,))], [4, 5]),
        "rows": (glide.glide_rows_matmul, "rows_matmul", [_rand((5, 64)), _rand((33, 64)), _rand((5, 33), F32)],
                 [2]),
        "block": (glide.glide_block_attn, "block_attn",
                  [_rand((B, L, H, 128)), caches[0][0], caches[1][0], _rand((B, L, H, 128)), 5, 0.0], [3]),
    }


NAMES = ["attn", "cross", "commit", "cape", "sample", "rows", "block"]


@pytest.mark.parametrize("name", NAMES)
def test_native_equals_python_path(name):
    require_gpu()
    torch.manual_seed(3)
    fn, native, args, outs = _calls()[name]
    fn(*args)  # workspaces exist from here on
    assert getattr(_lib._bind(), native)(*args, None) == 0
    torch.cuda.synchronize()
    got = [args[i].clone() for i in outs]
    for i in outs:
        args[i].fill_(77)
    fn(*args, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    for g, i in zip(got, outs):
        assert torch.equal(g, args[i])


@pytest.mark.parametrize("name", NAMES)
def test_native_declines_what_python_refuses(name):
    require_gpu()
    fn, native, args, _ = _calls()[name]
    nat = getattr(_lib._bind(), native)

    def refused(bad):
        assert nat(*bad, None) is None
        with pytest.raises((ValueError, TypeError, AttributeError)):
            fn(*bad)

    for i, a in enumerate(args):
        if isinstance(a, torch.Tensor):
            bad = [a.cpu(), a.to(torch.float16), a[1:].contiguous(), a.unsqueeze(0).contiguous(),
                   torch.stack([a, a], dim=-1)[..., 0], a.tolist()]
        elif isinstance(a, list):
            bad = [a[:1], a[:1] + [a[1].cpu()], a[:1] + [a[1][:, :, :-1].contiguous()], a[:1] + [a[1].to(F32)],
                   a[:1] + [torch.stack([a[1], a[1]], dim=-1)[..., 0]]]
        else:
            continue
        for x in bad:
            if name == "attn" and i == 4 or not (isinstance(x, torch.Tensor) and x.shape == a.shape
                                                 and x.dtype == a.dtype and x.is_cuda and x.is_contiguous()):
                refused(args[:i] + [x] + args[i + 1:])


@pytest.mark.parametrize("dtype", [BF, F32], ids=["bf16", "f32"])
def test_commit_moves_the_same_rows_on_either_path(dtype):
    """The commit of a path that skips nodes, so that rows move in every layer's
    K and V (three layers, five heads, other lengths in each sequence): every
    output and cache is the same on either path, and the rows are the accepted
    nodes' own."""
    require_gpu()
    torch.manual_seed(4)
    layers, heads, cap, path = 3, 5, 37, [1, 3, 5]
    parents = torch.tensor([[-1, -1, 0, 1, 1, 3]] * B, dtype=I32, device="cuda")
    tokens = torch.arange(10, 10 + B * N, dtype=I32, device="cuda").view(B, N)
    logits = _rand((B, N + 1, V), F32)
    for b in range(B):
        for n in path:
            logits[b, int(parents[b, n]) + 1, int(tokens[b, n])] = 50.0
    lens = torch.tensor([30, 11], dtype=I32, device="cuda")
    start = [[_rand((B, heads, cap, 128), dtype) for _ in range(layers)] for _ in range(2)]
    results = []
    for explicit in (False, True):   # an explicit stream takes the Python path
        caches = [[t.clone() for t in ts] for ts in start]
        outs = [_ints((B,)), _ints((B, N + 1)), _ints((B,)), _ints((B,)), _ints((B,)), _ints((B, N))]
        args = [logits, tokens, parents, *caches, lens, *outs]
        if explicit:
            glide.glide_verify_commit(*args, stream=torch.cuda.current_stream())
        else:
            assert _lib._bind().verify_commit(*args, None) == 0
        torch.cuda.synchronize()
        results.append(outs + caches[0] + caches[1])
    for x, y in zip(*results):
        assert torch.equal(x, y)
    assert results[0][2].tolist() == [3] * B and results[0][5][:, :3].tolist() == [path] * B
    for before, after in zip(start[0] + start[1], results[0][6:]):
        for b in range(B):
            L0 = int(lens[b])
            want = before[b].clone()
            want[:, L0:L0 + 3] = before[b][:, [L0 + n for n in path]]
            assert torch.equal(after[b], want)


def test_caches_outlive_their_lists_during_the_call():
    """The commit's cache tensors stay alive until the C call returns, also when
    the lists they were passed in are emptied meanwhile (as another thread
    could: the call runs without the GIL).  The C call is a stand-in that
    empties them and launches nothing."""
    require_gpu()
    args = _calls()["commit"][2]
    caches = [weakref.ref(t) for t in args[3] + args[4]]
    alive = []

    @ctypes.CFUNCTYPE(ctypes.c_int, *glide.load().glide_verify_commit.argtypes)
    def stand_in(*_):
        args[3].clear()
        args[4].clear()
        alive.extend(c() is not None for c in caches)
        return 0

    nat = _lib._bind()
    try:
        nat.bind((0, 0, ctypes.cast(stand_in, ctypes.c_void_p).value, 0, 0, 0, 0, 0), _lib._raw_stream,
                 _lib._ws_cache)
        glide.glide_verify_commit(*args)
    finally:
        _lib._native = None
        _lib._bind()
    assert alive == [True] * 4
    assert [c() for c in caches] == [None] * 4
