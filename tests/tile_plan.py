"""The plan of a call of the lm_head variant (csrc/lmhead_plan.hpp, which has no device code) as Python functions, so that a test
can say which tiles a shape takes and in how many chunks."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2507_19766_amd import build

_SOURCE = """
#include "lmhead_plan.hpp"
using namespace ulorl_detail;
extern "C" int forward(long N, long Hd, long V) { return forward_tile(0, N, Hd, V); }
extern "C" int backward(long N, long Hd, long V) { return backward_tile(0, N, Hd, V); }
extern "C" long chunk(long N, long Hd, long V, int vocab_chunk, unsigned long token_ws)
{
    return lmhead_layout(N, Hd, V, vocab_chunk, backward_tile(0, N, Hd, V), token_ws).chunk;
}
extern "C" unsigned long total(long N, long Hd, long V, int vocab_chunk, unsigned long token_ws)
{
    return lmhead_layout(N, Hd, V, vocab_chunk, 0, token_ws).total;
}
"""


@functools.lru_cache(None)
def _plan():
    with tempfile.TemporaryDirectory() as tmp:
        src, lib = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
        with open(src, "w") as f:
            f.write(_SOURCE)
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-fPIC", "-shared", "-I" + build.CSRC, src, "-o", lib])
        plan = ctypes.CDLL(lib)
    for name in ("chunk", "total"):
        getattr(plan, name).restype = ctypes.c_long
    return plan


def _sizes(*sizes):
    return [ctypes.c_long(n) for n in sizes]


def forward_is_large(N, Hd, V):
    return _plan().forward(*_sizes(N, Hd, V)) == 0


def backward_is_large(N, Hd, V):
    return _plan().backward(*_sizes(N, Hd, V)) == 0


def _token_ws(N, R):
    """Bytes of the token loss's own part of the workspace."""
    blocks = -(-N // 1024)
    return ctypes.c_ulong(sum(-(-n // 256) * 256 for n in (8, 8 * R, 4 * R, 8 * blocks, 32 * blocks, N, 4, 4)))


def workspace_bytes(N, Hd, V, R, vocab_chunk):
    return _plan().total(*_sizes(N, Hd, V), vocab_chunk, _token_ws(N, R))


def backward_chunks(N, Hd, V, vocab_chunk):
    """Launches of dz tiles in a backward call."""
    return -(-V // _plan().chunk(*_sizes(N, Hd, V), vocab_chunk, _token_ws(N, 1)))


def column_tiles(n):
    """Widths of the large tiles that share n columns."""
    tiles, units = -(-n // 256), -(-n // 32)
    return [32 * (units // tiles + (t < units % tiles)) for t in range(tiles)]
