"""Device memory of a policy, counted by a stand-in for the HIP allocator (a
small C library loaded ahead of the real runtime in a child process; nothing
touches a GPU).  The rows that only recompute_logprobs uses (chunks of up to
4096 rows) may add an eighth of the weights and the KV pool, or 32 MiB, to what
the largest step needs, and a device with room for the step alone still takes
the policy."""
import json
import os
import shutil
import subprocess
import sys

import pytest

from workload import ModelShape, get_config

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_02218_amd", "librollout.so")

ALLOCATOR = r"""
#include <stddef.h>
#include <stdlib.h>
static size_t used, room;
static char* next = (char*)0x100000000000;
void set_room(size_t n) { used = 0; room = n; }
size_t get_used(void) { return used; }
int hipMalloc(void** p, size_t n) {
  if (n > room - used) return 2;                  /* hipErrorOutOfMemory */
  used += n;
  *p = next;
  next += n + 4096;
  return 0;
}
int hipFree(void* p) { (void)p; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)d; (void)s; (void)n; (void)k; return 0; }
int hipMemcpy2D(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k) {
  (void)d; (void)dp; (void)s; (void)sp; (void)w; (void)h; (void)k; return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = malloc(n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipEventCreate(void** e) { *e = (void*)8; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = (void*)8; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)8; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipGetLastError(void) { return 0; }
"""

CHILD = r"""
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)       # found ahead of the real runtime's functions
fake.set_room.argtypes, fake.get_used.restype = [C.c_size_t], C.c_size_t
import paper_2606_02218_amd as rg
from paper_2606_02218_amd import _lib
lib = rg.load_library()
out = []
for shape, limits, room in json.load(sys.stdin):
    L = shape["n_layers"]
    cfg = _lib.rg_config(L, shape["d_model"], shape["n_q_heads"], shape["n_kv_heads"], shape["head_dim"],
                         shape["ffn_dim"], shape["vocab"], shape["vocab"] - 1, 1e4, 1e-6, int(shape["dtype"] == "bf16"))
    arr = (C.c_void_p * L)(*[4096] * L)
    per = C.cast(arr, _lib._PP)
    w = _lib.rg_weights(4096, 4096, 4096, *[per] * 9)
    lim = _lib.rg_limits(*limits, 0)
    h = C.c_void_p()
    fake.set_room(room)
    rc = lib.rg_policy_create(C.byref(cfg), C.byref(w), C.byref(lim), C.byref(h))
    n = int(lib.rg_policy_device_bytes(h)) if rc == 0 else -1
    assert rc != 0 or n == fake.get_used(), (n, fake.get_used())
    lib.rg_policy_destroy(h)
    out.append([rc, n])
print(json.dumps(out))
"""

SHAPES = [get_config(n).shape for n in ("tiny", "gpt2s", "1.5b", "7b")] + [
    ModelShape(1, 64, 1, 1, 64, 64, 16, 1e4, dtype="bf16"), ModelShape(2, 128, 4, 1, 128, 512, 50048, 1e4, dtype="f32")]
LIMITS = [(1, 1, 1, 2), (8, 2, 64, 1024), (8, 1, 4000, 9216), (64, 8, 700, 700), (512, 32, 16384, 4608)]
PLENTY = 1 << 50


def _create(cases, tmp):
    src, lib = os.path.join(tmp, "alloc.c"), os.path.join(tmp, "liballoc.so")
    with open(src, "w") as f:
        f.write(ALLOCATOR)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", lib, src], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, lib], input=json.dumps([[vars(s), lim, room] for s, lim, room in cases]),
                       capture_output=True, text=True, cwd=ROOT, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def _held(s, lim):
    """Weights, norm gains, RoPE table and KV pool, in bytes."""
    S, P, tokens, ctx = lim
    pages = -(-tokens // 16) + P + S * (-(-ctx // 16) + 1)
    weights = s.n_layers * s.matrix_params_per_layer() + 2 * s.vocab * s.d_model
    return (weights * s.elem_bytes + (2 * s.n_layers + 1) * s.d_model * 4 + ctx * s.head_dim * 4
            + pages * 16 * s.kv_bytes_per_token())


def _step_bytes(s, lim):
    """What the largest step's rows need: the residual, two operands, split
    partials, queries, sums of squares, attention partials of every row's
    chunks, logits of up to 1024 rows, and the integers."""
    S, P, tokens, ctx = lim
    M, widest = max(tokens, S), max(s.q_dim, s.ffn_dim, s.d_model)
    maxN = max(s.q_dim + 2 * s.kv_dim, 2 * s.ffn_dim, s.d_model)
    slots = max(M + 1024 + S * (16 + ctx // 1024 + 1), 4 * M, 2 * min(M, 2048) + 1024)
    words = M * (s.d_model + 2 * widest + s.q_dim + s.d_model // 32 + 1) + max(M, 32 * S) * maxN
    words += slots * (s.q_dim + 2 * s.n_q_heads) + max(S, P, min(M, 1024)) * s.vocab + 128 * max(S, P)
    pages = -(-tokens // 16) + P + S * (-(-ctx // 16) + 1)
    words += (3 * S + 2 * P) * (ctx // 16 + 2) + 4 * ctx + 16 * (M + S + P) + pages
    return 4 * words + (1 << 20)


@pytest.mark.skipif(not os.path.exists(LIB) or not shutil.which("gcc"), reason="library not built, or no C compiler")
def test_recompute_rows_cost_a_bounded_share(tmp_path):
    cases = [(s, lim, PLENTY) for s in SHAPES for lim in LIMITS]
    for (s, lim, _), (rc, n) in zip(cases, _create(cases, str(tmp_path))):
        held = _held(s, lim)
        bound = held + _step_bytes(s, lim) + max(32 << 20, held // 8)
        assert rc == 0 and n <= bound, (s, lim, n >> 20, bound >> 20)


@pytest.mark.skipif(not os.path.exists(LIB) or not shutil.which("gcc"), reason="library not built, or no C compiler")
def test_a_full_device_takes_the_step_alone(tmp_path):
    """With any room from what the step needs up to one byte less than the full
    workspace the policy is created, without the chunk's rows."""
    cases = [(s, lim, PLENTY) for s in SHAPES for lim in LIMITS]
    full = _create(cases, str(tmp_path))
    tight = [(s, lim, n - 1) for (s, lim, _), (_, n) in zip(cases, full)]
    smaller = 0
    for (s, lim, room), (rc, n) in zip(tight, _create(tight, str(tmp_path))):
        if max(lim[0], lim[2]) >= min(4096, lim[0] * lim[3]):   # the step holds a chunk already
            assert rc == -2, (s, lim, rc)
        else:
            assert rc == 0 and n <= room and n <= _held(s, lim) + _step_bytes(s, lim), (s, lim, rc, n, room)
            smaller += 1
    assert smaller >= len(cases) // 2
