"""CPU-only tests of the library's host side: the C ABI loads and exports every declared symbol,
argument validation that needs no GPU, and the host bookkeeping against the oracle."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from oracle import slicemoe_oracle as O
from paper_2512_12990_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "slicemoe.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(smoe_[a-z_0-9]+)\s*\(", hdr))
    assert len(declared) >= 20
    lib = B.lib()
    for name in declared:
        assert hasattr(lib, name), name
    assert declared == set(B.EXPORTS)


def test_strerror_and_bank_bytes_validation():
    lib = B.lib()
    assert lib.smoe_strerror(0) == b"ok"
    assert b"aligned" in lib.smoe_strerror(-3)
    d = B.BankDesc(64, 2048, 1408, 128, 8, 4, B.BF16, B.BF16)
    n = B.smoe_bank_bytes(d)
    # two nibble planes (= one 8-bit copy, no duplication) + 3 bytes of metadata per group; a row of
    # scales is padded to an even count (the down rows have 11 groups -> 12 stored)
    weights = 64 * 3 * 2048 * 1408
    groups = 64 * (2 * 1408 * 16 + 2048 * 11)
    pad = 64 * 2048 * 2
    assert weights + 3 * groups + pad <= n <= weights + 3 * groups + pad + 8 * 256 + 64 * 64
    nbytes = C.c_size_t()
    for bad, rc in [(B.BankDesc(0, 2048, 1408, 128, 8, 4, 0, 0), -2), (B.BankDesc(4, 2040, 1408, 128, 8, 4, 0, 0), -2),
                    (B.BankDesc(4, 2048, 1408, 100, 8, 4, 0, 0), -2), (B.BankDesc(4, 2048, 1408, 128, 8, 2, 0, 0), -6),
                    (B.BankDesc(4, 2048, 1408, 128, 4, 4, 0, 0), -2), (B.BankDesc(4, 2048, 1408, 128, 8, 4, 7, 0), -1),
                    (B.BankDesc(4, 2048, 1408, 128, 8, 4, 0, 0, 2), -1)]:
        assert lib.smoe_bank_bytes(C.byref(bad), C.byref(nbytes)) == rc
    # the lower nests store b_low bits per plane value: 3/4 and 1/2 of the plane bytes of the 8/4 nest
    for bh, bl in [(6, 3), (4, 2)]:
        nl = B.smoe_bank_bytes(B.BankDesc(64, 2048, 1408, 128, bh, bl, B.BF16, B.BF16))
        assert weights * bl // 4 + 3 * groups + pad <= nl <= weights * bl // 4 + 3 * groups + pad + 8 * 256 + 64 * 64
    assert lib.smoe_bank_bytes(None, C.byref(nbytes)) == -1
    assert lib.smoe_bank_bytes(C.byref(d), None) == -1


def test_topn_matches_oracle():
    rng = np.random.default_rng(0)
    for L, E in [(1, 4), (3, 5), (24, 60)]:
        hist = rng.integers(0, 6, size=(L, E)).astype(np.uint32)
        for n in [0, 1, L * E, L * E + 3, 2 * L * E, 2 * L * E + 10]:
            assert np.array_equal(B.smoe_topn_slices(hist, n), O.topn_slices(hist, n))


def test_cache_matches_oracle_in_lockstep():
    rng = np.random.default_rng(1)
    L, E, cap, k = 3, 16, 24, 4
    c, o = B.Cache(L, E, cap), O.SliceLRU(L, E, cap)
    hist = rng.integers(0, 9, size=(L, E)).astype(np.uint32)
    ids = O.topn_slices(hist, cap // 2)
    c.init_order(ids)
    o.init_order(ids)
    for step in range(300):
        l = int(rng.integers(L))
        idx = rng.choice(E, size=k, replace=False).astype(np.int32)
        wh = rng.integers(0, 2, size=k).astype(np.uint8)
        m1, b1 = c.snapshot(l, 1.0)
        m2, b2 = o.snapshot(l, 1.0)
        assert np.array_equal(m1, m2) and np.array_equal(b1, b2)
        c.access(l, idx, wh)
        o.access(l, idx, wh)
        assert c.order() == o.order
    assert c.stats() == o.stats
    assert len(c.order()) <= cap


def test_cache_argument_errors():
    lib = B.lib()
    h = C.c_void_p()
    assert lib.smoe_cache_create(1, 4, 1, C.byref(h)) == -2
    assert lib.smoe_cache_create(1, 4, 4, None) == -1
    c = B.Cache(2, 4, 4)
    bad = np.array([0, 9], np.int32)
    assert lib.smoe_cache_access(c.h, 0, 2, bad.ctypes.data_as(C.c_void_p), None) == -2
    assert lib.smoe_cache_access(c.h, 5, 1, bad.ctypes.data_as(C.c_void_p), None) == -2
    dup = np.array([1, 1], np.uint32)
    assert lib.smoe_cache_init_order(c.h, dup.ctypes.data_as(C.c_void_p), 2) == -1
    assert c.order() == []


def test_product_path_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2512_12990_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".hpp", ".cpp", ".h")):
                src = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in src.replace("the CPU oracle's tests", ""), f


def test_cache_all_layer_calls_match_per_layer_calls():
    """smoe_cache_snapshot_all / smoe_cache_access_all = the per-layer calls in layer order (and the oracle's LRU)."""
    rng = np.random.default_rng(3)
    L, E, cap, k = 5, 12, 30, 3
    a, b, o = B.Cache(L, E, cap), B.Cache(L, E, cap), O.SliceLRU(L, E, cap)
    masks, bias = np.empty((L, E), np.uint8), np.empty((L, E), np.float32)
    for t in range(60):
        idx = np.zeros((L, 16), np.int32)                         # padded rows, as a device buffer would have
        for l in range(L):
            idx[l, :k] = rng.choice(E, size=k, replace=False)
        want = (rng.random((L, k)) < 0.6).astype(np.uint8)
        a.snapshot_all(0.75, masks, bias)
        for l in range(L):
            m, bb = b.snapshot(l, 0.75)
            om, ob = o.snapshot(l, 0.75)
            assert np.array_equal(masks[l], m) and np.array_equal(bias[l], bb)
            assert np.array_equal(m, om) and np.array_equal(bb, ob)
        a.access_all(idx, k, want)
        for l in range(L):
            b.access(l, idx[l, :k], want[l])
            o.access(l, idx[l, :k], want[l])
        assert a.order() == b.order() == o.order and a.stats() == b.stats() == o.stats
    # an invalid index anywhere leaves the cache untouched
    bad = np.zeros((L, 16), np.int32)
    bad[L - 1, 1] = E
    before = a.order()
    with pytest.raises(B.SmoeError):
        a.access_all(bad, k, None)
    assert a.order() == before



def test_workspace_bytes_and_ctx_create_validation():
    lib = B.lib()
    # one token of the DeepSeek-V2-Lite-shaped layer: 64 KiB of records + (6 + 2) * 1408 floats
    assert B.smoe_workspace_bytes(1, 6, 1408, 2, 1408) == (64 << 10) + 8 * 1408 * 4
    # several tokens: vectors a fixed stride apart with room for the largest top-k (16)
    assert B.smoe_workspace_bytes(4, 6, 1408, 2, 1408) == (64 << 10) + 4 * (2 + 16) * 1408 * 4
    n = C.c_size_t()
    for args in [(0, 6, 1408, 2, 1408), (17, 6, 1408, 2, 1408), (1, 17, 1408, 0, 0), (1, 6, -1, 0, 0), (1, 6, 32, 9, 32)]:
        assert lib.smoe_workspace_bytes(*[C.c_int(a) for a in args], C.byref(n)) == -2
    assert lib.smoe_workspace_bytes(C.c_int(1), C.c_int(1), C.c_int(32), C.c_int(0), C.c_int(0), None) == -1
    # the context borrows its workspace: a null, misaligned or too small one is refused before any device call
    h = C.c_void_p()
    create = lib.smoe_ctx_create
    assert create(C.c_int(0), None, None, C.c_size_t(1 << 20), C.byref(h)) == -1
    assert create(C.c_int(0), None, C.c_void_p(0x1000 + 16), C.c_size_t(1 << 20), C.byref(h)) == -3
    assert create(C.c_int(0), None, C.c_void_p(0x1000), C.c_size_t(1024), C.byref(h)) == -4
    assert create(C.c_int(-1), None, C.c_void_p(0x1000), C.c_size_t(1 << 20), C.byref(h)) == -1


def test_single_launch_calls_reject_null_arguments():
    # (argument checks only: they return before any device call)
    lib = B.lib()
    n, t = C.c_longlong(), C.c_uint()
    assert lib.smoe_ctx_single_launch(None, C.c_int(1), C.c_int(0)) == -1
    assert lib.smoe_ctx_single_launch_status(None, C.byref(n), C.byref(t)) == -1


def test_no_device_allocation_in_the_library_sources():
    # the boundary's rule: device memory belongs to the caller
    csrc = os.path.join(ROOT, "paper_2512_12990_amd", "csrc")
    for name in os.listdir(csrc):
        text = open(os.path.join(csrc, name)).read()
        for call in ("hipMalloc", "hipFree", "hipMallocAsync", "hipExtMallocWithFlags", "hipHostMalloc"):
            assert not re.search(r"\b%s\s*\(" % call, text), (name, call)


def test_entry_division_is_exact_for_every_accepted_split(tmp_path):
    # The decode kernels turn an entry index into (slot, position) with a multiply-high by a launch
    # constant (csrc/fastdiv.hpp).  Checked here against integer division for EVERY row-pair count per
    # slot (cap) and every entry index the host lets through (slots * cap below the stated limit).
    src = tmp_path / "fastdiv_check.cpp"
    src.write_text(r'''
#include "fastdiv.hpp"
#include <stdio.h>
int main() {
  long long n = 0;
  for (int cap = 1; cap < SMOE_FASTDIV_LIMIT; cap++) {
    const uint32_t m = fastdiv_magic(cap);
    for (int e = 0; e < SMOE_FASTDIV_LIMIT; e++) {
      const int s = fastdiv(e, m);
      if (s != e / cap || e - s * cap != e % cap) { printf("FAIL cap=%d e=%d got %d want %d\n", cap, e, s, e / cap); return 1; }
      n++;
    }
  }
  printf("ok %lld\n", n);
  return 0;
}
''')
    exe = tmp_path / "fastdiv_check"
    import subprocess
    subprocess.run(["g++", "-O2", "-I", os.path.join(ROOT, "paper_2512_12990_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


def test_prefill_tiles_validation_and_heights():
    def bank(n, f, d=2048, nest=(8, 4), scale="bf16"):
        return B.BankDesc(n, d, f, 128, nest[0], nest[1], B.BF16, B._DT[scale], 0)

    lib, i = B.lib(), C.c_int()
    out = (C.byref(i), C.byref(i), C.byref(i))
    assert lib.smoe_prefill_tiles(None, None, 10, 1, 256, *out) == -1
    assert lib.smoe_prefill_tiles(C.byref(bank(8, 64)), None, 10, 1, 256, None, *out[1:]) == -1
    for T, k, n_cu in ((0, 1, 256), (10, 0, 256), (10, 9, 256), (10, 1, 0)):
        assert lib.smoe_prefill_tiles(C.byref(bank(8, 64)), None, T, k, n_cu, *out) == -2
    assert lib.smoe_prefill_tiles(C.byref(bank(8, 64)), C.byref(bank(1, 64, d=1024)), 10, 1, 256, *out) == -2
    # one tile of 32 or 64 rows for experts of few; the shared experts in the same launches, not with another nest or scale type
    dsv2, shared = bank(64, 1408), bank(2, 1408)
    assert B.smoe_prefill_tiles(dsv2, shared, 173, 6, 256) == (32, 32, True)
    assert B.smoe_prefill_tiles(dsv2, shared, 500, 6, 256)[0] == 64
    assert B.smoe_prefill_tiles(dsv2, bank(2, 1408, nest=(6, 3)), 173, 6, 256)[2] is False
    assert B.smoe_prefill_tiles(dsv2, bank(2, 1408, scale="f32"), 173, 6, 256)[2] is False
    # many rows per expert: tall tiles
    assert B.smoe_prefill_tiles(bank(60, 1408), bank(1, 5632), 4096, 4, 256) == (256, 256, True)
    assert B.smoe_prefill_tiles(bank(60, 1408), None, 1500, 4, 256) == (160, 0, False)


@pytest.mark.parametrize("E,d,f,k,T,ns,fs,nest,rows", [
    # heights that gain with one kind of routing what they lose with another (even, as a router makes it, popularity 1 / rank^1.1)
    (60, 2048, 1408, 4, 2048, 0, 0, (6, 3), 160),
    (60, 2048, 1408, 4, 2048, 0, 0, (4, 2), 160),
    (36, 896, 1024, 3, 3692, 0, 0, (4, 2), 160),
    (33, 512, 448, 8, 328, 0, 0, (8, 4), 96),
    # faster, or no slower, with each: taken
    (60, 2048, 1408, 4, 2048, 0, 0, (8, 4), 256),
    (60, 2048, 1408, 4, 3000, 0, 0, (8, 4), 256),
    (24, 2560, 2048, 8, 1000, 0, 0, (8, 4), 256),
    (64, 2048, 1408, 6, 2048, 2, 1408, (8, 4), 256),
    (16, 1024, 1024, 4, 3000, 0, 0, (8, 4), 256),
    (14, 256, 576, 6, 679, 1, 384, (4, 2), 96),
    (15, 448, 256, 3, 490, 2, 192, (6, 3), 96),
])
def test_prefill_heights_under_skewed_popularity(E, d, f, k, T, ns, fs, nest, rows):
    desc = lambda n, ff: B.BankDesc(n, d, ff, 64, nest[0], nest[1], B.BF16, B.BF16, 0)
    assert B.smoe_prefill_tiles(desc(E, f), desc(ns, fs) if ns else None, T, k, 256)[0] == rows


def test_library_handle_is_published_with_its_signatures(monkeypatch):
    """A second host thread may call lib() while the first one is still inside it: it must either load the library itself or get
    a handle on which every signature is set (without them ctypes passes a device pointer as a 32-bit int)."""
    handed_out = []

    class Function:
        def __init__(self):
            self.__dict__["set"] = set()

        def __setattr__(self, name, value):
            handed_out.append(B._lib)                    # what another thread would be handed at this moment
            self.set.add(name)

    class Library:
        def __init__(self, path):
            self.functions = {name: Function() for name in B.EXPORTS}

        def __getattr__(self, name):
            handed_out.append(B._lib)
            return self.functions[name]

    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B.C, "CDLL", Library)
    try:
        handle = B.lib()
    finally:
        monkeypatch.undo()
    assert handed_out and all(h is None for h in handed_out)
    assert all("argtypes" in handle.functions[name].set for name in B._SIGNATURES)


def test_inline_assembly_leaves_m0_to_the_compiler():
    """A direct load into LDS takes its address from M0.  The statement has to name that register as an operand: one that writes
    it unannounced may take it from under code the compiler placed around it."""
    csrc = os.path.join(ROOT, "paper_2512_12990_amd", "csrc")
    n_loads = 0
    for name in sorted(os.listdir(csrc)):
        if not name.endswith((".hip", ".hpp")):
            continue
        for stmt in re.findall(r"asm volatile\s*\((.*?)\);", open(os.path.join(csrc, name)).read(), flags=re.S):
            template = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', stmt.split(":")[0]))
            assert "m0" not in template, (name, stmt)
            if re.search(r"buffer_load\w+ .* lds", template):
                assert '"{m0}"(' in stmt, (name, stmt)
                n_loads += 1
    assert n_loads >= 3


def test_direct_lds_loads_keep_clear_of_vector_writes_to_their_scalars(tmp_path):
    """A memory instruction may read a scalar register five wait states after a vector instruction wrote it, not earlier.  The
    compiler sees to that for its own instructions but does not look into inline assembly, and a spilled scalar comes back by a
    vector instruction (v_readlane), so the distance is checked on the code that was built: back from every direct load into
    LDS, along every path."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    so = tmp_path / "lib.so"
    so.write_bytes(open(B.LIB_PATH, "rb").read())
    subprocess.run([objdump, "--offloading", str(so)], check=True, capture_output=True)

    def scalars(text):
        regs = set()
        for a, b, c in re.findall(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
            regs |= {int(c)} if c else set(range(int(a), int(b) + 1))
        return regs

    n_loads = 0
    for obj in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([objdump, "-d", str(obj)], check=True, capture_output=True, text=True).stdout
        if "offen lds" not in text:
            continue
        ins = [(m[1], int(m[2], 16)) for m in re.finditer(r"^\t(\S.*?)\s*// ([0-9A-F]+):", text, flags=re.M)]
        at = {addr: i for i, (_, addr) in enumerate(ins)}
        jumps_to = {}
        for i, (op, addr) in enumerate(ins):
            m = re.match(r"s_c?branch\w* (\d+)", op)
            if m:
                off = int(m[1]) - (65536 if int(m[1]) >= 32768 else 0)
                jumps_to.setdefault(at[addr + 4 + 4 * off], []).append(i)
        for i, (op, _) in enumerate(ins):
            if not (op.startswith("buffer_load") and op.endswith("lds")):
                continue
            n_loads += 1
            need, todo, seen = scalars(op), [(i, 0)], set()
            while todo:
                j, waited = todo.pop()
                before = list(jumps_to.get(j, []))
                if j and not re.match(r"s_branch|s_endpgm|s_setpc", ins[j - 1][0]):
                    before.append(j - 1)
                for b in before:
                    bop = ins[b][0]
                    written = scalars(bop.split(None, 1)[1].split(",")[0]) if bop.startswith("v_") and " " in bop else set()
                    assert not (written & need), (op, bop, waited)
                    w = waited + (int(bop.split()[1], 0) + 1 if bop.startswith("s_nop") else 1)
                    if w < 5 and (b, w) not in seen:
                        seen.add((b, w))
                        todo.append((b, w))
    assert n_loads > 0
