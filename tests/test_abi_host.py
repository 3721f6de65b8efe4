"""CPU-side checks of the C ABI: the library loads, exports every declared symbol, and the host
logic (configuration checks, memory sizing) behaves.  No compute call is made here."""
import ctypes as C
import os
import re

import pytest

from paper_2201_05500_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _cfg(**kw):
    d = dict(capacity_rows=1 << 16, dim=8, load_factor=0.5, n_replicas=1, lr=1e-3, beta1=0.9,
             beta2=0.999, eps=1e-8, init_seed=0, init_std=0.01, flags=0)
    d.update(kw)
    return B.ctr_config(*[d[f[0]] for f in B.ctr_config._fields_])


def test_library_exports_every_declared_symbol():
    from paper_2201_05500_amd import binding_mlp as BM
    lib = C.CDLL(B.LIB_PATH)
    for hdr, exported in (("ctr_sparse.h", B.EXPORTED), ("ctr_mlp.h", BM.EXPORTED)):
        header = open(os.path.join(ROOT, "include", hdr)).read()
        declared = set(re.findall(r"^\s*(?:int|size_t)\s+(ctr_\w+)\s*\(", header, re.M))
        assert declared == set(exported), hdr
        for name in declared:
            assert hasattr(lib, name), name


def test_mlp_host_logic():
    from paper_2201_05500_amd import binding_mlp as BM
    L = BM.lib()
    cfg = BM.make_config(19200, [1024, 512, 256])
    n = 19200 * 1024 + 1024 + 1024 * 512 + 512 + 512 * 256 + 256 + 256 + 1
    assert L.ctr_mlp_n_params(C.byref(cfg)) == n == 20318209
    assert L.ctr_mlp_bytes(C.byref(cfg)) >= n * (4 * 3 + 2)
    assert L.ctr_mlp_workspace_bytes(C.byref(cfg), 16384) >= 16384 * 19200 * 2
    assert L.ctr_mlp_workspace_bytes(C.byref(cfg), 100) == 0          # batch must be a multiple of 8
    assert L.ctr_mlp_workspace_bytes(C.byref(cfg), (1 << 20) + 8) == 0  # and at most CTR_MLP_MAX_BATCH
    for bad in (BM.make_config(100, [8]), BM.make_config(64, []), BM.make_config(64, [12]),
                BM.make_config(64, [8], n_replicas=2), BM.make_config(64, [8], lr=0.0)):
        assert L.ctr_mlp_bytes(C.byref(bad)) == 0
    out = C.c_void_p()
    assert L.ctr_mlp_create(C.byref(BM.make_config(64, [12])), 256, 1 << 30, None, C.byref(out)) == B.CTR_E_INVAL
    assert L.ctr_mlp_destroy(None) == B.CTR_E_INVAL


@pytest.mark.parametrize("in_dim,hidden", [(19200, [1024, 512, 256]), (624, [400, 200, 80]), (8, [8]), (8, [65536]),
                                           (8, [65536, 8, 65536]), (8, [65536, 8, 65536, 8, 65536]), (64, [8] * 6),
                                           (1024, [65536, 65536])])
@pytest.mark.parametrize("batch", [8, 4096, 1 << 16])
def test_mlp_workspace_needs_no_more_than_formerly(in_dim, hidden, batch):
    """Callers may hold a workspace sized when the output gradients of two layers, the logits and the partial sums of
    the widest layer had places of their own."""
    from paper_2201_05500_amd import binding_mlp as BM
    up = lambda b: (b + 255) & ~255
    dims, widest = [in_dim] + hidden + [1], max([8] + hidden)
    params = sum(a * b + b for a, b in zip(dims, dims[1:]))
    scratch = min(max(up(16 * max(a * b for a, b in zip(dims, hidden))), 32 << 20), 512 << 20)
    former = up(2 * batch * in_dim) + sum(up(2 * batch * h) for h in hidden) + 2 * up(2 * batch * widest) + \
        2 * up(4 * batch) + up(8 * batch) + up(4 * params) + up(4 * 64 * widest) + scratch
    assert 0 < BM.lib().ctr_mlp_workspace_bytes(C.byref(BM.make_config(in_dim, hidden)), batch) <= former


def test_config_struct_matches_header_layout():
    # uint64, uint32, float, uint32, 4 floats, uint64, float, uint32 with natural alignment
    assert C.sizeof(B.ctr_config) == 56
    assert B.ctr_config.init_seed.offset == 40 and B.ctr_config.flags.offset == 52


def test_table_bytes_accounts_for_every_array():
    R, D = 1 << 16, 8
    n = B.ctr_table_bytes(_cfg())
    slots = (1 << 17) * 16
    assert n >= slots + R * 8 + R * 4 + R * 3 * D * 4
    assert n < slots + R * 8 + R * 4 + R * 3 * D * 4 + 4096
    k = B.ctr_table_bytes(_cfg(n_replicas=8, flags=B.CTR_F_KSTEP))
    assert k - n >= 7 * R * 3 * D * 4 + R * D * 4
    # load factor decides the number of index slots (next power of two of R / lf)
    assert B.ctr_table_bytes(_cfg(load_factor=0.25)) - n == (1 << 17) * 16
    assert B.ctr_table_bytes(_cfg(load_factor=0.0)) == n            # 0 selects 0.5
    # AdaGrad rows hold two arrays instead of three; the prose merge needs no shared-denominator array
    assert n - B.ctr_table_bytes(_cfg(flags=B.CTR_F_ADAGRAD)) == R * D * 4
    assert k - B.ctr_table_bytes(_cfg(n_replicas=8, flags=B.CTR_F_KSTEP | B.CTR_F_KSTEP_PROSE)) == R * D * 4


def _workspace_with_spans_of_16(D, n):
    """Bytes of a batch's arrays when every batch below 2 M occurrences was walked in spans of 16: what a caller may
    have sized a workspace for by ctr_workspace_bytes of that time."""
    up = lambda b: (b + 255) & ~255
    words = (n + 31) // 32
    probe_tile = 2048 if n >= 4 << 20 else 256
    probe_tiles = -(-n // probe_tile)
    span = 128 if n >= 8 << 20 else 64 if n >= 4 << 20 else 32 if n >= 2 << 20 else 16
    spans = -(-n // span)
    lists = 6 * up(4 * n) + up(4 * 256 * 4096) + up(4 * 256)
    ranks = up(4 * (-(-words // 256) + 1)) + up(4 * (words + 1))
    pending = up(4 * probe_tile * (probe_tiles + 1)) + up(4 * (probe_tiles + 1))
    partials = 2 * up(8 * D * spans) + up(8 * D * -(-spans // 64)) + 2 * up(4 * spans)
    return max(lists + ranks + pending + partials, 256)


def test_fixed_scratch_of_the_lookup_holds_one_list():
    """The row of each key; segments are not recorded by a lookup.  (The header's constant, and the array in the
    library that it sizes.)"""
    import subprocess
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "s.c"), "w") as f:
            f.write('#include <stdio.h>\n#include "ctr_sparse.h"\n'
                    'int main(void) { printf("%zu %u", CTR_NOALLOC_SCRATCH_BYTES, CTR_NOALLOC_MAX_KEYS); return 0; }\n')
        exe = os.path.join(d, "s")
        subprocess.check_call(["gcc", "-I" + os.path.join(ROOT, "include"), os.path.join(d, "s.c"), "-o", exe])
        size, keys = map(int, subprocess.check_output([exe]).split())
    assert keys == B.CTR_NOALLOC_MAX_KEYS == 1 << 22 and size == 4 * keys


@pytest.mark.parametrize("rows", [1 << 16, 1 << 22, 1 << 24])
@pytest.mark.parametrize("D", [4, 8, 12, 16, 24, 32, 64, 100, 128, 132, 256])
def test_workspace_for_many_keys_serves_every_smaller_batch(D, rows):
    """Batches just below a size from which spans are longer need more than those at it: the answer for max_keys covers
    them, so it never falls as max_keys grows."""
    cfg = _cfg(dim=D, capacity_rows=rows)
    sizes = {2 ** e + d for e in range(9, 25) for d in (-1, 0, 1)} | {int(1.13 ** e) for e in range(10, 135)}
    sizes = sorted(sizes | {(k << 18) + d for k in range(4, 130) for d in (-1, 0)} | {2 * rows - 1, 2 * rows})
    answers = [B.ctr_workspace_bytes(cfg, n, 0) for n in sizes]
    assert all(a <= b for a, b in zip(answers, answers[1:]))
    assert all(B.ctr_debug_workspace_min_bytes(cfg, n) <= a for n, a in zip(sizes, answers))
    # room for the partial sums, 16 bytes per column and span, of the batch with the most spans up to max_keys
    most = 0
    for n, a in zip(sizes, answers):
        most = max(most, -(-n // B.ctr_debug_push_span(cfg, n)))
        assert a >= 16 * D * most, (n, a)


def test_spans_of_narrow_rows():
    """From 2 Mi occurrences on: 16 for rows of 4, 8 and 12 columns where the table's rows show that keys repeat, or where a power
    law over many keys does not lose by it; else 32, 64 and 128 from 2, 4 and 8 Mi on (profiles/push_spans.txt)."""
    few, many = 1 << 18, 1 << 24
    span = lambda D, rows, mi, d=0: B.ctr_debug_push_span(_cfg(dim=D, capacity_rows=rows), int(mi * (1 << 20)) + d)
    lines = {4: [(2, 16), (3.5, 32), (4, 16), (5, 64), (8, 16), (12, 128), (16, 16)],
             8: [(2, 16), (2.5, 32), (4, 64), (8, 16), (10, 128), (12, 16)],
             12: [(2, 32), (4, 64), (5.5, 16), (8, 128), (10.5, 16)],
             16: [(2, 32), (4, 16)], 20: [(2, 32), (10, 64)], 32: [(2, 32), (10, 64)], 36: [(2, 32), (4, 64), (8, 128)],
             256: [(2, 32), (4, 64), (8, 128)]}
    for D, steps in lines.items():
        for (at, want), end in zip(steps, [s[0] for s in steps[1:]] + [2047]):
            assert span(D, many, at) == span(D, many, end, -1) == want, (D, at)
    for D, steps in {4: [(2, 16)], 8: [(2, 16), (2.5, 32), (3, 16)], 12: [(2, 32), (4, 16)], 16: [(2, 32), (4, 16)]}.items():
        for (at, want), end in zip(steps, [s[0] for s in steps[1:]] + [2047]):
            assert span(D, few, at) == span(D, few, end, -1) == want, (D, at)
    for D in (4, 8, 12):  # twice as many occurrences as rows
        rows = {4: 6 << 20, 8: 2 << 20, 12: 9 << 19}[D]
        assert span(D, rows, 2 * rows / (1 << 20)) == 16 and span(D, rows, 2 * rows / (1 << 20), -1) == {4: 16, 8: 32, 12: 128}[D]
    assert B.ctr_debug_push_span(_cfg(dim=6), 10) == B.ctr_debug_push_span(_cfg(), 1 << 31) == 0


def test_workspaces_of_the_former_sizes_are_accepted():
    sizes = set(range(0, 70)) | {2 ** e + d for e in range(6, 31) for d in (-257, -1, 0, 1, 300)}
    sizes |= {(k << 24) // 8 + d for k in range(1, 1024, 5) for d in (-4097, -77440, 0, 2048)}   # lists of whole sort chunks
    sizes |= {16702448, 16683000, 33300000, 49900000, 66500000, 300000, 300001, 500001, 1000001, 1750001, 2 ** 31 - 1}
    sizes |= {int(1.37 ** e) for e in range(20, 68)}
    for D in (4, 8, 64, 100, 256):
        for n in sorted(n for n in sizes if 0 <= n < 2 ** 31):
            least = B.ctr_debug_workspace_min_bytes(_cfg(dim=D), n)
            assert 0 < least <= B.ctr_workspace_bytes(_cfg(dim=D), n, 0), (D, n)
            assert least <= _workspace_with_spans_of_16(D, n), (D, n, least)
    assert B.ctr_debug_workspace_min_bytes(_cfg(dim=6), 10) == 0
    assert B.ctr_debug_workspace_min_bytes(_cfg(), 2 ** 31) == 0


@pytest.mark.parametrize("bad", [
    dict(dim=0), dict(dim=6), dict(dim=260), dict(capacity_rows=0), dict(capacity_rows=(1 << 30) + 1),
    dict(n_replicas=0), dict(n_replicas=32), dict(load_factor=0.95), dict(load_factor=-1.0),
    dict(flags=16), dict(flags=B.CTR_F_KSTEP_PROSE), dict(flags=B.CTR_F_ADAGRAD | B.CTR_F_KSTEP),
    dict(flags=B.CTR_F_ADAGRAD, n_replicas=2), dict(flags=B.CTR_F_BIAS_CORRECTION | B.CTR_F_KSTEP),
    dict(n_replicas=2), dict(lr=0.0), dict(beta1=1.0), dict(beta2=-0.1), dict(eps=0.0),
])
def test_invalid_configurations_are_rejected(bad):
    assert B.ctr_table_bytes(_cfg(**bad)) == 0
    assert B.ctr_workspace_bytes(_cfg(**bad), 1000, 10) == 0
    out = C.c_void_p()
    st = B.lib().ctr_table_create(C.byref(_cfg(**bad)), 256, 1 << 30, None, C.byref(out))
    assert st == B.CTR_E_INVAL


def test_workspace_bytes_grow_with_keys_and_dim():
    a = B.ctr_workspace_bytes(_cfg(), 10000, 100)
    b = B.ctr_workspace_bytes(_cfg(), 20000, 100)
    c = B.ctr_workspace_bytes(_cfg(dim=64), 10000, 100)
    assert 0 < a < b and a < c
    assert B.ctr_workspace_bytes(_cfg(), 0, 0) >= 256
    assert B.ctr_workspace_bytes(_cfg(), 1 << 31, 10) == 0           # n_keys limit


def test_workspace_bytes_never_shrink_with_the_batch_size():
    """The work geometry changes at 2, 4 and 8 Mi occurrences, of 20 to 32 columns at 10 Mi (shorter spans below each
    threshold need more partial sums): a workspace sized for max_keys must cover every smaller batch."""
    for dim in (16, 24, 32, 64):
        sizes = [1, 1000, (1 << 20), (2 << 20) - 1, 2 << 20, (3 << 20), (4 << 20) - 1, 4 << 20, (6 << 20),
                 (8 << 20) - 1, 8 << 20, (10 << 20) - 1, 10 << 20, 12 << 20, 40 << 20]
        need = [B.ctr_workspace_bytes(_cfg(dim=dim), n, 10) for n in sizes]
        assert all(a <= b for a, b in zip(need, need[1:])), (dim, need)
        assert all(n > 0 for n in need)


def test_null_and_misaligned_arguments():
    L = B.lib()
    out = C.c_void_p()
    assert L.ctr_table_create(None, 256, 1 << 30, None, C.byref(out)) == B.CTR_E_INVAL
    assert L.ctr_table_create(C.byref(_cfg()), None, 1 << 30, None, C.byref(out)) == B.CTR_E_INVAL
    assert L.ctr_table_create(C.byref(_cfg()), 264, 1 << 30, None, C.byref(out)) == B.CTR_E_INVAL
    assert L.ctr_table_create(C.byref(_cfg()), 256, 1024, None, C.byref(out)) == B.CTR_E_NOMEM
    assert L.ctr_table_destroy(None) == B.CTR_E_INVAL
    assert L.ctr_kstep_merge(None, None) == B.CTR_E_INVAL
    assert L.ctr_push_adam(None, 0, None, None, 0, None) == B.CTR_E_INVAL
    assert L.ctr_last_status(None, None) == B.CTR_E_INVAL
    assert L.ctr_debug_set_geometry(None, 0, 0) == B.CTR_E_INVAL
    assert L.ctr_debug_set_push_order(None, 32, 0, 0) == B.CTR_E_INVAL


def test_headers_are_plain_c99(tmp_path):
    """The boundary is a C ABI: both headers compile as strict C99 on their own."""
    import os
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = tmp_path / "hdr.c"
    src.write_text('#include "ctr_sparse.h"\n#include "ctr_mlp.h"\nint main(void) { return 0; }\n')
    subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I" + os.path.join(root, "include"),
                           "-fsyntax-only", str(src)])


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    """No CPU fallback exists: without the built HIP library the binding raises instead of computing."""
    from paper_2201_05500_amd import binding as B
    from paper_2201_05500_amd import binding_mlp as BM
    monkeypatch.setattr(B, "LIB_PATH", str(tmp_path / "libctr_sparse.so"))
    monkeypatch.setattr(B, "_lib", None)
    with pytest.raises(RuntimeError, match="missing"):
        B.lib()
    with pytest.raises(RuntimeError, match="missing"):          # the tower's binding loads the same library
        BM.lib()


def test_geometry_set_after_a_reservation_has_its_room():
    """ctr_debug_set_geometry may need a larger workspace for the keys that room was reserved for before."""
    import types

    import torch
    t = object.__new__(B.CtrTable)
    t._torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda device: None), empty=torch.empty, uint8=torch.uint8)
    t.device, t.cfg, t._handle = torch.device("cpu"), _cfg(), None
    t._ws, t._ws_of_live_batch, t.ws_bytes, t._ws_keys, t._ws_need = None, None, 0, -1, 0
    t.reserve(1000, 10)
    first = t.ws_bytes
    assert first == B.ctr_workspace_bytes(t.cfg, 1000, 10)
    t.set_geometry(4, 8)
    t.reserve(1000, 10)
    assert t.ws_bytes == first + (1 << 20) and t._ws.numel() == t.ws_bytes
    t.set_geometry(0, 0)
    t.reserve(1000, 10)
    assert t.ws_bytes == first + (1 << 20)
