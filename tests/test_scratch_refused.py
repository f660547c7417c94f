"""What the library's host code does when the device has no room for a work buffer, and what it launches: without a GPU, against a HIP runtime that
launches nothing (stub_hip.cpp).  A refused allocation is the call's own business: where there is another way it is taken, else the call returns
Z2Z_ENOMEM, and neither leaves an error behind that a later launch -- the library's or the program's -- would report as its own."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys, types
sys.path.insert(0, {root!r})
sys.modules["torch"] = types.ModuleType("torch")          # (only the binding's structs are used)
stub = ctypes.CDLL({stub!r}, ctypes.RTLD_GLOBAL)
stub.stub_capacity.argtypes = [ctypes.c_size_t]
stub.stub_used.restype = stub.stub_most.restype = ctypes.c_size_t
stub.stub_log.restype = ctypes.c_char_p
from paper_2506_01084_amd import api
lib = api.load_library()
P = 1 << 20                                               # (a device pointer that nothing follows)
MB = 1 << 20

def context(B, V, M, cap, d, dtype=api.BF16):
    stub.stub_capacity(1 << 40)
    cfg, h = api.Config(), ctypes.c_void_p()
    cfg.B, cfg.V, cfg.M, cfg.cap, cfg.d, cfg.dtype = B, V, M, cap, d, dtype
    assert lib.z2z_create(ctypes.byref(h), ctypes.byref(cfg)) == 0
    stub.stub_clear_log()
    return h

def room(mb):                                             # for this much more
    stub.stub_capacity(stub.stub_used() + mb * MB)

def launches():
    out = [(l.rsplit(" ", 1)[0], int(l.rsplit(" ", 1)[1])) for l in stub.stub_log().decode().splitlines()]
    stub.stub_clear_log()
    return out

def named(log, what):
    return [g for n, g in log if what in n]

def clean():
    assert stub.stub_last_error() == 0, "an error is left behind"

def encoder(d, layers=2, ff=None):
    arr = (api.EncoderLayer * layers)()
    for lay in arr:
        for name, _ in api.EncoderLayer._fields_:
            setattr(lay, name, P)
    e = api.EncoderDesc()
    e.n_layers, e.n_heads, e.d_ff, e.attention_only = layers, max(d // 64, 1), ff or 4 * d, 0
    e.layers = ctypes.cast(arr, ctypes.POINTER(api.EncoderLayer))
    e.keep = arr
    return e

def nll_backward(h, B, rows_per_seq):
    return lib.z2z_extended_nll_backward(h, P, B * rows_per_seq, rows_per_seq, P, P, P, P, P, P, P, P, None)
"""


@pytest.fixture(scope="session")
def without_a_device(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("stub") / "stub_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "stub_hip.cpp")], check=True)
    prelude = PRELUDE.format(root=ROOT, stub=lib)

    def run(body):
        r = subprocess.run([sys.executable, "-c", prelude + body], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


def test_products_go_on_whole_where_the_parts_have_no_room(without_a_device):
    without_a_device("""
h = context(B=1, V=4096, M=3, cap=100, d=128)
room(40)                                                  # the parts of cut tiles take 64 MiB
assert nll_backward(h, 1, 300) == 0
clean()
log = launches()
assert len(named(log, "logits_fast_kernel")) == 5 and not named(log, "tile_sum"), log
stub.stub_capacity(1 << 40)
assert nll_backward(h, 1, 300) == 0
assert named(launches(), "tile_sum")
""")


def test_a_layer_of_the_encoder_goes_on_whole_where_the_parts_have_no_room(without_a_device):
    without_a_device("""
h, enc = context(B=4, V=512, M=3, cap=200, d=2048), encoder(2048, ff=2048)
need = 4 * 200 * 3 * (8 * 2048 + 12 * 2048)
room(need // MB + 40)
assert lib.z2z_hyper_encode(h, P, ctypes.byref(enc), P, None, 0, None) == 0
clean()
assert not named(launches(), "tile_sum")
stub.stub_capacity(1 << 40)
assert lib.z2z_hyper_encode(h, P, ctypes.byref(enc), P, None, 0, None) == 0
assert named(launches(), "tile_sum")
""")


def test_a_refused_call_leaves_no_error_to_the_next(without_a_device):
    without_a_device("""
h, big = context(B=4, V=40000, M=3, cap=1024, d=128), context(B=64, V=40000, M=3, cap=1024, d=128)
step = lambda: lib.z2z_extended_logits(h, P, 4, 1, P, P, P, P, P, None, None)
room(2)
assert lib.z2z_extended_sample(big, P, 64, 1, P, P, 1.0, 50, 0.9, 1, 2, P, P, None) == api.E_NOMEM
clean()
assert nll_backward(big, 64, 20) == api.E_NOMEM
clean()
assert lib.z2z_hyper_encode(big, P, ctypes.byref(encoder(128)), P, None, 0, None) == api.E_NOMEM
clean()
assert step() == 0
h = ctypes.c_void_p()
cfg = api.Config()
cfg.B, cfg.V, cfg.M, cfg.cap, cfg.d, cfg.dtype = 1024, 40000, 3, 4096, 128, api.BF16
room(8)
assert lib.z2z_create(ctypes.byref(h), ctypes.byref(cfg)) == api.E_NOMEM and not h
clean()
""")


@pytest.mark.parametrize("B,rows_per_seq,V,cap,d,cut", [
    (8, 4096, 128256, 2048, 4096, 1),                    # tiles an XCD: dH 256, hyper 256, dW_hyper 128, whole rounds of 32; dW_base 1002, 10 left
    (8, 3300, 32000, 2048, 1024, 0),                     # 52, 62 and 63, 52: more than half a round left; 32
    (8, 3300, 32000, 2048, 4096, 2),                     # 208 (dH and its hyper part): 16 left; 250, 128
    (1, 300, 4096, 100, 128, 1),                         # dH: 2 tiles, 64 slabs
    (1, 2816, 4096, 100, 3072, 1),                       # dH: 16 tiles, 17 on some: whole; dW_base 24; dW_hyper 12 tiles in all, 44 slabs
])
def test_a_sum_is_launched_where_something_may_be_cut(without_a_device, B, rows_per_seq, V, cap, d, cut):
    without_a_device(f"""
h = context(B={B}, V={V}, M=3, cap={cap}, d={d})
assert nll_backward(h, {B}, {rows_per_seq}) == 0
log = launches()
assert len(named(log, "logits_fast_kernel")) == 5 and len(named(log, "tile_sum")) == {cut}, log
""")


def test_the_encoder_takes_shorter_passes_where_long_ones_have_no_room(without_a_device):
    """40 sequences of up to 600 entries of 3 slots: one pass of 72000 rows, or two (546 and 54 entries) of up to 65520."""
    without_a_device("""
enc = encoder(512)
run = lambda h: lib.z2z_hyper_encode(h, P, ctypes.byref(enc), P, None, 0, None)
row = 8 * 512 + 2 * (5 * 512 + 2048 + 64)                  # bytes of a slot row, and some more
parts = 64 * MB
h = context(B=40, V=512, M=3, cap=600, d=512)
assert run(h) == 0 and len(named(launches(), "enc_rows")) == 1
h = context(B=40, V=512, M=3, cap=600, d=512)
room((65600 * row + parts) // MB)
assert run(h) == 0
clean()
assert len(named(launches(), "enc_rows")) == 2
stub.stub_most()
stub.stub_capacity(1 << 40)
assert run(h) == 0 and len(named(launches(), "enc_rows")) == 2          # (once refused, the buffer stays as it is)
assert stub.stub_most() == stub.stub_used()

# under capture nothing grows: the buffer of a call with 546 new entries holds the shorter passes of a whole one, not the long one
h = context(B=40, V=512, M=3, cap=600, d=512)
assert lib.z2z_hyper_encode(h, P, ctypes.byref(enc), P, None, 546, None) == 0
launches()
stub.stub_capturing(1)
assert run(h) == 0 and len(named(launches(), "enc_rows")) == 2
h2 = context(B=40, V=512, M=3, cap=600, d=512)
assert run(h2) == api.E_CAPTURE
stub.stub_capturing(0)

h = context(B=40, V=512, M=3, cap=600, d=512)
room(64000 * row // MB)
assert run(h) == api.E_NOMEM
clean()
""")
