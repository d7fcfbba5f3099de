"""Host side of libnt on a HIP runtime that runs nothing (hip_stub.c): which kernels a call launches with which grids, what a
load puts on the device, and what happens when the device reports an error.  Each case is a child process, because the stub
has to be loaded before the library."""
import io
import json
import os
import re
import subprocess
import sys

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PREAMBLE = """
import ctypes as C, json, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
stub.stub_func.restype = stub.stub_launch.restype = C.c_char_p
import numpy as np
import nt_synth
import paper_2109_08003_amd as nt

class Stream:
    cuda_stream = 0

def config(**kw):
    return dict(nt_synth.model_config("C1"), vocab=256, max_len=256, **kw)

def load(cfg, tokens=4096, lanes=1):
    return nt.Model(cfg, np.zeros(nt.param_count(cfg), dtype=np.float16), max_batch_tokens=tokens, stream=Stream, pipeline_lanes=lanes)

def encode(model, rows, length):
    # the launches of one encode: (kernel, blocks)
    a = np.zeros(1, dtype=np.int32)
    stub.stub_clear()
    nt.binding._check(nt.binding.lib().nt_encode(model._h, a.ctypes.data, a.ctypes.data, rows, length, None))
    return launches()

def launches():
    grid, out = (C.c_uint32 * 3)(), []
    for i in range(stub.stub_n_launches()):
        out.append((stub.stub_launch(i, grid).decode(), grid[0] * grid[1] * grid[2]))
    return out
"""


@pytest.fixture(scope="session")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", "-o", so, os.path.join(ROOT, "tests", "hip_stub.c")], check=True)

    def run(code, timeout=300):
        """Runs code after the preamble; returns what it printed last, as JSON."""
        res = subprocess.run([sys.executable, "-c", PREAMBLE + code, so], cwd=ROOT, timeout=timeout, capture_output=True, text=True,
                             env=dict(os.environ, PYTHONPATH=ROOT))
        assert res.returncode == 0, res.stderr
        return json.loads(res.stdout.strip().splitlines()[-1])

    return run


# one lane, a large budget, and four lanes; batches of one sentence each, so that every staging set is used several times
@pytest.mark.parametrize("lanes,budget", [(1, 16), (4, 32768), (4, 16)])
def test_translate_returns_a_device_error(host, lanes, budget):
    """Every event reports a launch failure: the call ends with NT_EHIP and does not wait for what never becomes ready."""
    rc, message = host(f"""
model = load(config(), lanes={lanes})
offsets = np.arange(0, 16 * 13, 16, dtype=np.int64)
C.c_int.in_dll(stub, "stub_event_status").value = 719
try:
    model.translate_batch(np.full(192, 5, dtype=np.int32), offsets, {budget}, max_rows=1, stream=Stream)
    print(json.dumps((0, "")))
except nt.NtError as e:
    print(json.dumps((e.code, str(e))))
""", timeout=180)
    assert rc == -5 and "stub error" in message


@pytest.mark.parametrize("kw,i16", [(dict(), True), (dict(n_heads=8, d_ffn=64), False), (dict(dec_n_heads=2), False)])
def test_a_layer_holds_the_matrices_its_kernels_read(host, kw, i16):
    """One more encoder layer costs its own matrices and no others; one more decoder layer those of its two attentions and its
    caches (several decoder layers are never folded, so the matrices for folding are not there either)."""
    d, F = 512, kw.get("d_ffn", 0)
    enc, dec = host(f"""
size = lambda **kw: load(config(**dict({kw!r}, **kw)), tokens=64).device_bytes()
print(json.dumps((size(n_enc=3) - size(n_enc=2), size(n_enc=1, n_dec=3) - size(n_enc=1, n_dec=2))))
""")
    norm, parts = 2 * 4 * d, 40                       # parts: each is rounded up to 256 bytes
    attention = norm + 2 * (4 * d * d * 2) + 4 * 4 * d  # four matrices in two layouts, four biases
    ffn = norm + 2 * (2 * d * F) + 2 * d * F + 4 * (F + d) if F else 0  # the second matrix, K = 64, has no fragment order
    positions = 64, (6 * 64 + 4) // 5 + 3 * 64 + 8    # of the cross and of the self cache
    caches = positions[0] * 2 * d * 2 + positions[1] * 2 * d * (2 if i16 else 4) + (8 * sum(positions) if i16 else 0)
    assert abs(enc - attention - ffn) <= 256 * parts, enc
    assert abs(dec - 2 * attention - ffn - caches) <= 256 * parts, dec


def test_a_load_copies_what_the_host_makes(host):
    """The vectors and matrices of the folded caches are made on the device: 128 more positions are 128 more rows of the position table to
    copy, and none of the four rows each that the folded layer's start reads; the device has both (and the first layer's table)."""
    d = 512
    copied, there = host("""
out = []
for max_len in (128, 256):
    before = C.c_int64.in_dll(stub, "stub_copied").value
    model = load(dict(config(n_enc=1), max_len=max_len), tokens=64)
    out.append((C.c_int64.in_dll(stub, "stub_copied").value - before, model.device_bytes()))
print(json.dumps([b - a for a, b in zip(*out)]))
""")
    assert copied == 128 * d * 4
    assert there == 128 * d * 4 * (1 + 4 + 3)


def test_narrow_projections_are_one_round_of_workgroups(host):
    """The form with 32-column strips is for launches of at most 256 workgroups, whatever the matrix's width (an FFN of 192
    columns, an odd multiple of 64, has three groups of them), and for the matrix with one wide strip, of 64 columns."""
    got = host("""
out = []
for ffn in (0, 64, 192, 256, 2048):
    model = load(config(n_heads=8, d_ffn=ffn, n_enc=1), tokens=40000)
    for rows in (1, 85, 86, 100, 250, 640, 1000):
        out += [(ffn, rows, n, b) for n, b in encode(model, rows, 32) if "gemm_stream_kernel" in n]
print(json.dumps(out))
""")
    narrow = [x for x in got if re.search(r"gemm_stream_kernelILi\d+ELi\d+ELb.ELb.ELb.ELi\d+ELi1EE", x[2])]
    assert len(narrow) > 10 and len(got) - len(narrow) > 10
    assert max(blocks for ffn, _, _, blocks in narrow if ffn != 64) <= 256
    first = lambda ffn: {rows for f, rows, name, _ in narrow if f == ffn and "Li512ELb0ELb1" in name}  # fp16 out: the FFN's first matrix
    assert first(192) == {1, 85} and first(64) == {1, 85, 86, 100, 250, 640, 1000} and first(2048) == {1}


def test_decoder_layer_forms_are_all_in_use(host):
    """Every decoder layer kernel in the library's code object is launched by some row count of some model (those that reach
    their rows through a row map are the EOS mode's, whose loop waits for the device: the same forms)."""
    used = host("""
out = set()
for kw in (dict(), dict(dec_d_ffn=512), dict(n_heads=8), dict(n_dec=2), dict(n_dec=2, dec_d_ffn=512), dict(d_model=256),
           dict(d_model=256, dec_d_ffn=256), dict(d_model=256, n_dec=2), dict(d_model=256, n_dec=2, dec_d_ffn=256)):
    model = load(config(**dict(kw, n_enc=1)), tokens=33000)
    a = np.zeros(33000, dtype=np.int32)
    for rows, length in [(rows, 2) for rows in (1, 64, 65, 256, 257, 512, 513, 1023, 1024, 2000)] + [(300, 110)]:
        encode(model, rows, length)
        nt.binding._check(nt.binding.lib().nt_decode_greedy(model._h, rows, 1, None, a.ctypes.data, None))
        out |= {n for n, _ in launches() if "dec1_kernel" in n}
print(json.dumps(sorted(out)))
""")
    with open(os.path.join(ROOT, "paper_2109_08003_amd", "libnt.so"), "rb") as f:
        built = {n.decode() for n in re.findall(rb"_ZN2nt11dec1_kernelI(?:Li\d+E)+(?:Lb[01]E)+EEvNS_8Dec1ArgsE", f.read())}
    rows_direct = {n for n in built if re.search(r"Li\d+ELb0E", n)}
    assert len(used) > 10 and rows_direct == set(used)


def test_decoder_layer_without_folding_keeps_its_arguments_out_of_the_pick():
    """A form that can pick reads its arguments again afterwards: kept across the pick they were 59 and 85 spilled scalar registers (d = 512,
    two and eight rows per workgroup), in launches that do not pick as well."""
    with open(os.path.join(ROOT, "paper_2109_08003_amd", "libnt.so"), "rb") as f:
        so = f.read()
    spilled = {}
    for at in (m.start() for m in re.finditer(rb"AMDGPU\0\0\x83", so)):  # code objects' notes: a map of three
        for kernel in msgpack.Unpacker(io.BytesIO(so[at + 8:]), raw=False).unpack()["amdhsa.kernels"]:
            spilled[kernel[".name"]] = kernel[".sgpr_spill_count"]
    form = re.compile(r"_ZN2nt11dec1_kernelILi\d+ELi(2ELi8|8ELi16)ELi4ELi0ELb0ELb[01]ELb0ELb0E")
    got = {n: v for n, v in spilled.items() if form.match(n)}
    assert len(got) == 8 and max(got.values()) <= 32, got


def test_folded_caches_end_at_512_rows_and_32768_tokens(host):
    """The decoder layer's form with folded caches, on both sides of both lines."""
    got = host("""
model, out = load(config(n_enc=1), tokens=40000), []
a = np.zeros(40000, dtype=np.int32)
for rows, length in ((512, 1), (513, 1), (512, 64), (512, 65), (256, 128), (256, 129), (163, 201), (164, 201)):
    encode(model, rows, length)
    stub.stub_clear()
    nt.binding._check(nt.binding.lib().nt_decode_greedy(model._h, rows, 1, None, a.ctypes.data, None))
    out.append([n for n, _ in launches() if "dec1_kernel" in n])
print(json.dumps(out))
""")
    folded = [bool(re.search(r"Lb[01]ELb0ELb1ELb0EEE", names[0])) for names in got]
    assert [len(names) for names in got] == [1] * 8
    assert folded == [True, False, True, False, True, False, True, False]


def test_arg_max_of_17_to_32_rows(host):
    """More than 256 strips of the output matrix, up to 32 rows: the kernel that reads all of it; but from 17 rows on (256-wide models: 25)
    the scout where the pick is no launch, that is in fixed-length decoding of one head, in one layer without an FFN, and from 17 rows on
    in every batch of a call that has several."""
    got = host("""
out, kinds = [], lambda: sorted({k for n, _ in launches() for k in ("vocab_wide", "vocab_scout_few", "vocab_pick") if k in n})
for name, kw in (("one head", dict()), ("narrow", dict(d_model=256)), ("deep", dict(n_dec=2)), ("ffn", dict(dec_d_ffn=512)), ("heads", dict(n_heads=8))):
    model = load(dict(config(n_enc=1, **kw), vocab=16450), tokens=4096, lanes=2)
    a = np.zeros(4096, dtype=np.int32)
    for rows in (16, 17, 24, 25, 32, 33):
        for mode in ("fixed", "eos"):
            encode(model, rows, 2)
            stub.stub_clear()
            args = model._h, rows, 2, None
            if mode == "eos":  # (two steps: the host does not wait for the device yet)
                nt.binding._check(nt.binding.lib().nt_decode_greedy_eos(*args, 2, a.ctypes.data, a.ctypes.data, None))
            else:
                nt.binding._check(nt.binding.lib().nt_decode_greedy(*args, a.ctypes.data, None))
            out.append((name, rows, mode, kinds()))
        for batches in (1, 2):
            stub.stub_clear()
            model.translate_batch(np.full(2 * rows * batches, 5, dtype=np.int32), np.arange(0, 2 * rows * batches + 1, 2, dtype=np.int64), 4096,
                                  max_rows=rows, stream=Stream)
            out.append((name, rows, "several" if batches > 1 else "fixed", kinds()))
print(json.dumps(out))
""")
    for name, rows, mode, kinds in got:
        line = 16 if mode == "several" else 32 if mode == "eos" or name in ("deep", "ffn", "heads") else 24 if name == "narrow" else 16
        assert kinds == (["vocab_wide"] if rows <= line else ["vocab_pick", "vocab_scout_few"]), (name, rows, mode, kinds)  # (the last step's pick)


def test_integer_folded_layers_are_one_round_of_workgroups(host):
    """At d = 512, where a CU holds two of them, the forms with the fewest rows per workgroup end at 512 rows."""
    got = host("""
out = []
for ffn in (-1, 512):
    model = load(config(n_enc=1, dec_d_ffn=ffn), tokens=40000)
    a = np.zeros(40000, dtype=np.int32)
    for rows in (512, 513, 1023):
        encode(model, rows, 32800 // rows + 1)  # past the fp32 caches' 32,768 tokens
        stub.stub_clear()
        nt.binding._check(nt.binding.lib().nt_decode_greedy(model._h, rows, 1, None, a.ctypes.data, None))
        out += [(rows, n, b) for n, b in launches() if "dec1_kernel" in n]
print(json.dumps(out))
""")
    form = lambda n: tuple(int(x) for x in re.search(r"dec1_kernelILi512ELi(\d+)ELi(\d+)ELi\d+ELi1ELb0", n).groups())
    assert [(rows, *form(n), b) for rows, n, b in got] == [(512, 1, 4, 512), (513, 2, 4, 257), (1023, 2, 4, 512),
                                                          (512, 2, 8, 256), (513, 4, 16, 129), (1023, 4, 16, 256)]


def test_lanes_with_different_sentence_lengths_share_a_kernel(host):
    """Four threads meet the tiled encoder attention for the first time with four lengths: none may lower the LDS limit under
    another's launches."""
    rc, message = host("""
model = load(config(n_enc=4), lanes=4)
C.c_int.in_dll(stub, "stub_slow_limits").value = 1
lens = np.array([199, 190, 150, 140, 135, 134, 131, 130])
offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
try:
    model.translate_batch(np.full(offsets[-1], 5, dtype=np.int32), offsets, 200, stream=Stream)
    assert any("enc_attention_kernel" in n for n, _ in launches())
    print(json.dumps((0, "")))
except nt.NtError as e:
    print(json.dumps((e.code, str(e))))
""")
    assert rc == 0, message
