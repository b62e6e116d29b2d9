"""The library's kernels and launchers, compiled as plain C++ against the CPU stand-in
for the HIP device environment in tests/simt/ and run under the address sanitizer:
small end-to-end cases (prefill compress, one chunk, decode attention over cache +
buffer, decompress) through the C ABI and the Key selection by itself, compared with the oracle.  This checks the host
logic (grids, LDS sizes, arena and workspace layout) and that no kernel reads or
writes outside its buffers or its LDS; it does not replace the GPU parity tests (the
emulation knows nothing of the real compiler's code or the hardware's timing)."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import gear_workloads as gw
from oracle import gear_oracle as go
from tests import parity_util as pu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SIMT = os.path.join(ROOT, "tests", "simt")
CSRC = os.path.join(ROOT, "paper_2403_05527_amd", "csrc")
SOURCES = ["gear_api", "compress_filter", "compress_values", "lowrank", "decode", "decompress_export"]


def find_clang():
    for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")):
        if c and os.path.exists(c):
            return c
    return None


@pytest.fixture(scope="module")
def build(tmp_path_factory):
    """build(name): the library and tests/simt/<name>.cpp as one program."""
    cxx = find_clang()
    if cxx is None:
        pytest.skip("no clang++ to build the CPU emulation")
    out = tmp_path_factory.mktemp("simt")
    # -ffp-contract=fast: the host compiler may fuse every multiply-add it finds, except where the sources
    # switch contraction off (the quantizer's decision sequence), which the bit-exact code comparison checks
    flags = ["-std=c++17", "-O1", "-gline-tables-only", "-ffp-contract=fast", "-fsanitize=address", "-fno-omit-frame-pointer", "-pthread",
             "-I", SIMT, "-I", os.path.join(ROOT, "include"), "-I", CSRC]

    def objects(names, extra=()):
        procs = []
        suffix = ".d.o" if extra else ".o"
        for s in names:
            src = ["-x", "c++", "-c", os.path.join(CSRC, s + ".hip")] if s in SOURCES else ["-c", os.path.join(SIMT, s + ".cpp")]
            procs.append(subprocess.Popen([cxx] + src + ["-o", str(out / (s + suffix))] + flags + list(extra), stderr=subprocess.PIPE,
                                          text=True))
        for p in procs:
            err = p.communicate()[1]
            assert p.returncode == 0, err[-3000:]
        return [str(out / (s + suffix)) for s in names]

    common = objects(SOURCES + ["simt_rt"])

    def program(name, device=False):
        """device: the choice of a read's launch as on the device (the stand-in lowers its limits for the small cases)."""
        exe = str(out / name)
        if not os.path.exists(exe):
            parts = list(common)
            if device:
                parts[SOURCES.index("decode")] = objects(["decode"], ["-O0", "-fno-sanitize=address", "-DGEAR_CUS=256", "-DGEAR_SINGLE_WAVES=16",
                                                                      "-DGEAR_MERGE_16=16", "-DGEAR_MERGE_32=32"])[0]
            r = subprocess.run([cxx] + parts + objects([name]) + ["-o", exe] + flags, capture_output=True, text=True)
            assert r.returncode == 0, r.stderr[-3000:]
        return exe
    return program


@pytest.fixture(scope="module")
def emulator(build):
    return build("run_pipeline")


def test_dynamic_lds_is_raised_on_every_device(build):
    r = subprocess.run([build("check_devices", device=True)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


def test_copies_to_lds_arrive_at_the_wait(build):
    r = subprocess.run([build("check_copies")], capture_output=True, text=True, timeout=120, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("size,launch", [
    # bits, group, B, H_kv, H_q, n, rank, n_buf, n_buf_cap, chunks: the kernel, the blocks that share a slab's columns.  The single
    # launch of four columns would need more LDS than there is (factor rows staged, groups of 32): two columns per block fit.
    ("2 32 32 8 32 877 7 12 20 4", "single 2"),
    ("2 32 32 8 32 1765 7 0 20 1", "single 2"),
    ("2 32 64 4 16 1049 7 11 20 5", "single 2"),
    ("2 32 64 2 16 789 7 3 20 6", "single 4"),         # eight columns: neither fits as a whole nor in two parts
    ("4 32 16 8 64 1091 7 16 20 5", "single 4"),
    ("4 64 1 32 32 512 4 7 20 0", "single 1"),
    ("2 64 5 8 64 3001 4 13 20 2", "split 2"),
])
def test_read_is_launched_as_planned(build, size, launch):
    """The choice of the kernel and that of the parts rest on the same LDS size: where one block's LDS does not hold the single
    launch, the parts are those that are best without it."""
    r = subprocess.run([build("list_reads", device=True)], input=size + "\n", capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    kernel, parts, lds = r.stdout.split()
    assert kernel + " " + parts == launch and int(lds) <= 160 * 1024


@pytest.mark.parametrize("slots", [512, 16])
def test_workspace_holds_exactly_the_most_strips(tmp_path, slots):
    """The bound by which the workspace of the Gram matrices is sized is reached and never passed, at the device's number of
    block slots and at the stand-in's."""
    cxx = find_clang()
    if cxx is None:
        pytest.skip("no clang++")
    exe = str(tmp_path / "check_strips")
    r = subprocess.run([cxx, "-std=c++17", "-O2", "-pthread", "-DGEAR_BLOCK_SLOTS=%d" % slots, os.path.join(SIMT, "check_strips.cpp"), "-o", exe,
                        "-I", SIMT, "-I", os.path.join(ROOT, "include"), "-I", CSRC], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


# B, H, Hq, n, bits, g, ppm, rank, n_buf, per_head, chunk_n, n_b, n_lowrank
CASES = [
    (1, 4, 8, 290, 2, 64, 20000, 4, 5, False, 20, 20, -1),     # the method as stated; n > 256: Gram-matrix power iteration
    (1, 2, 2, 140, 4, 0, 30000, 2, 3, True, 20, 20, -1),       # per-vector groups and the per-head Value Filter
    (1, 8, 8, 70, 2, 64, 20000, 2, 3, False, 20, 20, -1),      # eight KV heads: Value token rows of 1024 entries, four per wave
    (1, 2, 2, 200, 4, 32, 30000, 2, 3, False, 20, 20, -1),     # two KV heads by the same kernel, 4-bit codes, groups of 32
    (1, 1, 2, 70, 2, 64, 20000, 2, 255, False, 255, 255, -1),  # the largest streaming buffer: 255 live rows, a flushed
                                                           # segment of 255 tokens (two 128-row pieces in the decode kernel)
    (1, 2, 8, 1100, 2, 128, 10000, 8, 7, False, 20, 20, -1),   # n > 1024: Key vectors selected in registers; rank 8, four
                                                           # query heads per KV head, groups of 128
    (1, 3, 3, 1030, 2, 64, 20000, 2, 3, False, 20, 20, -1),    # more Key rows: selected by lists of candidates
    (1, 1, 8, 150, 4, 64, 20000, 3, 4, False, 33, 40, -1),     # eight query heads per KV head, a rank that is not one read
                                                           # (factor rows staged in LDS), a flushed segment of 33 tokens
    (1, 2, 4, 330, 2, 64, 20000, 4, 6, False, 20, 20, 100),  # the low-rank term on the last 100 of 330 tokens only
    # blocks that walk several tiles of 128 tokens, a ragged one at the end (as the 1100-token case; in the one above the
    # low-rank term begins inside a strip's second tile):
    (1, 1, 1, 390, 4, 32, 50000, 2, 3, False, 20, 20, -1),     # groups of 32, long overflow lists
    (1, 1, 1, 390, 2, 0, 20000, 4, 3, True, 20, 20, 250),      # per-vector groups, the per-head Value Filter, a late low-rank term
    (1, 1, 2, 600, 2, 64, 20000, 2, 3, False, 20, 20, -1),     # a merge of four records
]


def _run_case(exe, d, B, H, Hq, n, bits, g, ppm, rank, n_buf, per_head, chunk_n, n_b, n_lowrank):
    """Writes a case's inputs to d and runs it: (the process's result, the oracle's cache, the inputs of its reads)."""
    w = gw.Workload("emu", B=B, H_kv=H, H_q=Hq, n=n, bits=bits, group=g, outlier_ppm=ppm, rank=rank,
                    rank_chunk=2, n_b=n_b, steps=1, seed=5)
    a = lambda t: t.numpy()
    oc = go.OracleCache(B, H, Hq, 128, bits, g, ppm, per_head)
    K, V, ib = a(gw.make_keys(w, n, 0)), a(gw.make_values(w, n, 0)), a(gw.make_init_B(w, rank, 0))
    for name, x in (("K", K), ("V", V), ("ib", ib)):
        x.tofile(os.path.join(d, name + ".bin"))
    if n_lowrank >= 0:
        oc.compress(K, V, rank, 3, ib, n_lowrank=n_lowrank)
    else:
        oc.compress(K, V, rank, 3, ib)
    Kc, Vc, ibc = a(gw.make_keys(w, chunk_n, 1)), a(gw.make_values(w, chunk_n, 1)), a(gw.make_init_B(w, 2, 1))
    for name, x in (("Kc0", Kc), ("Vc0", Vc), ("ibc0", ibc)):
        x.tofile(os.path.join(d, name + ".bin"))
    oc.compress(Kc, Vc, 2, 3, ibc)
    q, Kb, Vb = a(gw.make_queries(w, 0)), a(gw.make_keys(w, n_b, 50)), a(gw.make_values(w, n_b, 50))
    for name, x in (("q", q), ("Kb", Kb), ("Vb", Vb)):
        x.tofile(os.path.join(d, name + ".bin"))
    q2 = np.stack([q[:, :, 0], a(gw.make_queries(w, 1))[:, :, 0]], axis=2)       # two query rows per head
    q2.tofile(os.path.join(d, "q2.bin"))
    with open(os.path.join(d, "meta.txt"), "w") as f:
        f.write(" ".join(str(x) for x in [B, H, Hq, bits, g, ppm, n, rank, 1, chunk_n, 2, n_buf, n_b, 3, 1 if per_head else 0, n_lowrank]) + "\n")
    r = subprocess.run([exe, d], capture_output=True, text=True, timeout=900,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    return r, oc, q, q2, Kb, Vb


LAUNCHED = set()   # the kernels that this module's runs have launched


@pytest.fixture(scope="module")
def pipeline_runs(request, emulator, tmp_path_factory):
    def one(case):
        d = str(tmp_path_factory.mktemp("case"))
        return (d,) + _run_case(emulator, d, *case)
    selected = {tuple(i.callspec.params["case"]) for i in request.session.items
                if getattr(i, "originalname", "") == "test_pipeline_under_address_sanitizer"}
    pool = ThreadPoolExecutor(3)   # (an emulated run is bound by its barriers: a few at a time)
    return {c: pool.submit(one, c) for c in CASES if c in selected}


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_pipeline_under_address_sanitizer(pipeline_runs, case):
    B, H, Hq, n, bits, g, ppm, rank, n_buf, per_head, chunk_n, n_b, n_lowrank = case
    d, r, oc, q, q2, Kb, Vb = pipeline_runs[case].result()
    LAUNCHED.update(re.findall(r"^launch (\w+)", r.stderr, re.M))
    assert r.returncode == 0, r.stderr[-4000:]
    assert "AddressSanitizer" not in r.stderr
    out = np.fromfile(os.path.join(d, "out.bin"), np.float16).reshape(B, Hq, 1, 128)
    oc.decode_attn(q, Kb, Vb, n_buf)
    pu.check_attention(out, oc.last_attn_f64)
    Ko, Vo = oc.decompress()
    Kg = np.fromfile(os.path.join(d, "Khat.bin"), np.float16).reshape(Ko.shape).astype(np.float64)
    Vg = np.fromfile(os.path.join(d, "Vhat.bin"), np.float16).reshape(Vo.shape).astype(np.float64)
    for got, want in ((Kg, Ko.astype(np.float64)), (Vg, Vo.astype(np.float64))):
        assert np.linalg.norm(got - want) <= 1e-3 * np.linalg.norm(want)
    # codes, scales and zero-points bit for bit, although this build lets the compiler contract
    for name, segs in (("K", oc.K), ("V", oc.V)):
        o_codes = np.concatenate([s.codes for s in segs], axis=2)
        o_scale = np.concatenate([s.scale for s in segs], axis=2)
        o_zero = np.concatenate([s.zero for s in segs], axis=2)
        codes = np.fromfile(os.path.join(d, name + "codes.bin"), np.uint8).reshape(o_codes.shape)
        scale = np.fromfile(os.path.join(d, name + "scale.bin"), np.float16).reshape(o_scale.shape)
        zero = np.fromfile(os.path.join(d, name + "zero.bin"), np.float16).reshape(o_zero.shape)
        assert np.array_equal(scale.view(np.uint16), o_scale.view(np.uint16)), name
        assert np.array_equal(zero.astype(np.float32), o_zero.astype(np.float32)), name
        assert np.array_equal(codes, o_codes), name
        # the sparse matrix: support and values bit for bit, as a dense view and in coordinate form
        o_mask = np.concatenate([s.mask for s in segs], axis=2)
        o_vals = np.concatenate([s.svals for s in segs], axis=2)
        mask = np.fromfile(os.path.join(d, name + "mask.bin"), np.uint8).reshape(o_mask.shape).astype(bool)
        vals = np.fromfile(os.path.join(d, name + "svals.bin"), np.uint16).reshape(o_mask.shape)
        assert np.array_equal(mask, o_mask), name
        assert np.array_equal(vals[o_mask], o_vals.view(np.uint16)[o_mask]) and not vals[~o_mask].any(), name
        want = np.flatnonzero(o_mask)
        assert np.array_equal(np.fromfile(os.path.join(d, name + "coo_idx.bin"), np.int64), want), name
        assert np.array_equal(np.fromfile(os.path.join(d, name + "coo_val.bin"), np.uint16),
                              o_vals.view(np.uint16).reshape(-1)[want]), name
    # the exported factors of the prefill segment give the oracle's low-rank product (bar of the GPU tests)
    if rank > 0:
        for name, seg in (("K", oc.K[0]), ("V", oc.V[0])):
            A = np.fromfile(os.path.join(d, name + "_A.bin"), np.float16).reshape(B, H, n, rank).astype(np.float64)
            Bf = np.fromfile(os.path.join(d, name + "_B.bin"), np.float16).reshape(B, H, 128, rank).astype(np.float64)
            got = A @ np.swapaxes(Bf, -1, -2)
            want = seg.A.astype(np.float64) @ np.swapaxes(seg.Bf.astype(np.float64), -1, -2)
            assert np.linalg.norm(got - want) <= pu.LOWRANK_REL_TOL * np.linalg.norm(want), name
    if 2 * (Hq // H) <= 8 and n_buf >= 2:
        out2 = np.fromfile(os.path.join(d, "out2.bin"), np.float16).reshape(B, Hq, 2, 128)
        pu.check_attention(out2, go.decode_attn_multi(oc, q2, Kb, Vb, n_buf, True), "two query rows")


SELECTIONS = [   # kind of values, slabs, tokens, outliers in ppm, per-vector groups
    ("normal", 1, 3003, 20000, 1),          # the sample is the whole segment
    ("normal", 1, 5003, 20000, 0),          # ... is one row of each stretch, 16 channels per block
    ("normal", 1, 9001, 10000, 1),          # ... 8 channels per block
    ("normal", 3, 4100, 20000, 0),          # more than one round of blocks of 1024 threads: blocks of 512
    ("normal", 1, 40, 50000, 1),            # a flushed buffer, without its Values
    ("cliff", 1, 3003, 20000, 1), ("two channels", 1, 4100, 20000, 0), ("coarse grid", 1, 5003, 20000, 1), ("one sign", 1, 3003, 20000, 0),
    ("constant", 1, 9001, 20000, 0), ("falling", 1, 4100, 20000, 1), ("grid", 1, 9001, 150000, 0),   # the last: from a channel-major copy
]


@pytest.fixture(scope="module")
def selection_runs(request, build, tmp_path_factory):
    exe = build("select_keys")

    def one(case):
        kind, slabs, n, ppm, per_vector = case
        K = pu.values_of_kind(kind, (1, slabs, n, 128), n + ppm).numpy()
        f = str(tmp_path_factory.mktemp("keys") / "k")
        K.tofile(f)
        return K, f, subprocess.run([exe], input="%s %d %d %d %d\n" % (f, slabs, n, ppm, per_vector), capture_output=True, text=True,
                                    timeout=900, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    selected = {tuple(i.callspec.params["case"]) for i in request.session.items if getattr(i, "originalname", "") == "test_key_selection_under_address_sanitizer"}
    pool = ThreadPoolExecutor(3)
    return {c: pool.submit(one, c) for c in SELECTIONS if c in selected}


@pytest.mark.parametrize("case", SELECTIONS, ids=lambda c: "-".join(map(str, c)))
def test_key_selection_under_address_sanitizer(selection_runs, case):
    kind, slabs, n, ppm, per_vector = case
    K, f, r = selection_runs[case].result()
    assert r.returncode == 0 and "AddressSanitizer" not in r.stderr, r.stderr[-4000:]
    LAUNCHED.update(re.findall(r"^launch (\w+)", r.stdout, re.M))
    got = np.unpackbits(np.fromfile(f + ".mask", np.uint8).reshape(1, slabs, n, 16), axis=-1, bitorder="little").astype(bool)
    want = go.filter_keys(K, ppm)
    assert np.array_equal(got, want)
    if per_vector:
        y = np.where(want, np.float16(0), K).astype(np.float32)
        lo, hi = y.min(axis=2), y.max(axis=2)
        sz = np.fromfile(f + ".sz", np.float16).reshape(1, slabs, 128, 2).astype(np.float32)
        assert np.array_equal(sz[..., 0], ((hi - lo) / np.float32(3)).astype(np.float16).astype(np.float32))
        assert np.array_equal(sz[..., 1], lo)


def test_every_form_of_the_merge_ran(pipeline_runs):
    """The merge is built for 16, 32 and 64 records at once: split reads of the cases above go through each."""
    if len(pipeline_runs) < len(CASES):
        pytest.skip("not all cases were selected")
    forms = set()
    for run in pipeline_runs.values():
        forms |= set(re.findall(r"^launch decode_combine_kernel<(\d+)>", run.result()[1].stderr, re.M))
    assert forms == {"16", "32", "64"}


NOT_EMULATED = {"gram_sum_kernel",                                            # eight partial Gram matrices and more per slab
                "pi_sweep_kernel", "pi_update_kernel", "pi_finish_kernel"}    # a single round


def test_every_kernel_ran(request):
    """The cases above run each kernel of the library, those of both ways to read among them."""
    if sum(getattr(i, "originalname", "").endswith("under_address_sanitizer") for i in request.session.items) < len(CASES) + len(SELECTIONS):
        pytest.skip("not all cases were selected")
    kernels = set()
    for f in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, f)) as src:
            kernels |= set(re.findall(r"__global__(?:\s+__launch_bounds__\((?:[^()]|\([^()]*\))*\))?\s+void\s+(\w+)\(", src.read()))
    assert len(kernels) > 15
    assert kernels - LAUNCHED == NOT_EMULATED
