"""Graph-specialised kernels on the CPU: the generated HIP source compiles for gfx950 with the
run-time compiler, spills no registers, and uses no packed fp32 instructions."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2607_12324_amd import synth

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OPTS = [b"--offload-arch=gfx950", b"-O3", b"-std=c++17", b"-Xclang", b"-target-feature", b"-Xclang",
        b"-packed-fp32-ops"]


@pytest.fixture(scope="module")
def emo():
    from paper_2607_12324_amd import emo as mod
    return mod


@pytest.fixture(scope="module")
def hiprtc():
    return ctypes.CDLL("libhiprtc.so")


def compiler_runtime() -> int:
    """hipRuntimeGetVersion of the runtime whose hiprtc the tests compile with (the one the
    library uses: torch's, loaded first)."""
    rt = ctypes.c_int(0)
    lib = ctypes.CDLL("libamdhip64.so")
    assert lib.hipRuntimeGetVersion(ctypes.byref(rt)) == 0
    return rt.value


def compile_source(hiprtc, src: str, tmp_path) -> str:
    prog = ctypes.c_void_p()
    assert hiprtc.hiprtcCreateProgram(ctypes.byref(prog), src.encode(), b"k.hip", 0, None, None) == 0
    opts = (ctypes.c_char_p * len(OPTS))(*OPTS)
    rc = hiprtc.hiprtcCompileProgram(prog, len(OPTS), opts)
    n = ctypes.c_size_t()
    hiprtc.hiprtcGetProgramLogSize(prog, ctypes.byref(n))
    log = ctypes.create_string_buffer(n.value + 1)
    hiprtc.hiprtcGetProgramLog(prog, log)
    assert rc == 0, log.value.decode()[-3000:]
    hiprtc.hiprtcGetCodeSize(prog, ctypes.byref(n))
    code = ctypes.create_string_buffer(n.value)
    hiprtc.hiprtcGetCode(prog, code)
    hiprtc.hiprtcDestroyProgram(ctypes.byref(prog))
    path = os.path.join(str(tmp_path), "k.co")
    with open(path, "wb") as f:
        f.write(code.raw)
    return path


def kernel_notes(path):
    out = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
    names = re.findall(r"\.name:\s+(\S+)", out)
    spills = [int(x) for x in re.findall(r"\.vgpr_spill_count:\s+(\d+)", out)]
    vgprs = [int(x) for x in re.findall(r"\.vgpr_count:\s+(\d+)", out)]
    return dict(zip(names, zip(vgprs, spills)))


def kernel_bodies(asm: str) -> dict:
    out, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\w+)>:", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif name:
            out[name].append(line)
    return out


def check_code_object(path, expect, spill_ok=()):
    """spill_ok: kernels held to 128 VGPRs (4 waves per SIMD) that may keep a few long-lived
    values in scratch (at most 1 in 100 instructions)."""
    notes = kernel_notes(path)
    for k in expect:
        assert k in notes, (k, notes)
    asm = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", path], capture_output=True, text=True,
                         check=True).stdout
    bodies = kernel_bodies(asm)
    for name, (vgpr, spill) in notes.items():
        if any(name.startswith(p) for p in spill_ok):
            assert vgpr <= 128, (name, vgpr)
            n_scr = sum("scratch_" in l for l in bodies[name])
            if (compiler_runtime() < 70200000 and
                    len(bodies[name]) // 100 < n_scr <= len(bodies[name]) // 20):
                pytest.xfail(f"{name}: {n_scr} scratch accesses under the hiprtc of HIP runtime "
                             f"{compiler_runtime()} (ROCm 7.0, torch's bundle); the bound is "
                             "met under ROCm 7.2's")
            assert n_scr <= len(bodies[name]) // 100, f"{name}: {n_scr} scratch accesses"
        else:
            assert spill == 0, f"{name} spills {spill} VGPRs"
            assert not any("scratch_" in l for l in bodies[name]), name
    assert not re.search(r"v_pk_(add|mul|fma)_f32", asm), "packed fp32 arithmetic in specialised kernels"
    # level words and scratch rows are global loads (a flat load would also hold up LDS waits)
    assert "flat_load" not in asm and "flat_store" not in asm
    return notes, asm


@pytest.mark.parametrize("k", [1, 2, 3])
def test_workload_kernels_compile_without_spills(emo, hiprtc, tmp_path, k):
    g = synth.config_graph(k)
    src = emo.EmoGraph(g, device=-1).specialized_source()
    path = compile_source(hiprtc, src, tmp_path)
    expect = ["emo_sp_select"] + (["emo_sp_slack"] if g.num_packs <= 160 else [])
    notes, asm = check_code_object(path, expect)
    # the forward pass is straight-line: roughly five vector instructions per pack, plus a
    # fixed amount for the group loop and the selection loop over the latency targets
    body = asm.split("<emo_sp_select>:")[1].split("s_endpgm")[0]
    valu = len(re.findall(r"^\s+v_", body, flags=re.M))
    assert valu < 6.5 * g.num_packs + 300, valu


def test_large_graph_is_not_one_kernel(emo):
    g = synth.config_graph(4)
    gh = emo.EmoGraph(g, device=-1)
    with pytest.raises(emo.EmoError) as ei:
        gh.specialized_source()
    assert ei.value.status == 5
    small = emo.EmoGraph(synth.config_graph(2), device=-1)
    with pytest.raises(emo.EmoError) as ei:
        small.segmented_source()
    assert ei.value.status == 5
    with pytest.raises(emo.EmoError) as ei:
        small.cut_source()
    assert ei.value.status == 5


def test_cut_segment_kernels_compile(emo, hiprtc, tmp_path):
    """The cut-segment kernels of the 4096-pack graph (16 segments of 256 packs: all in one
    forward-only kernel, four per slack kernel): every segment kernel and the last kernel compile
    without spills, scratch or flat accesses, the slack kernels within 168 VGPRs (three waves per
    SIMD)."""
    g = synth.config_graph(4)
    src = emo.EmoGraph(g, device=-1).cut_source()
    k = len(re.findall(r"\bemo_ks(\d+)\(", src))
    assert k == 4 and len(re.findall(r"\bemo_kf(\d+)\(", src)) == 1
    path = compile_source(hiprtc, src, tmp_path)
    names = ["emo_kf0"] + [f"emo_ks{j}" for j in range(k)] + ["emo_kfin"]
    notes, _ = check_code_object(path, names)
    assert max(v for v, _ in notes.values()) <= 168, notes


@pytest.mark.parametrize("which", ["packed-4096p", "shuffled-F5"])
def test_segmented_kernels_compile(emo, hiprtc, tmp_path, which):
    """The chained segment kernels of a large graph (LDS table windows, staged slack) and of a
    graph with shuffled pack ids and five levels (device table, direct slack stores): every
    forward and backward kernel compiles without spills or scratch, within 128 VGPRs."""
    if which == "packed-4096p":
        g = synth.config_graph(4)
    else:
        g = synth.packed_graph(77, 700, 4, 5, sync_every=128, cross_p=0.05, shuffle_pack_ids=True)
    src = emo.EmoGraph(g, device=-1).segmented_source()
    m = len(re.findall(r"\bemo_cf(\d+)\(", src))
    assert m >= 2 and len(re.findall(r"\bemo_cb(\d+)\(", src)) == m
    path = compile_source(hiprtc, src, tmp_path)
    notes, _ = check_code_object(path, [f"emo_cf{j}" for j in range(m)] + [f"emo_cb{j}" for j in range(m)],
                                 spill_ok=("emo_cb",))
    assert max(v for v, _ in notes.values()) <= 128, notes


@pytest.mark.parametrize("seed", range(3))
def test_random_graph_kernels_compile(emo, hiprtc, tmp_path, seed):
    """Odd shapes: pack counts not multiple of 4 or 16, non-power-of-two level counts,
    shuffled pack ids (no staged slack output), fixed nodes between packs."""
    rng = np.random.default_rng(300 + seed)
    for i, (V, F) in enumerate([(7, 3), (40, 16), (90, 5), (150, 200)]):
        g = synth.random_dag(rng, V, 3.0 / V, 0.7, F, shuffle_packs=bool(i % 2))
        src = emo.EmoGraph(g, device=-1).specialized_source()
        path = compile_source(hiprtc, src, tmp_path)
        check_code_object(path, ["emo_sp_select"])


# table sizes around the workgroup sizes' borders (16, 32 and 40 KB), packs a multiple of 32, of 16 or neither
ONE_KERNEL_TABLES = [(128, 16), (125, 16), (131, 16), (128, 32), (126, 32), (130, 32), (144, 32), (157, 32), (80, 64),
                     (96, 48), (100, 48), (64, 64), (40, 128), (17, 256), (158, 32), (41, 128)]


@pytest.mark.parametrize("P,F", ONE_KERNEL_TABLES)
def test_one_kernel_slack_layouts_compile(emo, hiprtc, tmp_path, P, F):
    """Table, staged slack columns and selection arrays fit one workgroup's LDS at every workgroup size:
    the modules of per-pack and per-node slack compile (a sum past the limit is a compile error)."""
    table = (P * F + (0 if F & (F - 1) == 0 else 256)) * 8
    in_lds = table <= 40 * 1024
    gh = emo.EmoGraph(synth.stream_graph(P, P, 2, F), device=-1)
    for src, name, cols in ((gh.specialized_source(), "emo_sp_slack", P), (gh.node_source(), "emo_sp_nodes", gh.num_nodes)):
        kc = int(re.search(r"#define EMO_KC (\d+)", src).group(1))
        block = int(re.search(r"__launch_bounds__\((\d+)\)\s+" + name, src).group(1))
        waves = int(re.search(r"float stg_all\[(\d+)\]", src).group(1))
        assert kc == (16 if cols % 32 == 16 else min(32, (cols + 3) // 4 * 4))
        assert block == 64 * waves == (256 if not in_lds or table <= 16384 else 512)
        assert (table if in_lds else 0) + waves * (kc * 65 + 64) * 4 < 160 * 1024 - 512
        notes = kernel_notes(compile_source(hiprtc, src, tmp_path))
        assert name in notes and ("emo_sp_select" in notes) == (name == "emo_sp_slack"), notes


@pytest.mark.parametrize("k", [1, 2, 3])
def test_interval_kernels_compile(emo, hiprtc, tmp_path, k):
    """The time-interval kernel of the small workloads (the 512-pack graph's 64 KB table in LDS,
    the bucket table and the rows in dynamic LDS) compiles without spills, scratch, packed fp32
    or flat accesses."""
    g = synth.config_graph(k)
    src = emo.EmoGraph(g, device=-1).interval_source()
    path = compile_source(hiprtc, src, tmp_path)
    notes, asm = check_code_object(path, ["emo_iv"])


@pytest.mark.parametrize("kind, bound", [("training", 1024), ("chains-40", 1024), ("wide", 512), ("small-table", 256), ("large-table", 256)])
def test_interval_kernel_of_every_bound(emo, hiprtc, tmp_path, kind, bound):
    """The time-interval kernel is compiled once, for the largest workgroup that its live finish times
    leave enough registers for and a table of more than 16 KB to share, and spills none there."""
    g = {"training": lambda: synth.config_graph(3), "chains-40": lambda: synth.stream_graph(1, 400, 40, 8),
         "wide": lambda: synth.random_dag(np.random.default_rng(1), 300, 0.03, 0.8, 16, shuffle_ids=False,
                                          shuffle_packs=False),
         "small-table": lambda: synth.packed_graph(5, 500, 16, 4, sync_every=501),
         "large-table": lambda: synth.packed_graph(5, 600, 4, 24, sync_every=700)}[kind]()
    src = emo.EmoGraph(g, device=-1).interval_source()
    assert int(re.search(r"#define EMO_BLOCK (\d+)", src).group(1)) == bound
    notes, _ = check_code_object(compile_source(hiprtc, src, tmp_path), ["emo_iv"])
    assert notes["emo_iv"][0] <= 512 * 256 // bound, notes


@pytest.mark.parametrize("P,F,waves", [(300, 40, 5), (400, 24, 5), (600, 24, 4)])
def test_interval_kernel_with_device_table_keeps_its_waves(emo, hiprtc, tmp_path, P, F, waves):
    """A table past LDS: registers for five waves a SIMD up to 512 packs, for four above (fewer waves leave
    a batch a nearly empty last round)."""
    src = emo.EmoGraph(synth.packed_graph(P, P, 4, F, sync_every=P + 1, cross_p=0.05), device=-1).interval_source()
    notes, _ = check_code_object(compile_source(hiprtc, src, tmp_path), ["emo_iv"])
    assert notes["emo_iv"][0] <= 512 // waves // 8 * 8, notes
