"""How many replays a compute unit holds at once, from what the compiler wrote into the built library: registers (and how many
of them it keeps in memory) and fixed LDS of every replay kernel, and the dynamic LDS of a launch.  A replay takes its time however few run beside it, so
a population that does not fit at once takes a second round."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2602_11688_amd", "libgorgo.so")
LLVM = "/opt/rocm/llvm/bin"
TOOLS = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
LDS, PIECE, LANE_REGISTERS, WAVES = 160 * 1024, 1280, 512, 8        # of a compute unit; of one of its four SIMDs

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not all(map(os.path.exists, TOOLS)) or shutil.which("c++filt") is None,
                                reason="no built library, or no tools to read it")


@pytest.fixture(scope="module")
def notes(tmp_path_factory):
    """name -> (registers of a lane, fixed LDS, threads of a workgroup, registers of a lane kept in memory)."""
    tmp = tmp_path_factory.mktemp("code")
    fat, code = str(tmp / "fat"), str(tmp / "code")
    subprocess.run([TOOLS[0], f"--dump-section=.hip_fatbin={fat}", LIB, os.devnull], check=True)
    # (one bundle per source file, of which kernels.hip's is the one with kernels in it)
    data = open(fat, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    starts = [m.start() for m in re.finditer(magic, data)]
    found = {}
    for a, b in zip(starts, starts[1:] + [len(data)]):
        open(fat, "wb").write(data[a:b])
        subprocess.run([TOOLS[1], "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}",
                        f"--output={code}"], check=True)
        notes = subprocess.run([TOOLS[2], "--notes", code], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n  - ", notes):
            def field(key):
                m = re.search(rf"\.{key}:\s+(\S+)", block)
                return m.group(1) if m else None
            name = field("name")
            if name and field("vgpr_count"):
                found[name] = tuple(int(field(k)) for k in ("vgpr_count", "group_segment_fixed_size", "max_flat_workgroup_size",
                                                            "vgpr_spill_count"))
    names = list(found)
    plain = subprocess.run(["c++filt"], input="\n".join(names), check=True, capture_output=True, text=True).stdout.split("\n")
    return {p: found[n] for p, n in zip(plain, names)}


@pytest.fixture(scope="module")
def kernels(notes):
    """name -> (registers of a lane, fixed LDS, threads of a workgroup)."""
    return {name: kernel[:3] for name, kernel in notes.items()}


def test_registers_stay_registers(notes):
    """No replay kernel keeps a lane's registers in memory, and the four-wavefront kernel of imperfect proxy knowledge is away from the
    96 where it would begin to (engine model and tuner together need them all)."""
    replays = {name: kernel for name, kernel in notes.items() if re.search(r"replay_\w+_kernel<", name)}
    assert len(replays) >= 50
    assert not [(name, kernel) for name, kernel in replays.items() if kernel[3] != 0]
    proxy = {name: kernel[0] for name, kernel in replays.items()
             if re.search(r"replay_segments_kernel<(0, false|0, true|1, false), true, 1, false>", name)}
    assert len(proxy) == 3 and max(proxy.values()) <= 88, proxy


def _resident(kernel, dynamic):
    registers, fixed, threads = kernel
    waves = min(WAVES, LANE_REGISTERS // ((registers + 7) // 8 * 8)) * 4
    lds = -(-(fixed + dynamic) // PIECE) * PIECE
    return min(waves // (threads // 64), LDS // lds)


def _resident_of_six(kernel, dynamic):
    """Workgroups of six wavefronts: each takes the room of two on every SIMD (seven wavefronts of 72 registers fit a SIMD, and
    three such workgroups a compute unit)."""
    registers, fixed, threads = kernel
    assert threads == 384
    lds = -(-(fixed + dynamic) // PIECE) * PIECE
    return min(min(WAVES, LANE_REGISTERS // ((registers + 7) // 8 * 8)) // 2, LDS // lds)


def _queues(R, B, engine, window):
    """Dynamic LDS of a segment-row replay: its service slots, four sets of 64 or more, and the tuner's window."""
    return max(4, -(-R * B // 64)) * 64 * (44 if engine else 40) + (window + 7) // 8 * 64


# variants as the template arguments say: mode (1: online tuner), engine model, imperfect proxy knowledge
@pytest.mark.parametrize("R,B,window,least", [(32, 8, 128, 5), (64, 4, 128, 5), (32, 16, 128, 4), (64, 8, 128, 4), (48, 16, 0, 3),
                                              (32, 8, 1024, 4), (64, 16, 128, 2)])
def test_replays_of_a_compute_unit(kernels, R, B, window, least):
    seen = 0
    for name, kernel in kernels.items():
        seg = re.search(r"replay_segments_kernel<(\d), (true|false), (true|false), 1, false>", name)
        blk = re.search(r"replay_blocks_kernel<(\d), (true|false), (true|false)>", name)
        if not seg and not blk:
            continue
        mode, engine, _ = (seg or blk).groups()
        dynamic = _queues(R, B, engine == "true", window if mode == "1" else 0) + (0 if seg else 44 * R)
        assert _resident(kernel, dynamic) >= least, (name, kernel, dynamic)
        seen += 1
    assert seen >= 24


@pytest.mark.parametrize("R,B,window,few", [(12, 8, 128, True), (2, 64, 1024, True), (32, 8, 128, False), (64, 4, 128, False),
                                            (16, 16, 1024, False)])
def test_replays_of_six_wavefronts(kernels, R, B, window, few):
    """What the launch rule takes for granted: up to 768 replays (three per compute unit) with up to 12 replicas, but 512 with
    proxy, engine model and tuner together; 512 (two) with more."""
    seen = 0
    for name, kernel in kernels.items():
        apart = re.search(r"replay_apart_kernel<(\d), (true|false), (true|false), false>", name)
        if not apart:
            continue
        mode, engine, proxy = apart.groups()
        dynamic = _queues(R, B, engine == "true", window if mode == "1" else 0)
        all_three = (mode, engine, proxy) == ("1", "true", "true")
        assert _resident_of_six(kernel, dynamic) >= (3 if few and not all_three else 2), (name, kernel, dynamic)
        seen += 1
    assert seen == 14


@pytest.mark.parametrize("R,B,window,least", [(32, 8, 128, 4), (64, 4, 128, 4), (16, 8, 1024, 4), (32, 16, 128, 4)])
def test_replays_over_rows_of_stamps(kernels, R, B, window, least):
    """As many as with hashed tables: four per compute unit, five in the variants of up to 96 registers."""
    seen = 0
    for name, kernel in kernels.items():
        rows = re.search(r"replay_rows_kernel<(\d), (true|false), (true|false)>", name)
        if not rows:
            continue
        mode, engine, proxy = rows.groups()
        dynamic = _queues(R, B, engine == "true", window if mode == "1" else 0) + R * (16 + 25 * 4) + 4
        all_three = (mode, engine, proxy) == ("1", "true", "true")
        assert _resident(kernel, dynamic) >= least + (0 if all_three or R * B > 256 else 1), (name, kernel, dynamic)
        seen += 1
    assert seen == 14


@pytest.mark.parametrize("R,B,window,pairs", [(32, 8, 128, 2), (16, 16, 128, 2), (32, 16, 128, 2), (32, 32, 128, 1)])
def test_pairs_of_replays(kernels, R, B, window, pairs):
    """Workgroups of eight wavefronts with two replays: two per compute unit, one with 1,024 service slots."""
    seen = 0
    for name, kernel in kernels.items():
        apart = re.search(r"replay_apart_pairs_kernel<(\d), (true|false), (true|false)>", name)
        if not apart:
            continue
        mode, engine, proxy = apart.groups()
        dynamic = 2 * _queues(R, B, engine == "true", window if mode == "1" else 0)
        assert kernel[2] == 512 and min(_resident(kernel, dynamic), 2) == pairs, (name, kernel, dynamic)
        seen += 1
    assert seen == 10
