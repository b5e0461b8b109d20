"""How many replays a compute unit holds at once, from what the compiler wrote into the built library: registers and
fixed LDS of every replay kernel, and the dynamic LDS of a launch.  A replay takes its time however few run beside it, so
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
def kernels(tmp_path_factory):
    """name -> (registers of a lane, fixed LDS, threads of a workgroup)."""
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
                found[name] = (int(field("vgpr_count")), int(field("group_segment_fixed_size")), int(field("max_flat_workgroup_size")))
    names = list(found)
    plain = subprocess.run(["c++filt"], input="\n".join(names), check=True, capture_output=True, text=True).stdout.split("\n")
    return {p: found[n] for p, n in zip(plain, names)}


def _resident(kernel, dynamic):
    registers, fixed, threads = kernel
    waves = min(WAVES, LANE_REGISTERS // ((registers + 7) // 8 * 8)) * 4
    lds = -(-(fixed + dynamic) // PIECE) * PIECE
    return min(waves // (threads // 64), LDS // lds)


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
