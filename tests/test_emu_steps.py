"""sim_kernel's source on the CPU under AddressSanitizer and
UndefinedBehaviorSanitizer (emu/emu_steps.cpp, one OS thread per GPU thread,
buffers of exactly the host's sizes): per-trial thresholds and tables, one-step
burns and turn-off times, windows and whole lattices, bitsets in LDS and in
global memory, queues that spill, widths at word boundaries, fires from corners.
Every simulation must equal the oracle's on the tables the source itself makes.
"""
import os
import pathlib
import shutil
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_1701_03549_amd import synth

EMU = pathlib.Path(__file__).resolve().parent / "emu"
REPO = pathlib.Path(__file__).resolve().parents[1]
SEED = 0x5EED0001


@pytest.fixture(scope="module")
def binaries(tmp_path_factory):
    cxx = next((c for c in ("/opt/rocm/llvm/bin/clang++", "clang++") if shutil.which(c)), None)
    if cxx is None:
        pytest.skip("no clang++ for the host")
    sys.path.insert(0, str(EMU))
    try:
        import mkkernel
    finally:
        sys.path.pop(0)
    out = tmp_path_factory.mktemp("emu_steps")
    mkkernel.generate(out / "kernel.inc")
    procs = {}
    for block in (64, 128):
        procs[block] = subprocess.Popen(
            [cxx, "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-pthread",
             "-ffp-contract=off", f"-DEMU_BLOCK={block}", f"-I{out}", f"-I{EMU}", f"-I{REPO / 'include'}",
             str(EMU / "emu_steps.cpp"), "-o", str(out / f"emu_{block}")],
            stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    for block, p in procs.items():
        err = p.communicate()[1]
        assert p.returncode == 0, err[-4000:]
    return {block: out / f"emu_{block}" for block in procs}


# width, height, threads, window, queue entries, global bitset
SHAPES = [(32, 40, 64, 0, 64, 0), (33, 37, 64, 0, 64, 1), (64, 33, 128, 0, 64, 0), (1, 70, 64, 0, 64, 1),
          (70, 1, 64, 0, 64, 0), (98, 97, 64, 64, 64, 0), (130, 90, 128, 64, 128, 1)]


@pytest.mark.parametrize("table", [1, 0])
@pytest.mark.parametrize("turn_off", [0, 1])
@pytest.mark.parametrize("W,H,threads,window,cap,glob", SHAPES)
def test_emulated_steps_match_oracle(binaries, tmp_path, W, H, threads, window, cap, glob, turn_off, table):
    """beta 2.5 ignites whole squares (fronts of hundreds of cells, past every
    form's limit and the queues of 64 entries), beta 0 every second neighbour;
    a row of NaN covariates for the filter (slopes of 120)."""
    from paper_1701_03549_amd import fire
    ls = synth.random_small_landscape(W, H, 7 * W + H, p_blocked=0.05)
    ls["slope_deg"][H // 3] = 120.0
    ign = [(0, 0), (W - 1, H - 1), (min(31, W - 1), H // 2)]
    for x, y in ign:
        ls["veg"][y, x] = 2
    betas = np.array([(2.5, 0.0, 0.0, 0.3, 0.0), (0.0, 0.2, 0.1, 0.4, 0.1)])
    steps = np.full(256, 3, dtype=np.uint8)
    steps[2] = 1
    sims = fire.make_sims(6, 0, -1, np.array(ign * 2), param_index=np.repeat([0, 1], 3))
    sims["max_steps"][4] = 7
    ls["veg"].astype(np.uint8).tofile(tmp_path / "veg.bin")
    for key, name in (("elev_m", "elev"), ("slope_deg", "slope"), ("aspect_deg", "aspect"), ("wind_to_deg", "wind")):
        np.ascontiguousarray(ls[key], dtype=np.float32).tofile(tmp_path / f"{name}.bin")
    betas.tofile(tmp_path / "betas.bin")
    steps.tofile(tmp_path / "steps.bin")
    sims.view(np.uint8).tofile(tmp_path / "sims.bin")
    r = subprocess.run([str(binaries[threads]), str(tmp_path), str(W), str(H), str(window), str(cap), "2", hex(SEED),
                        str(table), str(turn_off), str(glob)], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    if window:
        assert 0 < int(r.stdout.split("re-runs ")[1].split(" ")[0])
    T = np.fromfile(tmp_path / "tables.bin", np.uint32).reshape(2, H, W, 8)
    got = np.fromfile(tmp_path / "results.bin", np.uint8).view(fire.RESULT_DTYPE)
    maps = np.fromfile(tmp_path / "maps.bin", np.uint32).reshape(6, H, -1)
    for i, sd in enumerate(sims):
        o = oracle.simulate(ls["veg"], T[int(sd["param_index"])], (int(sd["ign_x"]), int(sd["ign_y"])),
                            int(sd["sim_index"]), SEED, int(sd["max_steps"]), burn_steps=steps if turn_off else None)
        assert (int(got["burnt"][i]), int(got["steps"][i]), int(got["trials"][i])) == \
            (o["burnt"], o["steps"], o["trials"]), i
        assert np.array_equal(maps[i], o["map"]), i
