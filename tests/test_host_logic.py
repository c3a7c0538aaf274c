"""Host-side logic that needs no GPU: the index arithmetic the kernels rely on."""
import os
import re
import struct
import subprocess

import numpy as np
import pytest


def _magic(d):
    return 0 if d <= 1 else (1 << 32) // d + 1


def _udiv_magic(u, d, m):
    """The kernels' division by a precomputed reciprocal, emulated with exact integers: high word of the
    32 x 32 product, then one multiply-and-compare."""
    if m == 0:
        return u
    q = (u * m) >> 32
    q &= 0xFFFFFFFF
    return q - 1 if ((q * d) & 0xFFFFFFFF) > u else q


def test_reciprocal_division_is_exact_over_the_admitted_range():
    """Sub-tile ids are below 2^30 / 16 and divisors (sub-tiles per image, per row) are arbitrary: the corrected
    form must be exact where the bare high-word estimate is not (power-of-two grids with many streams)."""
    rng = np.random.default_rng(5)
    bad_plain = 0
    for d in [2, 3, 4, 7, 16, 49, 64, 196, 4096, 16384, 65536, 12345, 99991, (1 << 20) + 3]:
        m = _magic(d)
        us = {0, 1, d - 1, d, d + 1, (1 << 26) - 1, (1 << 26), (1 << 30) - 1}
        us |= {k * d - 1 for k in (2, 1000, (1 << 26) // d) if k * d - 1 > 0}
        us |= {k * d for k in (2, 1000, (1 << 26) // d)}
        us |= set(int(v) for v in rng.integers(0, 1 << 30, size=2000))
        for u in us:
            assert _udiv_magic(u, d, m) == u // d, (u, d)
            bad_plain += ((u * m) >> 32) != u // d
    assert bad_plain > 0  # the uncorrected estimate does fail in this range: the correction is needed
    # the advisor's cases: last sub-tile of stream >= 16 at 32 streams of 128 x 128 sub-tiles
    d = 16384
    u = 17 * d - 1
    assert ((u * _magic(d)) >> 32) != u // d and _udiv_magic(u, d, _magic(d)) == u // d


def test_position_kernel_unit_shapes_terminate_and_fit(tmp_path):
    """The work-unit choice of the position-gather kernel (pure host code): compiled alone and run over the
    benchmark shapes and a sweep; it must end, and what it picks must respect the kernel's limits (staged units
    and output positions per thread, LDS budget) and cover every output row and stream."""
    import os
    import re
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = tmp_path / "pos_shape_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(root, "include"), "-I",
                    os.path.join(root, "paper_1802_09723_amd", "csrc"), os.path.join(root, "tests", "host", "pos_shape_test.cpp"),
                    "-o", str(exe)], check=True)
    cases = [(1, 32, 32, 16, 16, 3, 1, 1, 1, 1), (512, 13, 13, 384, 384, 3, 1, 1, 1, 1), (512, 27, 27, 96, 256, 5, 2, 2, 1, 1),
             (257, 256, 256, 16, 4, 3, 1, 1, 1, 1), (3, 100, 100, 32, 8, 1, 0, 1, 1, 1)]
    for n in (1, 2, 64):
        for hw, c in ((56, 64), (28, 128), (14, 256), (7, 512)):
            cases.append((n, hw, hw, c, c, 3, 1, 1, 2, 2))
    rng = np.random.default_rng(9)
    for _ in range(60):
        k = int(rng.choice([1, 3, 5, 7]))
        hw = int(rng.integers(k, 80))
        grp = int(rng.choice([1, 2]))
        cases.append((int(rng.integers(1, 600)), hw, int(rng.integers(k, 80)), 16 * grp * int(rng.integers(1, 9)),
                      4 * grp * int(rng.integers(1, 70)), k, int(rng.integers(0, k)), grp, int(rng.choice([1, 2])), int(rng.choice([1, 2]))))
    eligible = 0
    for cse in cases:
        out = subprocess.run([str(exe)] + [str(v) for v in cse], check=True, capture_output=True, text=True, timeout=10).stdout
        if out.strip() == "no":
            continue
        eligible += 1
        f = {k: int(v) for k, v in re.findall(r"(\w+)=(\d+)", out)}
        n, h, w, ci, co, k, pad, grp, es, terms = cse
        ho, wo = h + 2 * pad - k + 1, w + 2 * pad - k + 1
        assert f["npos"] * 2 <= 256 * 10 and f["G"] * f["R"] * wo <= 512 * 2, (cse, f)
        assert f["lds"] <= 160 * 1024 - 1024, (cse, f)
        assert f["nbands"] * f["R"] >= ho and f["nsg"] * f["G"] >= n, (cse, f)
        assert f["units"] == f["nsg"] * f["nbands"] * grp * f["ncg"], (cse, f)
        assert f["RB"] == f["R"] + k - 1 and f["WP"] == w + pad and f["npos"] == f["G"] * f["RB"] * f["WP"] + pad
    assert eligible >= 20


def test_binary_band_geometry_terminates_fits_and_covers(tmp_path):
    """The band choice of the binary delta kernel (pure host code), compiled alone and run over the configuration
    shapes and a sweep: it must end; the bands cover every output row; a band's window, flags, list and sums fit
    the LDS budget; and where the single-launch step is allowed every input position lies in the window of the band
    that owns its row (else a change would be missed or counted twice)."""
    import os
    import re
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = tmp_path / "bin_shape_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(root, "include"), "-I",
                    os.path.join(root, "paper_1802_09723_amd", "csrc"), os.path.join(root, "tests", "host", "bin_shape_test.cpp"),
                    "-o", str(exe)], check=True)
    cases = [(1, 28, 28, 256, 256, 3, 1, 1, 1), (64, 28, 28, 256, 256, 3, 1, 1, 1), (1, 14, 14, 512, 512, 3, 1, 1, 1),
             (64, 14, 14, 512, 512, 3, 1, 1, 1), (1, 6, 300, 256, 16, 3, 1, 1, 1), (3, 30, 26, 128, 48, 3, 1, 1, 1),
             (1, 40, 40, 64, 32, 3, 1, 1, 1), (70000, 8, 8, 32, 8, 3, 1, 1, 1), (2, 11, 9, 128, 32, 3, 2, 1, 2),
             (1, 9, 9, 32, 8, 1, 2, 0, 1), (5, 200, 200, 32, 8, 5, 1, 2, 1)]
    # wide layers whose row fits only without the padding of the staged positions: bands, as long as a frame is small
    wide = [(1, 16, 350, 128, 128, 3, 1, 1, 1), (64, 4, 365, 128, 256, 3, 1, 1, 1), (3, 5, 335, 64, 130, 3, 1, 1, 1), (2, 4, 990, 128, 8, 1, 1, 0, 1),
            (1, 4, 1200, 128, 64, 1, 1, 0, 1), (2, 2, 470, 512, 65, 1, 1, 0, 1), (2, 3, 350, 256, 24, 3, 1, 1, 2)]
    cases += wide + [(1, 14, 14, 128, 512, 1, 1, 0, 1), (64, 28, 28, 128, 512, 1, 1, 0, 1), (128, 30, 30, 256, 256, 1, 1, 0, 1), (2, 9, 9, 288, 64, 1, 1, 0, 1)]
    rng = np.random.default_rng(17)
    for _ in range(80):
        k = int(rng.choice([1, 3, 5, 7]))
        grp = int(rng.choice([1, 2]))
        cases.append((int(rng.integers(1, 300)), int(rng.integers(k, 90)), int(rng.integers(k, 90)), 32 * grp * int(rng.integers(1, 9)),
                      grp * int(rng.integers(1, 130)), k, int(rng.choice([1, 2, 3])), int(rng.integers(0, k)), grp))
    banded = fused = 0
    for cse in cases:
        out = subprocess.run([str(exe)] + [str(v) for v in cse], check=True, capture_output=True, text=True, timeout=10).stdout
        if out.strip() == "no":
            continue
        f = {k: int(v) for k, v in re.findall(r"(\w+)=(\d+)", out)}
        n, h, w, ci, co, k, stride, pad, grp = cse
        assert f["ho"] == (h + 2 * pad - k) // stride + 1 and f["wo"] == (w + 2 * pad - k) // stride + 1
        assert cse not in wide or (f["R"] > 0 and f["bpitch"] < f["pitch"]), (cse, f)
        # the dense layer: on tiles without bands, for wide layers and for 1 x 1 filters of up to 256 channels (not on a chip full
        # of bands over mostly empty tiles)
        t1 = k == 1 and ci // grp <= 256 and not (f["vec4"] and n * f["nbands"] * grp * -(-co // grp // 64) >= 512
                                                  and 5 * f["ho"] * f["wo"] < 256 * -(-f["ho"] // 8) * -(-f["wo"] // 8))
        assert f["dtiles"] == int(f["R"] == 0 or f["bpitch"] < f["pitch"] or t1), (cse, f)
        if f["R"] == 0:
            continue
        banded += 1
        R, nb = f["R"], f["nbands"]
        assert nb * R >= f["ho"] and (nb - 1) * R < f["ho"], (cse, f)           # every output row in exactly one band
        assert n * nb <= 65535 and R * f["wo"] <= 65535, (cse, f)               # grid and 16-bit list entries
        assert f["lds"] <= 79 * 1024 and f["bpitch"] in (f["pitch"], 4 * f["nslab"]), (cse, f)
        assert f["bth"] == (R - 1) * stride + k and f["btw"] == (f["wo"] - 1) * stride + k, (cse, f)
        if f["fused"]:
            fused += 1
            assert f["vec4"] == 1
            # band b stages input rows [b R stride - pad, b R stride - pad + bth) and all columns [-pad, -pad + btw);
            # it owns rows [b R stride, (b + 1) R stride), the last band up to h
            assert -pad + f["btw"] >= w, (cse, f)
            for b in range(nb):
                lo = b * R * stride
                hi = h if b == nb - 1 else (b + 1) * R * stride
                assert lo >= b * R * stride - pad and hi <= b * R * stride - pad + f["bth"], (cse, f, b)
    assert banded >= 40 and fused >= 10


@pytest.mark.parametrize("gone", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_the_current_stream_whatever_torch_names_it(monkeypatch, gone):
    """The raw stream comes from functions that are torch's own; without them from the stream object."""
    import types

    import torch
    from paper_1802_09723_amd.binding import _stream_ptr
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    for handle in (0x1230, 0):
        monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 1, raising=False)
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: handle if device == 1 else -1, raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=handle))
        for name in gone:
            monkeypatch.delattr(torch._C, name)
        assert _stream_ptr(None) == (handle or None)


def _gfx950_functions(path, tmp_path, name):
    """{kernel: [(address, instruction)]} of the library's gfx950 functions whose mangled name holds `name`."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    blob, found = open(path, "rb").read(), {}
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob)):
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + n] and name.encode() in blob[at + off:at + off + size]:
                obj = tmp_path / f"{at}.o"
                obj.write_bytes(blob[at + off:at + off + size])
                fn = None
                for line in subprocess.run([objdump, "-d", str(obj)], capture_output=True, text=True, check=True).stdout.splitlines():
                    if m := re.match(r"^[0-9a-f]+ <(.*)>:", line):
                        fn = m.group(1) if name in m.group(1) else None
                        if fn:
                            found[fn] = []
                    elif fn and (m := re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+): ", line)):
                        found[fn].append((int(m.group(2), 16), m.group(1)))
            pos += 24 + n
    return found


def test_short_k_loops_begin_where_they_are_fastest(tmp_path):
    """The one-term K loop of the window-tile kernel's shape of one channel block and eight slots begins eight bytes into a 32-byte
    line of instructions, in every form of the kernel (wherever else it lies it is up to 6 % slower)."""
    from paper_1802_09723_amd.binding import lib_path
    if not os.path.exists(lib_path()):
        pytest.skip("the library is not built")
    kernels = {k: v for k, v in _gfx950_functions(lib_path(), tmp_path, "conv_gather_kernel").items()
               if re.search(r"conv_gather_kernelILi\dELi\dELi1ELi8E", k)}
    assert len(kernels) >= 10
    for fn, code in kernels.items():
        loops = []  # (length, begin) of the loops around this kernel's four one-term products
        for at, text in code:
            m = re.match(r"s_c?branch\S* (\d+)", text)
            if m and int(m.group(1)) > 32767:
                begin = at + 4 + 4 * (int(m.group(1)) - 65536)
                if sum("v_mfma" in t for a, t in code if begin <= a <= at) == 4:
                    loops.append((at - begin, begin))
        assert loops and min(loops)[1] % 32 == 8, fn
