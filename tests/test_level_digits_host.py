"""The codebook's digits for the matrix-core logit kernel (build_level_digits):
the digits, summed as the kernel sums them, stand for every level to 2^-23 of
itself (twice the rounding of a float); one set of them does for the Lloyd-Max
codebooks at every width, at both ends of the range of floats too, further sets
for codebooks whose levels span orders of magnitude; and a level's mirror image
is exactly its negative.  Runs on the CPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2603_28430_amd", "csrc")


def test_level_digits(tmp_path):
    # host code with _Float16: the compiler that builds the library's host part
    cxx = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    if not os.path.exists(cxx) and (cxx := shutil.which("clang++")) is None:
        pytest.skip("no clang++")
    exe = tmp_path / "level_digits_check"
    subprocess.run([cxx, "-O2", "-std=c++17", f"-I{CSRC}", os.path.join(HERE, "native", "level_digits_check.cpp"),
                    os.path.join(CSRC, "isoq_host_params.cpp"), "-o", str(exe)], check=True, capture_output=True,
                   text=True)
    books = [(b, oracle.codebook(b, d), 1) for b in (2, 3, 4) for d in (1, 64, 80, 96, 128, 160, 192, 256, 512, 1024)]
    for b in (2, 3, 4):
        k = 1 << (b - 1)
        for ratio in (2.0, 50.0, 1e3, 1e6):
            pos = 0.3 * ratio ** (np.arange(k) / (k - 1) - 1.0)
            books.append((b, np.concatenate([-pos[::-1], pos]), None))
        zero = np.concatenate([[1e-60], 0.1 + np.arange(1, k) / 7.0])   # (a level that is zero as a float)
        books.append((b, np.concatenate([-zero[::-1], zero]), None))
        books.append((b, np.concatenate([-zero[::-1], zero]) * 1e-60, 1))
    # codebooks at the ends of the range of floats
    books += [(b, c * scale, sets) for b, c, sets in books[:30:5] for scale in (2.0 ** -115, 2.0 ** 120)]
    text = "".join("%d %s\n" % (b, " ".join("%.9g" % np.float32(v) for v in c)) for b, c, _ in books)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
    lines = out.strip().splitlines()
    assert len(lines) == len(books)
    for line, (b, c, sets) in zip(lines, books):
        n, narrow, *vals = line.split()
        vals, ref = np.array(vals, float), np.float32(c).astype(float)
        assert 1 <= int(n) < 8 and (sets is None or int(n) == sets), (b, n)
        assert np.all(np.abs(vals - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-30), (b, vals / ref - 1)
        assert np.array_equal(vals, -vals[::-1])
        # the short sum: the Lloyd-Max codebooks, not those of distant levels
        assert int(narrow) if sets else not (int(narrow) and ref[-1] > 64 * ref[len(ref) // 2])
