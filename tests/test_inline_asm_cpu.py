"""Inline assembly in the kernels (no GPU): the compiler adds no wait states for
the registers that an assembly block reads, and a vector instruction that
reads a matrix result too early gets an older value.  So no assembly block may
hold a vector instruction; the loads to LDS, waits and barriers stay.  Checked on
the assembly that the library's own flags give."""
import concurrent.futures as cf
import glob
import os
import re
import subprocess

from paper_2608_18656_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _assembly(src, out):
    flags = [*hip_build.HIPCC_FLAGS, *hip_build.PER_FILE_FLAGS.get(os.path.basename(src), [])]
    subprocess.run([hip_build.hipcc(), *flags, "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-S", src,
                    "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_no_vector_instruction_in_inline_assembly(tmp_path):
    sources = sorted(glob.glob(os.path.join(hip_build.CSRC, "*.hip")))
    with cf.ThreadPoolExecutor(len(sources)) as ex:
        texts = list(ex.map(lambda s: _assembly(s, str(tmp_path / (os.path.basename(s) + ".s"))), sources))
    blocks = 0
    for src, text in zip(sources, texts):
        for body in re.findall(r";#ASMSTART\n(.*?);;#ASMEND", text, re.S):
            blocks += 1
            vector = [line.strip() for line in body.splitlines() if line.strip().startswith("v_")]
            assert not vector, (os.path.basename(src), vector)
    assert blocks > 0
