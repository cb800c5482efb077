"""The host's splitting of decode batches over workgroups, asked through a small program compiled for the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_19867_amd", "csrc")

# A latent batch whose longest chunk touches every page that the kernel has room for: pages of 96 tokens, so that a chunk of
# 247 pages' tiles starts inside one.  Requests, context, page tokens, decode CUs.
FULL_CHUNK = (32, 48000, 96, 32)


def build(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path / "decode_split_dump")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, os.path.join(ROOT, "tests", "decode_split_dump.cpp"), "-o", exe], check=True)
    return exe


def split(exe, batches):
    """[(kind, page tokens, cus, kv heads, override, lengths)] -> (page ids, header words, [(n_wgs, max_chunks, chunk_units, items)])"""
    text = "".join(f"{k} {P} {cus} {hkv} {o} {len(lens)} {' '.join(map(str, lens))}\n" for k, P, cus, hkv, o, lens in batches)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=300).stdout.split("\n")
    pages, words = map(int, out[0].split())
    at, answers = 1, []
    for _ in batches:
        n_wgs, max_chunks, chunk_units, n = map(int, out[at].split())
        answers.append((n_wgs, max_chunks, chunk_units, [tuple(map(int, l.split())) for l in out[at + 1:at + 1 + n]]))
        at += 1 + n
    return pages, words, answers
