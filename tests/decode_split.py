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


class Split:
    """One batch's answer: workgroups, most chunks of a request, largest chunk, items (req, chunk, unit0, n_units, next), and the
    bytes of its records, of its metadata as the limit of the entry point that allocates nothing counts it, of its partials."""

    def __init__(self, head, items):
        self.n_wgs, self.max_chunks, self.chunk_units, _, self.record_bytes, self.metadata, self.partials = head
        self.items = items


def split(exe, batches):
    """[(kind, page tokens, cus, kv heads, q heads, append, override, lengths)] -> (page ids of a record, its header's words, bytes of
    a staging slot, cost of a chunk over bf16 pages, over FP8 pages), [Split]"""
    text = "".join(" ".join(map(str, (*b[:-1], len(b[-1]), *b[-1]))) + "\n" for b in batches)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=300).stdout.split("\n")
    at, answers = 1, []
    for _ in batches:
        head = tuple(map(int, out[at].split()))
        answers.append(Split(head, [tuple(map(int, l.split())) for l in out[at + 1:at + 1 + head[3]]]))
        at += 1 + head[3]
    return tuple(map(int, out[0].split())), answers
