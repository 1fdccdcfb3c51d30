"""Where the buffer loads of the kernels start (no GPU needed).

The hardware compares a lane's offset of a raw buffer load with the descriptor's size less the scalar offset; what a scalar offset
beyond the size reads is not described, so none may go out, also where the keys it would bring are hidden afterwards."""
import os
import re
import subprocess

import pytest

from paper_2510_21270_amd import build

# position of the scalar offset among the arguments
SCALAR_OFFSET = {"__builtin_amdgcn_raw_ptr_buffer_load_lds": 4, "__builtin_amdgcn_raw_buffer_load_b128": 2,
                 "__builtin_amdgcn_raw_buffer_load_b32": 2, "load_to_lds": 3}

# scalar offsets by which no load starts behind its descriptor, and why
WITHIN = {
    "attn_d64.hip": {
        "scalar_offset((slot0 + (c >> 1) * 16) * (D * 2), g.n * (D * 2))": "stops at the end",
        "from": "the same: load_kf forms it so",
        "slot0 * (D * 2) + c * 1024": "Vt holds whole blocks",
        "slot0 * (D * 2)": "Vt",
        "slot0 * 4": "the first slot of a pair comes from listed_slot: one of the n keys",
    },
    "attn_fp32.hip": {
        "at": "load_to_lds passes on what its callers give",
        "s0 * kKeyB": "s0 comes from listed_slot: one of the n keys",
        "s0 * 4": "the same",
        "values_at(s0) * kB": "Vt holds whole blocks",
    },
    "attn_fwd.hip": {
        "slot0 * 4": "slot0 stops at the n-th key",
        "scalar_offset(from, buf.n * 256)": "stops at the end",
        "scalar_offset(j * BLOCK + half * KT, buf.n) * 4": "the same",
        "from": "Vt holds whole blocks",
    },
    "attn_wide.hip": {
        "a.soff": "stage_load stops it at the end",
        "j * (BLOCK * 4)": "a block that is listed has at least one key",
        "k * 4": "a list's pieces of 64 entries, of which the first exists",
        "32 * k": "less than a row of Q'",
        "scalar_offset(nq * (BLOCK * 256) + k * 8192, a.g.n * 256)": "stops at the end",
    },
    "block_mask.hip": {},
    "key_scores.hip": {"soff": "issue_tile takes it from tile_offset, whose places the compiler goes through"},
}


def _arguments(text, at):
    """The arguments of the call whose opening bracket is text[at]."""
    depth, args, start = 0, [], at + 1
    for k in range(at, len(text)):
        if text[k] in "([{":
            depth += 1
        elif text[k] in ")]}":
            depth -= 1
            if depth == 0:
                return args + [text[start:k]]
        elif text[k] == "," and depth == 1:
            args.append(text[start:k])
            start = k + 1
    raise AssertionError("no closing bracket")


@pytest.mark.parametrize("name", sorted(WITHIN))
def test_no_load_starts_behind_its_descriptor(name):
    with open(os.path.join(build.CSRC, name)) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    found = 0
    for m in re.finditer(r"\b(%s)\(" % "|".join(SCALAR_OFFSET), text):
        if text[:m.start()].rstrip().endswith("void"):      # a definition
            continue
        offset = " ".join(_arguments(text, m.end() - 1)[SCALAR_OFFSET[m.group(1)]].split())
        found += 1
        assert offset == "0" or offset in WITHIN[name], (name, offset)
    assert found
    if name == "attn_wide.hip":
        assert re.search(r"a\.soff = scalar_offset\([^;]*, buf\.tile_bytes\);", text)
    if name == "key_scores.hip":
        assert "const int soff = tile_offset(t, wave, src.bytes);" in text
    if name == "attn_fwd.hip":
        assert set(re.findall(r"int slot0 = ([^;]*);", text)) == {"scalar_offset(j * BLOCK + half * KT, buf.n)"}
    if name == "attn_d64.hip":
        assert "const int from = scalar_offset(slot0 * (D * 2), g.n * (D * 2));" in text
    if name in ("attn_fp32.hip", "attn_d64.hip"):           # slots to load come from nowhere else
        slots = re.search(r"auto next_slot = .*?\n    };", text, re.S).group(0)
        assert set(re.findall(r"return ([^;]*);", slots)) == {"first", "-1"} and "first = listed_slot(" in slots


def test_listed_slots_are_keys_and_leave_none_out(tmp_path):
    code = """
#include <cstdio>
#include "load_places.h"
int main()
{
    for (int block = 16; block <= 128; block *= 2)
        for (int step = 16; step <= 64 && step <= block; step *= 2)
            for (int n = 1; n <= 3 * block + 1; ++n) {
                const int T = (n + block - 1) / block;
                for (int ni = 0; ni <= T; ++ni)
                    for (int j = -2; j <= T + 1; ++j) {
                        int keys = 0;
                        for (int part = 0; part < block / step; ++part) {
                            const int first = pbs::listed_slot(j, part, step, block, ni, n);
                            if (first == -1) continue;
                            if (first < 0 || first >= n || first != j * block + part * step) return 1;
                            keys += n - first < step ? n - first : step;
                        }
                        const int want = j < 0 || j >= ni ? 0 : n - j * block < block ? n - j * block : block;
                        if (keys != want) return 2;
                    }
            }
    for (int bytes = 0; bytes <= 4096; bytes += 128)
        for (int at = 0; at <= 8192; at += 128)
            if (pbs::scalar_offset(at, bytes) > bytes || (at <= bytes && pbs::scalar_offset(at, bytes) != at)) return 3;
    std::puts("all places hold");
}
"""
    src, exe = str(tmp_path / "places.cpp"), str(tmp_path / "places")
    with open(src, "w") as f:
        f.write(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", build.CSRC, src, "-o", exe], check=True)
    out = subprocess.run([exe], check=True, stdout=subprocess.PIPE, text=True).stdout
    assert "all places hold" in out
