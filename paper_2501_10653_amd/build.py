"""Build step for the HIP library (``libiqa_hip.so``, gfx950 only).

Run as ``python -m paper_2501_10653_amd.build``; ``__graft_entry__.build()``
calls :func:`build` too.  The library is built in-tree, next to this file.
"""

from __future__ import annotations

import os
import shutil
import subprocess
import sys
import time

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
# Each source is compiled on its own, with its own extra flags, then linked.
# The measurement probes are built with kernel-argument preloading: their
# scalar-argument kernels start with the arguments in SGPRs.
SOURCES = {
    os.path.join(PKG, "csrc", "iqa_kernels.hip"): [],
    os.path.join(PKG, "csrc", "iqa_server.hip"): [],
    os.path.join(PKG, "csrc", "iqa_probe.hip"): ["-mllvm", "-amdgpu-kernarg-preload-count=16"],
}
OBJDIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libiqa_hip.so")

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

# -ffp-contract=off: every multiply-add the kernels want is an explicit fmaf,
#   so compensated sums and the double-float finalisation round as written.
# -packed-fp32-ops off: no v_pk_* FP32 instructions are generated.
HIPFLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-pthread",
    "-I", os.path.join(ROOT, "include"),
]


TUNED_JSON = os.path.join(PKG, "tuned", "gfx950.json")
TUNED_INC = os.path.join(PKG, "csrc", "tuned_table.inc")


def _check_batch_geometry(key: str, cfg: dict) -> None:
    """Batch and server entries must be geometries the batch kernel runs:
    vec 4, ksplit 1, unroll 8, waves 1 or 4 (the library also skips any
    other at lookup)."""
    if not (cfg.get("vec") == 4 and cfg.get("ksplit") == 1 and cfg.get("unroll") == 8
            and cfg.get("waves") in (1, 4)):
        raise ValueError(f"tuned batch/serve entry {key}: {cfg} is not a batch geometry")


def write_tuned_table(json_path: str = TUNED_JSON, inc_path: str = TUNED_INC) -> int:
    """Turn the autotuner's JSON cache into the C table the library compiles
    in (single-pair shapes per (N, NT), batch geometry per NT, the server's
    geometry per (N, NT)).  Returns the
    number of entries; writes an empty table when there is no cache."""
    import json
    entries = []
    waves = 0
    if os.path.exists(json_path):
        with open(json_path) as fh:
            doc = json.load(fh)
        for key, rec in sorted(doc.get("single", {}).items()):
            N, NT = (int(v) for v in key.split("x"))
            entries.append((N, NT, 0, rec["cfg"]))
        for key, cfg in sorted(doc.get("batch", {}).items()):
            _check_batch_geometry(key, cfg)
            entries.append((0, int(key), 1, cfg))
        for key, cfg in sorted(doc.get("serve", {}).items()):
            _check_batch_geometry(key, cfg)
            N, NT = (int(v) for v in key.split("x"))
            entries.append((N, NT, 2, cfg))
        waves = int(doc.get("batch_waves", 0))
    fields = ("vec", "waves", "unroll", "seg", "rp", "ksplit")
    lines = ["// Generated by paper_2501_10653_amd/build.py from tuned/gfx950.json: launch",
             "// shapes by measurement on gfx950, the autotuner's and those of its `chosen`",
             "// section.  Do not edit.",
             "static const TunedEntry kTuned[] = {"]
    for N, NT, kind, cfg in entries:
        vals = ", ".join(str(int(cfg[f])) for f in fields)
        lines.append(f"    {{{N}, {NT}, {kind}, {{{vals}}}}},")
    if not entries:
        lines.append("    {-1, -1, -1, {0, 0, 0, 0, 0, 0}},")
    lines.append("};")
    lines.append(f"static const int kTunedCount = {len(entries)};")
    lines.append(f"static const int64_t kTunedBatchWaves = {waves};")
    text = "\n".join(lines) + "\n"
    if not os.path.exists(inc_path) or open(inc_path).read() != text:
        with open(inc_path, "w") as fh:
            fh.write(text)
    return len(entries)


def _hipcc(cmd: list) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 target feature: harmless
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{' '.join(cmd)}\n{err}")
    return err


def build(verbose: bool = False) -> str:
    """Compile every HIP source and link ``libiqa_hip.so`` (always recompiles)."""
    write_tuned_table()
    os.makedirs(OBJDIR, exist_ok=True)
    t0 = time.time()
    objs, msgs = [], []
    for src, extra in SOURCES.items():
        obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
        msgs.append(_hipcc([HIPCC, *HIPFLAGS, *extra, "-c", src, "-o", obj]))
        objs.append(obj)
    tmp = LIB + ".tmp"
    msgs.append(_hipcc([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", *objs,
                        "-o", tmp]))
    err = "\n".join(m for m in msgs if m.strip())
    if verbose and err.strip():
        print(err, file=sys.stderr)
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} in {time.time() - t0:.1f}s", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
