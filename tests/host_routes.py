"""Drives tests/host_abi/route_driver.cpp: the launches that the built library
makes for a plan, seen without a GPU."""

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2602_06688_amd")
BUILD = os.path.join(HERE, "host_abi", "_build")


def build():
    """The driver's path, or None without hipcc or the library."""
    cc = next((c for c in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)
    lib = os.path.join(PKG, "libpwfs.so")
    if not cc or not os.path.exists(lib):
        return None
    os.makedirs(BUILD, exist_ok=True)
    exe = os.path.join(BUILD, "route_driver")
    subprocess.run([cc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-w", "-rdynamic",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    os.path.join(HERE, "host_abi", "route_driver.cpp"), "-x", "none", lib,
                    "-Wl,-rpath," + PKG, "-o", exe], check=True)
    return exe


class Host:
    """One plan at a time; ``forward`` returns (status, launches), a launch as
    (kernel, workgroups, parts or None, bytes past the scratch or None)."""

    def __init__(self, exe):
        self.p = subprocess.Popen([exe], stdin=subprocess.PIPE, stdout=subprocess.PIPE, text=True)

    def _ask(self, line):
        self.p.stdin.write(line + "\n")
        self.p.stdin.flush()
        out = self.p.stdout.readline()
        assert out, "the driver ended"
        return out.split()

    def plan(self, sensors, frames):
        """(status, largest chunk accepted, chunk)"""
        from paper_2602_06688_amd import pwfs as P
        descs = " ".join(bytes(P.to_c(s)).hex() for s in sensors)
        return tuple(int(v) for v in self._ask(f"plan {frames} {len(sensors)} {descs}"))

    def tune(self, mode, chunk, row_groups=2048):
        return tuple(int(v) for v in self._ask(f"tune {mode} {chunk} {row_groups}"))

    def forward(self, frames):
        rc, *ls = self._ask(f"fwd {frames}")
        assert not any("!" in s for s in ls), ls
        out = []
        for s in ls:
            f = s.split(":")
            out.append((f[0], int(f[1]), *(int(v) for v in f[2:4])) if len(f) > 2 else (f[0], int(f[1]), None, None))
        return int(rc), out

    def scratch(self, sensor, delta=0):
        """Recorded bytes of a sensor's scratch, after a change of the record."""
        return int(self._ask(f"scratch {sensor} {delta}")[0])

    def points(self):
        """Points and x-tilts of the plan's sensors, counted and listed."""
        return [int(v) for v in self._ask("points")]

    def free(self):
        self._ask("free")

    def close(self):
        self.p.stdin.close()
        self.p.wait(timeout=60)
