"""Runs library calls on the host against tests/fake_hip.cpp and returns what they launched."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

HEAD = """
import ctypes, json, os, sys
sys.modules["torch"] = None        # the library must meet this runtime first
ctypes.CDLL(os.environ["FAKE_HIP_LIB"], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, os.environ["FAKE_HIP_ROOT"])
import numpy as np
from paper_1611_06797_amd import ltmp2 as L
"""


def build(directory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    lib = os.path.join(str(directory), "libfakehip.so")
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-o", lib,
                    os.path.join(HERE, "fake_hip.cpp")], check=True, capture_output=True)
    return lib


def run(lib, directory, code, timeout=100, **env):
    """Log lines (split) of a program that uses L (the bindings), and what it printed as JSON."""
    log = os.path.join(str(directory), "fake_hip.log")
    if os.path.exists(log):
        os.remove(log)
    r = subprocess.run([sys.executable, "-c", HEAD + code], capture_output=True, text=True,
                       timeout=timeout, env=dict(os.environ, FAKE_HIP_LIB=lib, FAKE_HIP_LOG=log,
                                                 FAKE_HIP_ROOT=ROOT, **env))
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [x.split() for x in open(log)] if os.path.exists(log) else []
    return lines, [json.loads(x) for x in r.stdout.splitlines() if x.startswith(("{", "["))]
