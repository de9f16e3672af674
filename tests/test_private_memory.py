"""The kernels ifcm_solve_noalloc launches need no private memory (spilled
registers), which the runtime would have to allocate: read from the metadata of
the built library's code objects."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2002_01981_amd", "libpifcm.so")
BIN = "/opt/rocm/llvm/bin"

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(os.path.join(BIN, "llvm-readelf")),
                                reason="needs the built library and the LLVM tools")


@pytest.fixture(scope="module")
def private_bytes(tmp_path_factory):
    """{mangled kernel name: bytes of private memory per lane}"""
    d = tmp_path_factory.mktemp("objects")
    fat = d / "fatbin"
    subprocess.run([os.path.join(BIN, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", LIB, os.devnull], check=True)
    data, magic, out = fat.read_bytes(), b"__CLANG_OFFLOAD_BUNDLE__", {}
    for k, at in enumerate(m.start() for m in re.finditer(magic, data)):
        n, pos = struct.unpack_from("<Q", data, at + len(magic))[0], at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if not target.startswith(b"hip") or not size:
                continue
            obj = d / f"{k}.elf"
            obj.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([os.path.join(BIN, "llvm-readelf"), "--notes", str(obj)], check=True,
                                   capture_output=True, text=True).stdout
            for kernel in re.split(r"\n  - \.", notes)[1:]:
                name = re.search(r"\.name:\s*(\S+)", kernel)
                private = re.search(r"\.private_segment_fixed_size:\s*(\d+)", kernel)
                if name and private:
                    out[name.group(1)] = int(private.group(1))
    return out


def _args(mangled, kernel):
    """Template arguments of an instance of `kernel`, or None."""
    m = re.match(r"_ZN5pifcm%d%sI((?:L[ib]\d+E)+)E" % (len(kernel), kernel), mangled)
    return [int(v) for v in re.findall(r"L[ib](\d+)E", m.group(1))] if m else None


def test_no_kernel_of_the_scratch_solve_spills(private_bytes):
    plain = ["k_invariants", "k_check_finite", "k_check_rows", "k_init_u", "k_labels", "k_fcm_x", "k_fcm_last", "k_finalize"]
    seen = set()
    for name, private in private_bytes.items():
        for k in plain:
            if re.match(r"_ZN5pifcm%d%s(?=[IE])" % (len(k), k), name):
                seen.add(k)
                assert private == 0, name
    assert seen == set(plain)
    # One particle per item, one run per tile; where there is an instance that
    # never spills, that one.  Steps with and without J, and the objective.
    step = {}
    for name, private in private_bytes.items():
        a = _args(name, "k_ifcm_gather")
        if a and a[4] == 1 and a[5] == 0:
            C, m2, nw, is_step, _, _, wj = a[:7]
            step.setdefault((C, m2, nw, is_step, wj), {})[a[7] if len(a) > 7 else 0] = private
    assert {k[0] for k in step} == set(range(2, 17)) and len({k for k in step if k[2] == 4}) == 15 * 2 * 3
    for key, by_lean in step.items():
        assert by_lean[max(by_lean)] == 0, key
