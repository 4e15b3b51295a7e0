"""Register spills of the built kernels, from the metadata in the library: the
row loop of the fused binning once kept 340 scalar registers in vector lanes
and moved them back one by one in every step."""
import os
import re
import struct
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def spills(lib: str, tmp: str) -> dict:
    """{kernel name: (scalar, vector) registers spilled}"""
    data, out, at = open(lib, "rb").read(), {}, 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                obj = os.path.join(tmp, "code.o")
                with open(obj, "wb") as f:
                    f.write(data[at + off:at + off + size])
                text = subprocess.run([READELF, "--notes", obj], capture_output=True, text=True, check=True).stdout
                for k in re.split(r"\n\s+- \.agpr_count", text)[1:]:
                    get = lambda key: re.search(rf"\.{key}:\s+(\S+)", k).group(1)  # noqa: E731
                    out[get("name")] = (int(get("sgpr_spill_count")), int(get("vgpr_spill_count")))
        at += len(magic)
    return out


def test_feature_kernels_keep_their_scalars(tmp_path):
    found = spills(os.path.join(ROOT, "paper_2609_35587_amd", "libhwsel.so"), str(tmp_path))
    features = {n: v for n, v in found.items() if "k_features" in n}
    assert len(features) >= 12, sorted(found)
    assert all(scalar == 0 and vector <= 16 for scalar, vector in features.values()), features
