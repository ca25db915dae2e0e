"""Private memory of the built kernels, from the metadata of the library's own
code objects: the kernels of the call that allocates no device memory must not
need any, since the runtime would have to find it at the launch."""
import os
import re
import struct
import subprocess

import pytest

import paper_1811_11007_amd as pt

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(tmp_path):
    """(name, bytes of private memory per lane) of every kernel in libpt.so."""
    path = os.path.join(os.path.dirname(pt.__file__), "libpt.so")
    data = open(path, "rb").read()
    at = [m.start() for m in re.finditer(b"\x7fELF", data)
          if struct.unpack_from("<H", data, m.start() + 18)[0] == 224]  # e_machine: AMD GPU
    assert at, "no code objects in the library"
    out = []
    for i, o in enumerate(at):
        f = tmp_path / "code_object"
        f.write_bytes(data[o:at[i + 1] if i + 1 < len(at) else len(data)])
        notes = subprocess.run([READELF, "--notes", str(f)], stdout=subprocess.PIPE, text=True).stdout
        for k in notes.split(".agpr_count:")[1:]:
            out.append((re.search(r"\.name:\s+(\S+)", k).group(1),
                        int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1))))
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_likelihood_kernels_need_no_private_memory(tmp_path):
    pt.lib()
    found = [k for k in kernels(tmp_path) if re.search("k_prune|k_pmat_lanes|k_tile_sums", k[0])]
    assert len(found) >= 27, found
    assert not [k for k in found if k[1]], [k for k in found if k[1]]
