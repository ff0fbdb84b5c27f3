"""What the built kernels take of a CU, from the metadata of the library's own code
objects: the pair of kernels that an eager call of long chains runs side by side
(CTR of 64-lane items, verification of 64-lane segments) fits one CU together."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(so, tmp):
    """{mangled name: {vgprs, spills, lds, threads}} of every kernel in the library's bundles."""
    data, out, at = open(so, "rb").read(), {}, 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (n,), o = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, o)
            target = data[o + 24:o + 24 + tl]
            o += 24 + tl
            if b"gfx950" not in target or not size:
                continue
            elf = os.path.join(tmp, "code_object")
            with open(elf, "wb") as f:
                f.write(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", elf], stdout=subprocess.PIPE, text=True, check=True).stdout
            for k in notes.split("- .agpr_count")[1:]:
                field = lambda name: re.search(r"\.%s:\s+(\S+)" % name, k).group(1)
                out[field("name")] = dict(vgprs=int(field("vgpr_count")), spills=int(field("vgpr_spill_count")),
                                          lds=int(field("group_segment_fixed_size")),
                                          threads=int(field("max_flat_workgroup_size")))
        at += 1
    return out


def test_the_eager_pair_shares_a_cu(tmp_path):
    import paper_2410_15240_amd as F
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    if not os.path.exists(F.library_path()):
        from paper_2410_15240_amd import build
        build.build()
    ks = kernels(F.library_path(), str(tmp_path))

    def gcm(lanes, split, mode):   # gcm_kernel<ENC = false, LL, SPLIT, MODE, RAG = false>
        (k,) = [v for n, v in ks.items() if "gcm_kernelILb0ELi%dELb%dELi%dELb0E" % (lanes, split, mode) in n]
        return k

    ctr, verify = gcm(6, 0, 1), gcm(6, 1, 2)
    assert ctr["lds"] + verify["lds"] <= 160 * 1024
    assert ctr["threads"] + verify["threads"] <= 2048
    # Four waves of each on a SIMD, registers given out in eights of its 512 a lane.
    assert 4 * sum(-(-k["vgprs"] // 8) * 8 for k in (ctr, verify)) <= 512
    streaming = [v for n, v in ks.items() if "gcm_kernel" in n]
    assert len(streaming) == 42
    assert all(k["spills"] == 0 and k["vgprs"] <= 128 for k in streaming)   # 16 waves per CU
