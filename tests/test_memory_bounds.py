"""Which memory the kernels touch, checked on the CPU: their sources are built for the host (tests/host_build) and run with every
operand, index list and workspace between two pages that nobody may touch, index lists exactly as long as their count."""
import ctypes as C
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import test_gpu_first
import test_gpu_group_se
import test_gpu_narrow
import test_gpu_pooled_lists
from paper_2308_15949_amd import binding as B
from paper_2308_15949_amd import build as build_rules

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_build")
CXX = "/opt/rocm/llvm/bin/clang++"


def host_source(name, s):
    """A kernel source with dynamic LDS as pointers, generic pointers only, and its inline assembly replaced or dropped."""
    s = re.sub(r"extern __shared__ (?:__align__\(16\) )?unsigned char (\w+)\[\];", r"unsigned char* const \1 = host::lds;", s)
    s = re.sub(r"extern __shared__ (?:__align__\(16\) )?float (\w+)\[\];", r"float* const \1 = (float*)host::lds;", s)
    s = re.sub(r"const __attribute__\(\(address_space\(\d\)\)\) ", "const ", s)
    s = s.replace("#if defined(__HIP_DEVICE_COMPILE__)", "#if 1")
    s = s.replace('asm volatile("s_waitcnt lgkmcnt(0)\\n\\ts_barrier" ::: "memory");', "host::barrier();")
    s = s.replace('asm volatile("s_barrier" ::: "memory");', "host::barrier();")
    if name == "laud_common.h":  # there is no kernel argument segment
        at = s.index("prefetch_args() {") + len("prefetch_args() {")
        s = s[:at] + s[s.index("\n}\n", at):]
    if name == "laud_tile_util.h":
        s = re.sub(r'asm volatile\("s_mov_b32 m0.*?;\n', "host::load_to_lds(rsrc, voff, soff, lds_base);\n", s, flags=re.S, count=1)
        s = re.sub(r'asm volatile\("s_mov_b32 m0.*?;\n', "host::load_dword_to_lds(rsrc, voff, soff, lds_base);\n", s, flags=re.S, count=1)
        s = re.sub(r"const f32x2 v = \{lo, hi\};\s*return [^;]*;", "return (unsigned)f32_to_bf16(lo) | ((unsigned)f32_to_bf16(hi) << 16);", s)
    return re.sub(r"\basm(?: volatile)?\s*\((?:[^()]|\((?:[^()]|\([^()]*\))*\))*\);", ";", s)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("host_build"))
    for name in os.listdir(build_rules.CSRC):
        if name.endswith((".h", ".hip")):
            with open(os.path.join(build_rules.CSRC, name)) as f:
                text = host_source(name, f.read())
            with open(os.path.join(d, name.replace(".hip", ".cpp")), "w") as f:
                f.write(text)
    flags = ["-O1", "-std=c++17", "-fPIC", "-w", "-fno-strict-aliasing", "-I", HERE, "-I", d, "-I", os.path.join(build_rules.ROOT, "include")]
    sources = [os.path.join(d, s.replace(".hip", ".cpp")) for s in build_rules.SOURCES if s != "laud_probe.hip"]
    sources.append(os.path.join(HERE, "host_run.cpp"))
    objects = [os.path.join(d, os.path.basename(s) + ".o") for s in sources]
    with ThreadPoolExecutor(8) as ex:
        list(ex.map(lambda so: subprocess.run([CXX, *flags, "-c", so[0], "-o", so[1]], check=True, capture_output=True), zip(sources, objects)))
    subprocess.run([CXX, "-shared", "-fPIC", *objects, "-o", os.path.join(d, "host.so")], check=True)
    return os.path.join(d, "host.so")


class Call:
    """Operands of one call and the call itself; runs in a process of its own."""

    def __init__(self, path, front):
        B.LIB_PATH, B._lib, B._stream = path, None, lambda: 0
        self.host = B.load()
        self.host.host_alloc.restype, self.host.host_alloc.argtypes = C.c_void_p, [C.c_size_t, C.c_int]
        self.host.host_init()
        self.front, self.rng, self.held = front, np.random.default_rng(1), []

    def buf(self, nbytes, data=None):
        p = self.host.host_alloc(max(int(nbytes), 4), self.front)
        if data is not None:
            C.memmove(p, data.ctypes.data, data.nbytes)
        return p

    def values(self, n, bf16):
        a = np.maximum(self.rng.standard_normal(n, dtype=np.float32), 0)
        a = (a.view(np.uint32) >> 16).astype(np.uint16) if bf16 else a
        return self.buf(a.nbytes, a)

    def ws(self, nbytes):
        w = self.buf(nbytes)
        C.memset(w, 0x7b, int(nbytes))

        class Workspace:
            data_ptr, numel, element_size = (lambda s: w), (lambda s: int(nbytes)), (lambda s: 1)
        return Workspace()

    def block(self, ci, m, co, gw, bf16, packed):
        t = [self.values(n, bf16) for n in (m * ci, m * 9 * (gw or m), co * m)] + [self.values(n, False) for n in (m, m, m, m, co, co)]
        p = B.Bottleneck(ci, m, co, *t, 1)
        nb = B.packed_weights_size(p, B.BF16 if bf16 else B.F32) if packed else 0
        if nb:
            p.packed = self.buf(nb)
            B.laud_pack_weights(p, B.BF16, p.packed)
        return p

    def launched(self):
        text = C.create_string_buffer(1 << 16)
        self.host.host_launched.restype, self.host.host_launched.argtypes = C.c_size_t, [C.c_char_p, C.c_size_t]
        assert self.host.host_launched(text, len(text)) < len(text)
        return text.value.decode()

    def list(self, patches, ratio):
        ids = np.flatnonzero(self.rng.random(patches) < ratio).astype(np.int32)
        return self.buf(ids.nbytes, ids), self.buf(4, np.array([len(ids)], np.int32))

    def se(self, m, gw, width):
        return B.GroupSE(gw, width, *([self.values(n, False) for n in (width * m, width, m * width, m)] if width else [None] * 4))

    def identity(self, kind, n, h, w, c, m, S, ratio, bf16=True, inplace=True, gw=None, se=0, packed=False, keep=False, D=0):
        fx, x, p = B.Fmap(n, h, w, c, B.BF16 if bf16 else B.F32), self.values(n * h * w * c, bf16), self.block(c, m, c, gw, bf16, packed)
        out, patches = x if inplace else self.buf(n * h * w * c * (2 if bf16 else 4)), n * (h // S) * (w // S)
        ws = self.ws(B.workspace_size(B.OP_CHANNEL_SKIP if kind == "channel" else B.OP_DYN_BOTTLENECK, fx, p, S))
        if kind == "channel":
            mask = (self.rng.random(n * D) < 0.5).astype(np.uint8)
            mask[:D], mask[-D:] = 1, 0
            B.laud_channel_skip_conv(x, fx, p, self.buf(n * D, mask), D, out, ws)
        elif kind == "masker":
            gate = self.buf(n, (self.rng.random(n) < 0.6).astype(np.uint8)) if keep else None
            w1 = self.rng.standard_normal(c, dtype=np.float32)
            B.laud_masker_dyn_bottleneck(x, fx, p, S, self.buf(w1.nbytes, w1), 0.01, gate, self.buf(patches), self.buf(4 * patches),
                                         self.buf(4), None, None if keep else self.buf(4 * patches), out, ws)
        elif gw:
            B.laud_dyn_group_se_bottleneck(x, fx, p, self.se(m, gw, se), S, *self.list(patches, ratio), out, ws)
        else:
            B.laud_dyn_bottleneck(x, fx, p, S, *self.list(patches, ratio), out, ws)

    def first(self, kind, n, hi, wi, ci, m, co, stride, S, ratio, bf16=True, gw=None, se=0, packed=False):
        h, w = (hi - 1) // stride + 1, (wi - 1) // stride + 1
        fx, x, p = B.Fmap(n, hi, wi, ci, B.BF16 if bf16 else B.F32), self.values(n * hi * wi * ci, bf16), self.block(ci, m, co, gw, bf16, packed)
        sc = self.values(co * ci, bf16), self.values(co, False), self.values(co, False)
        out = self.buf(n * h * w * co * (2 if bf16 else 4))
        if kind == "static":
            B.laud_static_bottleneck(x, fx, p, *sc, stride, out, self.ws(B.static_bottleneck_workspace(fx, p, stride)))
            return
        ws, ids = self.ws(B.dyn_projection_workspace(fx, p, stride)), self.list(n * (h // S) * (w // S), ratio)
        if gw:
            B.laud_dyn_group_se_projection_bottleneck(x, fx, p, self.se(m, gw, se), *sc, stride, S, *ids, out, ws)
        else:
            B.laud_dyn_projection_bottleneck(x, fx, p, *sc, stride, S, *ids, out, ws)

    def channel_wide(self, c_mid, G, bf16):
        """Channel skipping with more than 2 GiB of w2 (untouched pages, zero): one pixel that keeps the last group only."""
        c, D, eb = 8, c_mid // G, 2 if bf16 else 4
        fx, x = B.Fmap(1, 1, 1, c, B.BF16 if bf16 else B.F32), self.values(c, bf16)
        t = [self.values(c_mid * c, bf16), self.buf(9 * c_mid * c_mid * eb), self.values(c * c_mid, bf16)]
        assert 9 * c_mid * c_mid * eb > 1 << 31
        p = B.Bottleneck(c, c_mid, c, *t, *[self.values(n, False) for n in (c_mid, c_mid, c_mid, c_mid, c, c)], 1)
        mask = np.zeros(D, np.uint8)
        mask[-1] = 1
        B.laud_channel_skip_conv(x, fx, p, self.buf(D, mask), D, self.buf(c * eb), self.ws(B.workspace_size(B.OP_CHANNEL_SKIP, fx, p, D)))

    def masks(self, n, h, w, c, S, bf16=True, keep=False, D=4, m=16):
        """Spatial masker, compaction of its mask, gather with and without a halo, the unfused block, channel masker."""
        fx, x, patches = B.Fmap(n, h, w, c, B.BF16 if bf16 else B.F32), self.values(n * h * w * c, bf16), n * (h // S) * (w // S)
        w1 = self.rng.standard_normal(c, dtype=np.float32)
        gate = self.buf(n, (self.rng.random(n) < 0.6).astype(np.uint8)) if keep else None
        mask, idx, count = self.buf(patches), self.buf(4 * patches), self.buf(4)
        B.laud_mask_gen(x, fx, S, self.buf(w1.nbytes, w1), 0.01, gate, mask, idx, count, self.buf(4 * (n + 1)), self.buf(4 * patches),
                        self.ws(B.workspace_size(B.OP_MASK_GEN, fx, None, S)))
        B.laud_layer_skip_compact(mask, patches, self.buf(4 * patches), self.buf(4), self.ws(B.workspace_size(B.OP_COMPACT, fx, None, patches)))
        idx, count = self.list(patches, 0.4)
        for halo in (0, 1):
            B.laud_gather_patches(x, fx, S, halo, idx, count, self.buf(patches * (S + 2 * halo) ** 2 * c * (2 if bf16 else 4)))
        p = self.block(c, m, c, None, bf16, False)
        B.laud_dyn_bottleneck_unfused(x, fx, p, S, idx, count, self.buf(n * h * w * c * (2 if bf16 else 4)), self.ws(B.dyn_bottleneck_unfused_workspace(fx, p, S)))
        hidden = 16
        mlp = [self.values(k, False) for k in (hidden * c, hidden, 2 * D * hidden, 2 * D)]
        B.laud_channel_masker(x, fx, mlp[0], mlp[1], hidden, mlp[2], mlp[3], D, self.buf(n * D), self.buf(8 * n * D), self.ws(B.channel_masker_workspace(fx)))

    def stem(self, n, h, w, co, bf16=True, k=7):
        down = lambda v: (v - 1) // 2 + 1  # noqa: E731
        x, wt, s, t = self.values(n * h * w * 3, bf16), self.values(co * 3 * k * k, bf16), self.values(co, False), self.values(co, False)
        code, eb = (B.BF16, 2) if bf16 else (B.F32, 4)
        if k == 7:
            B.laud_stem(x, n, h, w, code, wt, s, t, co, self.buf(n * down(down(h)) * down(down(w)) * co * eb), self.ws(B.stem_workspace(n, h, w, co, code)))
        else:
            B.laud_stem3x3(x, n, h, w, code, wt, s, t, co, self.buf(n * down(h) * down(w) * co * eb))


CASES = {
    # small tiles; tiled kernels; index lists of one entry and of all
    "few_rows": ("identity", "dyn", 1, 7, 7, 136, 72, 1, 0.5),
    "few_rows_f32": ("identity", "dyn", 2, 5, 17, 24, 16, 1, 0.9, False, False),
    "tiled_128x64": ("identity", "dyn", 21, 28, 28, 72, 40, 4, 0.5, True, False),
    "tiled_64x128_split": ("identity", "dyn", 9, 28, 28, 200, 136, 7, 0.5, True, False),
    "tiled_128x128": ("identity", "dyn", 26, 28, 28, 80, 136, 4, 0.6, True, False),
    "tiled_128x128_f32": ("identity", "dyn", 26, 28, 28, 80, 136, 4, 0.6, False, False),
    "tiled_64x128_f32": ("identity", "dyn", 10, 28, 28, 264, 264, 4, 0.3, False),
    "tiled_64x64_f32": ("identity", "dyn", 42, 28, 28, 72, 40, 4, 0.3, False),
    "dense_first_split": ("identity", "dyn", 100, 7, 7, 520, 136, 1, 0.3, True, False),
    "last_128x64": ("identity", "dyn", 27, 28, 28, 136, 128, 4, 0.5),
    "last_f32": ("identity", "dyn", 12, 28, 28, 264, 64, 4, 0.5, False),
    "last_split": ("identity", "dyn", 100, 7, 7, 136, 520, 1, 0.3),
    "last_128x128": ("identity", "dyn", 32, 28, 28, 136, 328, 4, 0.3),
    "last_128x256": ("identity", "dyn", 16, 28, 28, 1032, 456, 4, 0.2),
    "tiled": ("identity", "dyn", 9, 28, 28, 64, 40, 7, 0.5, True, False),
    "tiled_f32": ("identity", "dyn", 20, 28, 28, 24, 40, 4, 0.3, False),
    "empty_list": ("identity", "dyn", 3, 14, 14, 64, 24, 2, 0.0, True, False),
    # 64-wide kernel, fused 3x3 -> 1x1 and register-weight first 1x1
    "narrow": ("identity", "dyn", 5, 56, 56, 256, 64, 4, 0.3, True, False),
    "narrow_static": ("first", "static", 1, 241, 239, 64, 64, 256, 2, 1, 1.0),
    "one_kernel_first": ("first", "static", 2, 27, 41, 64, 64, 256, 1, 1, 1.0),
    "one_kernel_first_one_row": ("first", "static", 1, 1, 1100, 64, 64, 256, 1, 1, 1.0),
    "one_kernel_first_walk": ("first", "static", 768, 4, 4, 64, 64, 256, 1, 1, 1.0),  # three rectangles a workgroup
    "narrow_projection": ("first", "dynamic", 5, 111, 112, 64, 64, 256, 2, 8, 0.4),
    "fused": ("identity", "dyn", 22, 14, 14, 1024, 256, 2, 0.3, True, False),
    "fused_packed": ("identity", "masker", 22, 14, 14, 1024, 256, 2, 0.5, True, True, None, 0, True, True),
    "projection_before_fused": ("first", "dynamic", 22, 14, 14, 320, 256, 1024, 1, 2, 0.5),
    # patches that are whole samples
    "samples_fused": ("identity", "dyn", 22, 14, 14, 1024, 256, 14, 0.3, True, False),
    "samples_fused_none": ("identity", "dyn", 22, 14, 14, 1024, 256, 14, 0.0, True, False),
    "samples_tiled": ("identity", "dyn", 26, 28, 28, 80, 136, 28, 0.1, True, False),
    "samples_first_split": ("identity", "dyn", 100, 7, 7, 520, 136, 7, 0.3, True, False),
    "samples_tiled_f32": ("identity", "dyn", 22, 28, 28, 24, 40, 28, 0.3, False),
    "samples_projection_f32": ("first", "dynamic", 22, 28, 27, 24, 16, 40, 2, 14, 0.4, False),
    # fused masker
    "masker": ("identity", "masker", 3, 12, 12, 72, 24, 4, 0.5),
    "masker_f32_gates": ("identity", "masker", 26, 14, 14, 32, 8, 1, 0.5, False, False, None, 0, False, True),
    "masker_128x64": ("identity", "masker", 40, 21, 21, 104, 72, 3, 0.5, True, False),
    "masker_128x128_f32": ("identity", "masker", 11, 28, 28, 24, 136, 4, 0.5, False),
    "masker_64x128_f32": ("identity", "masker", 6, 28, 28, 24, 200, 4, 0.5, False),
    "masker_64x64_f32": ("identity", "masker", 21, 28, 28, 24, 40, 4, 0.5, False),
    "masker_widest": ("identity", "masker", 3, 30, 30, 4096, 264, 2, 0.5),
    "masker_four_patches_a_thread": ("identity", "masker", 13, 32, 32, 16, 8, 4, 0.5, True, False, None, 0, False, True),
    "masker_two_blocks_of_patches": ("identity", "masker", 9, 24, 24, 16, 8, 2, 0.5),
    # first blocks
    "static": ("first", "static", 2, 13, 9, 40, 24, 96, 2, 1, 1.0),
    "static_shortcut_128x256": ("first", "static", 32, 28, 28, 8, 64, 264, 1, 1, 1.0),
    "static_3x3_split": ("first", "static", 9, 57, 55, 72, 136, 96, 2, 1, 1.0),
    "static_3x3_128x128": ("first", "static", 9, 129, 127, 16, 72, 80, 1, 1, 1.0),
    "static_3x3_256x128": ("first", "static", 9, 121, 123, 16, 72, 80, 2, 1, 1.0),
    "static_last_split": ("first", "static", 6, 28, 28, 16, 456, 136, 1, 1, 1.0),
    "static_last_128x128": ("first", "static", 16, 28, 28, 16, 328, 136, 1, 1, 1.0),
    "static_last_128x256": ("first", "static", 8, 28, 28, 16, 456, 1032, 1, 1, 1.0),
    "static_64x64_f32": ("first", "static", 42, 56, 56, 24, 40, 72, 2, 1, 1.0, False),
    "static_64x128_f32": ("first", "static", 10, 56, 56, 24, 264, 264, 2, 1, 1.0, False),
    "static_128x128_f32": ("first", "static", 14, 56, 56, 24, 136, 136, 2, 1, 1.0, False),
    "projection_f32": ("first", "dynamic", 3, 27, 14, 8, 16, 40, 2, 7, 0.4, False),
    # group convolution and SE, in one launch and in four
    "group_se": ("identity", "dyn", 3, 14, 14, 144, 144, 2, 0.5, True, True, 16, 36),
    "group_se_four_launches": ("identity", "dyn", 3, 6, 6, 392, 392, 2, 0.7, True, True, 8, 90),
    "group_se_projection": ("first", "dynamic", 2, 27, 28, 32, 104, 104, 2, 7, 0.5, True, 8, 26),
    "group_many_rows": ("identity", "dyn", 12, 28, 28, 144, 144, 2, 0.5, True, False, 16, 36),
    "group_many_rows_none": ("identity", "dyn", 12, 28, 28, 144, 144, 2, 0.0, True, True, 16, 36),
    "group_of_64": ("identity", "dyn", 5, 56, 56, 64, 64, 4, 0.5, True, True, 64),
    "group_of_8_odd": ("identity", "dyn", 9, 41, 37, 48, 48, 1, 0.5, True, True, 8),
    "group_many_rows_projection": ("first", "dynamic", 9, 55, 56, 32, 104, 104, 2, 7, 0.5, True, 8, 26),
    "group_fused": ("identity", "dyn", 3, 28, 28, 72, 72, 4, 0.6, True, False, 8, 20),
    "group_fused_strips": ("identity", "dyn", 3, 28, 42, 136, 136, 14, 0.6, True, True, 8, 20),
    "group_fused_walk": ("identity", "dyn", 57, 24, 24, 40, 40, 4, 1.0, True, True, 8),  # two tiles a workgroup
    "group_fused_none": ("identity", "dyn", 3, 28, 28, 72, 72, 4, 0.0, True, False, 8, 20),
    "group_fused_projection": ("first", "dynamic", 4, 27, 28, 104, 208, 208, 2, 2, 0.5, True, 16, 26),
    "group_fused_projection_strips": ("first", "dynamic", 2, 55, 56, 40, 104, 104, 2, 28, 0.9, True, 8),
    "group_fused_projection_walk": ("first", "dynamic", 12, 62, 61, 32, 24, 24, 2, 1, 0.9, True, 8),
    "group_many_rows_f32": ("identity", "dyn", 12, 28, 28, 136, 136, 4, 0.5, False, True, 8),
    "group_past_4096_channels": ("identity", "dyn", 3, 8, 8, 4104, 4104, 2, 0.5, True, True, 8),
    # channel skipping: groups of whole 16-byte chunks, the fused kernels, and groups that are not
    "channel": ("identity", "channel", 5, 7, 6, 64, 64, 1, 0, True, False, None, 0, False, False, 4),
    "channel_split": ("identity", "channel", 5, 7, 11, 1032, 136, 1, 0, True, False, None, 0, False, False, 17),
    "channel_128x64": ("identity", "channel", 5, 14, 14, 64, 64, 1, 0, True, False, None, 0, False, False, 4),
    "channel_64x64_f32": ("identity", "channel", 5, 9, 14, 64, 64, 1, 0, False, False, None, 0, False, False, 16),
    "channel_64x128_f32": ("identity", "channel", 5, 9, 14, 136, 136, 1, 0, False, False, None, 0, False, False, 17),
    "channel_128x128_f32": ("identity", "channel", 42, 14, 14, 136, 136, 1, 0, False, False, None, 0, False, False, 17),
    "channel_fused": ("identity", "channel", 6, 7, 7, 1024, 256, 1, 0, True, False, None, 0, False, False, 4),
    "channel_groups_of_9": ("identity", "channel", 6, 14, 3, 8, 72, 1, 0, True, False, None, 0, False, False, 8),
    "channel_groups_of_18": ("identity", "channel", 4, 14, 14, 288, 72, 1, 0, True, False, None, 0, False, False, 4),
    "channel_groups_of_33_f32": ("identity", "channel", 5, 12, 9, 264, 264, 1, 0, False, False, None, 0, False, False, 8),
    "channel_groups_of_1": ("identity", "channel", 3, 5, 5, 16, 8, 1, 0, True, False, None, 0, False, False, 8),
    "channel_wide": ("channel_wide", 10928, 16, True),
    "channel_wide_f32": ("channel_wide", 7728, 16, False),
    # maskers, index lists, gather, the unfused schedule
    "masks": ("masks", 3, 12, 20, 72, 4),
    "masks_f32_gates": ("masks", 5, 14, 14, 8, 7, False, True),
    "masks_long_lists": ("masks", 9, 32, 33, 8, 1),
    "masks_wide": ("masks", 1, 14, 7, 1032, 7),  # one lane a chunk column in the channel masker's pooling
    "masks_unfused_split": ("masks", 3, 12, 20, 72, 4, True, False, 4, 136),
    "masks_unfused_128x128": ("masks", 12, 56, 56, 8, 4, True, False, 4, 136),
    "masks_unfused_64x128_f32": ("masks", 3, 12, 20, 136, 4, False, False, 4, 136),
    "masks_unfused_128x128_f32": ("masks", 11, 28, 28, 136, 4, False, False, 4, 136),
    # stems
    "stem": ("stem", 2, 37, 45, 64),
    "stem_f32": ("stem", 1, 17, 9, 40, False),
    "stem3x3": ("stem", 2, 9, 66, 32, True, 3),
    "stem3x3_odd": ("stem", 2, 9, 65, 24, True, 3),
}


# Tiles that a case is there for (kernel, mode, type, rows x columns; "split": the K steps are shared by two groups of waves): a rule
# that sends the case elsewhere leaves them untested.  Every tile of k_pipe, k_group and k_group_fused is some case's,
# and every instance of k_narrow and k_first.
REACHES = {
    "narrow": ["narrow false"],
    "narrow_static": ["narrow true"],
    "narrow_projection": ["narrow false"],
    "one_kernel_first": ["first"],
    "one_kernel_first_one_row": ["first"],
    "one_kernel_first_walk": ["first"],
    "tiled_128x64": ["pipe CONV2 bf16 128x64", "pipe SD1 bf16 128x64", "pipe CONV3 bf16 128x64"],
    "tiled_64x128_split": ["pipe CONV2 bf16 64x128 split"],
    "tiled_128x128": ["pipe CONV2 bf16 128x128"],
    "tiled_128x128_f32": ["pipe CONV1 float 128x128", "pipe CONV2 float 128x128", "pipe CONV3 float 64x64"],
    "last_128x64": ["pipe CONV3 bf16 128x64"],
    "last_f32": ["pipe CONV3 float 64x128"],
    "tiled_64x128_f32": ["pipe CONV1 float 64x128", "pipe CONV2 float 64x128", "pipe CONV3 float 64x128"],
    "tiled_64x64_f32": ["pipe CONV1 float 64x64", "pipe CONV2 float 64x64"],
    "dense_first_split": ["pipe SD1 bf16 64x128 split"],
    "last_split": ["pipe CONV3 bf16 64x128 split"],
    "last_128x128": ["pipe SD1 bf16 128x256", "pipe CONV3 bf16 128x128"],
    "last_128x256": ["pipe CONV1 bf16 128x128", "pipe CONV3 bf16 128x256"],
    "samples_tiled": ["pipe CONV1 bf16 128x64"],
    "samples_first_split": ["pipe CONV1 bf16 64x128 split"],
    "masker_128x64": ["pipe DENSE1 bf16 128x64"],
    "masker_128x128_f32": ["pipe DENSE1 float 128x128"],
    "masker_64x128_f32": ["pipe DENSE1 float 64x128"],
    "masker_64x64_f32": ["pipe DENSE1 float 64x64"],
    "masker_widest": ["pipe DENSE1 bf16 128x128"],
    "static_shortcut_128x256": ["pipe SD2 bf16 128x64", "pipe SD3 bf16 128x64"],
    "static_3x3_split": ["pipe SD2 bf16 64x128 split"],
    "static_3x3_128x128": ["pipe SD2 bf16 128x128"],
    "static_3x3_256x128": ["pipe SD2 bf16 256x128"],
    "static_last_split": ["pipe SD3 bf16 64x128 split"],
    "static_last_128x128": ["pipe SD3 bf16 128x128"],
    "static_last_128x256": ["pipe SD3 bf16 128x256"],
    "static_64x64_f32": ["pipe SD1 float 64x64", "pipe SD2 float 64x64", "pipe SD3 float 64x64"],
    "static_64x128_f32": ["pipe SD1 float 64x128", "pipe SD2 float 64x128", "pipe SD3 float 64x128"],
    "static_128x128_f32": ["pipe SD2 float 128x128"],
    "group_many_rows": ["group 2"],
    "group_fused": ["group_fused 2"],
    "group_fused_strips": ["group_fused 2"],
    "group_fused_walk": ["group_fused 2"],
    "group_fused_projection": ["group_fused 1"],
    "group_fused_projection_strips": ["group_fused 1"],
    "group_fused_projection_walk": ["group_fused 1"],
    "group_of_64": ["group 4"],
    "group_many_rows_f32": ["pipe G2 float 64x64"],
    "group_past_4096_channels": ["pipe G2 bf16 128x64"],
    "channel": ["pipe CS1 bf16 64x128", "pipe CS2 bf16 64x128", "pipe CS3 bf16 64x128"],
    "channel_split": ["pipe CS1 bf16 64x128 split", "pipe CS2 bf16 64x128 split"],
    "channel_128x64": ["pipe CS1 bf16 128x64", "pipe CS2 bf16 128x64", "pipe CS3 bf16 128x64"],
    "channel_64x64_f32": ["pipe CS1 float 64x64", "pipe CS2 float 64x64", "pipe CS3 float 64x64"],
    "channel_64x128_f32": ["pipe CS1 float 64x128", "pipe CS2 float 64x128", "pipe CS3 float 64x128"],
    "channel_128x128_f32": ["pipe CS1 float 128x128", "pipe CS2 float 128x128", "pipe CS3 float 128x128"],
    "channel_groups_of_9": ["gemm CS1 bf16 64x64", "gemm CS2 bf16 64x64", "gemm CS3 bf16 64x64"],
    "channel_groups_of_18": ["gemm CS3 bf16 64x128"],
    "channel_groups_of_33_f32": ["gemm CS1 float 64x128", "gemm CS2 float 64x128", "gemm CS3 float 64x128"],
    "channel_wide": ["gemm CS2 bf16 64x128", "pipe CS3 bf16 64x128"],
    "channel_wide_f32": ["gemm CS2 float 64x128", "pipe CS3 float 64x64"],
    "masks": ["pipe U1 bf16 128x64", "pipe U2 bf16 128x64", "pipe U3 bf16 128x64"],
    "masks_f32_gates": ["pipe U1 float 64x64", "pipe U2 float 64x64", "pipe U3 float 64x64"],
    "masks_unfused_split": ["pipe U2 bf16 64x128 split"],
    "masks_unfused_128x128": ["pipe U2 bf16 128x128"],
    "masks_unfused_64x128_f32": ["pipe U1 float 64x128", "pipe U2 float 64x128", "pipe U3 float 64x128"],
    "masks_unfused_128x128_f32": ["pipe U1 float 128x128", "pipe U2 float 128x128", "pipe U3 float 128x128"],
}
# Threads of the last 1x1's workgroups that the LDS of a compute unit (160 KB) holds at least, where the reduction is short: its time is
# that of memory, and the copy of inactive patches runs in workgroups of the same size.
HELD = {"tiled_128x64": 1024, "last_128x64": 768, "last_f32": 768}
MODES = "CONV1 CONV2 CONV3 CS1 CS2 CS3 DENSE1 U1 U2 U3 SD1 SD2 SD3 G2".split()


def tiles(names):
    """The tiles among demangled kernel names, as REACHES has them."""
    names, found = names.replace("unsigned short", "bf16"), set()
    for kernel, mode, dtype, rows, columns, rest in re.findall(r"k_(pipe|gemm)<(\d+), (\w+), (\d+), (\d+), ([\d, ]+)>", names):
        found.add(f"{kernel} {MODES[int(mode)]} {dtype} {rows}x{columns}" + (" split" if rest.split(", ")[2:3] == ["2"] else ""))
    found |= {"first"} if "k_first(" in names else set()
    found |= {f"group_fused {k}" for k in re.findall(r"k_group_fused<(\d)>", names)}
    return found | {f"group {k}" for k in re.findall(r"k_group<(\d)>", names)} | {f"narrow {k}" for k in re.findall(r"k_narrow<(\w+)>", names)}


def test_every_tile_of_the_many_row_kernels_has_a_case(lib):
    symbols = subprocess.run(["nm", "-C", lib], check=True, capture_output=True, text=True).stdout
    built = {t for t in tiles(symbols) if not t.startswith("gemm")}
    assert len(built) > 60 and built == {t for case in REACHES.values() for t in case if not t.startswith("gemm")}


def in_a_process_of_its_own(body, capfd):
    """(a fault ends the process, with the kernel and the workgroup on stderr)"""
    pid = os.fork()
    if pid == 0:
        status = 1
        try:
            body()
            status = 0
        except BaseException as e:  # noqa: B902
            os.write(2, repr(e).encode())
        os._exit(status)
    _, status = os.waitpid(pid, 0)
    assert status == 0, capfd.readouterr().err


@pytest.mark.parametrize("front", [0, 1])
@pytest.mark.parametrize("name", CASES)
def test_kernels_stay_inside_their_buffers(lib, name, front, capfd):
    def body():
        method, *args = CASES[name]
        call = Call(lib, front)
        getattr(call, method)(*args)
        missing = set(REACHES.get(name, [])) - tiles(call.launched())
        assert not missing, (missing, call.launched())
        for lds, threads in re.findall(r"k_pipe<2, .*lds (\d+) threads (\d+)", call.launched()):
            assert (160 << 10) // int(lds) * int(threads) >= HELD.get(name, 0), (lds, threads)
    in_a_process_of_its_own(body, capfd)


# Static blocks of 64 -> 64 -> 256 channels, bf16: the kernel of the whole block, whose rectangles are mostly empty on small and on thin
# maps, only where it needs few rounds of them for the rows there are (256 workgroups, 128 rows each).
ONE_KERNEL = [
    (2, 41, 25), (128, 56, 56), (50, 72, 72), (1, 1100, 1), (65, 4, 4),       # full rectangles; at most one a workgroup
    (285, 3, 3), (492, 5, 5), (768, 4, 4), (286, 7, 7),                       # small tiles: a second round from 2560 rows on, a third from 12288
    (300, 7, 7), (512, 8, 8), (768, 8, 8), (694, 12, 12), (4669, 9, 9),       # ahead of the 64-wide kernel's tiles: 2 rounds for 1, 3 for 2, 6 for 4, 19 for 12
]
NOT_ONE_KERNEL = [
    (1, 32, 32), (1100, 1, 1), (257, 2, 2), (284, 3, 3), (683, 3, 3), (767, 4, 4), (769, 4, 4), (13, 1100, 1),
    (600, 5, 5), (30000, 1, 1), (1875, 4, 4), (612, 7, 7), (1024, 8, 8), (1562, 8, 8), (2778, 12, 12), (25000, 4, 4), (27, 1100, 1), (667, 300, 2),
]


@pytest.mark.parametrize("case", [(*c, 1, "first") for c in ONE_KERNEL + test_gpu_first.CASES] +
                         [(*c, 1, None) for c in NOT_ONE_KERNEL] + [(*c, "narrow true") for c in test_gpu_narrow.STATIC_CASES])
def test_static_block_takes_the_whole_block_kernel_where_a_map_fills_it(lib, case, capfd):
    """(the sizes of the GPU tests of both kernels too: that they are about the kernel they name)"""
    n, h, w, stride, kernel = case

    def body():
        call = Call(lib, 0)
        call.host.host_record_only()
        call.first("static", n, h, w, 64, 64, 256, stride, 1, 1.0)
        found = tiles(call.launched())
        assert kernel in found if kernel else "first" not in found, call.launched()
    in_a_process_of_its_own(body, capfd)


@pytest.mark.parametrize("case", test_gpu_group_se.FUSED + test_gpu_group_se.FUSED_PROJ)
def test_group_blocks_take_first_1x1_and_3x3_in_one_launch(lib, case, capfd):
    """(the sizes of the GPU test of that kernel: that they are about it)"""
    def body():
        call = Call(lib, 0)
        call.host.host_record_only()
        if len(case) == 10:
            n, h, w, c, g, se, S = case[:7]
            call.identity("dyn", n, h, w, c, c, S, 0.5, gw=g, se=se)
        else:
            n, h, w, ci, co, g, se, stride, S = case[:9]
            call.first("dynamic", n, h, w, ci, co, co, stride, S, 0.5, gw=g, se=se)
        assert f"group_fused {2 if len(case) == 10 else 1}" in tiles(call.launched()), call.launched()
    in_a_process_of_its_own(body, capfd)


class Untouched:
    """A workspace of zeros whose pages stay untouched."""

    def __init__(self, call, nbytes):
        p = call.buf(nbytes)
        self.data_ptr, self.numel, self.element_size = (lambda: p), (lambda: int(nbytes)), (lambda: 1)


def bf16(a):
    return (np.asarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def wide_projection(call, n, h, w, ids):
    """The fused 3x3 -> last 1x1 kernel of a first block of 256 -> 256 -> 1024 channels (stride 1, S = 1), weights and h1 zero: onto the
    shortcut, which is not run, it adds the last 1x1's shift.  The shortcut is 256 (i + 1) in the i-th listed pixel; returns `out`."""
    call.host.host_run_only.argtypes = [C.c_char_p]
    call.host.host_run_only(b"k_tail")
    ci, m, co = 256, 256, 1024
    weights = [call.buf(k * 2) for k in (m * ci, 9 * m * m, co * m)]
    affine = [call.buf(4 * k, np.full(k, v, np.float32)) for k, v in ((m, 1), (m, 0), (m, 1), (m, 0), (co, 1), (co, 64))]
    p = B.Bottleneck(ci, m, co, *weights, *affine, 1)
    p.packed = call.buf(B.packed_weights_size(p, B.BF16))
    fx, out, ids = B.Fmap(n, h, w, ci, B.BF16), call.buf(n * h * w * co * 2), np.array(ids, np.int32)
    for i, pixel in enumerate(ids):
        row = bf16(np.full(co, 256 * (i + 1)))
        C.memmove(out + int(pixel) * co * 2, row.ctypes.data, co * 2)
    B.laud_dyn_projection_bottleneck(call.buf(n * h * w * ci * 2), fx, p, call.buf(co * ci * 2), affine[4], affine[5], 1, 1, call.buf(ids.nbytes, ids),
                                     call.buf(4, np.array([len(ids)], np.int32)), out, Untouched(call, B.dyn_projection_workspace(fx, p, 1)))
    return out


@pytest.mark.parametrize("n", [64, 65, 129])
def test_outputs_of_the_fused_kernel_past_2_gib(lib, n, capfd):
    """First blocks whose output is wider than what the size rule counts (c_in, c_mid): 64 samples of 128 x 128 are 2 GiB of output, 65
    more, the last of 129 lies past 4 GiB.  (The threads of a wave run one after the other here: of what they hand each other through LDS
    some values come late, so that a result is the shortcut plus the shift or, where it came late, plus nothing.)"""
    pixels = n * 128 * 128
    ids = sorted({0, 1, 16383, 777777, (1 << 20) - 1, pixels - 16384, pixels - 2, pixels - 1} | ({1 << 20, (1 << 20) + 5} if n > 64 else set()) |
                 ({1 << 21} if n > 128 else set()))

    def body():
        call = Call(lib, 0)
        out = wide_projection(call, n, 128, 128, ids)
        rows = lambda pixel: np.ctypeslib.as_array((C.c_uint16 * 1024).from_address(out + pixel * 2048))  # noqa: E731
        assert "k_tail" in call.launched()
        for i, pixel in enumerate(ids):
            got = set(rows(pixel).tolist())
            assert got <= set(bf16([256 * (i + 1), 256 * (i + 1) + 64]).tolist()) and len(got) > 1, (pixel, got)
        for pixel in {2, 3, 5, 8, 4096, 16384, 16386, 32768} - set(ids):  # (an offset that wraps lands in the first samples)
            assert not rows(pixel).any(), pixel
    in_a_process_of_its_own(body, capfd)


# First blocks of few rows with groups (n, h, w, c_in, c, group width, stride, S): those whose shortcut and first 1x1 are faster in one launch
# than the 3x3 with the first 1x1, and the nearest ones that are not.
SHORTCUT_PAIR = [(1, 4, 4, 112, 16, 8, 1, 2), (2, 14, 14, 144, 320, 16, 1, 1), (4, 7, 7, 208, 440, 8, 1, 1), (33, 4, 4, 64, 288, 16, 1, 2),
                 (63, 8, 8, 64, 16, 16, 1, 4), (95, 8, 8, 128, 16, 16, 1, 4), (1, 7, 7, 8, 8, 8, 1, 7), (4, 16, 16, 96, 48, 16, 2, 2), (63, 8, 8, 136, 16, 16, 2, 2),
                 (159, 8, 8, 328, 16, 16, 2, 4)]
NOT_SHORTCUT_PAIR = [(64, 8, 8, 64, 16, 16, 1, 4), (96, 8, 8, 128, 16, 16, 1, 4), (4, 16, 16, 64, 48, 16, 2, 2), (5, 16, 16, 96, 48, 16, 2, 2), (64, 8, 8, 136, 16, 16, 2, 2), (160, 8, 8, 328, 16, 16, 2, 4),
                     (1, 112, 112, 32, 64, 16, 2, 4), (1, 56, 56, 64, 144, 16, 2, 2), (3, 28, 28, 144, 320, 16, 2, 2)]


@pytest.mark.parametrize("case", SHORTCUT_PAIR + NOT_SHORTCUT_PAIR)
def test_small_first_blocks_keep_shortcut_and_first_1x1_in_one_launch(lib, case, capfd):
    n, h, w, ci, c, g, stride, S = case

    def body():
        call = Call(lib, 0)
        call.host.host_record_only()
        call.first("dynamic", n, h, w, ci, c, c, stride, S, 0.5, gw=g, se=0)
        names = call.launched()
        assert ("k_skinny_pair" in names, "k_group_fused" in names) == (case in SHORTCUT_PAIR, case in NOT_SHORTCUT_PAIR), names
    in_a_process_of_its_own(body, capfd)


# Where the masker's decision of the patches and their list are made (n, h, w, S, with gates): in one launch up to a number of patches (less with
# gates where a patch is one pixel), in two past it.
POOL_ROUTES = [
    ((8, 32, 32, 1, True), "k_pool_compact<1, 8>"), ((9, 32, 32, 1, True), "k_pool_mask"), ((12, 32, 32, 1, True), "k_pool_mask"),
    ((12, 32, 32, 1, False), "k_pool_compact<1, 8>"), ((13, 32, 32, 1, False), "k_pool_mask"),
    ((32, 32, 32, 2, True), "k_pool_compact<2, 8>"), ((33, 32, 32, 2, True), "k_pool_mask"), ((32, 32, 32, 4, True), "k_pool_compact<4, 1>"),
    ((33, 32, 32, 4, False), "k_pool_mask"),
]


@pytest.mark.parametrize("case,kernel", POOL_ROUTES)
def test_masker_decides_its_patches_in(lib, case, kernel, capfd):
    n, h, w, S, keep = case

    def body():
        call = Call(lib, 0)
        call.host.host_record_only()
        call.identity("masker", n, h, w, 16, 8, S, 0.5, keep=keep)
        found = set(re.findall(r"k_pool_\w+(?:<\d, \d>)?", call.launched())) | set(re.findall(r"k_skinny<14", call.launched()))
        assert found == {kernel}, call.launched()
    in_a_process_of_its_own(body, capfd)


@pytest.mark.parametrize("case,threads", test_gpu_pooled_lists.PARTIAL)
def test_lists_of_less_than_a_block_are_launched_in_fewer_waves(lib, case, threads, capfd):
    """(the sizes of the GPU test of that launch: that they are about it)"""
    def body():
        n, h, w, c, m, S = case[:6]
        call = Call(lib, 0)
        call.host.host_record_only()
        call.identity("masker", n, h, w, c, m, S, 0.5)
        assert re.findall(r"k_pool_compact<(\d), \d>.* threads (\d+)", call.launched()) == [(str(S), str(threads))], call.launched()
    in_a_process_of_its_own(body, capfd)


@pytest.mark.parametrize("case,threads", test_gpu_pooled_lists.IN_3X3)
def test_few_patches_are_decided_in_the_3x3(lib, case, threads, capfd):
    def body():
        n, h, w, c, m, S, dtype = case[:7]
        call = Call(lib, 0)
        call.host.host_record_only()
        call.identity("masker", n, h, w, c, m, S, 0.5, dtype == B.BF16)
        assert re.findall(r"k_skinny<14, .* threads (\d+)", call.launched()) == [str(threads)] and "k_pool" not in call.launched(), call.launched()
    in_a_process_of_its_own(body, capfd)


@pytest.mark.parametrize("apart,kernel", [(-40, "k_skinny<14"), (40, "k_skinny<14"), (0, "k_pool_compact<4, 1>"), (39, "k_pool_compact<4, 1>"), (-39, "k_pool_compact<4, 1>")])
@pytest.mark.parametrize("n", [40, 1100])
def test_masks_over_their_gates_are_decided_by_one_reader_a_gate(lib, n, apart, kernel, capfd):
    """Every workgroup of the 3x3, and every later block of the list's launch, reads the gates again: not where the mask is written over
    them (gates `apart` of n bytes from the mask's)."""
    def body():
        call = Call(lib, 0)
        call.host.host_record_only()
        fx, x, p = B.Fmap(n, 4, 4, 16, B.BF16), call.values(n * 256, True), call.block(16, 8, 16, None, True, False)
        both = call.buf(3 * n)
        mask, gates = both + n, both + n + (apart if abs(apart) < 40 else n if apart > 0 else -n)
        B.laud_masker_dyn_bottleneck(x, fx, p, 4, call.values(16, False), 0.01, gates, mask, call.buf(4 * n), call.buf(4), None, None, x,
                                     call.ws(B.workspace_size(B.OP_DYN_BOTTLENECK, fx, p, 4)))
        found = set(re.findall(r"k_pool_\w+(?:<\d, \d>)?", call.launched())) | set(re.findall(r"k_skinny<14", call.launched()))
        assert found == {kernel if n == 40 else "k_pool_compact<4, 1>" if abs(apart) == 40 else "k_pool_mask"}, call.launched()
    in_a_process_of_its_own(body, capfd)
