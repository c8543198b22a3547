"""The C-ABI library without a GPU: it loads, exports what include/moe.h declares, sizes
workspaces, and rejects bad arguments on the host before any launch."""
import ctypes as C
import os
import re
import struct
import subprocess

import pytest

import paper_2503_00245_amd as pkg
from paper_2503_00245_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "moe.h")).read()
    return re.findall(r"MOE_API\s+[\w\s\*]+?\b(moe_\w+)\s*\(", text)


def test_library_exports_every_declared_symbol():
    names = _declared()
    assert set(names) == set(pkg.EXPORTS) and len(names) == 15
    L = pkg.lib()
    for n in names:
        assert getattr(L, n) is not None


def test_status_strings():
    assert pkg.status_string(0) == "ok"
    assert len({pkg.status_string(s) for s in (0, -1, -2, -3, -4, -99)}) == 6


def test_workspace_bytes_by_shape():
    small = pkg.moe_workspace_bytes(pkg.make_shape(32, 128, 256, 4, 2, 0, pkg.MOE_F32))
    big = pkg.moe_workspace_bytes(pkg.make_shape(2048, 2048, 5632, 8, 2, 0, pkg.MOE_BF16))
    assert 0 < small < big
    # the phone prefill workspace must hold h [P,F] and y_perm [P,d] in bf16
    assert big >= 4096 * (5632 + 2048) * 2
    assert big % 256 == 0
    assert pkg.moe_workspace_bytes(pkg.make_shape(0, 128, 256, 4, 2)) > 0


@pytest.mark.parametrize("d,F,E,k,r,act,flags", [
    (2048, 5632, 8, 2, 0, pkg.MOE_BF16, 0), (1024, 2816, 8, 2, 0, pkg.MOE_BF16, 0), (1440, 3840, 16, 4, 0, pkg.MOE_BF16, 0),
    (432, 1152, 4, 1, 0, pkg.MOE_BF16, 0), (8, 4096, 64, 40, 0, pkg.MOE_BF16, 0),
    (2048, 5632, 8, 2, 1024, pkg.MOE_BF16, 0), (520, 1040, 8, 3, 1064, pkg.MOE_BF16, 0), (400, 1064, 8, 2, 200, pkg.MOE_BF16, 0),
    (2048, 5632, 8, 2, 64, pkg.MOE_BF16, 1), (264, 520, 4, 1, 1064, pkg.MOE_BF16, 1), (64, 2056, 8, 8, 40, pkg.MOE_BF16, 1),
    (128, 256, 4, 2, 0, pkg.MOE_F32, 0), (512, 1408, 8, 2, 256, pkg.MOE_F32, 1),
])
def test_a_workspace_for_more_tokens_holds_fewer(d, F, E, k, r, act, flags):
    # a server sizes one workspace for its largest batch: the size must not fall as the tokens grow
    tokens = list(range(1, 1200)) + list(range(1200, 20000, 13))
    sizes = [pkg.moe_workspace_bytes(pkg.make_shape(t, d, F, E, k, r, act, flags)) for t in tokens]
    falls = [t for t, a, b in zip(tokens[1:], sizes, sizes[1:]) if b < a]
    assert not falls, f"{len(falls)} token counts need less than the one before, first {falls[:5]}"
    # one token takes no part of the grouped products' cuts: what a step of its own kind needs
    es = 4 if act == pkg.MOE_F32 else 2
    per_token = k * (F + 3 * r + d) * es + (3 * F + d) * es * (flags & 1) + d * es + 5 * 4 * k
    assert sizes[0] <= per_token + 4 * k * (F + 3 * r) + 4 * E + 16 * 256


def test_parts_keep_within_the_allocation_free_entry_points_array():
    # largest batches of the shapes that the array holds (no parts there), and the ones behind them
    for (d, F, E, k, r, flags), t in (((2048, 5632, 8, 2, 0, 0), 239), ((1024, 2816, 8, 2, 0, 0), 479),
                                      ((2048, 5632, 8, 2, 1024, 0), 176), ((2048, 5632, 8, 2, 64, 1), 113)):
        assert pkg.moe_workspace_bytes(pkg.make_shape(t, d, F, E, k, r, pkg.MOE_BF16, flags)) <= pkg.STATIC_WORKSPACE_BYTES
        assert pkg.moe_workspace_bytes(pkg.make_shape(t + 1, d, F, E, k, r, pkg.MOE_BF16, flags)) > pkg.STATIC_WORKSPACE_BYTES


@pytest.mark.parametrize("kw,status", [
    (dict(top_k=0), -1), (dict(top_k=5), -1), (dict(n_tokens=-1), -1), (dict(rank=-8), -1),
    (dict(flags=1), -1),                 # shared base without a rank
    (dict(flags=8), -1),                 # unknown flag
    (dict(n_experts=65, top_k=2), -2), (dict(d_model=100), -2), (dict(d_ff=100), -2),
    (dict(rank=12), -2), (dict(act_dtype=7), -2), (dict(n_tokens=1 << 23), -2),
])
def test_bad_shapes_are_rejected_on_the_host(kw, status):
    base = dict(n_tokens=8, d_model=128, d_ff=256, n_experts=4, top_k=2, rank=0,
                act_dtype=pkg.MOE_BF16, flags=0)
    base.update(kw)
    shape = pkg.make_shape(**base)
    assert pkg.moe_workspace_bytes(shape) == 0
    L = pkg.lib()
    dummy = C.c_void_p(4096)
    assert L.moe_route(C.byref(shape), dummy, dummy, None, dummy, dummy, None, None) == status
    assert L.moe_combine(C.byref(shape), dummy, dummy, dummy, None, dummy, None) == status
    w = pkg.MoeWeights()
    assert L.moe_forward(C.byref(shape), C.byref(w), dummy, dummy, None, None, dummy, 1 << 30,
                         None) == status


def test_null_misaligned_and_short_workspace_arguments():
    L = pkg.lib()
    shape = pkg.make_shape(8, 128, 256, 4, 2)
    ok, odd = C.c_void_p(4096), C.c_void_p(4100)
    assert L.moe_route(C.byref(shape), None, ok, None, ok, ok, None, None) == -1
    assert L.moe_route(C.byref(shape), odd, ok, None, ok, ok, None, None) == -1
    assert L.moe_route(None, ok, ok, None, ok, ok, None, None) == -1
    assert L.moe_combine(C.byref(shape), ok, ok, ok, odd, ok, None) == -1
    assert L.moe_permute(C.byref(shape), ok, None, ok, ok, None, None, ok, 1 << 20, None) == -1
    assert L.moe_permute(C.byref(shape), ok, ok, ok, ok, ok, None, ok, 1 << 20, None) == -1
    w = pkg.MoeWeights()
    assert L.moe_forward(C.byref(shape), C.byref(w), ok, ok, None, None, ok, 1 << 30, None) == -1
    for n in ("router_w", "w_gate", "w_up", "w_down"):
        setattr(w, n, 4096)
    need = pkg.moe_workspace_bytes(shape)
    y = C.c_void_p(8192)
    assert L.moe_forward(C.byref(shape), C.byref(w), ok, y, None, None, ok, need - 1, None) == -3
    assert L.moe_forward(C.byref(shape), C.byref(w), ok, y, None, None, None, need, None) == -3
    assert L.moe_forward(C.byref(shape), C.byref(w), ok, ok, None, None, ok, need, None) == -1  # y aliases x
    assert L.moe_expert_ffn(C.byref(shape), C.byref(w), ok, ok, ok, ok, 16, None) == -3
    w.rg = 4096  # factors without a rank are ignored, a dense block without the flag is not
    wd = pkg.make_shape(8, 128, 256, 4, 2, rank=16)
    assert L.moe_forward(C.byref(wd), C.byref(w), ok, C.c_void_p(8192), None, None, ok, 1 << 30, None) == -1
    assert L.moe_stack_forward(C.byref(shape), C.byref(w), 0, ok, C.c_void_p(8192), None, ok, 1 << 30, None) == -1


def test_zero_tokens_is_a_no_op_without_touching_pointers():
    L = pkg.lib()
    shape = pkg.make_shape(0, 128, 256, 4, 2)
    assert L.moe_route(C.byref(shape), None, None, None, None, None, None, None) == 0
    assert L.moe_combine(C.byref(shape), None, None, None, None, None, None) == 0
    w = pkg.MoeWeights()
    for n in ("router_w", "w_gate", "w_up", "w_down"):
        setattr(w, n, 4096)
    assert L.moe_forward(C.byref(shape), C.byref(w), None, None, None, None, None, 0, None) == 0
    assert L.moe_expert_ffn(C.byref(shape), C.byref(w), None, None, None, None, 0, None) == 0


def test_trace_metric_entry_points_reject_bad_shapes_on_the_host():
    L = pkg.lib()
    ok = C.c_void_p(4096)
    assert L.moe_expert_replacements(ok, 1, 8, 3, 2, ok, ok, None) == -1      # K > E
    assert L.moe_expert_replacements(ok, 1, 8, 2, 65, ok, ok, None) == -2     # E > 64
    assert L.moe_expert_replacements(None, 1, 8, 2, 8, ok, ok, None) == -1
    assert L.moe_offload_counters(ok, 0, 8, 2, 8, ok, ok, None) == -1
    assert L.moe_offload_counters(ok, 2, 8, 2, 8, None, ok, None) == -1
    assert pkg.moe_bles_workspace_bytes(4, 128, 8) >= 8 * 65 + 4 * (4 * 127 * 8 // 256)
    assert pkg.moe_bles_workspace_bytes(4, 128, 65) == 0
    assert L.moe_bles_loss(ok, ok, 4, 128, 2, 8, ok, ok, 16, None) == -3       # short workspace
    assert L.moe_bles_loss(ok, ok, 4, 128, 2, 8, None, ok, 1 << 20, None) == -1


def test_static_entry_point_refuses_what_its_scratch_cannot_hold():
    # checked on the host, before the scratch array is even looked up
    L = pkg.lib()
    w = pkg.MoeWeights()
    for n in ("router_w", "w_gate", "w_up", "w_down"):
        setattr(w, n, 4096)
    ok, y = C.c_void_p(4096), C.c_void_p(8192)
    big = pkg.make_shape(2048, 2048, 5632, 8, 2)
    assert pkg.moe_workspace_bytes(big) > pkg.STATIC_WORKSPACE_BYTES
    assert L.moe_forward_static(C.byref(big), C.byref(w), ok, y, None, None, None) == -3
    assert L.moe_forward_static(C.byref(big), C.byref(w), ok, ok, None, None, None) == -1  # y aliases x
    assert L.moe_forward_static(C.byref(pkg.make_shape(8, 100, 256, 4, 2)), C.byref(w), ok, y, None, None, None) == -2
    one = pkg.make_shape(1, 2048, 5632, 8, 2)
    assert 0 < pkg.moe_workspace_bytes(one) <= pkg.STATIC_WORKSPACE_BYTES


def test_a_product_planned_in_parts_has_a_kernel_that_writes_them(tmp_path):
    # host code alone, on the library's own objects: every width up to matrices of 4 GB and more, every kind of layer
    objs = [os.path.join(hip_build.OBJ, src.replace(".hip", ".o")) for src in hip_build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        hip_build.build()
    main, exe = str(tmp_path / "check.o"), str(tmp_path / "check")
    subprocess.run([hip_build._hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    hip_build.CSRC, "-c", os.path.join(ROOT, "tests", "split_plan_check.cpp"), "-o", main], check=True)
    subprocess.run([hip_build._hipcc(), main, *objs, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


def _host_check(source, tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run([hip_build._hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    hip_build.CSRC, os.path.join(ROOT, "tests", source), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


def test_a_launch_has_a_workgroup_for_every_tile(tmp_path):
    _host_check("tile_grid_check.cpp", tmp_path)


def test_a_single_tokens_rows_are_taken_once_and_lie_together(tmp_path):
    _host_check("unit_order_check.cpp", tmp_path)


def test_the_combine_of_a_layer_without_a_base_leaves_a_cu_eight_workgroups(tmp_path):
    # eight workgroups of 256 threads are eight waves a SIMD, of 512 registers a lane
    out = str(tmp_path / "combine.s")
    subprocess.run([hip_build._hipcc(), *hip_build.FLAGS, "--offload-device-only", "-S", os.path.join(hip_build.CSRC, "combine.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    used = {n: int(v) for n, v in re.findall(r"\.name:\s+(_ZN3moe14combine_kernel\S+)[\s\S]*?\.vgpr_count:\s+(\d+)", text)}
    small = {n: v for n, v in used.items() if not re.search(r"Li\d+ELi2EE", n)}  # (the last argument: fp32 parts of an addend)
    assert max(small.values()) <= 64, small
    assert len(used) > len(small)


def test_a_first_stage_without_a_rest_does_without_the_order_of_one(tmp_path):
    # the instances for layers of whole turns read no count of turns: what stands ahead of their first request is what it was without the order
    out = str(tmp_path / "one.s")
    subprocess.run([hip_build._hipcc(), *hip_build.FLAGS, "--offload-device-only", "-S", os.path.join(hip_build.CSRC, "expert_gemv_one.hip"), "-o", out],
                   check=True, capture_output=True)
    read = {}  # kernel: the dwords of its arguments that it loads
    for name, body in re.findall(r"^(_ZN3moe19decode_first_kernel\w+):[^\n]*\n([\s\S]*?)\.end_amdhsa_kernel", open(out).read(), re.M):
        read[name] = {int(at, 16) + 4 * i for n, at in re.findall(r"s_load_dword(x\d+)? s\S+, s\S+, (0x[0-9a-f]+)", body)
                      for i in range(int(n[1:] or 1))}
    pairs = [(n, n.replace("ELb1EEEv", "ELb0EEEv")) for n in read if "ELb1EEEv" in n]  # (the last template argument: with a rest)
    assert len(pairs) == 16  # two types, four row lengths, with and without SwiGLU
    for spread, plain in pairs:
        assert read[spread] - read[plain], spread


def _device_objects():
    """The gfx950 code objects of the built library, one per source file."""
    data = open(hip_build.ensure_built(), "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(magic))[0]):
            offset, size, n = struct.unpack_from("<3Q", data, pos)
            if data[pos + 24:pos + 24 + n].endswith(b"gfx950"):
                yield data[at + offset:at + offset + size]
            pos += 24 + n
        at = data.find(magic, at + 1)


def test_no_wait_stands_between_the_prefill_kernels_matrix_instructions(tmp_path):
    # the fragments have landed before the barrier that begins a phase's products
    obj = str(tmp_path / "device.o")
    products = 0
    for code in _device_objects():
        if b"gemm_pp_kernel" not in code:
            continue
        open(obj, "wb").write(code)
        objdump = os.path.join(os.path.dirname(os.path.realpath(hip_build._hipcc())), "..", "lib", "llvm", "bin", "llvm-objdump")
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--no-leading-addr", obj], check=True, capture_output=True, text=True).stdout
        text = re.sub(r"\s*//.*", "", text)
        products += text.count("v_mfma")
        assert not re.findall(r"v_mfma[^\n]*\n\s*s_waitcnt lgkmcnt[^\n]*\n(?=\s*v_mfma)", text)
    assert products > 1000
