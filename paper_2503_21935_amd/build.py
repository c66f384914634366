"""Build libme.so for gfx950.

Steps: run the process generator into ``csrc/gen/``, write one translation
unit per process and the process table, compile each with hipcc
(``--offload-arch=gfx950``) and link the shared library in-tree.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
GEN = os.path.join(CSRC, "gen")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libme.so")

PROCESSES = ["ee_mumu", "gg_tt", "gg_ttg", "gg_ttgg", "gg_ttggg", "gux_taptamux", "gux_taptamgux",
             "gux_taptamggux"]

# processes whose colour-flow amplitudes live in LDS (workgroup kernel of me_coop.h)
COOP = {"gg_ttggg"}

# one-wave processes that also get the float64 form with the colour sum on the
# matrix cores (needs a multiple of 4 colour flows); the workgroup processes
# always get it
CM = {"gg_ttgg"}

# kernels of the float64 sum over spins with real polarisation vectors
WAVE = {"gg_tt": "k_me_gg2_pol", "gg_ttg": "k_me_gg3_pol", "gg_ttgg": "k_me_gg4_wave", "gg_ttggg": "k_me_gg5_wave"}
# events per wave of those that hold several
EVENTS_PER_WAVE = {"gg_tt": 64, "gg_ttg": 8}

# Calibration of the mixed form's amplitude error estimate (multiplies
# u32 * 2 lambda_max(|N|) |S| |J| / Q); fixed by comparing float32 results
# with the oracle (see the mixed-precision tests).
MIXED_CEST = {"gg_tt": 8.0, "gg_ttg": 8.0, "gg_ttgg": 8.0, "gg_ttggg": 8.0}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HIPFLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-variable",
    "-Wno-unused-function", "-Wno-unknown-pragmas",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", CSRC,
]

_TU_QEW = """// Generated translation unit: kernels of {name} (quark line + lepton pair).
#include "me_qew_pol.h"
{include}

static hipError_t launch_sum(const double* mom, int64_t nevt, double* out, unsigned, const me_params& prm,
                             const int* idx, const int* count, bool, hipStream_t s) {{
    me_each_launch(nevt, 64 >> {proc}::ngluon, 64, [&](int64_t first, unsigned blocks) {{
        hipLaunchKernelGGL((k_me_qew_pol<{proc}>), dim3(blocks), dim3(64), 0, s, mom, nevt, out, prm, idx, count,
                           first);
    }});
    return hipGetLastError();
}}

static hipError_t launch_f64(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                             const me_params& prm, double* qhel, int lg, hipStream_t s) {{
    const dim3 grid((unsigned)(((nevt << lg) + ME_BLOCK - 1) / ME_BLOCK));
    hipLaunchKernelGGL((k_me_qew<{proc}>), grid, dim3(ME_BLOCK), 0, s, mom, nevt, out, hels, nh, prm, qhel, lg);
    return hipGetLastError();
}}

#ifndef __HIP_DEVICE_COMPILE__  // the table entry holds host function pointers
extern const me_process_desc me_desc_{name} = {{
    "{name}", ME_KIND_QEW, {proc}::npart, {proc}::ndiag, {proc}::ncol, {proc}::nhel,
    {proc}::flops_amp, {proc}::flops_colour, {proc}::flops_executed, launch_f64, nullptr, nullptr, 8.0,
    nullptr, nullptr, 0, nullptr, launch_sum, nullptr, false, 65536}};
#endif
"""

_TU = """// Generated translation unit: kernels of {name}.
#include "me_mixed.h"
{include}

{f64}{mixed}{cm}
#ifndef __HIP_DEVICE_COMPILE__  // the table entry holds host function pointers
extern const me_process_desc me_desc_{name} = {{
    "{name}", {kind}, {proc}::npart, {proc}::ndiag, {proc}::ncol, {proc}::nhel,
    {proc}::flops_amp, {proc}::flops_colour, {proc}::flops_executed, launch_f64, {idx_ptr}, {mixed_ptr}, {cest},
    {cm_ptr}, {mc_ptr}, {mc_n}, {mc_desc}, {sum_ptr}, {chan_ptr},
    {mixed_part}, {hel_turn}}};
#endif
"""

_F64_GG = """static hipError_t launch_f64(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                             const me_params& prm, double* qhel, int lg, hipStream_t s) {{
    const dim3 grid((unsigned)(((nevt << lg) + ME_BLOCK - 1) / ME_BLOCK));
    hipLaunchKernelGGL((k_me_gg<{proc}>), grid, dim3(ME_BLOCK), 0, s, mom, nevt, out, hels, nh, prm, qhel, lg);
    return hipGetLastError();
}}
"""

_F64_EE = """static hipError_t launch_f64(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                             const me_params& prm, double* qhel, int lg, hipStream_t s) {{
    const dim3 grid((unsigned)(((nevt << lg) + ME_BLOCK - 1) / ME_BLOCK));
    hipLaunchKernelGGL((k_me_ee<{proc}>), grid, dim3(ME_BLOCK), 0, s, mom, nevt, out, hels, nh, prm,
                       qhel, nullptr, nullptr, lg);
    return hipGetLastError();
}}

static hipError_t launch_f64_idx(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                 const me_params& prm, const int* idx, const int* count, hipStream_t s) {{
    const dim3 grid((unsigned)((nevt + ME_BLOCK - 1) / ME_BLOCK));
    hipLaunchKernelGGL((k_me_ee<{proc}>), grid, dim3(ME_BLOCK), 0, s, mom, nevt, out, hels, nh, prm,
                       nullptr, idx, count, 0);
    return hipGetLastError();
}}
"""

_MC_DECL = """
#ifndef __HIP_DEVICE_COMPILE__
// the multi-channel kernel is compiled in a translation unit of its own
hipError_t me_launch_mc_{name}(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                               const me_params& prm, const int* chan, double* alpha, hipStream_t s);
hipError_t me_launch_chan_{name}(const double* mom, int64_t nevt, double* out, const me_params& prm, const int* chan,
                                 double* alpha, hipStream_t s);
extern const int me_nchan_{name};
extern const char* const* const me_chan_desc_{name};
#endif
"""

_WAVE_DECL = """
#ifndef __HIP_DEVICE_COMPILE__
hipError_t me_launch_sum_{name}(const double* mom, int64_t nevt, double* out, unsigned spins, const me_params& prm,
                                const int* idx, const int* count, bool mfma, hipStream_t s);
#endif
"""

_TU_WAVE = """// Generated translation unit: spin-summed float64 kernel of {name} (one event per wave).
#include "{header}"
#include "gen/proc_{name}.h"

hipError_t me_launch_sum_{name}(const double* mom, int64_t nevt, double* out, unsigned spins, const me_params& prm,
                                const int* idx, const int* count, bool mfma, hipStream_t s) {{
{launch}    return hipGetLastError();
}}
"""

# one wave per block, one or two events at a time
_LAUNCH_WAVE = """    const int eb = me_wave_events(nevt);
    const int64_t turns = (nevt + eb - 1) / eb;
    const dim3 grid((unsigned)(turns < ME_WAVE_BLOCKS ? turns : ME_WAVE_BLOCKS));
    if (mfma)
        hipLaunchKernelGGL(({kernel}<proc_{name}, true>), grid, dim3(64), 0, s, mom, nevt, out, spins, prm, idx,
                           count, eb);
    else
        hipLaunchKernelGGL(({kernel}<proc_{name}, false>), grid, dim3(64), 0, s, mom, nevt, out, spins, prm, idx,
                           count, eb);
"""
# one event per workgroup
_LAUNCH_GROUP = """    const dim3 grid((unsigned)(nevt < ME_GROUP_BLOCKS ? nevt : ME_GROUP_BLOCKS));
    if (mfma)
        hipLaunchKernelGGL(({kernel}<proc_{name}, true>), grid, dim3(w5::THREADS), 0, s, mom, nevt, out, spins, prm,
                           idx, count);
    else
        hipLaunchKernelGGL(({kernel}<proc_{name}, false>), grid, dim3(w5::THREADS), 0, s, mom, nevt, out, spins, prm,
                           idx, count);
"""
# the same with four times the lanes per event, one for each spin pair, while the call is
# within one wave per SIMD that way
_LAUNCH_FEW = """    if (nevt <= 1024 * {per} / 4) {{
        me_each_launch(nevt, {per} / 4, 64, [&](int64_t first, unsigned blocks) {{
            hipLaunchKernelGGL(({kernel}<proc_{name}, void, 4 * 64 / {per}>), dim3(blocks), dim3(64), 0, s, mom, nevt,
                               out, spins, prm, idx, count, first, nullptr, nullptr);
        }});
        return hipGetLastError();
    }}
"""
# several events per wave
_LAUNCH_LANES = """    (void)mfma;
    me_each_launch(nevt, {per}, 64, [&](int64_t first, unsigned blocks) {{
        hipLaunchKernelGGL(({kernel}<proc_{name}>), dim3(blocks), dim3(64), 0, s, mom, nevt, out, spins, prm, idx,
                           count, first, nullptr, nullptr);
    }});
"""


def _wave_tu(name):
    if name in EVENTS_PER_WAVE:
        launch = _LAUNCH_FEW + _LAUNCH_LANES
        return _TU_WAVE.format(name=name, header="me_gg_pol.h",
                               launch=launch.format(name=name, kernel=WAVE[name], per=EVENTS_PER_WAVE[name]))
    group = name in COOP
    launch = (_LAUNCH_GROUP if group else _LAUNCH_WAVE).format(name=name, kernel=WAVE[name])
    return _TU_WAVE.format(name=name, header="me_wave5.h" if group else "me_wave.h", launch=launch)


_TU_MC = """// Generated translation unit: multi-channel kernel of {name}.
#include "me_kernels.h"
#include "gen/proc_{name}_mc.h"

hipError_t me_launch_mc_{name}(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                               const me_params& prm, const int* chan, double* alpha, hipStream_t s) {{
    const dim3 grid((unsigned)((nevt + ME_BLOCK - 1) / ME_BLOCK));
    hipLaunchKernelGGL((k_me_gg_mc<proc_{name}_mc>), grid, dim3(ME_BLOCK), 0, s, mom, nevt, out, hels, nh, prm,
                       chan, alpha);
    return hipGetLastError();
}}

#ifndef __HIP_DEVICE_COMPILE__
extern const int me_nchan_{name} = proc_{name}_mc::nchan;
extern const char* const* const me_chan_desc_{name} = channel_desc_{name};
#endif
"""

_TU_CHAN = """// Generated translation unit: multi-channel form of {name} with shared wavefunctions.
#include "{header}"
#include "gen/proc_{name}.h"
#include "gen/proc_{name}_mc.h"

hipError_t me_launch_sum_{name}(const double* mom, int64_t nevt, double* out, unsigned spins, const me_params& prm,
                                const int* idx, const int* count, bool mfma, hipStream_t s);

hipError_t me_launch_chan_{name}(const double* mom, int64_t nevt, double* out, const me_params& prm, const int* chan,
                                 double* alpha, hipStream_t s) {{
{launch}    return hipGetLastError();
}}
"""

# weights in a kernel of their own
_LAUNCH_CHAN_WAVE = """    const hipError_t e = me_launch_sum_{name}(mom, nevt, out, 0xfu, prm, nullptr, nullptr, false, s);
    if (e != hipSuccess) return e;
    const int eb = me_wave_events(nevt);
    const int64_t turns = (nevt + eb - 1) / eb;
    const dim3 grid((unsigned)(turns < ME_WAVE_BLOCKS ? turns : ME_WAVE_BLOCKS));
    hipLaunchKernelGGL((k_me_gg4_chan<chan_ids_{name}>), grid, dim3(64), 0, s, mom, nevt, chan, alpha, prm, eb);
"""
# with |M|^2 in one kernel
_LAUNCH_CHAN_LANES = """    me_each_launch(nevt, {per}, 64, [&](int64_t first, unsigned blocks) {{
        hipLaunchKernelGGL(({kernel}<proc_{name}, chan_ids_{name}>), dim3(blocks), dim3(64), 0, s, mom, nevt, out, 0xfu,
                           prm, nullptr, nullptr, first, chan, alpha);
    }});
"""


def _chan_tu(name):
    if name in EVENTS_PER_WAVE:
        launch = _LAUNCH_CHAN_LANES.format(name=name, kernel=WAVE[name], per=EVENTS_PER_WAVE[name])
        return _TU_CHAN.format(name=name, header="me_gg_pol.h", launch=launch)
    return _TU_CHAN.format(name=name, header="me_chan.h", launch=_LAUNCH_CHAN_WAVE.format(name=name))


_CM = """
static hipError_t launch_f64_cm(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                const me_params& prm, double* qhel, int lg, hipStream_t s) {{
    const dim3 grid((unsigned)(((nevt << lg) + ME_BLOCK - 1) / ME_BLOCK));
    hipLaunchKernelGGL((k_me_gg_cm<{proc}>), grid, dim3(ME_BLOCK), 0, s, mom, nevt, out, hels, nh, prm, qhel, lg);
    return hipGetLastError();
}}
"""

_TU_COOP = """// Generated translation unit: kernels of {name} (workgroup form, J in LDS).
#include "me_coop.h"
{include}

static hipError_t launch_f64(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                             const me_params& prm, double* qhel, int lg, hipStream_t s) {{
    const dim3 grid((unsigned)(((nevt << lg) + ME_TILE - 1) / ME_TILE));
    hipLaunchKernelGGL((k_me_gg_coop<{proc}>), grid, dim3(ME_TILE * {proc}::waves), 0, s, mom, nevt, out, hels,
                       nh, prm, qhel, lg);
    return hipGetLastError();
}}

#ifndef __HIP_DEVICE_COMPILE__  // the table entry holds host function pointers
// the mixed-precision launcher and the matrix-core colour form are compiled in
// translation units of their own
hipError_t me_launch_mixed_{name}(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                  const me_params& prm, float tol, float cest, int* flag_count, int* flag_idx,
                                  float* err_out, unsigned char* flag_out, float2* part, hipStream_t s);
hipError_t me_launch_f64_cm_{name}(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                   const me_params& prm, double* qhel, int lg, hipStream_t s);
hipError_t me_launch_sum_{name}(const double* mom, int64_t nevt, double* out, unsigned spins, const me_params& prm,
                                const int* idx, const int* count, bool mfma, hipStream_t s);
extern const me_process_desc me_desc_{name} = {{
    "{name}", ME_KIND_GG, {proc}::npart, {proc}::ndiag, {proc}::ncol, {proc}::nhel,
    {proc}::flops_amp, {proc}::flops_colour, {proc}::flops_executed, launch_f64, nullptr, me_launch_mixed_{name}, {cest},
    me_launch_f64_cm_{name}, nullptr, 0, nullptr, me_launch_sum_{name}, nullptr, false, 16384}};
#endif
"""

_TU_COOP_CM = """// Generated translation unit: float64 kernel of {name} with the colour sum on the matrix cores.
#include "me_coop.h"
{include}

hipError_t me_launch_f64_cm_{name}(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                   const me_params& prm, double* qhel, int lg, hipStream_t s) {{
    const dim3 grid((unsigned)(((nevt << lg) + ME_TILE - 1) / ME_TILE));
    hipLaunchKernelGGL((k_me_gg_coop<{proc}, true>), grid, dim3(ME_TILE * {proc}::waves), 0, s, mom, nevt, out,
                       hels, nh, prm, qhel, lg);
    return hipGetLastError();
}}
"""

_TU_COOP_MIXED = """// Generated translation unit: mixed-precision kernel of {name} (workgroup form).
#include "me_coop_mixed.h"
{include}

hipError_t me_launch_mixed_{name}(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                  const me_params& prm, float tol, float cest, int* flag_count, int* flag_idx,
                                  float* err_out, unsigned char* flag_out, float2*, hipStream_t s) {{
    if (flag_count) hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, s, flag_count);
    const dim3 grid((unsigned)((nevt + ME_TILE - 1) / ME_TILE));
    hipLaunchKernelGGL((k_me_gg_coop_mixed<{proc}>), grid, dim3(ME_TILE * {proc}::waves), 0, s, mom, nevt, out,
                       hels, nh, prm, tol, cest, flag_count, flag_idx, err_out, flag_out);
    return hipGetLastError();
}}
"""

_MIXED = """
static hipError_t launch_mixed(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                               const me_params& prm, float tol, float cest, int* flag_count, int* flag_idx,
                               float* err_out, unsigned char* flag_out, float2* part, hipStream_t s) {{
    if (flag_count) hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, s, flag_count);
    const unsigned tiles = (unsigned)((nevt + ME_BLOCK - 1) / ME_BLOCK);
    const int per = part ? mixed_per_block(nevt, nh) : nh;
    if (per >= nh) part = nullptr;
    hipLaunchKernelGGL((k_me_gg_mixed<{proc}>), dim3(tiles, part ? (unsigned)((nh + per - 1) / per) : 1u), dim3(ME_BLOCK),
                       0, s, mom, nevt, out, hels, nh, prm, tol, cest, flag_count, flag_idx, err_out, flag_out, part, per);
    if (part)
        hipLaunchKernelGGL((k_mixed_sum<{proc}>), dim3(tiles), dim3(64), 0, s, part, nevt, nh, tol, cest, out, flag_count,
                           flag_idx, err_out, flag_out);
    return hipGetLastError();
}}
"""

_REG = """// Generated process table.
#include <cstring>
#include "me_launch.h"
{decls}
static const me_process_desc* const table[] = {{{ptrs}}};

const me_process_desc* me_find_process(const char* name) {{
    for (const me_process_desc* d : table)
        if (std::strcmp(d->name, name) == 0) return d;
    return nullptr;
}}
"""


def _write(path, text):
    old = open(path).read() if os.path.exists(path) else None
    if old != text:
        with open(path, "w") as f:
            f.write(text)


def generate_sources(processes):
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2503_21935_amd.gen import MULTICHANNEL, QEW_SPECS, generate

    info = generate(GEN, [p for p in processes if p.startswith("gg_") or p in QEW_SPECS])
    tus = []
    for name in processes:
        if name in QEW_SPECS:
            path = os.path.join(GEN, f"tu_{name}.hip")
            _write(path, _TU_QEW.format(name=name, include=f'#include "gen/proc_{name}.h"', proc=f"proc_{name}"))
            tus.append(path)
            continue
        if name == "ee_mumu":
            inc, proc, kind = "", "proc_ee_mumu", "ME_KIND_EE"
            mixed, mixed_ptr = "", "nullptr"
        else:
            inc, proc, kind = f'#include "gen/proc_{name}.h"', f"proc_{name}", "ME_KIND_GG"
            mixed, mixed_ptr = _MIXED.format(proc=proc), "launch_mixed"
        path = os.path.join(GEN, f"tu_{name}.hip")
        if name in COOP:
            _write(path, _TU_COOP.format(name=name, include=inc, proc=proc, cest=MIXED_CEST.get(name, 8.0)))
            tus.append(path)
            path_m = os.path.join(GEN, f"tu_{name}_mixed.hip")
            _write(path_m, _TU_COOP_MIXED.format(name=name, include=inc, proc=proc))
            tus.append(path_m)
            path_c = os.path.join(GEN, f"tu_{name}_cm.hip")
            _write(path_c, _TU_COOP_CM.format(name=name, include=inc, proc=proc))
            tus.append(path_c)
            path_w = os.path.join(GEN, f"tu_{name}_wave.hip")
            _write(path_w, _wave_tu(name))
            tus.append(path_w)
            continue
        cm, cm_ptr = ("", "nullptr")
        if name in CM:
            cm, cm_ptr = _CM.format(proc=proc), "launch_f64_cm"
        mc_ptr, mc_n, mc_desc, chan_ptr = "nullptr", "0", "nullptr", "nullptr"
        if name in MULTICHANNEL:
            cm += _MC_DECL.format(name=name)
            mc_ptr, mc_n, mc_desc = f"me_launch_mc_{name}", f"me_nchan_{name}", f"me_chan_desc_{name}"
            path_mc = os.path.join(GEN, f"tu_{name}_mc.hip")
            _write(path_mc, _TU_MC.format(name=name))
            tus.append(path_mc)
            path_ch = os.path.join(GEN, f"tu_{name}_chan.hip")
            _write(path_ch, _chan_tu(name))
            tus.append(path_ch)
            chan_ptr = f"me_launch_chan_{name}"
        sum_ptr = "nullptr"
        if name in WAVE:
            cm += _WAVE_DECL.format(name=name)
            sum_ptr = f"me_launch_sum_{name}"
            path_w = os.path.join(GEN, f"tu_{name}_wave.hip")
            _write(path_w, _wave_tu(name))
            tus.append(path_w)
        f64 = (_F64_EE if name == "ee_mumu" else _F64_GG).format(proc=proc)
        idx_ptr = "launch_f64_idx" if name == "ee_mumu" else "nullptr"
        _write(path, _TU.format(name=name, include=inc, f64=f64, idx_ptr=idx_ptr, proc=proc, kind=kind, mixed=mixed,
                                mixed_ptr=mixed_ptr, cest=MIXED_CEST.get(name, 8.0), cm=cm,
                                cm_ptr=cm_ptr, mc_ptr=mc_ptr, mc_n=mc_n, mc_desc=mc_desc, sum_ptr=sum_ptr, chan_ptr=chan_ptr,
                                mixed_part="false" if mixed_ptr == "nullptr" else "true",
                                hel_turn=0 if name == "ee_mumu" else 65536))
        tus.append(path)
    decls = "\n".join(f"extern const me_process_desc me_desc_{n};" for n in processes)
    ptrs = ", ".join(f"&me_desc_{n}" for n in processes)
    reg = os.path.join(GEN, "registry.cpp")
    _write(reg, _REG.format(decls=decls, ptrs=ptrs))
    return tus + [reg, os.path.join(CSRC, "me_api.cpp"), os.path.join(CSRC, "mlp.hip"),
                  os.path.join(CSRC, "me_unweight.hip"), os.path.join(CSRC, "ps_rambo.hip")], info


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    lang = ["-x", "hip"] if src.endswith((".hip", ".cpp")) else []
    cmd = [HIPCC] + HIPFLAGS + lang + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr[-4000:]}")
    return obj


def build(processes=None, jobs: int = 8, verbose: bool = True):
    processes = processes or PROCESSES
    os.makedirs(GEN, exist_ok=True)
    os.makedirs(OBJ, exist_ok=True)
    srcs, info = generate_sources(processes)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return info


if __name__ == "__main__":
    procs = sys.argv[1:] or None
    build(procs)
