"""Writes the kernel-instance units: zk_batch_{row,col}_{f64,f32}.hip and, so
that they compile in parallel, their further parts ..._1.hip, ..._2.hip, ....
Each part holds a table of its kernels by team shape (T, E, padded) and form;
the first one also lists the tables of all parts.  Run from any directory; the
units are committed, this script regenerates them."""
import os

HERE = os.path.dirname(os.path.abspath(__file__))
# power-of-two axes: padded iff E % 3 == 0
POW2 = ([(T, E) for T in (2, 4, 8, 16) for E in (2, 3, 4, 6)]
        + [(T, E) for T in (32, 64, 128, 256) for E in (2, 3, 4, 6, 8, 12)]
        + [(512, E) for E in (2, 3, 4, 6)] + [(1024, E) for E in (2, 3)])
SHAPES = [(T, E, E % 3 == 0) for T, E in POW2]
# axes of n = 3 2^k and 5 2^k points: teams of n / 2 threads, E = 3 padded and 2 base (FP64 only)
ODD = sorted([3 * 2 ** k for k in range(1, 9)] + [5 * 2 ** k for k in range(1, 8)])
SHAPES += [(T, E, E == 3) for T in ODD for E in (2, 3)]
# and teams of a power of two: E = 9 padded and 6 base, E = 15 padded and 10 base
SHAPES += ([(T, 9, True) for T in (2, 4, 8, 16, 32, 64, 128, 256)]
           + [(T, 6, False) for T in (2, 4, 8, 16, 32, 64, 128, 256)])
SHAPES += [(T, 15, True) for T in (2, 4, 8, 16, 32, 64, 128)] + [(T, 10, False) for T in (2, 4, 8, 16, 32, 64, 128)]
PARTS = {"row_f64": 7, "row_f32": 5, "col_f64": 2, "col_f32": 2}


def team_slot(T):
    """as team_slot() in zk_kernels.hpp"""
    return 1 << (T - 1).bit_length() if T <= 64 else (T + 63) // 64 * 64


def block_threads(T):
    """as block_threads() in zk_kernels.hpp"""
    return team_slot(T) if team_slot(T) > 128 else 256


def lanes_ok(T, E, pad, real_bytes):
    """as row_lanes_ok() in zk_kernels.hpp"""
    N, tpb = T * E, block_threads(T) // team_slot(T)
    return (pad and E % 5 != 0 and T % 64 == 0 and T & (T - 1) == 0 and T <= 1024
            and 2 * tpb * N * 2 * real_bytes <= 100 * 1024)


def fold_team_shape(f64, T, E, pad):
    """as fold_team_shape() in zk_kernels.hpp"""
    return pad and E == 3 and 3 * ((T + 63) // 64 * 64) <= 1024 and (T >= 16 if f64 else T in (64, 128, 256))


def compiled(T, E, pad):
    """as row_compiled_shapes() in zk_kernels.hpp"""
    return pad and ((E == 3 and T >= 16) or (E == 6 and 128 <= T <= 512))


def early(T, E, pad, f64):
    """as early_row_shape() in zk_kernels.hpp"""
    return E == 3 and compiled(T, E, pad) and T <= (128 if f64 else 32)


def b(v):
    return "true" if v else "false"


def instances(kind, real):
    """(weight, T, E, pad, form, kernel) of every instance; the weight is a rough compile time"""
    out = []
    for T, E, pad in SHAPES:
        if T in ODD and real == "float":
            continue
        if kind == "row":
            if T % 8 or (T * E * 2 // 3 if pad else T * E) % 16:  # no x axis has this shape
                if T not in (2, 4):
                    continue
            out.append((30 if compiled(T, E, pad) else E, T, E, pad, "KF_PLAIN", f"row_kernel_batch<{real}, {T}, {E}, {b(pad)}>"))
            if early(T, E, pad, real == "double"):
                out.append((30, T, E, pad, "KF_EARLY", f"row_kernel_batch<{real}, {T}, {E}, true, false, true>"))
            if lanes_ok(T, E, pad, 8 if real == "double" else 4):
                out.append((8, T, E, pad, "KF_LANES", f"row_kernel_batch<{real}, {T}, {E}, true, true>"))
        else:
            out.append((E, T, E, pad, "KF_PLAIN", f"col_kernel_batch<{real}, {T}, {E}, false, {b(pad)}>"))
            if not pad:
                out.append((E, T, E, pad, "KF_LIFTSYM", f"col_kernel_batch<{real}, {T}, {E}, true, false>"))
            if fold_team_shape(real == "double", T, E, pad):
                out.append((4, T, E, pad, "KF_FOLDS", f"col_kernel_folds<{real}, {T}, {E}>"))
    return out


for kind in ("row", "col"):
    for real, tag in (("double", "f64"), ("float", "f32")):
        parts = [[] for _ in range(PARTS[f"{kind}_{tag}"])]
        load = [0] * len(parts)
        for inst in sorted(instances(kind, real), reverse=True):
            k = load.index(min(load))
            parts[k].append(inst[1:])
            load[k] += inst[0]
        for k, part in enumerate(parts):
            name = f"zk_batch_{kind}_{tag}" + (f"_{k}" if k else "")
            lines = [f"// {name}.hip -- batched {kind}-pass kernel instances ({real} transforms);",
                     "// written by gen_batch_units.py.", '#include "zk_kernels.hpp"', "", "namespace zk {", "",
                     f"extern const KernelEntry {kind}_{tag}_{k}[];", f"const KernelEntry {kind}_{tag}_{k}[] = {{"]
            for T, E, pad, form, fn in sorted(part):
                lines.append(f"    {{{T}, {E}, {b(pad)}, {form}, reinterpret_cast<const void *>(&{fn})}},")
            lines += ["    {0, 0, false, 0, nullptr}};", ""]
            if k == 0:
                lines += [f"extern const KernelEntry {kind}_{tag}_{j}[];" for j in range(1, len(parts))]
                lines += [f"const KernelEntry *const {kind}_kernels_{tag}[] = {{"
                          + "".join(f"{kind}_{tag}_{j}, " for j in range(len(parts))) + "nullptr};", ""]
            lines += ["}  // namespace zk", ""]
            with open(os.path.join(HERE, name + ".hip"), "w") as f:
                f.write("\n".join(lines))
